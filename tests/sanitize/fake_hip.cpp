#include "fake_hip.h"

#include <algorithm>
#include <deque>
#include <map>
#include <mutex>
#include <set>

namespace {
enum Kind { LAUNCH, RECORD, WAIT, HOLD };
struct Op {
  Kind kind;
  long id;  // RECORD: its own number; WAIT: the record waited for
};
struct Stream {
  std::deque<Op> ops;
  bool caller = false, capturing = false;
};

std::mutex mu;
std::map<hipStream_t, Stream> streams;     // null stream and per-thread stream come with their first use
std::map<hipEvent_t, long> events;         // number of the latest record, 0: none
std::set<hipStream_t> took_kernels;
std::set<long> reached;
long next_record = 0, next_object = 0x1000;
int bad = 0, creations_left = -1;

template <typename T>
T new_handle() {
  return reinterpret_cast<T>(next_object += 16);
}
Stream* find(hipStream_t s) {
  auto it = streams.find(s);
  if (it != streams.end()) return &it->second;
  if (s == nullptr || s == hipStreamPerThread) return &streams[s];
  ++bad;
  return nullptr;
}
}  // namespace

namespace fake {
hipStream_t caller_stream() {
  std::lock_guard<std::mutex> lk(mu);
  hipStream_t s = new_handle<hipStream_t>();
  streams[s].caller = true;
  return s;
}
void hold(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  if (Stream* q = find(s)) q->ops.push_back({HOLD, 0});
}
void release(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  if (Stream* q = find(s))
    q->ops.erase(std::remove_if(q->ops.begin(), q->ops.end(), [](const Op& o) { return o.kind == HOLD; }),
                 q->ops.end());
}
void capture(hipStream_t s, bool on) {
  std::lock_guard<std::mutex> lk(mu);
  if (Stream* q = find(s)) q->capturing = on;
}
void launch(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  took_kernels.insert(s);
  if (Stream* q = find(s)) q->ops.push_back({LAUNCH, 0});
}
void run() {
  std::lock_guard<std::mutex> lk(mu);
  for (bool moved = true; moved;) {
    moved = false;
    for (auto& [h, q] : streams) {
      while (!q.ops.empty()) {
        const Op o = q.ops.front();
        if (o.kind == HOLD || (o.kind == WAIT && !reached.count(o.id))) break;
        if (o.kind == RECORD) reached.insert(o.id);
        q.ops.pop_front();
        moved = true;
      }
    }
  }
}
bool idle(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  Stream* q = find(s);
  return q && q->ops.empty();
}
std::vector<hipStream_t> launched_on() {
  std::lock_guard<std::mutex> lk(mu);
  std::vector<hipStream_t> v(took_kernels.begin(), took_kernels.end());
  took_kernels.clear();
  return v;
}
int misuse() {
  std::lock_guard<std::mutex> lk(mu);
  return bad;
}
int live_streams() {
  std::lock_guard<std::mutex> lk(mu);
  int n = 0;
  for (auto& [h, q] : streams) n += h != nullptr && h != hipStreamPerThread && !q.caller;
  return n;
}
int live_events() {
  std::lock_guard<std::mutex> lk(mu);
  return (int)events.size();
}
void fail_stream_create_after(int n) {
  std::lock_guard<std::mutex> lk(mu);
  creations_left = n;
}
}  // namespace fake

extern "C" {
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  if (creations_left == 0) return hipErrorOutOfMemory;
  if (creations_left > 0) --creations_left;
  *s = new_handle<hipStream_t>();
  streams[*s];
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  auto it = streams.find(s);
  if (it == streams.end() || it->second.caller) {
    ++bad;
    return hipErrorInvalidHandle;
  }
  if (!it->second.ops.empty()) ++bad;  // its work may be lost, or the call may wait for it
  streams.erase(it);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  std::lock_guard<std::mutex> lk(mu);
  Stream* q = find(s);
  if (!q) return hipErrorInvalidHandle;
  *st = q->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  Stream* q = find(s);
  auto it = events.find(e);
  if (!q || it == events.end()) {
    ++bad;
    return hipErrorInvalidHandle;
  }
  if (it->second) q->ops.push_back({WAIT, it->second});
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  *e = new_handle<hipEvent_t>();
  events[*e] = 0;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::lock_guard<std::mutex> lk(mu);
  if (!events.erase(e)) ++bad;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  std::lock_guard<std::mutex> lk(mu);
  Stream* q = find(s);
  auto it = events.find(e);
  if (!q || it == events.end()) {
    ++bad;
    return hipErrorInvalidHandle;
  }
  it->second = ++next_record;
  q->ops.push_back({RECORD, it->second});
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}
}
