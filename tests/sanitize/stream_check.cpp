// The stage schedule's streams against a stand-in for the HIP runtime
// (fake_hip.h): which calls may wait for which, and how long the library's
// streams live.  `stream_check <scenario>` runs one of the scenarios below.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <thread>
#include <vector>

#include "fake_hip.h"
#include "merak_stage.h"

#define EXPECT(c)                                                             \
  do {                                                                        \
    if (!(c)) {                                                               \
      fprintf(stderr, "check failed at %s:%d: %s\n", __FILE__, __LINE__, #c); \
      exit(1);                                                                \
    }                                                                         \
  } while (0)

namespace {
// Device memory is never touched on the host: any aligned address will do.
void* dev(uintptr_t k) { return reinterpret_cast<void*>((uintptr_t)0x100000000 + k * 0x1000000); }

merak_stage_config config() {
  merak_stage_config c{};
  c.n_blocks = 3;
  c.hidden = 256;
  c.n_heads = 4;
  c.ffn = 1024;
  c.seq_len = 128;
  c.micro_batch = 4;
  c.tp_degree = 1;
  c.n_sub_microbatches = 2;
  c.recompute_mask = 1;
  c.dtype = MERAK_BF16;
  c.ln_eps = 1e-5f;
  return c;
}

struct Pair {
  hipStream_t s0, s1;
};
Pair pair() { return {fake::caller_stream(), fake::caller_stream()}; }

merak_stage_t create(int k) {
  const merak_stage_config c = config();
  size_t ws = 0, rc = 0;
  EXPECT(merak_stage_workspace_bytes(&c, &ws, &rc) == MERAK_OK);
  merak_stage_t h = nullptr;
  EXPECT(merak_stage_create(&c, dev(100 + 2 * k), ws, dev(101 + 2 * k), rc, &h) == MERAK_OK);
  return h;
}

void backward(merak_stage_t h, Pair p) {
  EXPECT(merak_stage_bwd(h, dev(1), dev(2), dev(3), static_cast<float*>(dev(4)), 0, nullptr, p.s0, p.s1) == MERAK_OK);
}
void step(merak_stage_t h, Pair p) {
  EXPECT(merak_stage_fwd(h, dev(1), dev(5), dev(6), nullptr, p.s0, p.s1) == MERAK_OK);
  EXPECT(merak_stage_recompute(h, dev(1), p.s0, p.s1) == MERAK_OK);
  backward(h, p);
}

// A handle is destroyed once its own work is done; another handle that has
// used the same stream of the library keeps its queued work.
void lifetime() {
  merak_stage_t a = create(0), b = create(1);
  const Pair x = pair();
  step(a, x);
  fake::run();
  EXPECT(fake::idle(x.s0) && fake::idle(x.s1));
  fake::hold(x.s0);
  step(b, x);
  fake::run();
  EXPECT(merak_stage_destroy(a) == MERAK_OK);
  EXPECT(fake::misuse() == 0);
  fake::release(x.s0);
  fake::run();
  EXPECT(fake::idle(x.s0) && fake::idle(x.s1));
  step(b, x);
  fake::run();
  EXPECT(fake::idle(x.s0) && fake::idle(x.s1));
  EXPECT(merak_stage_destroy(b) == MERAK_OK);
}

// Calls on one pair of caller streams never wait for what another pair's streams
// wait for, also where a handle has used both.
void moved() {
  merak_stage_t a = create(0), b = create(1), c = create(2);
  const Pair x = pair(), y = pair(), z = pair();
  step(a, x);
  step(b, x);
  fake::run();
  fake::hold(x.s0);
  step(b, x);  // waits on x
  step(a, y);  // and what it has to receive, a sends on y
  step(c, z);
  fake::run();
  EXPECT(!fake::idle(x.s0));
  EXPECT(fake::idle(y.s0) && fake::idle(y.s1));
  EXPECT(fake::idle(z.s0) && fake::idle(z.s1));
  // the other way round, and with only the second stream held back
  fake::release(x.s0);
  fake::run();
  EXPECT(fake::idle(x.s0));
  fake::hold(y.s1);
  step(a, y);
  step(c, y);
  step(b, z);
  step(b, x);
  fake::run();
  EXPECT(!fake::idle(y.s0));
  EXPECT(fake::idle(x.s0) && fake::idle(z.s0));
  fake::release(y.s1);
  fake::run();
  EXPECT(fake::idle(y.s0) && fake::idle(y.s1));
  for (merak_stage_t h : {a, b, c}) EXPECT(merak_stage_destroy(h) == MERAK_OK);
}

// The library's streams that took kernels since the last call.
std::vector<hipStream_t> aux_streams(std::vector<Pair> callers) {
  std::vector<hipStream_t> v;
  for (hipStream_t s : fake::launched_on()) {
    bool caller = false;
    for (const Pair& p : callers) caller |= s == p.s0 || s == p.s1;
    if (!caller) v.push_back(s);
  }
  return v;
}

// Handles on one pair share a stream, under graph capture too: every call on it is
// then captured.  Calls on other streams use another meanwhile.
void captured() {
  merak_stage_t h[3] = {create(0), create(1), create(2)};
  const Pair x = pair(), y = pair();
  aux_streams({});
  for (merak_stage_t k : {h[0], h[1]}) step(k, x);
  const std::vector<hipStream_t> shared = aux_streams({x});
  EXPECT(shared.size() == 1);
  fake::run();
  fake::capture(x.s0, true);
  for (merak_stage_t k : {h[0], h[1]}) step(k, x);
  EXPECT(aux_streams({x}) == shared);
  step(h[2], y);  // eager
  const std::vector<hipStream_t> other = aux_streams({y});
  EXPECT(other.size() == 1 && other != shared);
  fake::capture(x.s0, false);
  for (merak_stage_t k : h) step(k, x);
  EXPECT(aux_streams({x}) == shared);
  fake::run();
  for (merak_stage_t k : h) EXPECT(merak_stage_destroy(k) == MERAK_OK);
}

// Host threads at once, each with handles of its own: on pairs of their own, and
// all on one pair.
void threads() {
  const Pair shared = pair();
  for (bool one_pair : {false, true}) {
    std::vector<std::thread> ts;
    for (int t = 0; t < 4; ++t)
      ts.emplace_back([=] {
        const Pair mine = one_pair ? shared : pair();
        for (int round = 0; round < 20; ++round) {
          merak_stage_t a = create(2 * t), b = create(2 * t + 1);
          for (int i = 0; i < 5; ++i) {
            step(a, mine);
            step(b, mine);
          }
          fake::run();
          EXPECT(merak_stage_destroy(a) == MERAK_OK);
          step(b, mine);
          fake::run();
          EXPECT(merak_stage_destroy(b) == MERAK_OK);
        }
      });
    for (std::thread& t : ts) t.join();
    fake::run();
    EXPECT(fake::idle(shared.s0) && fake::idle(shared.s1));
  }
}

// Which stream a call takes: a handle alone takes its own from pair to pair; with
// more pairs than handles the calls on the others run on the caller's streams; the
// per-thread stream (whose value names another stream in each thread) is not shared.
void many_pairs() {
  merak_stage_t a = create(0);
  std::vector<Pair> ps;
  for (int i = 0; i < 12; ++i) ps.push_back(pair());
  ps.push_back({nullptr, nullptr});
  aux_streams({});
  step(a, ps[0]);
  const std::vector<hipStream_t> own = aux_streams(ps);
  EXPECT(own.size() == 1);
  for (const Pair& p : ps) {
    step(a, p);
    EXPECT(aux_streams(ps) == own);
    fake::run();
    EXPECT(fake::idle(p.s0) && fake::idle(p.s1));
  }
  merak_stage_t b = create(1);
  for (int turn = 0; turn < 2; ++turn)
    for (const Pair& p : ps) {
      step(a, p);
      step(b, p);
      fake::run();
      EXPECT(fake::idle(p.s0) && fake::idle(p.s1));
    }
  EXPECT(fake::live_streams() == 2);
  merak_stage_t c = create(2), d = create(3);
  const Pair per_thread{hipStreamPerThread, hipStreamPerThread};
  aux_streams({});
  step(c, per_thread);
  const std::vector<hipStream_t> sc = aux_streams({per_thread});
  step(d, per_thread);
  const std::vector<hipStream_t> sd = aux_streams({per_thread});
  EXPECT(sc.size() == 1 && sd.size() == 1 && sc[0] != sd[0]);
  step(a, per_thread);
  EXPECT(aux_streams({per_thread}).empty());
  fake::run();
  EXPECT(fake::idle(hipStreamPerThread));
  for (merak_stage_t h : {a, b, c, d}) EXPECT(merak_stage_destroy(h) == MERAK_OK);
}

// A creation that fails part-way leaves nothing behind.
void failed_create() {
  const merak_stage_config c = config();
  size_t ws = 0, rc = 0;
  EXPECT(merak_stage_workspace_bytes(&c, &ws, &rc) == MERAK_OK);
  fake::fail_stream_create_after(0);
  merak_stage_t h = nullptr;
  EXPECT(merak_stage_create(&c, dev(100), ws, dev(101), rc, &h) == MERAK_ERR_HIP && h == nullptr);
  EXPECT(fake::live_streams() == 0 && fake::live_events() == 0);
  fake::fail_stream_create_after(-1);
}

const struct {
  const char* name;
  void (*run)();
} kScenarios[] = {
    {"lifetime", lifetime},
    {"moved", moved},
    {"captured", captured},
    {"threads", threads},
    {"many_pairs", many_pairs},
    {"failed_create", failed_create},
};
}  // namespace

int main(int argc, char** argv) {
  for (const auto& s : kScenarios)
    if (argc == 2 && !strcmp(argv[1], s.name)) {
      s.run();
      // every scenario destroys its handles after their work
      EXPECT(fake::misuse() == 0);
      EXPECT(fake::live_streams() == 0 && fake::live_events() == 0);
      printf("%s passed\n", s.name);
      return 0;
    }
  fprintf(stderr, "no such scenario\n");
  return 2;
}
