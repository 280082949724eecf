// A stand-in for the HIP runtime calls that the stage schedule makes, for checks
// of its streams and events without a GPU.  Streams are queues of operations;
// nothing runs until fake::run(), which executes every operation whose stream
// has reached it, whose awaited event records have been reached and that no hold
// precedes.  Misuse (a destroyed stream or event used again, a stream destroyed
// with work still in it) is counted, not fatal.
#pragma once
#include <hip/hip_runtime_api.h>

#include <vector>

namespace fake {
hipStream_t caller_stream();                 // a stream of the caller's
void hold(hipStream_t s);                    // keeps s at this point (a receive that has not arrived)
void release(hipStream_t s);                 // lets every hold on s pass
void capture(hipStream_t s, bool on);        // what hipStreamIsCapturing reports for s
void launch(hipStream_t s);                  // a kernel (called by the launch stubs)
void run();                                  // execute whatever can run
bool idle(hipStream_t s);                    // s has no operation left
std::vector<hipStream_t> launched_on();      // streams that took kernels since the last call, each once
int misuse();                                // misuses so far
int live_streams();                          // the library's streams not yet destroyed
int live_events();
void fail_stream_create_after(int n);        // the (n + 1)-th creation fails (< 0: none)
}  // namespace fake
