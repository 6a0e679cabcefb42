// The slice scheduler against a model of the GPU's streams, without a GPU.  The runtime functions it calls are defined
// here and take the place of the HIP runtime's: a stream is a thread that carries out what was enqueued on it, in order,
// while its gate is open.  Launches come from the checks themselves; they do to the progress words what a kernel does.
// Usage: scheduler_check <check>; the exit status says whether it held.  A check that blocks is ended by the caller.
#include "vkv_internal.h"

#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <random>
#include <thread>

using namespace vkv;

#define CHECK(cond)                                                            \
  do {                                                                         \
    if (!(cond)) {                                                             \
      std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #cond);          \
      std::_Exit(1);                                                           \
    }                                                                          \
  } while (0)

namespace {

std::mutex mu;
std::condition_variable changed;
int unfinished = 0, most_unfinished = 0;
int launched = 0;

struct Event {
  uint64_t recorded = 0, done = 0;
};

struct Stream {
  std::deque<std::function<void()>> todo;   // run without the lock
  bool open = true, busy = false, capturing = false;
  hipError_t failed = hipSuccess;
  std::thread worker;
  Stream() {
    worker = std::thread([this]() {
      std::unique_lock<std::mutex> lock(mu);
      for (;;) {
        changed.wait(lock, [&]() { return open && !todo.empty(); });
        auto what = std::move(todo.front());
        todo.pop_front();
        busy = true;
        lock.unlock();
        what();
        lock.lock();
        busy = false;
        changed.notify_all();
      }
    });
    worker.detach();
  }
};

std::map<hipStream_t, Stream*> streams;
Stream* stream(hipStream_t s) {   // with the lock held
  Stream*& p = streams[s];
  if (!p) p = new Stream;
  return p;
}
void push(hipStream_t s, std::function<void()> what) {
  std::lock_guard<std::mutex> lock(mu);
  stream(s)->todo.push_back(std::move(what));
  changed.notify_all();
}
void gate(hipStream_t s, bool open) {
  std::lock_guard<std::mutex> lock(mu);
  stream(s)->open = open;
  changed.notify_all();
}
void wait_idle(hipStream_t s) {
  std::unique_lock<std::mutex> lock(mu);
  changed.wait(lock, [&]() { return stream(s)->todo.empty() && !stream(s)->busy; });
}

hipStream_t handle(int n) { return (hipStream_t)(uintptr_t)(0x1000 + 64 * n); }

bool drop_uploads = false;
int kernels = 0, fail_kernel = 0;   // runtime launches so far; the one that fails, 0 = none
int pause_us = 0;   // how long a launch takes, 0 = as short as it gets

// what a slice kernel does for the scheduler
void launch(vkv_pool* p, hipStream_t on, int longest) {
  static uint32_t header[64];
  const Report r = next_report(p, header);
  {
    std::lock_guard<std::mutex> lock(mu);
    most_unfinished = std::max(most_unfinished, ++unfinished);
    ++launched;
  }
  if (stream(on)->capturing) {
    CHECK(!r.started && !r.finished);
    std::lock_guard<std::mutex> lock(mu);
    --unfinished;
    return;
  }
  const int us = longest ? rand() % longest : pause_us;
  push(on, [r, us]() {
    if (r.started) __atomic_store_n(r.started, r.seq, __ATOMIC_RELEASE);
    if (us) std::this_thread::sleep_for(std::chrono::microseconds(us));
    {
      std::lock_guard<std::mutex> lock(mu);
      --unfinished;
    }
    if (r.finished) __atomic_store_n(r.finished, r.seq, __ATOMIC_RELEASE);
  });
}

struct Call {
  bool may_overlap = false, end_events = false;
  int n_tail = 0;
};

int run(vkv_pool* p, hipStream_t hs, int n, int max_inflight, Call c = {}, int longest = 0, int32_t* cursor = nullptr) {
  int32_t own = 0;
  return run_slices(p, cursor ? cursor : &own, n, max_inflight, hs, "check",
                    [&](int32_t, hipStream_t on) {
                      launch(p, on, longest);
                      return VKV_OK;
                    },
                    c.n_tail,
                    [&](int32_t) {
                      launch(p, hs, longest);
                      return VKV_OK;
                    },
                    c.n_tail > 0, c.may_overlap, c.end_events);
}

vkv_pool* make_pool() {
  vkv_pool_config c{};
  c.num_layers = c.num_q_heads = c.num_kv_heads = c.num_blocks = c.blocks_per_handle = 1;
  c.head_dim = 64;
  c.block_tokens = 16;
  vkv_pool* p = nullptr;
  CHECK(kv_pool_init(&c, &p) == VKV_OK);
  CHECK(ensure_plan_stage(p, 4096) == VKV_OK);   // as a bind does
  return p;
}

const Call kDecodeTwo{true, true, 0}, kPrefillTwo{true, false, 0}, kPrefillMerged{true, false, 2}, kOne{false, false, 0};

// Calls of every kind in any order and with any limit: never more launches unfinished than the call at hand allows.
void bound() {
  vkv_pool* p = make_pool();
  srand(7);
  for (int rep = 0; rep < 400; ++rep) {
    CHECK(kv_sched_set_overlap(p, rand() % 4 != 0) == VKV_OK);
    const Call kinds[4] = {kDecodeTwo, kPrefillTwo, kPrefillMerged, kOne};
    const int max_inflight = 1 + rand() % 8;
    {   // what is unfinished when the call comes may have been allowed by a higher limit
      std::lock_guard<std::mutex> lock(mu);
      most_unfinished = 0;
    }
    CHECK(run(p, handle(0), 1 + rand() % 12, max_inflight, kinds[rand() % 4], rand() % 3 ? 60 : 1) == VKV_OK);
    std::lock_guard<std::mutex> lock(mu);
    CHECK(most_unfinished <= max_inflight);
  }
}

// A lower limit than the call before had, with the caller's stream held up and the second one not: what ended on the
// second stream says nothing about the caller's.
void lower_limit() {
  vkv_pool* p = make_pool();
  CHECK(kv_sched_set_overlap(p, 1) == VKV_OK);
  CHECK(run(p, handle(0), 2, 2, kPrefillTwo) == VKV_OK);   // the streams are there
  wait_idle(handle(0));
  std::thread later;
  CHECK(run_slices(p, [] { static int32_t at = 0; return &at; }(), 8, 8, handle(0), "check",
                   [&](int32_t s, hipStream_t on) {
                     if (s == 0) gate(handle(0), false);   // behind the fork
                     launch(p, on, 0);
                     return VKV_OK;
                   }, 0, nullptr, false, true, false) == VKV_OK);
  std::this_thread::sleep_for(std::chrono::milliseconds(30));   // the second stream's four are done, the others wait
  {
    std::lock_guard<std::mutex> lock(mu);
    CHECK(unfinished >= 4);
    most_unfinished = 0;
    pause_us = 200;
  }
  later = std::thread([]() {
    std::this_thread::sleep_for(std::chrono::milliseconds(30));
    gate(handle(0), true);
  });
  CHECK(run(p, handle(0), 6, 2, kPrefillTwo) == VKV_OK);
  later.join();
  std::lock_guard<std::mutex> lock(mu);
  CHECK(most_unfinished <= 2);
}

// Decode and prefill, one stream and two, taking turns: while there is room under the limit no call waits for the GPU.
void taking_turns() {
  vkv_pool* p = make_pool();
  CHECK(kv_sched_set_overlap(p, 1) == VKV_OK);
  CHECK(run(p, handle(0), 2, 2, kPrefillTwo) == VKV_OK);
  wait_idle(handle(0));
  gate(handle(0), false);
  CHECK(run(p, handle(0), 2, 8, kOne) == VKV_OK);
  CHECK(run(p, handle(0), 2, 8, kDecodeTwo) == VKV_OK);
  CHECK(run(p, handle(0), 1, 8, kOne) == VKV_OK);
  CHECK(run(p, handle(0), 2, 8, kPrefillTwo) == VKV_OK);
  CHECK(launched == 9 && unfinished == 7);
  gate(handle(0), true);
  // more turns than the ring has places, now that the GPU runs
  for (int rep = 0; rep < 50; ++rep)
    for (Call c : {kOne, kDecodeTwo, kPrefillMerged, kOne, kPrefillTwo}) {
      most_unfinished = 0;
      CHECK(run(p, handle(0), 3, 3, c, 40) == VKV_OK);
      CHECK(most_unfinished <= 3);
    }
}

// A yield finds launches of every kind in flight; when it returns none is left.
void yield_between() {
  vkv_pool* p = make_pool();
  CHECK(kv_sched_set_overlap(p, 1) == VKV_OK);
  const Call kinds[4] = {kOne, kDecodeTwo, kPrefillTwo, kPrefillMerged};
  for (int a = 0; a < 4; ++a)
    for (int b = 0; b < 4; ++b) {
      pause_us = 300;
      CHECK(run(p, handle(0), 3, 8, kinds[a]) == VKV_OK);
      CHECK(run(p, handle(0), 2, 8, kinds[b]) == VKV_OK);
      CHECK(kv_yield_request(p) == VKV_OK);
      int32_t cursor = 1;
      const int before = launched;
      CHECK(run(p, handle(0), 6, 8, kinds[a], 0, &cursor) == VKV_YIELDED);
      CHECK(cursor == 1 && launched == before && unfinished == 0);
      CHECK(kv_yield_clear(p) == VKV_OK);
      CHECK(run(p, handle(0), 6, 8, kinds[a], 0, &cursor) == VKV_OK);
      CHECK(cursor == 6 + kinds[a].n_tail && launched == before + 5 + kinds[a].n_tail);
    }
}

// Decode on one stream, prefill on another, both on one pool: a launch that starts late on one of them does not take
// back what the other's have reported.
void late_start() {
  vkv_pool* p = make_pool();
  for (int rep = 0; rep < 20; ++rep) {
    gate(handle(1), false);
    CHECK(run(p, handle(1), 1, 3) == VKV_OK);
    CHECK(run(p, handle(2), 2, 3) == VKV_OK);
    wait_idle(handle(2));
    gate(handle(1), true);   // starts only now, with an earlier number than the two that have ended
    wait_idle(handle(1));
    CHECK(run(p, handle(2), 5, 3) == VKV_OK);
    wait_idle(handle(2));
  }
}

void fail(hipStream_t s, hipError_t e) {
  std::lock_guard<std::mutex> lock(mu);
  stream(s)->failed = e;
  stream(s)->open = false;
}

// A stream that fails reports nothing any more: the call that waits for it, or for an upload on it, says so.
void failed_stream() {
  for (int max_inflight : {1, 2}) {
    vkv_pool* p = make_pool();
    const hipStream_t s = handle(max_inflight);
    CHECK(run(p, s, 2, max_inflight) == VKV_OK);
    wait_idle(s);
    fail(s, hipErrorLaunchFailure);
    CHECK(run(p, s, 4, max_inflight) == VKV_E_HIP);
    CHECK(std::strstr(vkv_last_error(), "hipStreamQuery"));
    CHECK(kv_yield_request(p) == VKV_OK);
    CHECK(run(p, s, 4, max_inflight) == VKV_E_HIP);
  }
  vkv_pool* p = make_pool();
  static char to[4096];
  CHECK(stage_upload(p->stage, to, sizeof to, handle(3)) == VKV_OK);
  CHECK(ensure_plan_stage(p, 64) == VKV_OK);
  fail(handle(3), hipErrorLaunchFailure);
  CHECK(stage_upload(p->stage, to, sizeof to, handle(3)) == VKV_OK);
  CHECK(ensure_plan_stage(p, 64) == VKV_E_HIP);
  // a kernel that never ran on a stream that has nothing left to do
  p = make_pool();
  drop_uploads = true;
  CHECK(stage_upload(p->stage, to, sizeof to, handle(4)) == VKV_OK);
  CHECK(ensure_plan_stage(p, 64) == VKV_E_HIP);
}

// Long waits end where the work does, however long it takes.
void long_waits() {
  vkv_pool* p = make_pool();
  pause_us = 12000;
  for (int max_inflight : {1, 2, 3}) CHECK(run(p, handle(0), 6, max_inflight) == VKV_OK);
  static char to[4096];
  CHECK(stage_upload(p->stage, to, sizeof to, handle(0)) == VKV_OK);
  CHECK(ensure_plan_stage(p, 64) == VKV_OK && unfinished == 0);
}

// Recorded into a graph a layer of any length goes through whole and leaves the launches in flight alone.
void recorded() {
  vkv_pool* p = make_pool();
  CHECK(kv_sched_set_overlap(p, 1) == VKV_OK);
  CHECK(run(p, handle(0), 3, 2, kOne) == VKV_OK);
  for (Call c : {kOne, kDecodeTwo, kPrefillMerged}) {
    for (int max_inflight : {1, 2, 8}) {
      {
        std::lock_guard<std::mutex> lock(mu);
        stream(handle(5))->capturing = stream(handle(9))->capturing = true;
      }
      const int before = launched;
      CHECK(run(p, handle(5), 40, max_inflight, c) == VKV_OK);
      CHECK(launched == before + 40 + c.n_tail);
      {
        std::lock_guard<std::mutex> lock(mu);
        stream(handle(5))->capturing = stream(handle(9))->capturing = false;
      }
      CHECK(run(p, handle(0), 3, max_inflight, c) == VKV_OK);
    }
  }
}

// A launch that fails leaves the caller's stream behind everything that went to the second one.
void failed_launch() {
  for (Call c : {kDecodeTwo, kPrefillTwo}) {
    vkv_pool* p = make_pool();
    CHECK(kv_sched_set_overlap(p, 1) == VKV_OK);
    gate(handle(9), false);
    int32_t cursor = 0;
    CHECK(run_slices(p, &cursor, 6, 8, handle(0), "check",
                     [&](int32_t s, hipStream_t on) {
                       if (s == 3) { set_error("slice 3"); return (int)VKV_E_HIP; }
                       launch(p, on, 0);
                       return (int)VKV_OK;
                     }, 0, nullptr, false, c.may_overlap, c.end_events) == VKV_E_HIP);
    CHECK(!std::strcmp(vkv_last_error(), "slice 3"));
    std::atomic<bool> passed{false};
    push(handle(0), [&]() { passed = true; });
    std::this_thread::sleep_for(std::chrono::milliseconds(30));
    CHECK(!passed);
    gate(handle(9), true);
    wait_idle(handle(0));
    CHECK(passed && unfinished == 0);
  }
}

// A relocation whose copy cannot be launched: the remap's staging buffer is free again only if its upload was part of
// that launch.
void failed_copy() {
  alignas(16) static char memory[64 * 4096];
  for (bool listed : {true, false}) {
    vkv_pool_config c{};
    c.num_layers = c.num_q_heads = c.num_kv_heads = c.blocks_per_handle = 1;
    c.head_dim = 64;
    c.block_tokens = 16;
    c.num_blocks = 64;
    c.base = memory;
    c.bytes = sizeof memory;
    vkv_pool* p = nullptr;
    CHECK(kv_pool_init(&c, &p) == VKV_OK && p->block_bytes == 4096);
    const int32_t ids[3] = {1, 2, 3};
    CHECK(kv_pool_adopt(p, ids, 3) == VKV_OK);
    const hipStream_t s = handle(listed ? 1 : 2);
    gate(s, false);
    static int32_t remap[64], table[1] = {1};
    fail_kernel = kernels + (listed ? 1 : 2);
    CHECK(kv_reclaim_range(p, 0, 8, table, 1, listed ? 0 : 4096, 0, s, s, remap, 0, nullptr) == VKV_E_HIP);
    CHECK(p->broken && p->remap.n_flags == (listed ? 0 : 1));
    gate(s, true);
    CHECK(stage_wait(p->remap) == VKV_OK && p->remap.n_flags == 0);
    CHECK(listed || remap[1] != 1);
  }
}

// Which decode layers go over two streams: long ones cut into several slices that are worth a launch each, or as told.
void overlap_rule() {
  const uint64_t mib = 1ull << 20;
  CHECK(!decode_overlaps(1, 5, 5000 * mib) && decode_overlaps(1, 6, 6000 * mib) && decode_overlaps(1, 9, 4264 * mib));
  CHECK(decode_overlaps(1, 34, 34000 * mib) && decode_overlaps(1, 6, 2000000000) && !decode_overlaps(1, 6, 1999999999));
  CHECK(decode_overlaps(1, 20, 2400 * mib) && !decode_overlaps(1, 20, 2400 * mib - 1) && !decode_overlaps(1, 7, 1000 * mib) && !decode_overlaps(1, 0, 0));
  CHECK(decode_overlaps(2, 2, 2) && decode_overlaps(2, 14, 1000 * mib));
}

}  // namespace

// ---- the runtime functions the library calls ----
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
static thread_local std::vector<Config> configs;

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  configs.push_back({grid, block, lds, s});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = configs.back().grid;
  *block = configs.back().block;
  *lds = configs.back().lds;
  *s = configs.back().stream;
  configs.pop_back();
  return hipSuccess;
}
// the kernels launched here: an upload by workgroups of 256, and one thread that stores a number
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void** args, size_t, hipStream_t s) {
  if (++kernels == fail_kernel) return hipErrorInvalidConfiguration;
  if (block.x == 256) {
    const UploadShare u = *(UploadShare*)args[0];
    push(s, [u, grid]() {
      if (drop_uploads) return;
      std::memcpy(u.dst, u.src, u.bytes);
      for (unsigned i = 0; i < grid.x; ++i) __atomic_store_n(u.flags + i, u.seq, __ATOMIC_RELEASE);
    });
    return hipSuccess;
  }
  CHECK(grid.x == 1 && block.x == 1);
  uint32_t* word = *(uint32_t**)args[0];
  const uint32_t value = *(uint32_t*)args[1];
  push(s, [word, value]() { __atomic_store_n(word, value, __ATOMIC_RELEASE); });
  return hipSuccess;
}
hipError_t hipGetLastError() { return fail_kernel && kernels == fail_kernel ? hipErrorInvalidConfiguration : hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = handle(9);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
  std::lock_guard<std::mutex> lock(mu);
  *status = stream(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) {
  std::lock_guard<std::mutex> lock(mu);
  Stream* st = stream(s);
  if (st->failed != hipSuccess) return st->failed;
  return st->todo.empty() && !st->busy ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new Event;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Event* ev = (Event*)e;
  uint64_t n;
  {
    std::lock_guard<std::mutex> lock(mu);
    n = ++ev->recorded;
  }
  push(s, [ev, n]() {
    std::lock_guard<std::mutex> lock(mu);
    ev->done = std::max(ev->done, n);
    changed.notify_all();
  });
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Event* ev = (Event*)e;
  uint64_t n;
  {
    std::lock_guard<std::mutex> lock(mu);
    n = ev->recorded;
  }
  push(s, [ev, n]() {
    std::unique_lock<std::mutex> lock(mu);
    changed.wait(lock, [&]() { return ev->done >= n; });
  });
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Event* ev = (Event*)e;
  std::unique_lock<std::mutex> lock(mu);
  const uint64_t n = ev->recorded;
  changed.wait(lock, [&]() { return ev->done >= n; });
  return hipSuccess;
}
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> checks = {
      {"bound", bound}, {"lower_limit", lower_limit}, {"taking_turns", taking_turns}, {"yield_between", yield_between},
      {"late_start", late_start}, {"failed_stream", failed_stream}, {"long_waits", long_waits},
      {"recorded", recorded}, {"failed_launch", failed_launch}, {"failed_copy", failed_copy},
      {"overlap_rule", overlap_rule}};
  if (argc != 2 || !checks.count(argv[1])) return 2;
  checks.at(argv[1])();
  std::printf("%s holds\n", argv[1]);
  std::fflush(stdout);
  std::_Exit(0);   // the streams' threads are still there
}
