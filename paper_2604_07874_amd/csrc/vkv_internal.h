// Internal declarations shared by the translation units of libvalvekv.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>

#include <atomic>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <functional>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "valvekv.h"

namespace vkv {

void set_error(const char* fmt, ...);
int  hip_fail(hipError_t e, const char* what);

#define VKV_HIP(call)                                         \
  do {                                                        \
    hipError_t e_ = (call);                                   \
    if (e_ != hipSuccess) return vkv::hip_fail(e_, #call);    \
  } while (0)

constexpr int kMaxInflight = 8;
constexpr int kGroupTokens = 32;   // tokens one wave handles per loop iteration (two blocks)
constexpr int kMergeLdsBytes = 16 * 1024;   // LDS the last chunk may use for per-chunk (max, sum)
// a layer of at least this many slices merges its split sequences in one launch of its own after the last
// slice (kv_attn_run_layer) instead of inside the slices
constexpr int kDeferMergeMinSlices = 4;
// A decode layer goes over two streams (kv_sched_set_overlap 1) if it is long, in several slices, and they are not short.
// The second stream fills the end of each launch.  It costs a layer a fork and a join by events, 40-50 us and more where
// the layer is the only one of its step, and short slices suffer from the 25 us after which an event is seen.  Measured,
// one stream against two, us a layer, ragged contexts, eight layers a step: 4.5 GB (8 kv heads) in 3 slices 726 : 729,
// 5 728 : 703, 6 741 : 696, 9 807 : 700, 13 820 : 699; 2.2 GB (1 kv head) in 5 399 : 390, 6 419 : 385, 9 441 : 396, 13
// 453 : 442, 18 of 122 MB 452 : 472; 4.5 GB (32 kv heads of 64) in 5 731 : 755, 6 721 : 723, 9 744 : 729, 18 791 : 732;
// 1.1 GB (8 kv heads) in 6 208 : 214, 7 235 : 229, 9 of 118 MB 237 : 245, 13 of 81 MB 230 : 271.  One layer a step: 4.5 GB
// (8 kv heads) in 5 732 : 782, 6 743 : 745, 7 710 : 780, 9 809 : 773, 13 822 : 764; 2.2 GB in 5 404 : 470, 9 445 : 470.
// So what a model of many layers gains from five slices on, a step of one layer loses up to about eight: the line is six.
constexpr int kDecodeOverlapMinSlices = 6;
constexpr uint64_t kDecodeOverlapMinBytes = 2000000000ull, kDecodeOverlapMinSliceBytes = 120ull << 20;
inline bool decode_overlaps(int overlap, int32_t n_slices, uint64_t kv_bytes) {
  return overlap == 2 || (n_slices >= kDecodeOverlapMinSlices && kv_bytes >= kDecodeOverlapMinBytes &&
                          kv_bytes / (uint64_t)n_slices >= kDecodeOverlapMinSliceBytes);
}
constexpr int kMaxChunkTokens = 2048;   // an item's block ids fit two registers per lane

struct WorkItem {   // matches int4 on the device
  int32_t seq, kv_head, first_block, n_tokens;
};

// What one workgroup of a prefill slice has to do, all of it in one record so that the chain of loads before its
// first K rows is short.
struct PrefillItem {
  int32_t seq, row0, pos0, n_pos;          // the tile: sequence, first q row, first position, positions
  int32_t kv_head, first_block, n_tokens;
  int32_t partial;                         // where the partial result goes; -1: the item is all its tile can see
};

// Byte offsets of the pieces of the attention workspace.
struct WorkspaceLayout {
  uint64_t header = 0;       // 256 bytes; word 0 = bad-table-entry flag, words 16 .. 31 = Report::ended of the launches in flight
  uint64_t work = 0;         // WorkItem[n_items], in launch order (a permutation inside each slice)
  uint64_t seq_base = 0;     // int32[num_seqs + 1]: first item of each sequence
  uint64_t done = 0;         // int32[num_seqs][kv_heads]: chunks finished in the current layer
  uint64_t part_ml = 0;      // float[n_items][G][2]: running max (log2 units), sum of exponentials
  uint64_t part_acc = 0;     // float[n_items][G][D]: exp-weighted sum of V rows
  uint64_t total = 0;
  uint64_t upload_bytes = 0; // header + work + seq_base + done are written by kv_attn_bind
};

inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

inline WorkspaceLayout workspace_layout(int64_t n_items, int64_t num_seqs, int Hkv, int G, int D) {
  WorkspaceLayout w;
  w.header = 0;
  w.work = 256;
  w.seq_base = w.work + (uint64_t)n_items * sizeof(WorkItem);
  w.done = w.seq_base + (uint64_t)(num_seqs + 1) * 4;
  w.upload_bytes = w.done + (uint64_t)num_seqs * Hkv * 4;
  w.part_ml = align_up(w.upload_bytes, 256);
  w.part_acc = align_up(w.part_ml + (uint64_t)n_items * G * 2 * 4, 256);
  w.total = align_up(w.part_acc + (uint64_t)n_items * G * D * 4, 256);
  return w;
}

// What a launch reports to the scheduler (all NULL: nothing).
struct Report {
  uint32_t* started;    // pinned host memory: `seq`, stored when the launch starts
  uint32_t* finished;   // pinned host memory: `seq`, stored when the launch ends
  uint32_t* ended;      // device: workgroups of this launch that have come to their end, 0 between launches
  uint32_t seq;
};
// The first workgroup reports the start.
__device__ __forceinline__ void report_start(const Report& r) {
  if (r.started && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(r.started, r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// The end is reported by whichever workgroup comes to its end last.  A workgroup takes its ticket when it has only
// its results left to write (report_ticket) and looks at it behind the stores (report_end), so that the ticket's
// round trip of a microsecond does not hold its place on the compute unit.
__device__ __forceinline__ uint32_t report_ticket(const Report& r) {
  return r.finished && threadIdx.x == 0 ? __hip_atomic_fetch_add(r.ended, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
__device__ __forceinline__ void report_end(const Report& r, uint32_t ticket) {
  if (r.finished && threadIdx.x == 0 && ticket == gridDim.x - 1) {
    __hip_atomic_store(r.ended, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(r.finished, r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// A launch that may not have finished yet, and how its end is seen.
struct Launch {
  enum How : int32_t {
    kNone,
    kStart,   // it reports its start: the next launch that does has started behind it, or marker `mark` has run
    kEnd,     // it reports its end
    kEvent    // an event is recorded behind it
  } how = kNone;
  uint32_t number = 0;   // among the launches that report the same thing
  uint32_t mark = 0;     // number of the marker kernel behind it, 0 = none
  hipStream_t on = nullptr;
};

// Pinned host memory that the device is given a copy of.  A small kernel reads it over the link and writes the
// device copy, and each of its workgroups reports in pinned memory when it has read its share: a copy command with an
// event behind it, to know when the buffer may be written again, kept the stream's next kernel waiting for 15-20 us.
// Recorded into a graph an upload is a copy command, which reads the buffer at every replay.
struct Staging {
  static constexpr int kMaxFlags = 128;      // workgroups of an upload
  char* host = nullptr;                     // data
  char* dev = nullptr;                      // its device address
  size_t cap = 0;
  volatile uint32_t* flags = nullptr;       // kMaxFlags words behind the data: number of the upload each workgroup has read
  uint32_t* flags_dev = nullptr;
  uint32_t seq = 0;
  int n_flags = 0;                          // workgroups of the upload in flight, 0 = none
  hipStream_t on = nullptr;                 // the stream it went to
};
int stage_wait(Staging& s);                              // the buffer may be written again
// waits, and makes room: `cap` bytes (at least `bytes`) and the flags, `behind` more bytes after them; a block that is
// outgrown goes to *old (NULL: it is freed)
int stage_reserve(Staging& s, size_t bytes, size_t cap, size_t behind = 0, char** old = nullptr);
int stage_upload(Staging& s, void* dst, size_t bytes, hipStream_t st);
// What the workgroups of an upload do, for a kernel that uploads beside other work: its `grid` workgroups each call
// upload_share once.  stage_begin_upload says how many that are and counts the upload as in flight, so the launch must
// follow.  Not for streams that are being captured.
struct UploadShare {
  const char* src;
  char* dst;
  uint64_t bytes;
  uint32_t* flags;
  uint32_t seq;
};
UploadShare stage_begin_upload(Staging& s, void* dst, size_t bytes, hipStream_t on, int* workgroups);
// Bound by the link's latency (one trip for the sizes of plans and remaps); 4 KiB per workgroup and trip.
__device__ __forceinline__ void upload_share(const UploadShare& u, uint32_t block, uint32_t grid) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  if ((uintptr_t)u.dst % 16 == 0) {
    const uint64_t whole = u.bytes / 16 * 16;
    for (uint64_t at = (uint64_t)block * 4096 + threadIdx.x * 16; at < whole; at += (uint64_t)grid * 4096)
      *reinterpret_cast<u32x4*>(u.dst + at) = *reinterpret_cast<const u32x4*>(u.src + at);
    if (block == 0 && whole + threadIdx.x * 4 < u.bytes)   // sizes are multiples of four bytes
      *reinterpret_cast<uint32_t*>(u.dst + whole + threadIdx.x * 4) = *reinterpret_cast<const uint32_t*>(u.src + whole + threadIdx.x * 4);
  } else {
    for (uint64_t at = ((uint64_t)block * 256 + threadIdx.x) * 4; at < u.bytes; at += (uint64_t)grid * 1024)
      *reinterpret_cast<uint32_t*>(u.dst + at) = *reinterpret_cast<const uint32_t*>(u.src + at);
  }
  __syncthreads();   // everything this workgroup was to read it has read (it has been stored)
  if (threadIdx.x == 0) __hip_atomic_store(u.flags + block, u.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
void stage_free(Staging& s);
bool stream_capturing(hipStream_t st);

}  // namespace vkv

struct vkv_arena;

struct vkv_pool {
  vkv_pool_config cfg{};
  const vkv_arena* arena = nullptr;   // handle-backed memory under the pool, if the caller attached one
  int G = 1;
  uint64_t block_elems = 0;   // bf16 elements per block
  uint64_t block_bytes = 0;

  // occupancy
  std::vector<uint8_t> live;
  // handed-over ranges [first, second).  `clean` = every device block table the library was shown has
  // been rewritten and every slice that could hold an old entry has finished: only then may the
  // range's memory be unmapped.
  struct Range {
    int32_t first, second;
    bool clean;
    Range(int32_t a, int32_t b, bool c = true) : first(a), second(b), clean(c) {}
  };
  std::vector<Range> released;
  std::vector<uint8_t> handed;   // per block: 1 inside a handed-over range (kept in step with `released`)
  int64_t n_live = 0;
  void hand_over(int32_t lo, int32_t hi, bool clean) {
    released.emplace_back(lo, hi, clean);
    std::fill(handed.begin() + lo, handed.begin() + hi, (uint8_t)1);
  }

  // attention plan (host)
  bool has_plan = false;
  uint64_t plan_gen = 0;
  int32_t num_seqs = 0;
  int32_t chunk_tokens = 0;
  int32_t max_ctx_blocks = 0;                  // widest sequence in blocks
  uint64_t kv_bytes = 0;                       // K and V of one layer
  std::vector<vkv::WorkItem> work;
  std::vector<int32_t> slice_start;
  std::vector<int32_t> seq_base;
  std::vector<int32_t> order;            // launch order of the items (a permutation inside each slice)
  vkv::WorkspaceLayout ws{};

  // binding of the plan to a device workspace
  void* bound_ws = nullptr;
  uint64_t bound_gen = 0;

  // prefill plan (host) and its binding; see prefill.hip
  struct PrefillPlan {
    bool has_plan = false;
    uint64_t gen = 0, bound_gen = 0;
    void* bound_ws = nullptr;
    int32_t num_seqs = 0, total_q = 0, max_ctx_blocks = 0, gp_shift = 0, tile_positions = 0;
    std::vector<vkv::WorkItem> work;       // .seq holds the tile id
    std::vector<int32_t> slice_start;
    std::vector<int32_t> tiles;            // [n_tiles][4] = (sequence, first q row, first position, positions)
    std::vector<int32_t> tile_base;        // first item of each tile (+1 sentinel)
    std::vector<vkv::PrefillItem> items;   // the same items as the kernel reads them, in launch order
    std::vector<int32_t> merge_tiles;      // tiles with more than one chunk, rising
    std::vector<int32_t> merge_start;      // first entry of merge_tiles of each merge step (+1 sentinel)
    uint64_t off_items = 0, off_tiles = 0, off_tile_base = 0, off_merge_tiles = 0, off_ml = 0, off_acc = 0, upload_bytes = 0,
             total = 0;
  } pf;

  // pinned staging (allocated on first device use)
  vkv::Staging stage;          // plans (decode thread)
  vkv::Staging remap;          // remaps (memory thread)
  int32_t* remap_stage = nullptr;   // = remap.host
  hipEvent_t grace_ev = nullptr;

  // slice scheduler
  // ring of the launches that may still be running, oldest first; it persists across calls
  vkv::Launch inflight[vkv::kMaxInflight];
  hipEvent_t inflight_ev[vkv::kMaxInflight] = {};   // behind the launch in the same place, where it is one for which events are used
  int inflight_head = 0, inflight_count = 0;
  // second stream for overlapping consecutive slices of one layer (created on first use)
  int overlap = 0;               // as given to kv_sched_set_overlap: 0, 1 or 2
  hipStream_t aux_stream = nullptr;
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  std::atomic<int> yield_flag{0};
  // Progress words in pinned host memory that launches report to, so that the scheduler can bound
  // its lead over the GPU without an event between every two launches (an event record keeps the
  // next kernel from starting for several microseconds): word 1 = number of the newest marker that has run,
  // word 16 + n % 16 = number n of a launch that has ended (two streams: launches end in any order),
  // word 32 + n % 32 = number n of a launch that has started.
  volatile uint32_t* progress_host = nullptr;
  void* progress_block = nullptr;   // the allocation that holds them, freed with the pool
  uint32_t* progress_dev = nullptr;
  uint32_t start_seq = 0;        // launches numbered so far that report their start
  uint32_t end_seq = 0;          // launches numbered so far that report their end
  uint32_t mark_seq = 0;         // markers numbered so far
  vkv::Launch next;              // what the next launch reports, kNone between the scheduler's launches
  bool launched = false;         // set by whatever the scheduler calls to enqueue a kernel

  // per-launch timing (kv_profile_enable)
  std::vector<hipEvent_t> prof_ev;      // 2 per record: start, end
  std::vector<std::pair<int32_t, int32_t>> prof_tag;   // (kind, index)
  int32_t prof_cap = 0;
  int32_t prof_stride = 1, prof_tick = 0;   // only every prof_stride-th launch is bracketed
  std::mutex prof_mu;                  // the decode thread and the reclaim thread may both record

  bool broken = false;   // a HIP call failed mid-operation
};

namespace vkv {

bool in_released(const vkv_pool* p, int32_t b);
int  ensure_remap_stage(vkv_pool* p);

// Brackets one kernel launch with timing events while recording is on.
struct ProfScope {
  vkv_pool* p;
  hipStream_t st;
  int slot = -1;
  ProfScope(vkv_pool* pool, int32_t kind, int32_t index, hipStream_t stream) : p(pool), st(stream) {
    if (p->prof_cap > 0) {
      std::lock_guard<std::mutex> g(p->prof_mu);
      // sampling thins out the many slice launches; the few other launches are always bracketed
      const bool many = kind == VKV_PROF_SLICE || kind == VKV_PROF_PREFILL;
      if ((!many || p->prof_tick++ % p->prof_stride == 0) && (int32_t)p->prof_tag.size() < p->prof_cap) {
        slot = (int)p->prof_tag.size();
        p->prof_tag.emplace_back(kind, index);
      }
    }
    if (slot >= 0) (void)hipEventRecord(p->prof_ev[2 * slot], st);
  }
  ~ProfScope() {
    if (slot >= 0) (void)hipEventRecord(p->prof_ev[2 * slot + 1], st);
  }
};

// Timing of a single kernel launch while recording is on: the launch itself carries the two events
// (they take the dispatch's own start and end times), so nothing is enqueued between this kernel and
// its neighbours and the figure is the kernel's duration alone.
struct ProfKernel {
  vkv_pool* p;
  int slot = -1;
  ProfKernel(vkv_pool* pool, int32_t kind, int32_t index) : p(pool) {
    if (p->prof_cap > 0) {
      std::lock_guard<std::mutex> g(p->prof_mu);
      if (p->prof_tick++ % p->prof_stride == 0 && (int32_t)p->prof_tag.size() < p->prof_cap) {
        slot = (int)p->prof_tag.size();
        p->prof_tag.emplace_back(kind, index);
      }
    }
  }
  template <typename K, typename... Args>
  void launch(K kernel, dim3 grid, dim3 block, hipStream_t st, Args... args) {
    if (slot >= 0)
      hipExtLaunchKernelGGL(kernel, grid, block, 0, st, p->prof_ev[2 * slot], p->prof_ev[2 * slot + 1], 0, args...);
    else
      hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
  }
};

// Device address of the library's static scratch array on the current device (attn.hip);
// the first call on a device looks it up.
int static_scratch_for_current_device(void** out);

// Slice scheduler shared by decode and prefill (attn.hip).
// true if handles [first, last) of the arena all have physical memory behind them
bool arena_range_mapped(const vkv_arena* a, int32_t first, int32_t last);
int run_slices(vkv_pool* p, int32_t* cursor, int32_t n_slices, int32_t max_inflight, hipStream_t hs, const char* who,
               const std::function<int(int32_t, hipStream_t)>& launch, int32_t n_tail,
               const std::function<int(int32_t)>& tail, bool tail_launches, bool may_overlap, bool end_events,
               const std::function<int()>& after_slices = nullptr);
// the plans' staging buffer, with the progress words behind it when it is first made (one pinned allocation, not two)
int ensure_plan_stage(vkv_pool* p, size_t bytes);
// what the launch the scheduler is about to make reports; header = the workspace's first 256 bytes on the device
Report next_report(vkv_pool* p, void* header);

// Algorithm 1 on the host tables; evicted[r] != 0 for the requests that go.  See kv_select_handles.
int select_handles_impl(const vkv_pool* p, const int32_t* tables, int32_t n_rows, int32_t max_blk, const int64_t* cost,
                        int32_t k, int32_t* handles_out, std::vector<uint8_t>& evicted, int64_t* total_out, const char* who);
// Waits until work enqueued so far on `ds` (if it differs from `cs`) and on the pool's second stream
// has finished: slices launched before a table rewrite may still hold old entries.
int grace_wait(vkv_pool* p, hipStream_t cs, hipStream_t ds);
int launch_rewrite(vkv_pool* p, int32_t* tables, int64_t n, const int32_t* remap, int32_t nb, hipStream_t st);

// Host-side relocation plan; see kv_reclaim_plan.
int plan_relocation(const vkv_pool* p, int32_t lo, int32_t hi,
                    std::vector<int32_t>& src, std::vector<int32_t>& dst);

}  // namespace vkv
