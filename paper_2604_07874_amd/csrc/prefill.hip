// Preemptible causal attention of a chunk of new tokens over the paged KV pool (prefill).
//
// Long prefills are where coarse preemption costs most (paper Section 2.2: layer-level
// preemption delays of hundreds of milliseconds at 32k tokens; Section 5: bursts arriving
// during a long prefill iteration).  The same slicing as for decode bounds the time to the
// next yield point; here the work is compute-bound, so the MFMA units carry the load.
//
// Work split: the new tokens of a sequence are cut into query tiles of 128/GP positions
// (GP = group size rounded up to a power of two), so a tile has 128 (position, query head)
// columns; the tokens a tile can see (positions 0 .. its last position) are cut into chunks
// of chunk_tokens; one work item = (tile, kv head, chunk) = one workgroup.  Items of a tile
// are merged by a separate small kernel after the layer's last slice (prefill launches last
// milliseconds, so one more launch per layer is immaterial and needs no in-kernel
// cross-workgroup ordering).
//
// Kernel shape (wave64, gfx950): 4 waves; wave w owns columns [32w, 32w+32), one 32-column MFMA tile, and sees
// every token of the item.  Per 32-token group the workgroup brings K and V into LDS once for all four waves, with
// the 16-byte global->LDS loads of gfx950: wave w asks for rows 4w .. 4w+3 of both blocks of the group, K and V,
// four loads in all, which need no registers and are requested three steps ahead of their use.  The rows lie in LDS
// as in the pool (256 bytes per token), their 16-byte chunks permuted so that the operand reads meet no bank
// conflict.  A wave reads the 8 K operands (16-byte reads) and the V operands (16 transposing 8-byte reads, which
// hand each lane its own head dimension of four tokens) it needs for its 16 MFMAs (v_mfma_f32_32x32x16_bf16, 32
// cycles each) and runs online softmax per column with the causal mask applied by select.
//
// What bounds it, and why the step looks as it does: a wave issues at most one instruction every four cycles, so
// beside 18 matrix instructions (544 cycles) there is room for about 120 others before the issue and not the
// matrix unit is the limit.  Earlier the step had 263 instructions in phases that a wave went through one after
// the other (K reads, q.K, V reads, softmax, p.V): 2380 cycles with two waves per SIMD.  Now the softmax of group
// g stands between the q.K products of group g+1, operands are read half a step before they are needed, block
// addresses wait in LDS (two readlanes each instead of loads, selects and 64-bit adds), four steps per trip turn
// buffer offsets into immediates, and the step has about 140 instructions: 1350 cycles for two waves.  At that rate
// the chip's clock falls to 1.8-1.9 GHz (a loop of nothing but these matrix instructions on random data runs at 1.6).
// Counters over one layer of 64 sequences in 26 launches of 149 us: 1.93 GHz, matrix units busy 48 % of the cycles, 1.49
// of 2 waves resident per SIMD (items start and end, launches run out), no bank conflict.
// 32 prompts, the newest 2048 tokens of each: 2307 -> 1942 us; 4096 new tokens on 28k: 3007 -> 2182 us (945 TFLOP/s);
// one prompt of 1901 tokens: 68.1 -> 48.9 us.
#include "vkv_internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

namespace vkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileColumns = 128;   // (position, query head) columns of one query tile
constexpr int kMaxPrefillChunkTokens = 16384;   // bounds an item's run time, not a kernel limit
constexpr int kGroupsAhead = 5;     // K rows are requested this many groups ahead of the p.V products
// block addresses an item keeps in LDS: two per group, the groups requested past its end, whole windows of 64
constexpr int kMaxItemEntries = (kMaxPrefillChunkTokens / 16 + 2 * (kGroupsAhead + 1) + 63) / 64 * 64;
constexpr float kSlack = 8.0f;      // how far (log2 units) a score may exceed the running reference
constexpr float kNoMax = -1.0e30f;  // reference of a column that has seen no token yet (finite on purpose)

struct PrefillParams {
  const uint16_t* pool;       // pool base + layer offset (elements)
  const PrefillItem* items;   // in launch order: within a slice by falling token count
  const int32_t* tiles;       // [n_tiles][4] = (sequence, first q row, first position, positions)
  const int32_t* tile_base;   // [n_tiles + 1]
  const int32_t* merge_tiles; // tiles that were split into several chunks
  const uint16_t* q;          // [total_q][Hq][D]
  const int32_t* table;
  float* part_acc;            // [n_items][128][D]
  float* part_ml;             // [n_items][128][2]
  float* out;                 // [total_q][Hq][D]
  uint32_t* err;
  uint64_t block_elems;
  uint32_t v_off;
  int32_t item_first, merge_first, max_blk, Hq, Hkv, G, gp_shift, NB;
  float scale_log2;
  Report report;              // to the scheduler
};

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// LDS reads the compiler does not see as such.  It orders every LDS read it knows of behind all pending
// global->LDS loads (it cannot tell the staging buffers apart), which would wait for the groups that were
// requested ahead; these reads are ordered by hand instead: the loads of a buffer are waited for
// (s_waitcnt vmcnt) before the barrier that lets anyone read it.
template <int OFF>
__device__ __forceinline__ void lds_read_b128(u32x4& dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// transposing 8-byte read: within 16 lanes, lane i gets element i & 3 of the four 16-bit elements that lane
// 4 j + (i >> 2) points at, for j = 0..3
template <int OFF>
__device__ __forceinline__ void lds_read_tr16_b64(u32x2& dst, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// waits until at most LEFT of this wave's LDS reads are pending; they return in order, so the ones named have arrived
template <int LEFT>
__device__ __forceinline__ void lds_wait(u32x4 (&a)[8]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
               : "n"(LEFT) : "memory");
}
template <int LEFT>
__device__ __forceinline__ void lds_wait(u32x2 (&a)[8]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7])
               : "n"(LEFT) : "memory");
}
// Maximum of three as one instruction.  A NaN is passed on (fmaxf would ignore it, at the price of an
// instruction per operand that quiets it first); a column with a NaN score is NaN whatever its reference.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

template <int D>
__global__ __launch_bounds__(256, 2) void paged_prefill_attn_slice_kernel(const PrefillParams p) {
  static_assert(D == 128, "head_dim 128 only");
  constexpr int DT = D / 32;            // 32-row MFMA tiles of the output
  constexpr int KS = D / 16;            // MFMA k-steps of the score tile
  constexpr int ROW = D * 2;            // bytes of one token row of one head
  constexpr float NEG_INF = -INFINITY;

  // Four staging buffers of a 32-token group each, K rows and V rows as they lie in the pool (256 bytes
  // per token), written by the 16-byte global->LDS loads; no padding is possible there (a load places its
  // 64 lanes back to back), so the 16-byte chunks of a row are permuted instead, by the choice of the
  // global address each lane asks for: chunk c of K row r sits at position c ^ (r & 15), chunk c of V row r
  // at c ^ 4 (r & 3) (the LDS has 64 banks: 16 lanes of a 16-byte read, 32 lanes of an 8-byte read go together).
  constexpr int kBufs = 4;
  __shared__ __attribute__((aligned(16))) unsigned char k_lds4[kBufs][32 * ROW];
  __shared__ __attribute__((aligned(16))) unsigned char v_lds4[kBufs][32 * ROW];
  __shared__ uint64_t blk_addr[kMaxItemEntries];   // address of each of the item's blocks (this head's K rows)

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c32 = lane & 31, half = lane >> 5;

  report_start(p.report);

  // One record holds all an item needs (through order, item and tile lists the queries and the table row were two
  // loads later: 5.6 instead of 4.5 us from the start to the first products, 32 prompts 1942 -> 1893 us).
  const PrefillItem it = p.items[p.item_first + blockIdx.x];   // longest items of the slice start first
  const int row0 = it.row0, pos0 = it.pos0, n_pos = it.n_pos;
  const int ntok = it.n_tokens;
  const int tok_base = it.first_block * 16;          // position of the item's first token
  const int ngroups = (ntok + kGroupTokens - 1) / kGroupTokens;
  const int G = p.G, gp_mask = (1 << p.gp_shift) - 1;

  // this lane's column: position within the tile and query head
  const int col = wave * 32 + c32;
  const int cpos = col >> p.gp_shift, cg = col & gp_mask;
  const bool cvalid = cg < G && cpos < n_pos;
  bf16x8 qb[KS];   // B operand of the scores: column c32, k index 8 half + j <-> d = 16 ks + 8 half + j
  {
    const uint16_t* qrow = p.q + ((size_t)(row0 + (cvalid ? cpos : 0)) * p.Hq + (size_t)it.kv_head * G + (cvalid ? cg : 0)) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (cvalid) v = *reinterpret_cast<const u32x4*>(qrow + ks * 16 + half * 8);
      qb[ks] = __builtin_bit_cast(bf16x8, v);
    }
  }

  // The item's block ids become addresses in LDS once.  An entry outside the pool (a corrupted table, reported
  // here) and the entries past the item's end name the item's first block, whose rows exist: what they bring is
  // masked, cleared after it is read, or never used.
  const int32_t* trow = p.table + (size_t)it.seq * p.max_blk + it.first_block;
  const uint64_t kplane = (uint64_t)(uintptr_t)(p.pool + (size_t)it.kv_head * (16 * D));
  const int nblk_item = (ntok + 15) >> 4;
  const int32_t blk0 = trow[0];
  if (blk0 < 0 || blk0 >= p.NB) {   // nothing to fall back on: the whole workgroup leaves, before any barrier
    if (threadIdx.x == 0) atomicOr(p.err, 1u);
    report_end(p.report, report_ticket(p.report));
    return;
  }
  const int n_entries = (2 * (ngroups + kGroupsAhead + 1) + 63) & ~63;
  for (int e = threadIdx.x; e < n_entries; e += 256) {
    int32_t blk = e < nblk_item ? trow[e] : blk0;
    if (blk < 0 || blk >= p.NB) {
      atomicOr(p.err, 1u);
      blk = blk0;
    }
    blk_addr[e] = kplane + (uint64_t)(uint32_t)blk * (p.block_elems * 2);
  }

  f32x16 acc[DT];
  f32x4 accl = {0.f, 0.f, 0.f, 0.f};
  float m_run = kNoMax;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;

  // Row sums come from the matrix unit too, one 16x16x32 product per 16 tokens with the weights as they
  // stand in the operand of the 32x32x16 ones: there lane l holds 8 weights of column l & 31, so the 16-wide
  // instruction sees k-groups 0 and 2 of columns 0..15 and k-groups 1 and 3 of columns 16..31.  Row m of
  // its A operand is one on the k-groups of parity (m >> 2) & 1, zero on the others: register 0 of lane l
  // (row 4 (l >> 4)) is then the sum of column l & 31.
  bf16x8 pick;
#pragma unroll
  for (int i = 0; i < 8; ++i) pick[i] = (__bf16)(((lane >> 4) & 1) == ((lane >> 2) & 1) ? 1.0f : 0.0f);

  // ---- this wave's share of a group goes from the pool straight into LDS ----
  // Rows 4 wave .. 4 wave + 3 of both blocks of the group, K and V: four loads of 64 x 16 bytes.  Lane l
  // fills position l & 15 of row 4 wave + (l >> 4), so it asks for the chunk that belongs there.
  const int lrow = 4 * wave + (lane >> 4);                            // row within a block
  const uint32_t g_off_k = (uint32_t)(lrow * ROW + (((lane & 15) ^ (lrow & 15)) * 16));        // bytes
  const uint32_t g_off_v = (uint32_t)(lrow * ROW + (((lane & 15) ^ (4 * (lrow & 3))) * 16)) + p.v_off * 2;
  // The addresses of 32 groups at a time sit in two registers, one block per lane.
  uint32_t win_lo, win_hi;
  const uint32_t win_addr = lds_addr(blk_addr) + lane * 8;
  auto window = [&](int w) {   // a read the compiler does not see, see lds_read_b128
    u32x2 a;
    asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(a) : "v"(win_addr + (uint32_t)w * 512u) : "memory");
    win_lo = a[0];
    win_hi = a[1];
  };
  struct Blocks { uint64_t b[2]; };   // a group's two blocks
  auto blocks_of = [&](int grp) {
    Blocks r;
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      const int e = (grp * 2 + sb) & 63;
      r.b[sb] = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(win_hi, e) << 32) | (uint32_t)__builtin_amdgcn_readlane(win_lo, e);
    }
    return r;
  };
  // One 16-byte global->LDS load per lane: scalar base, 32-bit lane offset, destination in m0.  The instruction
  // needs one wait state behind the write of m0 and five behind a vector instruction's write of its scalar base
  // (v_readlane in blocks_of); the compiler keeps such distances for its own loads but does not look inside
  // assembly.  So block addresses pass through one of two statements between blocks_of and their first load, both
  // volatile, which keeps them and the loads in order: the prologue's waits the five states out (settled), and a
  // step's, at its start, has a wait, a barrier and six LDS reads behind it before the first load.  m0 cannot be named as overwritten (it is a
  // reserved register); the compiler keeps nothing in it and sets it ahead of each use of its own.
  auto load_lds = [&](uint32_t dst, uint64_t base, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst), "v"(off), "s"(base) : "memory");
  };
  auto settled = [&](Blocks& b0, Blocks& b1, Blocks& b2, Blocks& b3, Blocks& b4) {
    asm volatile("s_nop 4" : "+s"(b0.b[0]), "+s"(b0.b[1]), "+s"(b1.b[0]), "+s"(b1.b[1]), "+s"(b2.b[0]), "+s"(b2.b[1]),
                             "+s"(b3.b[0]), "+s"(b3.b[1]), "+s"(b4.b[0]), "+s"(b4.b[1]));
  };
  const uint32_t k_dst = __builtin_amdgcn_readfirstlane(lds_addr(&k_lds4[0][0]) + 4 * wave * ROW);
  const uint32_t v_dst = __builtin_amdgcn_readfirstlane(lds_addr(&v_lds4[0][0]) + 4 * wave * ROW);
  // slot: byte offset of the staging buffer
  auto load_k = [&](uint32_t slot, const Blocks& o, int sb) { load_lds(k_dst + slot + sb * 16 * ROW, o.b[sb], g_off_k); };
  auto load_v = [&](uint32_t slot, const Blocks& o, int sb) { load_lds(v_dst + slot + sb * 16 * ROW, o.b[sb], g_off_v); };

  // ---- operand reads of a staged group ----
  // K: row c32 of the operand is token c32 of the group; its chunk 2 ks + half sits at (2 ks + half) ^ (c32 & 15)
  uint32_t k_addr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_addr[ks] = lds_addr(&k_lds4[0][0]) + c32 * ROW + (((ks * 2 + half) ^ (c32 & 15)) << 4);
  // V: the operand of d-tile dt and k-step s (tokens 16 s .. 16 s + 15) comes from two transposing reads.  The
  // score registers hold tokens 8 (i >> 2) + 4 half + (i & 3), so element j of the operand has to be token
  // 16 s + 8 (j >> 2) + 4 half + (j & 3): read u = j >> 2 of the 16 lanes with (l >> 4) = 2 half + e points at
  // 8-byte pieces of rows 16 s + 8 u + 4 half .. + 3, d = 32 dt + 16 e .. + 15 (lane i at row + (i >> 2),
  // d + 4 (i & 3)), and gives each lane its own d of those four rows.
  const int v_rr = (lane >> 2) & 3;
  const uint32_t v_base = lds_addr(&v_lds4[0][0]) + (4 * half + v_rr) * ROW + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  uint32_t v_addr[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) v_addr[dt] = v_base + ((dt ^ v_rr) << 6);

  constexpr uint32_t SLOT = 32 * ROW;   // bytes of a staging buffer
  u32x4 ka[KS];
  u32x2 vh[2][8];   // [k-step s][2 dt + u]
  auto slot_of = [&](int grp) { return (uint32_t)(grp & (kBufs - 1)) * SLOT; };
  // Operand reads of buffer J, or, with J < 0, of the buffer at byte offset `slot`.
  auto read_k = [&](auto buf, uint32_t slot, int ks) {
    constexpr int J = decltype(buf)::value;
    if constexpr (J >= 0) lds_read_b128<J * (int)SLOT>(ka[ks], k_addr[ks]);
    else lds_read_b128<0>(ka[ks], k_addr[ks] + slot);
  };
  auto read_v = [&](auto buf, uint32_t slot, int s, int dt) {
    constexpr int J = decltype(buf)::value;
    const uint32_t a = J >= 0 ? v_addr[dt] : v_addr[dt] + slot;
    constexpr int O = J >= 0 ? J * (int)SLOT : 0;
    if (s == 0) {
      lds_read_tr16_b64<O>(vh[0][2 * dt], a);
      lds_read_tr16_b64<O + 8 * ROW>(vh[0][2 * dt + 1], a);
    } else {
      lds_read_tr16_b64<O + 16 * ROW>(vh[1][2 * dt], a);
      lds_read_tr16_b64<O + 24 * ROW>(vh[1][2 * dt + 1], a);
    }
  };
  // ---- mask (groups on the causal diagonal and a ragged last group only) and running reference ----
  const int limit = min(pos0 + cpos - tok_base, ntok - 1);   // last token index (within the item) this column sees
  auto mask = [&](int grp, f32x16& sc) {
    const int t0 = grp * kGroupTokens + 4 * half;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (t0 + 8 * (i >> 2) + (i & 3) > limit) sc[i] = NEG_INF;   // also drops NaN from rows past the end
  };
  auto max16 = [&](const f32x16& sc) {
    const float m0 = max3(sc[0], sc[1], sc[2]), m1 = max3(sc[3], sc[4], sc[5]), m2 = max3(sc[6], sc[7], sc[8]),
                m3 = max3(sc[9], sc[10], sc[11]), m4 = max3(sc[12], sc[13], sc[14]);
    return max3(max3(m0, m1, m2), max3(m3, m4, sc[15]), sc[15]);
  };
  auto reference = [&](float mx) {   // mx: this lane's largest score of the group
    if (__builtin_amdgcn_ballot_w64(fmaf(mx, p.scale_log2, -kSlack) > m_run) != 0ull) {
      const float mc = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mc * p.scale_log2);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      accl *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] *= alpha;
    }
  };
  // number of leading groups that are complete and visible to every column of this wave
  const int wave_limit = pos0 + ((wave * 32) >> p.gp_shift) - tok_base;
  const int n_interior = min(ntok, wave_limit + 1) >> 5;

  // One step of the software pipeline: the weights and p.V products of group grp (scores in `cur`) and the
  // scores of group grp + 1 (into `nxt`, K operands in ka since the step before), V operands of grp and K
  // operands of grp + 2 out of LDS, K rows of grp + 5 and V rows of grp + 3 into LDS (past the item's end: rows
  // of its first block, so that every step requests the same four loads and waits the same way).
  // A wave issues at most one instruction every four cycles and a matrix instruction holds the matrix unit for
  // 32, so a step of 18 of them (544 cycles) has room for about 120 other instructions; vector and LDS
  // instructions are placed between them by hand: exponentials and V reads in the first half, K reads and the
  // maximum in the second, the loads evenly over both.
  // buf = grp & 3 where it is known at compile time (then group grp + 1 exists and needs no mask), else -1.
  Blocks ahead1, ahead2;   // blocks of groups grp + 3 and grp + 4
  auto step = [&](int grp, f32x16& cur, f32x16& nxt, auto buf) {
    constexpr int J = decltype(buf)::value;
    constexpr bool kFast = J >= 0;
    const std::integral_constant<int, (J < 0 ? -1 : J & 3)> vbuf;
    const std::integral_constant<int, (J < 0 ? -1 : (J + 2) & 3)> kbuf;
    const uint32_t v_slot = slot_of(grp), k_slot = slot_of(grp + 2);
    const uint32_t v_to = kFast ? ((J + 3) & 3) * SLOT : slot_of(grp + 3), k_to = kFast ? ((J + 5) & 3) * SLOT : slot_of(grp + 5);
    if ((!kFast || J == 3) && ((grp + 5) & 31) == 0) window((grp + 5) >> 5);
    Blocks next = blocks_of(grp + 5);
    asm volatile("" : "+s"(next.b[0]), "+s"(next.b[1]));   // read before what follows, see load_lds
    // K rows of group grp + 2 and V rows of group grp have landed: this wave's loads here (those of the last
    // two steps may be pending), everybody's behind the barrier
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    // the barrier alone, without the fence of __syncthreads: that fence would wait for the loads ahead as
    // well; this wave's LDS reads of the previous step have returned, which is all the others need to know
    // before they overwrite those buffers
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const bool more = kFast || grp + 1 < ngroups;
    bf16x8 pb[2];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (more) {
        if (ks == 0) {
          f32x16 zero;
#pragma unroll
          for (int i = 0; i < 16; ++i) zero[i] = 0.f;
          nxt = zero;
        }
        nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[ks]), qb[ks], nxt, 0, 0, 0);
      }
      read_v(vbuf, v_slot, ks >> 2, ks & 3);
      if (ks == 2) load_k(k_to, next, 0);
      if (ks == 6) load_k(k_to, next, 1);
#pragma unroll
      for (int i = 2 * ks; i < 2 * ks + 2; ++i)
        pb[i >> 3][i & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(cur[i], p.scale_log2, -m_run));
      __builtin_amdgcn_sched_barrier(0);
    }
    auto pv = [&](int s, int dt) {
      const u32x4 va = {vh[s][2 * dt][0], vh[s][2 * dt][1], vh[s][2 * dt + 1][0], vh[s][2 * dt + 1][1]};
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), pb[s], acc[dt], 0, 0, 0);
    };
    auto clear_tail = [&](int s) {
      // the item's ragged last group: rows past the end hold whatever the pool holds there (maybe NaN);
      // their weights are zero, their V must be too
      if (kFast || grp * kGroupTokens + kGroupTokens <= ntok) return;
#pragma unroll
      for (int v = 0; v < 8; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (grp * kGroupTokens + 16 * s + 8 * (v & 1) + 4 * half + e >= ntok)
            vh[s][v][e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
    };
    lds_wait<8>(vh[0]);
    clear_tail(0);
    __builtin_amdgcn_sched_barrier(0);
    accl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick, pb[0], accl, 0, 0, 0);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      pv(0, dt);
      read_k(kbuf, k_slot, 2 * dt);
      read_k(kbuf, k_slot, 2 * dt + 1);
      if (dt == 2) load_v(v_to, ahead1, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_wait<8>(vh[1]);
    clear_tail(1);
    float mx = NEG_INF;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      pv(1, dt);
      if (dt == 0 && more) {
        if (!kFast && grp + 1 >= n_interior) mask(grp + 1, nxt);
        mx = max16(nxt);
      }
      if (dt == 2) load_v(v_to, ahead1, 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    accl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick, pb[1], accl, 0, 0, 0);
    ahead1 = ahead2;
    ahead2 = next;
    lds_wait<0>(ka);
    if (more) reference(mx);
  };

  // Prologue.  K rows lead V rows by two groups (four buffers each): at the barrier of step g every wave has
  // read K of group g+1 and V of group g-1, whose buffers take K of group g+5 and V of group g+3.
  constexpr std::integral_constant<int, 0> B0;
  constexpr std::integral_constant<int, 1> B1;
  constexpr std::integral_constant<int, 2> B2;
  constexpr std::integral_constant<int, 3> B3;
  constexpr std::integral_constant<int, -1> BX;
  __syncthreads();   // the addresses are in LDS
  window(0);
  {
    Blocks b0 = blocks_of(0), b1 = blocks_of(1), b2 = blocks_of(2);
    ahead1 = blocks_of(3);
    ahead2 = blocks_of(4);
    settled(b0, b1, b2, ahead1, ahead2);
    load_k(0 * SLOT, b0, 0);
    load_k(0 * SLOT, b0, 1);
    load_k(1 * SLOT, b1, 0);
    load_k(1 * SLOT, b1, 1);
    load_k(2 * SLOT, b2, 0);
    load_k(2 * SLOT, b2, 1);
    load_v(0 * SLOT, b0, 0);
    load_v(0 * SLOT, b0, 1);
    load_k(3 * SLOT, ahead1, 0);
    load_k(3 * SLOT, ahead1, 1);
    load_v(1 * SLOT, b1, 0);
    load_v(1 * SLOT, b1, 1);
    // K rows of groups 0 and 1 have landed (what was requested after them: K 2, V 0, K 3, V 1)
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) read_k(B0, 0, ks);
    lds_wait<0>(ka);
    __builtin_amdgcn_s_barrier();   // everybody has read K of group 0: its buffer takes group 4
    asm volatile("" ::: "memory");
    load_k(0 * SLOT, ahead2, 0);
    load_k(0 * SLOT, ahead2, 1);
    load_v(2 * SLOT, b2, 0);
    load_v(2 * SLOT, b2, 1);
  }
  f32x16 s0, s1;
#pragma unroll
  for (int i = 0; i < 16; ++i) s0[i] = s1[i] = 0.f;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[ks]), qb[ks], s0, 0, 0, 0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) read_k(B1, 0, ks);
  lds_wait<0>(ka);
  if (n_interior < 1) mask(0, s0);
  reference(max16(s0));
  int grp = 0;
  for (; grp + 4 < n_interior; grp += 4) {   // four buffers, two sets of score registers: four steps per trip
    step(grp, s0, s1, B0);
    step(grp + 1, s1, s0, B1);
    step(grp + 2, s0, s1, B2);
    step(grp + 3, s1, s0, B3);
  }
  for (; grp < ngroups; ++grp) {
    step(grp, s0, s1, BX);
    s0 = s1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the end too, before this LDS goes to another workgroup

  const uint32_t ticket = report_ticket(p.report);
  // ---- results: column-owned, no merge across waves; register i of d-tile dt is d = 32 dt + 8 (i >> 2) + 4 half + (i & 3) ----
  const float l = accl[0];
  const size_t item = (size_t)it.partial;
  if (it.partial < 0) {
    if (cvalid) {
      float* orow = p.out + ((size_t)(row0 + cpos) * p.Hq + (size_t)it.kv_head * G + cg) * D + 4 * half;
      const float inv = 1.0f / l;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          *reinterpret_cast<f32x4*>(orow + 32 * dt + 8 * k) =
              f32x4{acc[dt][4 * k], acc[dt][4 * k + 1], acc[dt][4 * k + 2], acc[dt][4 * k + 3]} * inv;
    }
  } else {
    float* prow = p.part_acc + (item * kTileColumns + col) * D + 4 * half;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<f32x4*>(prow + 32 * dt + 8 * k) =
            f32x4{acc[dt][4 * k], acc[dt][4 * k + 1], acc[dt][4 * k + 2], acc[dt][4 * k + 3]};
    if (half == 0) {
      p.part_ml[(item * kTileColumns + col) * 2 + 0] = m_run;
      p.part_ml[(item * kTileColumns + col) * 2 + 1] = l;
    }
  }
  report_end(p.report, ticket);
}

// Merge of the chunks of one split (tile, kv head): log-sum-exp merge in chunk order.  A workgroup
// takes a quarter of the tile's columns (kMergeCols), so that a merge step has four times the
// workgroups and a quarter of the dependent loads per thread: the kernel is nothing but memory latency.
// Pass 1, one thread per column: the maximum over the chunks, then the chunk weights 2^(m_c - M)
// into LDS (32 chunks at a time) and their weighted sum of the partial sums.
// Pass 2, one thread per (column, four output dims): the weighted partial accumulators, with the
// loads of four chunks in flight at a time.
constexpr int kMergeCols = 32;
template <int D>
__global__ __launch_bounds__(256) void prefill_merge_kernel(const PrefillParams p) {
  constexpr int kBatch = 32;
  constexpr int kParts = kTileColumns / kMergeCols;
  __shared__ float sm_w[kBatch][kMergeCols];
  __shared__ float sm_M[kMergeCols], sm_den[kMergeCols];
  report_start(p.report);
  // merge_first = first entry of the step in the list of split tiles
  const int unit = blockIdx.x / kParts, col0 = (blockIdx.x % kParts) * kMergeCols;
  const int tile = p.merge_tiles[p.merge_first + unit / p.Hkv], head = unit % p.Hkv;
  const int base = p.tile_base[tile];
  const int nch = (p.tile_base[tile + 1] - base) / p.Hkv;
  const int row0 = p.tiles[4 * tile + 1], n_pos = p.tiles[4 * tile + 3];
  const int G = p.G, gp_mask = (1 << p.gp_shift) - 1;
  auto item_col = [&](int c, int col) { return ((size_t)base + (size_t)c * p.Hkv + head) * kTileColumns + col; };
  const int tid = threadIdx.x;
  if (tid < kMergeCols) {
    float M = -INFINITY;
    for (int c = 0; c < nch; ++c) M = fmaxf(M, p.part_ml[item_col(c, col0 + tid) * 2]);
    sm_M[tid] = M;
    sm_den[tid] = 0.f;
  }
  constexpr int VPR = D / 4;                         // float4 per column
  constexpr int kIters = kMergeCols * VPR / 256;
  f32x4 num[kIters];
#pragma unroll
  for (int i = 0; i < kIters; ++i) num[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < nch; c0 += kBatch) {
    const int nb = min(kBatch, nch - c0);
    __syncthreads();                                 // sm_M ready / previous batch's weights consumed
    if (tid < kMergeCols) {
      const float M = sm_M[tid];
      float den = sm_den[tid];
      for (int j = 0; j < nb; ++j) {
        const size_t ic = item_col(c0 + j, col0 + tid);
        const float wt = __builtin_exp2f(p.part_ml[ic * 2] - M);   // 0 for a chunk this column cannot see
        sm_w[j][tid] = wt;
        den += wt * p.part_ml[ic * 2 + 1];
      }
      sm_den[tid] = den;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kIters; ++i) {
      const int e = i * 256 + tid, lc = e / VPR, v = e - lc * VPR;
      int j = 0;
      for (; j + 4 <= nb; j += 4) {
        f32x4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          x[u] = *reinterpret_cast<const f32x4*>(p.part_acc + item_col(c0 + j + u, col0 + lc) * D + v * 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) num[i] += sm_w[j + u][lc] * x[u];
      }
      for (; j < nb; ++j)
        num[i] += sm_w[j][lc] * *reinterpret_cast<const f32x4*>(p.part_acc + item_col(c0 + j, col0 + lc) * D + v * 4);
    }
  }
  __syncthreads();
  const uint32_t ticket = report_ticket(p.report);
#pragma unroll
  for (int i = 0; i < kIters; ++i) {
    const int e = i * 256 + tid, lc = e / VPR, v = e - lc * VPR;
    const int col = col0 + lc;
    const int cpos = col >> p.gp_shift, cg = col & gp_mask;
    if (cg >= G || cpos >= n_pos) continue;
    const float inv = 1.0f / sm_den[lc];
    *reinterpret_cast<f32x4*>(p.out + ((size_t)(row0 + cpos) * p.Hq + (size_t)head * G + cg) * D + v * 4) = num[i] * inv;
  }
  report_end(p.report, ticket);
}

// ---- host ---------------------------------------------------------------------------

static int pf_check_bound(vkv_pool* p, const void* workspace, const char* who) {
  if (!p) { set_error("%s: null pool", who); return VKV_E_INVAL; }
  if (p->broken) { set_error("%s: pool unusable after a HIP failure", who); return VKV_E_HIP; }
  if (!p->pf.has_plan) { set_error("%s: no plan; call kv_prefill_plan first", who); return VKV_E_STATE; }
  if (!workspace || workspace != p->pf.bound_ws || p->pf.bound_gen != p->pf.gen) {
    set_error("%s: workspace is not bound to the current plan; call kv_prefill_bind", who);
    return VKV_E_STATE;
  }
  return VKV_OK;
}

static int pf_check_args(vkv_pool* p, int32_t layer, const void* q, const int32_t* table, int32_t max_blk,
                         void* workspace, void* out, const char* who) {
  int st = pf_check_bound(p, workspace, who);
  if (st != VKV_OK) return st;
  if (!p->cfg.base) { set_error("%s: pool has no device memory", who); return VKV_E_INVAL; }
  if (p->cfg.head_dim != 128) { set_error("%s: prefill supports head_dim 128 only", who); return VKV_E_INVAL; }
  if (layer < 0 || layer >= p->cfg.num_layers) { set_error("%s: layer %d out of range", who, layer); return VKV_E_INVAL; }
  if (!q || !table || !out || (uintptr_t)q % 16 || (uintptr_t)out % 16) {
    set_error("%s: q, out (16-byte aligned) and block_table must be given", who);
    return VKV_E_INVAL;
  }
  if (max_blk < p->pf.max_ctx_blocks) {
    set_error("%s: block table has %d columns, the plan needs %d", who, max_blk, p->pf.max_ctx_blocks);
    return VKV_E_INVAL;
  }
  return VKV_OK;
}

static PrefillParams pf_params(vkv_pool* p, int32_t layer, const void* q, const int32_t* table, int32_t max_blk,
                               void* workspace, void* out, float scale) {
  const int D = p->cfg.head_dim;
  char* ws = (char*)workspace;
  PrefillParams a{};
  a.pool = (const uint16_t*)p->cfg.base + (uint64_t)layer * ((uint64_t)2 * p->cfg.num_kv_heads * 16 * D);
  a.items = (const PrefillItem*)(ws + p->pf.off_items);
  a.tiles = (const int32_t*)(ws + p->pf.off_tiles);
  a.tile_base = (const int32_t*)(ws + p->pf.off_tile_base);
  a.merge_tiles = (const int32_t*)(ws + p->pf.off_merge_tiles);
  a.q = (const uint16_t*)q;
  a.table = table;
  a.part_acc = (float*)(ws + p->pf.off_acc);
  a.part_ml = (float*)(ws + p->pf.off_ml);
  a.out = (float*)out;
  a.err = (uint32_t*)ws;
  a.block_elems = p->block_elems;
  a.v_off = (uint32_t)(p->cfg.num_kv_heads * 16 * D);
  a.max_blk = max_blk;
  a.Hq = p->cfg.num_q_heads;
  a.Hkv = p->cfg.num_kv_heads;
  a.G = p->G;
  a.gp_shift = p->pf.gp_shift;
  a.NB = p->cfg.num_blocks;
  a.scale_log2 = (scale != 0.f ? scale : 1.0f / std::sqrt((float)D)) * 1.4426950408889634f;
  return a;
}

static int pf_launch_slice(vkv_pool* p, int32_t layer, int32_t slice, const void* q, const int32_t* table,
                           int32_t max_blk, void* workspace, void* out, float scale, hipStream_t st) {
  PrefillParams a = pf_params(p, layer, q, table, max_blk, workspace, out, scale);
  a.item_first = p->pf.slice_start[slice];
  const int32_t count = p->pf.slice_start[slice + 1] - a.item_first;
  a.report = next_report(p, workspace);
  ProfKernel prof(p, VKV_PROF_PREFILL, slice);
  prof.launch(paged_prefill_attn_slice_kernel<128>, dim3((unsigned)count), dim3(256), st, a);
  VKV_HIP(hipGetLastError());
  return VKV_OK;
}

// merge step `step` covers tiles [merge_start[step], merge_start[step + 1])
static int pf_launch_merge(vkv_pool* p, int32_t step, void* workspace, void* out, hipStream_t st) {
  PrefillParams a = pf_params(p, 0, workspace, nullptr, 0, workspace, out, 0.f);
  a.merge_first = p->pf.merge_start[step];
  const int32_t n_tiles = p->pf.merge_start[step + 1] - a.merge_first;
  if (n_tiles == 0) return VKV_OK;   // no tile of this plan was split
  a.report = next_report(p, workspace);
  ProfScope prof(p, VKV_PROF_PREFILL_MERGE, step, st);
  hipLaunchKernelGGL(prefill_merge_kernel<128>, dim3((unsigned)(n_tiles * p->cfg.num_kv_heads * (kTileColumns / kMergeCols))),
                     dim3(256), 0, st, a);
  VKV_HIP(hipGetLastError());
  return VKV_OK;
}

}  // namespace vkv

using namespace vkv;

extern "C" {

int kv_prefill_plan(vkv_pool* p, const int32_t* ctx, const int32_t* q_len, int32_t S, uint64_t slice_bytes,
                    int32_t chunk_tokens, vkv_prefill_plan_info* info) {
  if (!p || !ctx || !q_len || S < 1) { set_error("kv_prefill_plan: bad argument"); return VKV_E_INVAL; }
  if (chunk_tokens < kGroupTokens || chunk_tokens % kGroupTokens || chunk_tokens > kMaxPrefillChunkTokens) {
    set_error("kv_prefill_plan: chunk_tokens must be a multiple of %d in [%d, %d]", kGroupTokens, kGroupTokens,
              kMaxPrefillChunkTokens);
    return VKV_E_INVAL;
  }
  const int Hkv = p->cfg.num_kv_heads, D = p->cfg.head_dim, B = p->cfg.block_tokens, G = p->G;
  if (D != 128) { set_error("kv_prefill_plan: prefill supports head_dim 128 only (pool has %d)", D); return VKV_E_INVAL; }
  int gp_shift = 0;
  while ((1 << gp_shift) < G) ++gp_shift;
  const int QP = kTileColumns >> gp_shift;   // positions per tile
  vkv_pool::PrefillPlan pl;
  pl.gp_shift = gp_shift;
  pl.tile_positions = QP;
  pl.num_seqs = S;
  int64_t row = 0;
  double flops = 0.0;
  uint64_t total = 0, max_slice = 0;
  for (int32_t s = 0; s < S; ++s) {
    if (q_len[s] < 1 || ctx[s] < q_len[s]) {
      set_error("kv_prefill_plan: sequence %d needs 1 <= q_len (%d) <= context length (%d)", s, q_len[s], ctx[s]);
      return VKV_E_INVAL;
    }
    pl.max_ctx_blocks = std::max(pl.max_ctx_blocks, (ctx[s] + B - 1) / B);
    const int32_t q0 = ctx[s] - q_len[s];
    for (int32_t t = 0; t * QP < q_len[s]; ++t) {
      const int32_t n_pos = std::min(QP, q_len[s] - t * QP), pos0 = q0 + t * QP, visible = pos0 + n_pos;
      const int32_t tile = (int32_t)pl.tile_base.size();
      pl.tiles.insert(pl.tiles.end(), {s, (int32_t)(row + (int64_t)t * QP), pos0, n_pos});
      pl.tile_base.push_back((int32_t)pl.work.size());
      for (int32_t first = 0; first < visible; first += chunk_tokens) {
        const int32_t nt = std::min(chunk_tokens, visible - first);
        for (int32_t h = 0; h < Hkv; ++h) pl.work.push_back(WorkItem{tile, h, first / B, nt});
      }
      if (pl.work.size() > 0x7FFFFF00u) { set_error("kv_prefill_plan: too many work items"); return VKV_E_INVAL; }
      for (int32_t i = 0; i < n_pos; ++i) flops += 4.0 * D * p->cfg.num_q_heads * (double)(pos0 + i + 1);
    }
    row += q_len[s];
  }
  if (row > 0x7FFFFFF0ll) { set_error("kv_prefill_plan: too many query rows"); return VKV_E_INVAL; }
  pl.total_q = (int32_t)row;
  pl.tile_base.push_back((int32_t)pl.work.size());
  const uint64_t token_bytes = (uint64_t)2 * D * 2;
  pl.slice_start.push_back(0);
  uint64_t acc = 0;
  for (size_t i = 0; i < pl.work.size(); ++i) {
    const uint64_t b = (uint64_t)pl.work[i].n_tokens * token_bytes;
    if ((int32_t)i > pl.slice_start.back() && acc + b > slice_bytes) {
      max_slice = std::max(max_slice, acc);
      pl.slice_start.push_back((int32_t)i);
      acc = 0;
    }
    acc += b;
    total += b;
  }
  max_slice = std::max(max_slice, acc);
  pl.slice_start.push_back((int32_t)pl.work.size());
  const uint64_t n_items = pl.work.size(), n_tiles = pl.tile_base.size() - 1;
  // The merge of split tiles is cut into steps as well, so that it cannot hold up a yield: a step
  // is a run of split tiles whose partial results and outputs amount to at most slice_bytes / 2.
  {
    const uint64_t tile_part = (uint64_t)kTileColumns * D * 4 * Hkv, bound = std::max<uint64_t>(slice_bytes / 2, tile_part);
    uint64_t acc_b = 0;
    pl.merge_start.push_back(0);
    for (size_t t = 0; t + 1 < pl.tile_base.size(); ++t) {
      const uint64_t nch = (uint64_t)(pl.tile_base[t + 1] - pl.tile_base[t]) / Hkv;
      if (nch <= 1) continue;
      const uint64_t b = (nch + 1) * tile_part;
      if (acc_b + b > bound && acc_b > 0) {
        pl.merge_start.push_back((int32_t)pl.merge_tiles.size());
        acc_b = 0;
      }
      pl.merge_tiles.push_back((int32_t)t);
      acc_b += b;
    }
    pl.merge_start.push_back((int32_t)pl.merge_tiles.size());
  }
  // What the kernel reads: one record per item.  Workgroups start in grid order: the longest items of a slice go
  // first so that the short ones fill the tail.  Results are stored by item id, so the order is invisible outside
  // the kernel.
  pl.items.reserve(n_items);
  for (size_t i = 0; i < n_items; ++i) {
    const WorkItem& w = pl.work[i];
    const int32_t* t = &pl.tiles[4 * (size_t)w.seq];
    const bool single = (pl.tile_base[w.seq + 1] - pl.tile_base[w.seq]) / Hkv == 1;
    pl.items.push_back(PrefillItem{t[0], t[1], t[2], t[3], w.kv_head, w.first_block, w.n_tokens, single ? -1 : (int32_t)i});
  }
  for (size_t sl = 0; sl + 1 < pl.slice_start.size(); ++sl)
    std::stable_sort(pl.items.begin() + pl.slice_start[sl], pl.items.begin() + pl.slice_start[sl + 1],
                     [](const PrefillItem& a, const PrefillItem& b) { return a.n_tokens > b.n_tokens; });
  pl.off_items = 256;
  pl.off_tiles = pl.off_items + n_items * sizeof(PrefillItem);
  pl.off_tile_base = pl.off_tiles + n_tiles * 16;
  pl.off_merge_tiles = pl.off_tile_base + (n_tiles + 1) * 4;
  pl.upload_bytes = pl.off_merge_tiles + pl.merge_tiles.size() * 4;
  pl.off_ml = align_up(pl.upload_bytes, 256);
  pl.off_acc = align_up(pl.off_ml + n_items * kTileColumns * 2 * 4, 256);
  pl.total = align_up(pl.off_acc + n_items * kTileColumns * (uint64_t)D * 4, 256);
  pl.has_plan = true;
  pl.gen = p->pf.gen + 1;
  p->pf = std::move(pl);
  if (info) {
    info->n_items = (int32_t)n_items;
    info->n_slices = (int32_t)p->pf.slice_start.size() - 1;
    info->n_tiles = (int32_t)n_tiles;
    info->tile_positions = QP;
    info->total_q = p->pf.total_q;
    info->n_merge_steps = (int32_t)p->pf.merge_start.size() - 1;
    info->workspace_bytes = p->pf.total;
    info->kv_bytes_per_layer = total;
    info->max_slice_kv_bytes = max_slice;
    info->flops_per_layer = flops;
  }
  return VKV_OK;
}

int kv_prefill_plan_read(vkv_pool* p, int32_t* work_out, int32_t* slice_start_out, int32_t* tiles_out,
                         int32_t* tile_base_out) {
  if (!p) { set_error("kv_prefill_plan_read: null pool"); return VKV_E_INVAL; }
  if (!p->pf.has_plan) { set_error("kv_prefill_plan_read: no plan"); return VKV_E_STATE; }
  if (work_out) std::memcpy(work_out, p->pf.work.data(), p->pf.work.size() * sizeof(WorkItem));
  if (slice_start_out) std::memcpy(slice_start_out, p->pf.slice_start.data(), p->pf.slice_start.size() * 4);
  if (tiles_out) std::memcpy(tiles_out, p->pf.tiles.data(), p->pf.tiles.size() * 4);
  if (tile_base_out) std::memcpy(tile_base_out, p->pf.tile_base.data(), p->pf.tile_base.size() * 4);
  return VKV_OK;
}

int kv_prefill_bind(vkv_pool* p, void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!p) { set_error("kv_prefill_bind: null pool"); return VKV_E_INVAL; }
  if (p->broken) { set_error("kv_prefill_bind: pool unusable after a HIP failure"); return VKV_E_HIP; }
  if (!p->pf.has_plan) { set_error("kv_prefill_bind: no plan"); return VKV_E_STATE; }
  if (!workspace || (uintptr_t)workspace % 256 || workspace_bytes < p->pf.total) {
    set_error("kv_prefill_bind: workspace must be 256-byte aligned and hold %llu bytes", (unsigned long long)p->pf.total);
    return VKV_E_INVAL;
  }
  int st = ensure_plan_stage(p, p->pf.upload_bytes);
  if (st != VKV_OK) return st;
  char* h = p->stage.host;
  std::memset(h, 0, 256);
  std::memcpy(h + p->pf.off_items, p->pf.items.data(), p->pf.items.size() * sizeof(PrefillItem));
  std::memcpy(h + p->pf.off_tiles, p->pf.tiles.data(), p->pf.tiles.size() * 4);
  std::memcpy(h + p->pf.off_tile_base, p->pf.tile_base.data(), p->pf.tile_base.size() * 4);
  std::memcpy(h + p->pf.off_merge_tiles, p->pf.merge_tiles.data(), p->pf.merge_tiles.size() * 4);
  if ((st = stage_upload(p->stage, workspace, p->pf.upload_bytes, (hipStream_t)stream)) != VKV_OK) return st;
  p->pf.bound_ws = workspace;
  p->pf.bound_gen = p->pf.gen;
  return VKV_OK;
}

int paged_prefill_attn_slice(vkv_pool* p, int32_t layer, int32_t slice, const void* q, const int32_t* table,
                             int32_t max_blk, void* workspace, void* out, float scale, void* stream) {
  int st = pf_check_args(p, layer, q, table, max_blk, workspace, out, "paged_prefill_attn_slice");
  if (st != VKV_OK) return st;
  if (slice < 0 || slice >= (int32_t)p->pf.slice_start.size() - 1) {
    set_error("paged_prefill_attn_slice: slice %d out of range [0,%d)", slice, (int)p->pf.slice_start.size() - 1);
    return VKV_E_INVAL;
  }
  return pf_launch_slice(p, layer, slice, q, table, max_blk, workspace, out, scale, (hipStream_t)stream);
}

int kv_prefill_merge(vkv_pool* p, int32_t step, void* workspace, void* out, void* stream) {
  int st = pf_check_bound(p, workspace, "kv_prefill_merge");
  if (st != VKV_OK) return st;
  if (!out) { set_error("kv_prefill_merge: null output"); return VKV_E_INVAL; }
  if (step < 0 || step >= (int32_t)p->pf.merge_start.size() - 1) {
    set_error("kv_prefill_merge: step %d out of range [0,%d)", step, (int)p->pf.merge_start.size() - 1);
    return VKV_E_INVAL;
  }
  return pf_launch_merge(p, step, workspace, out, (hipStream_t)stream);
}

int kv_prefill_run_layer(vkv_pool* p, int32_t layer, int32_t* cursor, const void* q, const int32_t* table,
                         int32_t max_blk, void* workspace, void* out, float scale, int32_t max_inflight,
                         void* stream) {
  int st = pf_check_args(p, layer, q, table, max_blk, workspace, out, "kv_prefill_run_layer");
  if (st != VKV_OK) return st;
  hipStream_t hs = (hipStream_t)stream;
  return run_slices(p, cursor, (int32_t)p->pf.slice_start.size() - 1, max_inflight, hs, "kv_prefill_run_layer",
                    [&](int32_t s, hipStream_t on) {
                      return pf_launch_slice(p, layer, s, q, table, max_blk, workspace, out, scale, on);
                    },
                    (int32_t)p->pf.merge_start.size() - 1,
                    [&](int32_t step) { return pf_launch_merge(p, step, workspace, out, hs); }, !p->pf.merge_tiles.empty(),
                    true,   // two streams: few, long items per slice, 2300 : 1940 us in 20 slices, no worse in 3
                    false);  // ends reported: events 2-3 % faster in 3 to 5 slices of 400-670 items, as fast or up to 8 % slower elsewhere
}

int kv_prefill_check(vkv_pool* p, void* workspace, void* stream) {
  int st = pf_check_bound(p, workspace, "kv_prefill_check");
  if (st != VKV_OK) return st;
  VKV_HIP(hipStreamSynchronize((hipStream_t)stream));
  uint32_t flag = 0;
  VKV_HIP(hipMemcpy(&flag, workspace, 4, hipMemcpyDeviceToHost));
  if (flag) { set_error("kv_prefill_check: a slice met a block-table entry outside the pool"); return VKV_E_STATE; }
  return VKV_OK;
}

}  // extern "C"
