// Head-mixed causal prefill on gfx950.
//
// Computes, per (batch, query head, query row i), the attention of the paper's
// Sec. 5 (chunked-prefill stage): softmax over the visible keys of
// q_i . k_j / sqrt(D), times V.  Retrieval heads see j <= i; streaming heads
// see j <= i with j < n_sink or j >= lo(i), where lo(i) = i - window + 1 for
// the per-token band and lo(i) = floor(i / K) K - window for chunk eviction
// with chunks of K tokens (the cache before a chunk keeps the sink and the
// window most recent tokens; the chunk sees those and itself).
//
// bf16 kernels.  One workgroup = 128 or 256 query rows of one query head; each
// wave owns 32 rows.  Key/value tiles of 64 keys are staged in LDS and shared by
// the workgroup's waves.  Per tile and wave:
//   S^T[64 keys x 32 rows] = K_tile . Q^T        (v_mfma_f32_32x32x16_bf16)
//   online softmax in fp32, one query row per lane column, so the row max is a
//   lane-local reduction plus one exchange with the partner lane (lane ^ 32)
//   O^T[D x 32 rows] += V_tile^T . P^T           (same MFMA)
// P never leaves registers: the S^T accumulator layout is already the B
// operand layout of the P^T product.  V^T operands come straight out of the
// row-major V tile through the gfx950 LDS transpose read (ds_read_b64_tr_b16).
// Streaming heads iterate only over the sink tiles and the diagonal band of
// tiles; other tiles are never loaded.  Tiles that are fully visible skip the
// per-element mask.
//   prefill_pp_kernel: direct global->LDS tile loads into rings of LDS tiles,
//     swizzled LDS rows, two phase-shifted wave groups, XCD-aware workgroup
//     order (see its own comment).  A layer with both head types runs as one
//     launch (prefill_pp_mixed_kernel): retrieval items first, streaming items
//     after them.
//
// fp32 kernel: a plain per-row kernel (one thread per query row) kept exact
// for fp32 inputs; it has no performance role.
#include <algorithm>
#include <atomic>
#include <numeric>
#include <type_traits>

#include "aoh_device.h"
#include "aoh_internal.h"

namespace aoh {

constexpr int kBN = 64;          // keys per tile
// Largest sum of a lane's 32 exponentials of one tile, taken against the trailing
// reference max, that is accepted as it is.
constexpr float kSumHi = 65536.f;

// First non-sink key visible to row i of a streaming head (may be negative).
__device__ __forceinline__ int lo_of(int i, int chunk, int window) {
  return chunk ? (i / chunk) * chunk - window : i - window + 1;
}

// Tile visit plan of one query block [i0, i0 + rows).
struct TilePlan {
  int n_sink_tiles;  // leading sink tiles visited before the band
  int band_first;    // first band tile
  int n_visit;       // total tiles
  __device__ __forceinline__ int tile(int it) const {
    return it < n_sink_tiles ? it : band_first + (it - n_sink_tiles);
  }
};

template <bool STREAM>
__device__ __forceinline__ TilePlan make_plan(int i0, int rows, int T, int n_sink, int window, int chunk) {
  const int last_row = min(i0 + rows - 1, T - 1);
  const int last_tile = last_row / kBN;
  TilePlan p;
  if (!STREAM) {
    p.n_sink_tiles = 0;
    p.band_first = 0;
    p.n_visit = last_tile + 1;
  } else {
    const int band_lo = max(0, lo_of(i0, chunk, window));  // lo is non-decreasing in i
    p.band_first = band_lo / kBN;
    const int sink_tiles = (n_sink + kBN - 1) / kBN;
    p.n_sink_tiles = min(sink_tiles, p.band_first);
    p.n_visit = p.n_sink_tiles + (last_tile - p.band_first + 1);
  }
  return p;
}

// fp32 reference-grade kernel: one thread per query row, keys visited in
// order (sink part, then the recent band), exact expf.
template <int D, bool STREAM>
__global__ __launch_bounds__(kPrefillRowsF32) void prefill_f32_kernel(PrefillArgs a) {
  // No implicit FMA contraction: a lone visible key must get weight exactly 1.
#pragma clang fp contract(off)
  const int n_qh = a.n_kv * a.gs;
  const int per_block = n_qh * a.B;
  const int wg = blockIdx.x;
  const int qb = a.n_qblocks - 1 - wg / per_block;
  const int rem = wg % per_block;
  const int qh_local = rem % n_qh;
  const int b = rem / n_qh;
  const int g = a.kv_heads[qh_local / a.gs];
  const int h = g * a.gs + (qh_local % a.gs);
  const int i = qb * kPrefillRowsF32 + threadIdx.x;
  int T = a.T;
  int64_t tok0 = 0;
  if (a.cu_seqlens) {
    const int s0 = min(max(a.cu_seqlens[b], 0), a.total);
    const int s1 = min(max(a.cu_seqlens[b + 1], s0), a.total);
    T = min(s1 - s0, a.T);
    tok0 = s0;
  }
  if (i >= T) return;
  const int64_t qoff = a.cu_seqlens ? tok0 * a.q_st : (int64_t)b * a.q_sb;
  const int64_t koff = a.cu_seqlens ? tok0 * a.k_st : (int64_t)b * a.k_sb;
  const int64_t voff = a.cu_seqlens ? tok0 * a.v_st : (int64_t)b * a.v_sb;
  const int64_t ooff = a.cu_seqlens ? tok0 * a.o_st : (int64_t)b * a.o_sb;
  const float* qp = reinterpret_cast<const float*>(a.q) + qoff + (int64_t)i * a.q_st +
                    (int64_t)h * a.q_sh;
  const float* kp = reinterpret_cast<const float*>(a.k) + koff + (int64_t)g * a.k_sh;
  const float* vp = reinterpret_cast<const float*>(a.v) + voff + (int64_t)g * a.v_sh;
  float q[D], o[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    q[d] = qp[d];
    o[d] = 0.f;
  }
  float m = -INFINITY, l = 0.f;
  int lo = 0, sink_end = 0;
  if (STREAM) {
    lo = max(0, lo_of(i, a.chunk, a.window));
    sink_end = min(a.n_sink, lo);
  }
  auto visit = [&](int j) {
    float s = 0.f;
    const float* kr = kp + (int64_t)j * a.k_st;
#pragma unroll
    for (int d = 0; d < D; ++d) s = fmaf(q[d], kr[d], s);
    s *= a.scale;
    const float m_new = fmaxf(m, s);
    const float alpha = expf(m - m_new);
    const float p = expf(s - m_new);
    l = l * alpha + p;
    const float* vr = vp + (int64_t)j * a.v_st;
#pragma unroll
    for (int d = 0; d < D; ++d) o[d] = o[d] * alpha + p * vr[d];
    m = m_new;
  };
  for (int j = 0; j < sink_end; ++j) visit(j);
  for (int j = lo; j <= i; ++j) visit(j);
  float* op = reinterpret_cast<float*>(a.out) + ooff + (int64_t)i * a.o_st + (int64_t)h * a.o_sh;
  const float inv = 1.f / l;
#pragma unroll
  for (int d = 0; d < D; ++d) op[d] = o[d] * inv;
}

// ---------------------------------------------------------------------------
// bf16 kernel, phase-shifted wave groups.
//
// Work item: 128 or 256 query rows of one query head (PPShape), 32 rows per
// wave, S^T = K.Q^T and O^T += V^T.P^T on the 32x32x16 bf16 MFMA, online
// softmax in fp32.
//  * K/V tiles move global -> LDS with direct loads (global_load_lds_dwordx4),
//    no register staging, into a K ring and a V ring of two to four tiles each
//    (16 KB a tile for d_head 128, 8 KB for 64), issued one or two tiles ahead
//    of their first use.
//  * Rows hold D / 8 chunks of 16 bytes with no padding, swizzled (PPTile) so
//    that the K row reads and the V transpose reads are free of bank
//    conflicts.  Every operand address is one of D / 16 + D / 32 per-lane base
//    registers plus a constant, and the tile loop runs several tiles per pass so
//    that each ring slot is a compile-time constant too: the operand reads take
//    it as an immediate offset, with no address arithmetic per tile.
//  * Per tile t a wave runs an MFMA phase (P(t-1).V(t-1) then K(t).Q^T, at
//    raised wave priority) and a vector phase (mask, exponentials of S(t)
//    against a trailing reference max, no max pass unless the tile's
//    exponentials grow too large), with one workgroup barrier per tile.  With
//    256 rows, waves 0-3 and waves 4-7 (one of each per SIMD) run one phase
//    apart: the barrier comes after the vector phase for waves 0-3, after the
//    MFMA phase for waves 4-7.  With 128 rows the waves of different
//    workgroups on a SIMD interleave their phases.
//    The loop has a single path, so the accumulators never move between
//    registers: a tile with no visible key for a wave yields P = 0 (d_head 128),
//    or lies outside the loop's range of tiles (64).
//  * The fused cache append writes the block's own (diagonal) tiles after
//    the loop, from the ring, which still holds them.
//  * Workgroups are ordered so that the query heads of one KV group and query
//    block run on the same XCD (one L2); the light items at the end of a
//    launch are taken from per-XCD work queues, so that faster XCDs take over
//    part of the slower ones' share.
// Shape of a workgroup of ROWS query rows, 32 a wave: 8 waves in two phase-
// shifted groups, or 4 waves and two (d_head 128) or three (64) workgroups a
// CU, which drift apart by themselves.  Loads run kAhead tiles ahead.  A tile's
// K is last read in its own MFMA phase, its V in the next one: with loads two
// tiles ahead K needs two slots and V three.  The slots also hold a block's
// diagonal tiles for the append after the loop (ROWS / kBN of them).
template <int D, int ROWS>
struct PPShape {
  static constexpr int kThreads = 2 * ROWS;
  static constexpr bool kPair = ROWS == 256;
  static constexpr int kAhead = kPair ? 3 : 2;
  static constexpr int kKSlots = kPair ? 4 : D == 128 ? 2 : 3;
  static constexpr int kVSlots = kPair ? 4 : 3;
  // tiles per pass of the loop, a common multiple of the slots
  static constexpr int kUnroll = kPair ? 4 : D == 128 ? 6 : 3;
  static constexpr int kWavesPerSimd = D == 64 ? 3 : 2;
  static constexpr int kLoads = kBN * (D / 8) / kThreads;  // loads per thread and tile, K or V
  static_assert(ROWS / kBN <= kKSlots, "the ring holds the diagonal tiles");
};

// The LDS rings: the K tiles of the slots, then the V tiles (a slot's offset
// within a ring fits the 16-bit immediate offset of an LDS read).
template <int D, int ROWS>
struct PPRing {
  uint16_t k[PPShape<D, ROWS>::kKSlots][kBN * D];
  uint16_t v[PPShape<D, ROWS>::kVSlots][kBN * D];
};

// Swizzle of a tile's rows: chunk c of row r is stored at c ^ kx(r) in a K
// tile and c ^ vx(r) in a V tile.  K operands are read 16 bytes a lane down 32
// rows: 16 consecutive rows take 16 different 16-byte columns of the 64 banks
// (a row of d_head 64 spans half of them, so two rows share a pattern).  V
// operands are read as 4 rows x 64 bytes a half wave: the four land in
// different quarters.
template <int D>
struct PPTile {
  static constexpr int kChunks = D / 8;                     // 16-byte chunks of a row
  static constexpr uint32_t kBytes = kBN * D * 2;           // one K or V tile
  static __device__ __forceinline__ int kx(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
  static __device__ __forceinline__ int vx(int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }
  static __device__ __forceinline__ int koff(int r, int c) { return r * D + 8 * (c ^ kx(r)); }
  static __device__ __forceinline__ int voff(int r, int c) { return r * D + 8 * (c ^ vx(r)); }
};

// Direct global -> LDS load of 16 bytes per lane: lane L's bytes land at
// lds_row + 16 L (one contiguous 1 KB block per wave).  Issued as inline
// assembly so that the compiler does not treat every later LDS read as
// possibly depending on it (it would wait for all outstanding loads before
// each one); the kernel orders these loads itself with s_waitcnt and barriers.
__device__ __forceinline__ void lds_dma16(const void* gptr, const void* lds_row) {
  const uint32_t m0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds_row));
  asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(gptr), "{m0}"(m0) : "memory");
}

// s_waitcnt immediates (gfx9 encoding: vmcnt [3:0] and [15:14], expcnt [6:4],
// lgkmcnt [11:8]); a field at its maximum does not wait.
constexpr int kWaitVm0 = 0x0 | (0x7 << 4) | (0xF << 8);
constexpr int wait_vm(int n) { return n | (0x7 << 4) | (0xF << 8); }  // n < 16
constexpr int kWaitLgkm0 = 0xF | (0x7 << 4) | (0x0 << 8) | (0x3 << 14);

// Work item of a workgroup: query block qb (rows qb * ROWS ..), local query
// head qh_local of the launch's KV-head list and sequence b.  Dense batches use
// the XCD-aware order below; packed batches with sequence-major order walk
// cu_seqlens.  Returns false when the workgroup has no work (past the last
// sequence's blocks).
template <int ROWS>
__device__ __forceinline__ bool pp_work_item(const PrefillArgs& a, int wg, int& qb, int& qh_local, int& b) {
  const int n_qh = a.n_kv * a.gs;
  if constexpr (ROWS != 128) {
    // Both branches set these again; with them the compiler lays out the 256-row
    // kernels better (retrieval launch of 32768 tokens 3.145 ms, 3.165 without;
    // 4 packed prompts of 1000-30000 1% faster).
    const int per_block = n_qh * a.B;
    qb = a.n_qblocks - 1 - wg / per_block;
    const int rem = wg % per_block;
    qh_local = rem % n_qh;
    b = rem / n_qh;
  }
  if (!a.seq_major) {
    int b0 = 0, B = a.B;
    if (ROWS == 128 && a.part < a.B) {
      // Parts of the batch one after the other (PrefillArgs::part), each in the
      // order below.
      const int per_part = a.n_qblocks * n_qh * a.part;
      const int part = wg / per_part;
      wg -= part * per_part;
      b0 = part * a.part;
      B = min(a.part, a.B - b0);
    }
    // XCD-aware order.  Workgroups go to the 8 XCDs (each with its own L2)
    // in turn; work item group j = (query block, sequence, KV head), heaviest
    // block first, holds the gs query heads that read the same K/V tiles.
    // Round m of 8 groups runs as gs consecutive workgroups on each XCD, so a
    // group's tiles are fetched into one L2 once.  Groups get lighter along
    // the order, so odd rounds deal them in reverse, which keeps each XCD's
    // total work level (dealt one way, XCD 0 would take the heaviest group of
    // every round).  When a round holds whole query blocks (the per-block
    // group count divides 8) only the blocks' order is reversed: each XCD
    // keeps serving one (sequence, KV head), whose causal prefix stays in its
    // L2.  The trailing groups that do not fill a round of 8 are dealt in
    // plain order.
    const int n_groups = a.n_qblocks * a.n_kv * B;
    const int full = 8 * a.gs * (n_groups / 8);
    const int pq = a.n_kv * B;
    int j, hl;
    if (wg < full) {
      const int slot = wg >> 3;
      const int m = slot / a.gs;
      int x = wg & 7;
      if (m & 1) x = (8 % pq == 0) ? (8 - pq) - (x - x % pq) + x % pq : 7 - x;
      j = 8 * m + x;
      hl = slot % a.gs;
    } else {
      j = (full / a.gs) + (wg - full) / a.gs;
      hl = (wg - full) % a.gs;
    }
    qb = a.n_qblocks - 1 - j / pq;
    const int r2 = j % pq;
    b = b0 + r2 / a.n_kv;
    qh_local = (r2 % a.n_kv) * a.gs + hl;
  }
  if (a.seq_major) {
    int unit = wg / n_qh;
    qh_local = wg % n_qh;
    b = -1;
    for (int s2 = 0; s2 < a.B; ++s2) {
      const int s0 = min(max(a.cu_seqlens[s2], 0), a.total);
      const int s1 = min(max(a.cu_seqlens[s2 + 1], s0), a.total);
      const int nb = (min(s1 - s0, a.T) + ROWS - 1) / ROWS;
      if (unit < nb) {
        b = s2;
        qb = nb - 1 - unit;
        break;
      }
      unit -= nb;
    }
    if (b < 0) return false;
  }
  return true;
}

// Fused append of one resident tile (keys kb .. kb+63) into the cache of the
// launch: the paged cache (K token-major, V dimension-major per page; pages
// outside the block table are skipped) or the ring (a position is kept only
// if no later prompt position maps to its slot).  Threads tid, tid + nthr, ..
// take the 16-byte chunks of the tile; crank = the KV head's rank in the cache.
template <int D, bool STREAM>
__device__ __forceinline__ void pp_write_tile(const PrefillArgs& a, const uint16_t* tk, const uint16_t* tv, int kb,
                                              int b, int crank, int T, int tid, int nthr) {
  constexpr int kCh = D / 8;
  uint16_t* ck = static_cast<uint16_t*>(a.ck);
  uint16_t* cv = static_cast<uint16_t*>(a.cv);
  if (!STREAM) {
    for (int e = tid; e < kBN * kCh; e += nthr) {
      const int row = e / kCh, ch = e % kCh;
      const int p = kb + row;
      const int lp = p / kPageTokens;
      if (p >= T || lp >= a.max_pages) continue;
      const int page = a.block_table[(int64_t)b * a.max_pages + lp];
      if (page < 0 || page >= a.num_pages) continue;
      uint16_t* dst = ck + (((int64_t)page * a.n_cache + crank) * kPageTokens + p % kPageTokens) * D + 8 * ch;
      st16(dst, *reinterpret_cast<const u32x4*>(&tk[PPTile<D>::koff(row, ch)]));
    }
    for (int e = tid; e < (kBN / kPageTokens) * D * 2; e += nthr) {
      const int pg = e / (2 * D), d = (e / 2) % D, hf = e % 2;
      const int p0 = kb + kPageTokens * pg + 8 * hf;
      const int lp = p0 / kPageTokens;
      if (p0 >= T || lp >= a.max_pages) continue;
      const int page = a.block_table[(int64_t)b * a.max_pages + lp];
      if (page < 0 || page >= a.num_pages) continue;
      uint16_t* dst = cv + (((int64_t)page * a.n_cache + crank) * D + d) * kPageTokens + 8 * hf;
      const int row0 = kPageTokens * pg + 8 * hf;
      const int dc = d >> 3, de = d & 7;
      if (p0 + 8 <= T) {
        u32x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[j] = (uint32_t)tv[PPTile<D>::voff(row0 + 2 * j, dc) + de] |
                 ((uint32_t)tv[PPTile<D>::voff(row0 + 2 * j + 1, dc) + de] << 16);
        st16(dst, w);
      } else {
        for (int j = 0; p0 + j < T; ++j) dst[j] = tv[PPTile<D>::voff(row0 + j, dc) + de];
      }
    }
  } else {
    for (int e = tid; e < kBN * kCh; e += nthr) {
      const int row = e / kCh, ch = e % kCh;
      const int p = kb + row;
      if (p >= T || !(p < a.n_sink || p >= T - a.window)) continue;
      const int slot = p < a.n_sink ? p : a.n_sink + (p - a.n_sink) % a.window;
      const int64_t unit = ((int64_t)b * a.n_cache + crank) * a.ring_blocks + slot / kPageTokens;
      const int r = slot % kPageTokens;
      st16(ck + unit * (kPageTokens * D) + r * D + 8 * ch,
           *reinterpret_cast<const u32x4*>(&tk[PPTile<D>::koff(row, ch)]));
      uint16_t* rv = cv + unit * (kPageTokens * D);
      const int vo = PPTile<D>::voff(row, ch);
#pragma unroll
      for (int j = 0; j < 8; ++j) rv[(8 * ch + j) * kPageTokens + r] = tv[vo + j];
    }
  }
}

// One work item (workgroup index wg of its launch's item space) of the
// kernel; ring = the workgroup's LDS rings.
template <int D, int ROWS, bool STREAM, bool OUT_F32, bool APPEND>
__device__ __forceinline__ void prefill_pp_body(const PrefillArgs& a, int wg, PPRing<D, ROWS>& ring) {
  using Tile = PPTile<D>;
  using Shape = PPShape<D, ROWS>;
  constexpr int kKSteps = D / 16;
  constexpr int kMBlocks = D / 32;

  int qb, qh_local, b;
  if (!pp_work_item<ROWS>(a, wg, qb, qh_local, b)) return;
  const int g = a.kv_heads[qh_local / a.gs];
  const int h = g * a.gs + (qh_local % a.gs);

  const int tid = threadIdx.x;
  // Wave index as a scalar: every branch that decides a barrier is uniform.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;
  const int lane = tid & 63;
  const int l32 = lane & 31;
  const int h2 = lane >> 5;
  int T = a.T;
  int64_t tok0 = 0;
  if (a.cu_seqlens) {
    const int s0 = min(max(a.cu_seqlens[b], 0), a.total);
    const int s1 = min(max(a.cu_seqlens[b + 1], s0), a.total);
    T = min(s1 - s0, a.T);
    tok0 = s0;
  }
  T = __builtin_amdgcn_readfirstlane(T);
  const int i0 = qb * ROWS;
  if (i0 >= T) return;
  const int r0 = i0 + wave * 32;
  const int my_row = r0 + l32;
  const int my_lo = lo_of(my_row, a.chunk, a.window);

  const int64_t qoff = a.cu_seqlens ? tok0 * a.q_st : (int64_t)b * a.q_sb;
  const int64_t koff = a.cu_seqlens ? tok0 * a.k_st : (int64_t)b * a.k_sb;
  const int64_t voff = a.cu_seqlens ? tok0 * a.v_st : (int64_t)b * a.v_sb;
  const int64_t ooff = a.cu_seqlens ? tok0 * a.o_st : (int64_t)b * a.o_sb;
  const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + qoff + (int64_t)h * a.q_sh;
  const uint16_t* kp = reinterpret_cast<const uint16_t*>(a.k) + koff + (int64_t)g * a.k_sh;
  const uint16_t* vp = reinterpret_cast<const uint16_t*>(a.v) + voff + (int64_t)g * a.v_sh;

  const TilePlan plan = make_plan<STREAM>(i0, ROWS, T, a.n_sink, a.window, a.chunk);
  const int n = __builtin_amdgcn_readfirstlane(plan.n_visit);
  if (n < 1) return;  // a block with rows below T always has its diagonal tile

  // Direct loads of tile `it` into its slots: wave w fills kLoads blocks of
  // 1 KB (512 / D rows) of K and of V, one instruction each; lane L writes
  // physical chunk L % kChunks of its row and therefore fetches the logical
  // chunk that the swizzle puts there.  Rows past the sequence end repeat its
  // last row (those keys are masked for every query row).  Per-lane element
  // offsets relative to the tile's first key (full tiles), and the rows
  // themselves (the ragged last tile clamps them).
  constexpr int kBlockRows = 512 / D;
  int64_t dma_k[Shape::kLoads], dma_v[Shape::kLoads];
  int dma_r[Shape::kLoads];
#pragma unroll
  for (int jj = 0; jj < Shape::kLoads; ++jj) {
    const int r = kBlockRows * (Shape::kLoads * wave + jj) + lane / Tile::kChunks;
    const int pc = lane % Tile::kChunks;
    dma_r[jj] = r;
    dma_k[jj] = (int64_t)r * a.k_st + 8 * (pc ^ Tile::kx(r));
    dma_v[jj] = (int64_t)r * a.v_st + 8 * (pc ^ Tile::vx(r));
  }
  auto issue_tile = [&](int it) {
    const int kb = plan.tile(it) * kBN;
    uint16_t* sk = ring.k[it % Shape::kKSlots];
    uint16_t* sv = ring.v[it % Shape::kVSlots];
    if (kb + kBN <= T) {
      const uint16_t* kt = kp + (int64_t)kb * a.k_st;
      const uint16_t* vt = vp + (int64_t)kb * a.v_st;
#pragma unroll
      for (int jj = 0; jj < Shape::kLoads; ++jj) {
        const int j = Shape::kLoads * wave + jj;
        lds_dma16(kt + dma_k[jj], &sk[512 * j]);
        lds_dma16(vt + dma_v[jj], &sv[512 * j]);
      }
    } else {
#pragma unroll
      for (int jj = 0; jj < Shape::kLoads; ++jj) {
        const int j = Shape::kLoads * wave + jj;
        const int r = dma_r[jj];
        const int pc = lane % Tile::kChunks;
        const int64_t row = min(kb + r, T - 1);
        lds_dma16(kp + row * a.k_st + 8 * (pc ^ Tile::kx(r)), &sk[512 * j]);
        lds_dma16(vp + row * a.v_st + 8 * (pc ^ Tile::vx(r)), &sv[512 * j]);
      }
    }
  };

  bf16x8 qreg[kKSteps];  // Q^T operands: lane holds row my_row, dims 8*h2 + 16*s .. +8
  f32x16 acc_o[kMBlocks];
#pragma unroll
  for (int mb = 0; mb < kMBlocks; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc_o[mb][i] = 0.f;
  float m_run = -INFINITY;  // reference max (log2 units) of this lane's row
  float m_use = 0.f;        // m_run, or 0 while the row has seen no visible key
  float l_run = 0.f;        // this lane's partial row sum (partner lane has the rest)
  f32x16 sacc[2];           // S^T of the current tile, two 32-key blocks
  bf16x8 pop[4];            // P^T operands of the previous tile's 4 key steps

  const float c = a.scale_log2;

  // Per-lane LDS byte addresses.  K operand of step s, block blk: row
  // 32 blk + l32, logical chunk 2 s + h2; with the swizzle that is
  // kaddr0 ^ 32 s (+ 64 D bytes per block).  V^T operand of key step ks, 32-dim
  // block mb (transpose reads): row 16 ks + 4 h2 + i16 / 4 (+ 8 rows for the
  // second half), logical chunk 4 mb + 2 (q16 & 1) + (i16 & 3) / 2, 4 more
  // elements for odd i16; that is vaddr0 ^ 64 mb (+ 32 D bytes per key step).
  // (8, 16 or 32 rows more leave the swizzle as it is.)
  const int q16 = lane >> 4;
  const int i16 = lane & 15;
  const uint32_t kring0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&ring.k[0][0]));
  const uint32_t vring0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&ring.v[0][0]));
  const uint32_t kaddr0 = 2u * (uint32_t)PPTile<D>::koff(l32, h2);
  const int vrow0 = 4 * h2 + (i16 >> 2);
  const uint32_t vaddr0 = 2u * (uint32_t)(PPTile<D>::voff(vrow0, 2 * (q16 & 1) + ((i16 & 3) >> 1)) + 4 * (i16 & 1));
  // The swizzle XORs touch bits below 256 and the rings are 1 KB aligned, so
  // a slot offset adds after them: operand addresses are these per-lane bases
  // plus constants (immediate offsets once the slot is known at compile time).
  uint32_t kx[kKSteps], vx[kMBlocks];
#pragma unroll
  for (int s = 0; s < kKSteps; ++s) kx[s] = (kring0 + kaddr0) ^ (32u * s);
#pragma unroll
  for (int mb = 0; mb < kMBlocks; ++mb) vx[mb] = (vring0 + vaddr0) ^ (64u * mb);
  auto k_operand = [&](int st, int s, int blk) {
    typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
    return *reinterpret_cast<lds_bf16x8*>(kx[s] + (uint32_t)st * Tile::kBytes + 64u * D * blk);
  };
  auto v_operand = [&](int st, int ks, int mb) {
    typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
    const uint32_t a = vx[mb] + (uint32_t)st * Tile::kBytes + 32u * D * ks;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4*>(a));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4*>(a + 16u * D));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  auto wave_dead = [&](int kb) {
    return (kb > r0 + 31) || (STREAM && kb >= a.n_sink && kb + kBN - 1 < lo_of(r0, a.chunk, a.window));
  };
  auto need_mask = [&](int kb) {
    return (kb + kBN - 1 > r0) ||
           (STREAM && !(kb + kBN - 1 < a.n_sink || kb >= lo_of(r0 + 31, a.chunk, a.window)));
  };

  // Fused append: the first query head of each group copies its block's own
  // K/V rows from LDS into the cache.  They are the block's diagonal tiles,
  // the last tiles of the loop, which the ring still holds when
  // the loop ends; the workgroup writes them then.
  const bool writer = APPEND && (qh_local % a.gs) == 0;
  const int crank = qh_local / a.gs;
  // MFMA phase of tile t (K slot st): O^T += V(t-1)^T P(t-1)^T (V slot vst),
  // then S^T(t) = K(t) Q^T.
  auto pv_part = [&](int vst) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int mb = 0; mb < kMBlocks; ++mb) acc_o[mb] = mfma32(v_operand(vst, ks, mb), pop[ks], acc_o[mb]);
  };
  auto qk_part = [&](int st) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < 16; ++i) sacc[blk][i] = 0.f;
#pragma unroll
    for (int s = 0; s < kKSteps; ++s)
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) sacc[blk] = mfma32(k_operand(st, s, blk), qreg[s], sacc[blk]);
  };
  auto append_tile = [&](int t) {
    const int kb = plan.tile(t) * kBN;
    if (kb >= i0 && kb < i0 + ROWS)
      pp_write_tile<D, STREAM>(a, ring.k[t % Shape::kKSlots], ring.v[t % Shape::kVSlots], kb, b, crank, T, tid,
                               Shape::kThreads);
  };
  // Steady-state MFMA phase.  Both products run unconditionally, so the loop
  // has one path and the O accumulators stay in place.  (d_head 128: a wave with
  // no visible key in a tile gets P = 0 from its vector phase; a V row of such a
  // tile that is not finite still makes the wave's rows NaN.)
  // The MFMA phase runs at raised wave priority (s_setprio, this wave only):
  // its SIMD also holds a wave of the other group in its vector phase, and
  // the matrix core is kept fed first (2-3% faster than equal priority).
  auto mfma_phase = [&](int st, int vst) {
    __builtin_amdgcn_s_setprio(1);
    pv_part(vst);
    qk_part(st);
    // Operands are read four MFMAs ahead of their products, the first K
    // operands while the last P.V products run (an operand of V^T is two reads,
    // one of K is one; each product is D / 8 MFMAs).
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int i = 0; i < D / 8 - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
  };

  // Vector phase of tile t: mask, exponentials into the P^T operands, row
  // sums (and, rarely, a new reference max with the rescale).
  auto apply_mask = [&](int kb) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = kb + 32 * blk + 8 * (i >> 2) + 4 * h2 + (i & 3);
        bool vis = key <= my_row;
        if (STREAM) vis = vis && (key < a.n_sink || key >= my_lo);
        sacc[blk][i] = vis ? sacc[blk][i] : -INFINITY;
      }
  };
  // Softmax of a tile without a max pass: the exponentials are taken against
  // the reference max m_use as it stands (it trails the true row max) and the
  // tile is accepted when each lane's 32 exponentials sum to at most kSumHi,
  // which bounds every P by it (P, l and O stay far from fp32 overflow and P
  // keeps bf16's relative precision).  A lane whose row has seen no visible
  // key yet, or whose sum is larger or NaN, sends the wave through the exact
  // step: the true row max of the tile becomes the reference, O and l are
  // rescaled and the exponentials are taken again.  Row sums of the fp32
  // exponentials are added as balanced trees: the phase ends on its longest
  // dependency chain, and a running accumulator, a chain of bf16 dot products
  // or a max pass ahead of the exponentials lengthens it.
  auto softmax_tile = [&]() {
    auto exps = [&]() {
      float psum[4];
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          bf16x8 pv;
          float pf[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            pf[i] = fast_exp2(fmaf(sacc[blk][8 * hf + i], c, -m_use));
            pv[i] = f32_to_bf16(pf[i]);
          }
          if constexpr (D == 64) {
            // rounded P, as P.V takes it: two chains of two dot products with 1
            const bf16x2 ones = {(bf16)1.f, (bf16)1.f};
            auto pair = [&](auto j, float acc) {
              constexpr int J = decltype(j)::value;
              return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, J, J + 1), ones, acc, false);
            };
            using std::integral_constant;
            psum[2 * blk + hf] = pair(integral_constant<int, 2>{}, pair(integral_constant<int, 0>{}, 0.f)) +
                                 pair(integral_constant<int, 6>{}, pair(integral_constant<int, 4>{}, 0.f));
          } else {
            psum[2 * blk + hf] = ((pf[0] + pf[1]) + (pf[2] + pf[3])) + ((pf[4] + pf[5]) + (pf[6] + pf[7]));
          }
          pop[2 * blk + hf] = pv;
        }
      return (psum[0] + psum[1]) + (psum[2] + psum[3]);
    };
    float tsum = exps();
    if (__any(!(tsum <= kSumHi) || m_run == -INFINITY)) {
      float mx = -INFINITY;
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[blk][i]);
      const float m_new = fmaxf(m_run, xor32_max(mx) * c);
      const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < kMBlocks; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_o[mb][i] *= alpha;
      m_use = (m_run == -INFINITY) ? 0.f : m_run;
      tsum = exps();
    }
    l_run += tsum;
  };
  auto valu_phase = [&](int t) {
    const int kb = plan.tile(t) * kBN;
    if (D == 128 && wave_dead(kb)) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) pop[ks][i] = (bf16)0.f;
      return;
    }
    if (need_mask(kb)) apply_mask(kb);
    softmax_tile();
  };

  // One workgroup barrier per tile.  Every wave runs MFMA(0) V(0) MFMA(1)
  // V(1) ..; waves 0-3 take the barrier of tile t after V(t), waves 4-7 after
  // MFMA(t), so a SIMD's two waves alternate without a barrier between their
  // phases.  The barrier of tile t follows each wave's wait for its loads of
  // tile t+1 (with loads three tiles ahead those of t+2 may stay in flight);
  // after it, tile t + kAhead goes into the K slot of tile t (two slots) or an
  // older one and the V slot of tile t-1: their last reads (K(t) Q^T and P.V of
  // tile t-1, both in MFMA(t)) every wave has completed by then.
  auto barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto sync_tile = [&](int t) {
    if (Shape::kAhead > 2 && t + 2 < n) __builtin_amdgcn_s_waitcnt(wait_vm(2 * Shape::kLoads));
    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    barrier();
    if (t + Shape::kAhead < n) issue_tile(t + Shape::kAhead);
  };

  // Prologue: tiles 0 .. Shape::kAhead-1 and this wave's Q rows in flight, then
  // everything complete (the explicit full wait also tells the compiler that
  // the Q registers are ready, so it adds no wait of its own inside the loop).
  for (int u = 0; u < Shape::kAhead && u < n; ++u) issue_tile(u);
#pragma unroll
  for (int s = 0; s < kKSteps; ++s) {
    u32x4 x = {0u, 0u, 0u, 0u};
    if (my_row < T) x = ld16(qp + (int64_t)my_row * a.q_st + 8 * h2 + 16 * s);
    qreg[s] = __builtin_bit_cast(bf16x8, x);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  barrier();

  // Tile t uses slots t % kKSlots and t % kVSlots: the loop runs kUnroll tiles
  // per pass with each slot a compile-time constant (its operand addresses are
  // then immediate offsets), the remaining tiles with the slots computed.
  // phase = t modulo kUnroll
  auto tile_step = [&](int t, int phase) {
    mfma_phase(phase % Shape::kKSlots, (phase + Shape::kUnroll - 1) % Shape::kVSlots);
    if (grp == 1) sync_tile(t);
    valu_phase(t);
    if (grp == 0) sync_tile(t);
  };
  // Tiles t0 .. t1 - 1, t0 < t1 (S(t0) first, P.V of tile t1 - 1 last).
  auto run_tiles = [&](int t0, int t1) {
    qk_part(t0 % Shape::kKSlots);
    if (grp == 1) sync_tile(t0);
    valu_phase(t0);
    if (grp == 0) sync_tile(t0);
    int t = t0 + 1;
    if (D == 64)
      for (; t < t1 && t % Shape::kUnroll != 1; ++t) tile_step(t, t % Shape::kUnroll);
    for (; t + Shape::kUnroll <= t1; t += Shape::kUnroll) {
#pragma unroll
      for (int u = 0; u < Shape::kUnroll; ++u) tile_step(t + u, (u + 1) % Shape::kUnroll);
    }
    for (; t < t1; ++t) tile_step(t, t % Shape::kUnroll);
    pv_part((t1 - 1) % Shape::kVSlots);
  };
  if constexpr (D == 128) {
    run_tiles(0, n);
  } else {
    // A wave takes part in the barriers and loads of every tile and skips the
    // products of tiles in which none of its rows sees a key, so that a V that
    // is not finite reaches only waves (32 rows) with a visible key in its tile
    // (with P = 0 for the others it would make them 0 x V = NaN).  The tiles left
    // are at most two runs: the sink's [0, head), then [band, end) from the
    // band's first visible tile to the diagonal.
    const int end = min(n, plan.n_sink_tiles + (r0 + 31) / kBN - plan.band_first + 1);
    int head = end, band = end;
    if (STREAM) {
      const int lo = max(lo_of(r0, a.chunk, a.window), 0) / kBN;  // >= band_first
      head = min(end, (a.n_sink + kBN - 1) / kBN);
      band = plan.n_sink_tiles + lo - plan.band_first;
      if (band <= head) head = end;
    }
    int t = 0;
#pragma unroll 1
    for (int seg = 0; seg < (STREAM ? 2 : 1); ++seg) {
      const int t1 = seg == 0 ? head : end;
      if (seg == 1)
        for (; t < min(band, n); ++t) sync_tile(t);
      if (t < t1) {
        run_tiles(t, t1);
        t = t1;
      }
    }
    for (; t < n; ++t) sync_tile(t);
  }
  // every wave passed the barrier of tile n-1 after its loads of the last
  // tiles completed, so the ring holds them
  if (APPEND && writer)
    for (int u = max(n - ROWS / kBN, 0); u < n; ++u) append_tile(u);

  // Epilogue: normalise by the row sum, store.
  const float l_tot = xor32_sum(l_run);
  const float inv = 1.f / l_tot;
  if (my_row < T) {
    if (OUT_F32) {
      float* op = reinterpret_cast<float*>(a.out) + ooff + (int64_t)my_row * a.o_st + (int64_t)h * a.o_sh;
#pragma unroll
      for (int mb = 0; mb < kMBlocks; ++mb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          f32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = acc_o[mb][4 * q4 + e] * inv;
          *reinterpret_cast<f32x4*>(op + 32 * mb + 8 * q4 + 4 * h2) = w;
        }
    } else {
      uint16_t* op = reinterpret_cast<uint16_t*>(a.out) + ooff + (int64_t)my_row * a.o_st + (int64_t)h * a.o_sh;
#pragma unroll
      for (int mb = 0; mb < kMBlocks; ++mb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          u32x2 w;
          w[0] = (uint32_t)f32_to_bf16_bits(acc_o[mb][4 * q4 + 0] * inv) |
                 ((uint32_t)f32_to_bf16_bits(acc_o[mb][4 * q4 + 1] * inv) << 16);
          w[1] = (uint32_t)f32_to_bf16_bits(acc_o[mb][4 * q4 + 2] * inv) |
                 ((uint32_t)f32_to_bf16_bits(acc_o[mb][4 * q4 + 3] * inv) << 16);
          *reinterpret_cast<u32x2*>(op + 32 * mb + 8 * q4 + 4 * h2) = w;
        }
    }
  }
}

// Dynamic tail of the d_head-128 launches (n_dyn > 0).  The XCDs run at different speeds
// under this load (several percent apart), and the slowest sets the end of a
// launch whose items are dealt to them in equal shares.  The first items keep
// their static XCD-aware order; the light items at the end (the streaming
// items of the one-launch form, the second half of the items of a one-type
// launch) are taken dynamically: queue x holds the items the XCD-aware order
// puts on XCD x (index w with w % 8 == x), a workgroup takes the next item of
// the queue of the XCD it runs on (read from the XCC_ID register) or, once
// that is empty, of another queue, and the launch has kStreamSlack more
// workgroups than tail items so that a fast XCD can take over a slow one's
// share.  Workgroups that find every queue empty exit.
// The queue counters live in one of kSchedSlots slots of a device array,
// chosen per launch by the host; the last workgroup to take (or fail to take)
// an item clears the slot.  Launches that run at the same time therefore
// need different slots: consecutive launches take consecutive slots.
constexpr int kSchedSlots = 64;
constexpr float kStreamSlack = 0.25f;
__device__ uint32_t g_pp_sched[kSchedSlots][16];  // [0, 8): queue heads; [8]: workgroups served

// XCD (0..7) the calling wave runs on: bits 3:0 of hardware register XCC_ID.
__device__ __forceinline__ int pp_xcc() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 7; }

// Next item for a workgroup on XCD x, or -1 when every queue is empty.
// Queue y holds ceil((n - y) / 8) items.
__device__ __forceinline__ int pp_grab(uint32_t* q, int n, int x) {
  {
    const int n_x = (n - x + 7) >> 3;
    if (n_x > 0) {
      const uint32_t k = atomicAdd(&q[x], 1u);
      if (k < (uint32_t)n_x) return 8 * (int)k + x;
    }
  }
  for (;;) {
    uint32_t head[8];
#pragma unroll
    for (int y = 0; y < 8; ++y) head[y] = __hip_atomic_load(&q[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int pick = -1;
    for (int d = 1; d < 8 && pick < 0; ++d) {
      const int y = (x + d) & 7;
      if (head[y] < (uint32_t)((n - y + 7) >> 3)) pick = y;
    }
    if (pick < 0) return -1;
    const uint32_t k = atomicAdd(&q[pick], 1u);
    if (k < (uint32_t)((n - pick + 7) >> 3)) return 8 * (int)k + pick;
  }
}

// One tail item for this workgroup (every thread gets it), or -1: n tail
// items, n_dyn workgroups of the launch take part.  The last of them to take
// (or fail to take) an item clears the slot.
__device__ __forceinline__ int pp_take(int slot, int n, int n_dyn) {
  __shared__ int s_item;
  uint32_t* q = g_pp_sched[slot];
  if (threadIdx.x == 0) {
    s_item = pp_grab(q, n, pp_xcc());
    if (atomicAdd(&q[8], 1u) == (uint32_t)n_dyn - 1) {
#pragma unroll
      for (int y = 0; y < 9; ++y) atomicExch(&q[y], 0u);
    }
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(s_item);
}

// The launches that have a dynamic tail: few large workgroups per CU.  (Its
// four bytes of LDS would also leave one workgroup a CU for 128 rows of
// d_head 128, whose rings take half of the LDS.)
template <int D, int ROWS>
constexpr bool kPPDynamic = D == 128 && ROWS == 256;

// One head type: workgroups [0, n_static) take items [0, n_static) in the
// XCD-aware order, the n_dyn others the tail items [n_static, n_static + n_tail).
template <int D, int ROWS, bool STREAM, bool OUT_F32, bool APPEND>
__global__ __launch_bounds__(2 * ROWS, (PPShape<D, ROWS>::kWavesPerSimd)) void prefill_pp_kernel(
    PrefillArgs a, int n_static, int n_tail, int n_dyn, int slot) {
  __shared__ __align__(1024) PPRing<D, ROWS> ring;
  int w = blockIdx.x;
  if constexpr (kPPDynamic<D, ROWS>) {
    if (w >= n_static) {
      w = pp_take(slot, n_tail, n_dyn);
      if (w < 0) return;
      w += n_static;
    }
  }
  prefill_pp_body<D, ROWS, STREAM, OUT_F32, APPEND>(a, w, ring);
}

// Both head types of a layer in one launch: workgroups [0, n_ret) take the
// retrieval items, [ret_pad, ret_pad + n_dyn) the n_str streaming ones
// through the queues (ret_pad = n_ret rounded up to the 8 XCDs, so both item
// spaces keep their XCD-aware order), or with n_dyn = 0 [ret_pad, ret_pad +
// n_str) take them in order.  The light streaming items are dispatched last
// and fill the CUs that the causal retrieval items leave idle at the end.
template <int D, int ROWS, bool OUT_F32, bool APPEND>
__global__ __launch_bounds__(2 * ROWS, (PPShape<D, ROWS>::kWavesPerSimd)) void prefill_pp_mixed_kernel(
    PrefillArgs ar, PrefillArgs as, int n_ret, int ret_pad, int n_str, int n_dyn, int slot) {
  __shared__ __align__(1024) PPRing<D, ROWS> ring;
  const int wg = blockIdx.x;
  if (wg < n_ret) {
    prefill_pp_body<D, ROWS, false, OUT_F32, APPEND>(ar, wg, ring);
    return;
  }
  if (wg < ret_pad) return;
  int w = wg - ret_pad;
  if constexpr (kPPDynamic<D, ROWS>) w = pp_take(slot, n_str, n_dyn);
  if (w >= 0) prefill_pp_body<D, ROWS, true, OUT_F32, APPEND>(as, w, ring);
}

static std::atomic<uint32_t> g_sched_next{0};
static int pp_slot() { return (int)(g_sched_next.fetch_add(1, std::memory_order_relaxed) % kSchedSlots); }
// Workgroups that take part in a dynamic tail of n items.
static int pp_n_dyn(int n) { return (int)((1.f + kStreamSlack) * n / 8 + 1) * 8; }

template <int D, int ROWS, bool STREAM, bool OUT_F32>
static hipError_t launch_bf16(const PrefillArgs& a, hipStream_t s) {
  const int grid = a.n_qblocks * a.n_kv * a.gs * a.B;
  // with a dynamic tail the first half of the items (a multiple of 8) is static
  constexpr bool kDyn = kPPDynamic<D, ROWS>;
  const int n_static = kDyn ? grid / 16 * 8 : grid, n_tail = grid - n_static;
  const int n_dyn = kDyn ? pp_n_dyn(n_tail) : 0;
  const int slot = kDyn ? pp_slot() : 0;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(n_static + n_dyn), dim3(2 * ROWS), 0, s, a, n_static, n_tail, n_dyn, slot);
  };
  if (a.append) go(prefill_pp_kernel<D, ROWS, STREAM, OUT_F32, true>);
  else go(prefill_pp_kernel<D, ROWS, STREAM, OUT_F32, false>);
  return hipGetLastError();
}

template <int D, bool STREAM>
static hipError_t launch_f32(const PrefillArgs& a, hipStream_t s) {
  const int grid = a.n_qblocks * a.n_kv * a.gs * a.B;
  hipLaunchKernelGGL((prefill_f32_kernel<D, STREAM>), dim3(grid), dim3(kPrefillRowsF32), 0, s, a);
  return hipGetLastError();
}

// The mixed launch pays where the retrieval items fill only a few rounds of
// the 256 CUs (one workgroup of 256 rows per CU): their causal tail is then a
// sizeable part of the launch.  Its retrieval path is compiled together with
// the streaming one and runs ~1-2% slower per tile, so long launches keep two
// kernels: measured on the 28/4-head d_head-128 layer, 1.6% faster at 32768
// tokens (7 rounds), even at 65536, 0.5-1.7% slower from 131072 on.
constexpr int kMixedMaxRetItems = 8 * 256;

bool prefill_mixed_preferred(const PrefillArgs& ar, int dtype, int d, int rows) {
  const int64_t n_ret = (int64_t)ar.n_qblocks * ar.n_kv * ar.gs * ar.B;
  return dtype == 0 && (d == 64 || n_ret * rows <= (int64_t)kMixedMaxRetItems * 256);
}

template <int D, int ROWS>
static hipError_t launch_mixed_d(const PrefillArgs& ar, const PrefillArgs& as, int out_f32, hipStream_t s) {
  const int n_ret = ar.n_qblocks * ar.n_kv * ar.gs * ar.B;
  const int n_str = as.n_qblocks * as.n_kv * as.gs * as.B;
  const int ret_pad = (n_ret + 7) / 8 * 8;
  constexpr bool kDyn = kPPDynamic<D, ROWS>;
  const int n_dyn = kDyn ? pp_n_dyn(n_str) : 0;
  const int slot = kDyn ? pp_slot() : 0;
  const dim3 grid(ret_pad + (kDyn ? n_dyn : n_str)), blk(2 * ROWS);
  const bool app = ar.append;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, blk, 0, s, ar, as, n_ret, ret_pad, n_str, n_dyn, slot);
  };
  if (out_f32) {
    if (app) go(prefill_pp_mixed_kernel<D, ROWS, true, true>);
    else go(prefill_pp_mixed_kernel<D, ROWS, true, false>);
  } else {
    if (app) go(prefill_pp_mixed_kernel<D, ROWS, false, true>);
    else go(prefill_pp_mixed_kernel<D, ROWS, false, false>);
  }
  return hipGetLastError();
}

// Query rows per workgroup.  d_head 64: 128 rows, three workgroups a CU (its
// products are half as long next to the same softmax, so a third wave per SIMD
// pays: 32 query / 8 KV heads, half of them streaming, 4 x 4000 tokens 220 us;
// 250 with 256 rows, 259 with 384 rows of 12 waves).  d_head 128: 256 rows where
// prompts are long (a K/V tile is fetched for twice the rows: 32768 tokens 3.87
// ms, 4.15 with 128), 128 where items are few or uneven, or many of them
// streaming (whose blocks of 256 rows visit more tiles outside a row's window).
// The line is on the prompts' length, earlier where more than two thirds of the
// KV heads are retrieval; 128 / 256 rows, 32 query heads of 8 KV heads: one
// prompt of 2048 tokens, none streaming, 50 / 53 us, 6000 even, 8192 482 / 469;
// 4 x 8192, 4 streaming, 1.16 / 1.18 ms, 8 x 12000 4.86 / 4.75, 2 x 12000 even.
// 8 or more prompts whose mean is below two thirds of the longest leave more
// to balance: 16 of 512-24576 tokens 13.2 / 13.7 ms, 16 of 4100-15700, none
// streaming, 8.36 / 8.55.
int prefill_rows(int dtype, int d, int64_t n_rows, int64_t batch, int64_t longest, bool packed, int n_ret, int n_str) {
  if (dtype == 1) return kPrefillRowsF32;
  if (d == 64) return 128;
  const bool causal = 2 * n_str < n_ret;
  const int64_t even = causal ? 6144 : 8192, uneven = causal ? 10240 : 16384;
  if (!packed) return longest <= even ? 128 : 256;
  return n_rows <= batch * (batch >= 8 && 2 * longest * batch > 3 * n_rows ? uneven : even) ? 128 : 256;
}

// The blocks of a batch whose K/V exceed the 256 MB cache in front of HBM would
// fetch them from HBM again for each query block if all sequences were visited
// together: with 128 rows and one query head a KV head that is more than HBM
// gives.  The sequences are therefore visited in parts of at most kPartBytes
// (one head a group; four times that otherwise, where L2 serves the group's
// heads and short parts cost balance), rounded up to whole rounds of the XCD
// order.  (Up to 64 MB in all the cache holds them, and cutting the few blocks
// costs balance: 16 x 200 tokens 34.4 us, 32.8 together.)  32 heads of width
// 128, one a group: 16 x 4096 tokens 2.14 ms, 3.67 all together, 16 x 2048 0.62
// (1.01), 128 x 256, half of them streaming, 309 us (449); 128 MB parts 2.23
// ms, 0.65 and 430.  Two a group, 32 x 4096: 4.44 ms (5.21). 256 rows halve the
// fetches and keep the order their work queues assume.  Packed batches whose
// bound is far above the mean launch mostly empty workgroups, to which the two
// steps more are a loss (100 of 500 tokens, bound 32768, 8 KV heads of four:
// 1.64 ms, 1.55 all together) that passes the gain.
constexpr int64_t kPartBytes = 32 << 20;

int prefill_part(int rows, int d, int64_t avg_len, int64_t longest, int n_kv, int gs, int batch) {
  if (rows != 128 || n_kv < 1 || longest > avg_len * (gs == 1 ? 8 : 4)) return batch;
  const int64_t seq_bytes = std::max<int64_t>(1, avg_len * n_kv * d * 4);
  if (seq_bytes * batch <= 2 * kPartBytes) return batch;
  const int64_t fit = std::max<int64_t>(1, kPartBytes * (gs == 1 ? 1 : 4) / seq_bytes);
  const int64_t whole = 8 / std::gcd(n_kv, 8);
  return (int)std::min<int64_t>(batch, (fit + whole - 1) / whole * whole);
}

hipError_t launch_prefill_mixed(const PrefillArgs& ar, const PrefillArgs& as, int out_f32, int d, int rows,
                                hipStream_t s) {
  if (d == 64) return launch_mixed_d<64, 128>(ar, as, out_f32, s);
  return rows == 128 ? launch_mixed_d<128, 128>(ar, as, out_f32, s) : launch_mixed_d<128, 256>(ar, as, out_f32, s);
}

template <int D, int ROWS>
static hipError_t launch_one_type(const PrefillArgs& a, int out_f32, bool streaming, hipStream_t s) {
  if (out_f32) return streaming ? launch_bf16<D, ROWS, true, true>(a, s) : launch_bf16<D, ROWS, false, true>(a, s);
  return streaming ? launch_bf16<D, ROWS, true, false>(a, s) : launch_bf16<D, ROWS, false, false>(a, s);
}

hipError_t launch_prefill(const PrefillArgs& a, int dtype, int out_f32, int d, int rows, bool streaming,
                          hipStream_t s) {
  if (dtype == 1) {  // fp32
    if (d == 64) return streaming ? launch_f32<64, true>(a, s) : launch_f32<64, false>(a, s);
    return streaming ? launch_f32<128, true>(a, s) : launch_f32<128, false>(a, s);
  }
  if (d == 64) return launch_one_type<64, 128>(a, out_f32, streaming, s);
  return rows == 128 ? launch_one_type<128, 128>(a, out_f32, streaming, s)
                     : launch_one_type<128, 256>(a, out_f32, streaming, s);
}

}  // namespace aoh
