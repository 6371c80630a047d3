// KV-cache append (paper Sec. 5: retrieval heads retain every token; streaming
// heads evict all but the sink and the most recent tokens).
//
// One workgroup per (16-position page-aligned chunk, KV head, sequence).  The
// chunk is logical page start_pos/16 + blockIdx.x, clipped to the appended
// range [start, start + n_new), so the grid depends only on n_new and the
// start position is read on the device.
//   retrieval head -> paged cache: K rows copied as 16-byte vectors; V staged
//     in LDS and written dimension-major ([D][16] per page), only for the
//     positions of this append (a page may already hold earlier tokens), or,
//     for token-major V pages, copied like K.
//   streaming head -> ring: a position is written only if no later position of
//     the same append maps to its slot (p < n_sink or p >= end - window), so
//     the final state is independent of the order in which lanes write.
// All copies are bit-exact.
#include "aoh_device.h"
#include "aoh_internal.h"

namespace aoh {

// Bound: memory, and for short appends the chain start position -> (rows,
// block table) -> stores.  The rows are loaded before the block table entry is
// known.  A chunk that fills a page (or ring block) writes V through the LDS
// tile as 16-byte vectors, 8 positions of a dimension each.  4 x 4096 tokens, 8
// KV heads of width 128, half of them streaming: 17.3 us a call, 23.1 with
// 2-byte stores of V.  Several positions of a page that is not filled pass
// through the tile too, so that a dimension's 2-byte stores are contiguous (64 x
// 16 tokens at odd positions, 8 heads of width 128: 4.5 us, 6.6 without, where
// a single position is faster straight from the row: 2.5, 3.3).
template <int D, typename T>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a) {
  constexpr int kVec = 16 / sizeof(T);          // elements per 16-byte vector
  constexpr int kVecPerRow = D / kVec;
  constexpr int kItems = kPage * kVecPerRow;    // 16-byte vectors per 16-position chunk
  constexpr int kPer = (kItems + 255) / 256;    // per thread
  __shared__ __align__(16) T vtile[kPage][D + kVec];

  const int g = blockIdx.y;
  const int b = blockIdx.z;
  const int start = (a.start_pos ? a.start_pos[b] : 0) + a.start_bias;
  if (start < 0) return;  // invalid start position: write nothing
  const int end = start + a.n_new;
  const int lp = start / kPage + (int)blockIdx.x;
  const int p_lo = max(lp * kPage, start);
  const int p_hi = min(lp * kPage + kPage, end);
  if (p_lo >= p_hi) return;
  const bool streaming = (a.streaming_mask >> g) & 1ull;
  const int rank = a.rank[g];
  // ring: a later position of this append overwrites all others
  auto kept = [&](int p) { return !streaming || p < a.n_sink || p >= end - a.window; };
  if (!kept(p_lo) && !kept(p_hi - 1)) return;
  // Positions beyond the block table are skipped: a write never leaves the cache.
  if (!streaming && lp >= a.max_pages) return;

  const int tid = threadIdx.x;
  const T* kn = reinterpret_cast<const T*>(a.k_new) + (int64_t)b * a.k_sb + (int64_t)g * a.k_sh;
  const T* vn = reinterpret_cast<const T*>(a.v_new) + (int64_t)b * a.v_sb + (int64_t)g * a.v_sh;
  u32x4 kv[kPer], vv[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int it = tid + 256 * u;
    const int p = lp * kPage + it / kVecPerRow, cv = it % kVecPerRow;
    if (it < kItems && p >= p_lo && p < p_hi && kept(p)) {
      kv[u] = ld16(kn + (int64_t)(p - start) * a.k_st + cv * kVec);
      vv[u] = ld16(vn + (int64_t)(p - start) * a.v_st + cv * kVec);
    }
  }

  // The cache unit and row of position p: a page, or a ring block.
  auto slot_of = [&](int p) { return p < a.n_sink ? p : a.n_sink + (p - a.n_sink) % a.window; };
  int64_t unit0;
  bool whole = p_hi - p_lo == kPage;  // the chunk is one whole unit
  bool v_token_major = false;
  T* ck;
  T* cv_;
  if (!streaming) {
    // unmapped or invalid pages are skipped
    const int page = a.block_table[(int64_t)b * a.max_pages + lp];
    if (page < 0 || page >= a.num_pages) return;
    unit0 = (int64_t)page * a.n_ret + rank;
    ck = reinterpret_cast<T*>(a.pk);
    cv_ = reinterpret_cast<T*>(a.pv);
    v_token_major = a.v_token_major;
  } else {
    int first = 0;
    whole = whole && kItems >= 256;  // bf16 of width 64 leaves half of the threads idle there
    if (whole) {
      first = slot_of(p_lo);
      whole = kept(p_lo) && kept(p_hi - 1) && first % kPage == 0 && slot_of(p_hi - 1) == first + kPage - 1 &&
              (p_hi <= a.n_sink || p_lo >= max(a.n_sink, end - a.window));
    }
    unit0 = ((int64_t)b * a.n_str + rank) * a.ring_blocks + (whole ? first / kPage : 0);
    ck = reinterpret_cast<T*>(a.rk);
    cv_ = reinterpret_cast<T*>(a.rv);
  }

  if (v_token_major || whole || (!streaming && p_hi - p_lo > 1)) {
    T* uk = ck + unit0 * (kPage * D);
    T* uv = cv_ + unit0 * (kPage * D);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int it = tid + 256 * u;
      const int row = it / kVecPerRow, cv = it % kVecPerRow, p = lp * kPage + row;
      if (it < kItems && p >= p_lo && p < p_hi) {
        st16(uk + (int64_t)row * D + cv * kVec, kv[u]);
        if (v_token_major) st16(uv + (int64_t)row * D + cv * kVec, vv[u]);
        else *reinterpret_cast<u32x4*>(&vtile[row][cv * kVec]) = vv[u];
      }
    }
    if (v_token_major) return;  // uniform across the workgroup
    __syncthreads();
    // Dimension-major V unit: element (d, r) at uv[d * 16 + r].
    if (!whole) {  // part of a page
      for (int e = tid; e < D * kPage; e += 256) {
        const int d = e / kPage, r = e % kPage, p = lp * kPage + r;
        if (p >= p_lo && p < p_hi) uv[(int64_t)d * kPage + r] = vtile[r][d];
      }
      return;
    }
    for (int e = tid; e < D * (kPage / kVec); e += 256) {
      const int d = e / (kPage / kVec), r0 = (e % (kPage / kVec)) * kVec;
      T w[kVec];
#pragma unroll
      for (int i = 0; i < kVec; ++i) w[i] = vtile[r0 + i][d];
      u32x4 x;
      __builtin_memcpy(&x, w, 16);
      st16(uv + (int64_t)d * kPage + r0, x);
    }
  } else {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int it = tid + 256 * u;
      const int p = lp * kPage + it / kVecPerRow, cv = it % kVecPerRow;
      if (!(it < kItems && p >= p_lo && p < p_hi && kept(p))) continue;
      const int slot = streaming ? slot_of(p) : p % kPage;
      const int64_t unit = unit0 + slot / kPage;
      const int r = slot % kPage;
      T* uk = ck + unit * (kPage * D);
      T* uv = cv_ + unit * (kPage * D);
      st16(uk + (int64_t)r * D + cv * kVec, kv[u]);
      const T* ve = reinterpret_cast<const T*>(&vv[u]);
#pragma unroll
      for (int e = 0; e < kVec; ++e) uv[(int64_t)(cv * kVec + e) * kPage + r] = ve[e];
    }
  }
}

template <int D, typename T>
static hipError_t launch(const AppendArgs& a, hipStream_t s) {
  dim3 grid(a.n_chunks, a.Hkv, a.B);
  hipLaunchKernelGGL((append_kernel<D, T>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_append(const AppendArgs& a, int dtype, int d, hipStream_t s) {
  if (dtype == 1) return d == 64 ? launch<64, float>(a, s) : launch<128, float>(a, s);
  return d == 64 ? launch<64, uint16_t>(a, s) : launch<128, uint16_t>(a, s);
}

}  // namespace aoh
