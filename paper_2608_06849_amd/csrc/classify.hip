// The effective-rank head classifier (paper Sec. 4, Eqs. 2-7 and Algorithm 1;
// group-level classification of the GQA appendix) on gfx950.
//
// For query head h of KV group g the method needs the singular values of
// M_h = W_K^g^T W_Q^h, obtained from the d_head x d_head proxy
// C_h = (W_Q W_Q^T)(W_K W_K^T) (Eq. 5): sigma_k^2 = lambda_k(C_h).  C_h is not
// symmetric, so instead of a general eigensolver this path uses the congruent
// symmetric matrix B_h = L_g^T (W_Q W_Q^T) L_g, where W_K W_K^T = L_g L_g^T
// (Cholesky): B_h = L^T QQ L is similar to QQ L L^T = C_h, so it has the same
// eigenvalues, and being symmetric positive semidefinite they are computed by
// Householder tridiagonalisation and Sturm-sequence bisection (Golub and Van
// Loan, Matrix Computations, Alg. 8.3.1 and Sec. 8.4.1).
//
// Kernels, in stream order:
//   gram_kernel      per (layer, head): G = W W^T over d_model, bf16 MFMA with
//                    fp32 accumulation, for the Hq query slices and Hkv key slices;
//   chol_kernel      per (layer, group): L_g from G_K in fp64 registers;
//   tridiag_kernel   per (layer, query head): B = L^T (QQ L) on the fp64 matrix
//                    cores and its tridiagonal form;
//   spectrum_kernel  per (layer, query head): all eigenvalues of that, sigma =
//                    sqrt(max(lambda, 0)) and eff_rank = exp(-sum p log p),
//                    p = sigma / sum sigma (Eq. 4);
//   select_kernel    per layer: group means and the k lowest groups as retrieval
//                    (stable: the lower group index wins a tie).
#include <type_traits>

#include "aoh_device.h"
#include "aoh_internal.h"

namespace aoh {
namespace {

constexpr int kGramBK = 64;  // d_model columns per main-loop iteration

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 x) { return __builtin_bit_cast(bf16x8, x); }

// G = W W^T for one d x d_model slice (W row-major, row stride rs elements).
// The slice is streamed through LDS 64 columns at a time: eight lanes load the
// 128 bytes of a row, so that an instruction touches whole cache lines, two
// stages ahead of the MFMAs (28 layers of 32 heads of width 128, d_model 3584:
// 177 us, 4.6 TB/s; half rows a thread and one stage ahead took 190).  Wave w
// owns 32-row block w as the A operand and computes the 32x32 tiles (w, c) for
// c >= w; each tile is written with its transpose, so G is exactly symmetric.
// The sum over d_model is order-free, so both operands use the same k mapping
// (k = k0 + 32 * half + 8 * s + j for MFMA step s, element j).
constexpr int kGramRowPad = kGramBK + 8;  // bf16 per LDS row (bank spread)

template <int D>
__global__ __launch_bounds__(64 * (D / 32)) void gram_kernel(ClassifyArgs a) {
  constexpr int NRB = D / 32;
  __shared__ __align__(16) bf16 stage[2][D][kGramRowPad];
  const int n_heads = a.Hq + a.Hkv;
  const int u = blockIdx.x % n_heads;
  const int layer = blockIdx.x / n_heads;
  const bf16* w;
  int64_t rs;
  if (u < a.Hq) {
    w = static_cast<const bf16*>(a.wq) + layer * a.wq_sl + (int64_t)u * D * a.wq_sr;
    rs = a.wq_sr;
  } else {
    w = static_cast<const bf16*>(a.wk) + layer * a.wk_sl + (int64_t)(u - a.Hq) * D * a.wk_sr;
    rs = a.wk_sr;
  }
  const int t = threadIdx.x;
  const int wave = t >> 6;
  const int lane = t & 63;
  const int l32 = lane & 31;
  const int half = lane >> 5;
  const int lrow = t >> 3, lcol = (t & 7) * 8;  // this thread's parts of a stage: rows lrow + D / 4 * s
  const bf16* src = w + (int64_t)lrow * rs + lcol;
  const int64_t part = (int64_t)(D / 4) * rs;

  f32x16 acc[NRB];
#pragma unroll
  for (int c = 0; c < NRB; ++c) acc[c] = f32x16{};

  u32x4 ld[2][4];
  auto gload = [&](int it, u32x4 (&x)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = ld16_stream(src + it * kGramBK + s * part);
  };
  auto lstore = [&](int buf, const u32x4 (&x)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) st16(&stage[buf][lrow + D / 4 * s][lcol], x[s]);
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 xa = as_bf16x8(*reinterpret_cast<const u32x4*>(&stage[buf][32 * wave + l32][32 * half + 8 * s]));
#pragma unroll
      for (int c = 0; c < NRB; ++c)
        if (c >= wave) {
          const bf16x8 xb = as_bf16x8(*reinterpret_cast<const u32x4*>(&stage[buf][32 * c + l32][32 * half + 8 * s]));
          acc[c] = mfma32(xa, xb, acc[c]);
        }
    }
  };

  // Stage `it` sits in LDS buffer it & 1, stage it + 1 in ld[1 ^ it & 1], and
  // stage it + 2 is loaded into the registers that stage `it` left.
  const int n_it = a.d_model / kGramBK;
  gload(0, ld[0]);
  if (n_it > 1) gload(1, ld[1]);
  lstore(0, ld[0]);
  __syncthreads();
  for (int it = 0; it < n_it; it += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (it + u >= n_it) break;
      if (it + u + 2 < n_it) gload(it + u + 2, ld[u]);
      compute(u);
      if (it + u + 1 < n_it) lstore(u ^ 1, ld[u ^ 1]);
      __syncthreads();
    }
  }

  float* g = a.gram + ((int64_t)layer * n_heads + u) * D * D;
#pragma unroll
  for (int c = 0; c < NRB; ++c) {
    if (c < wave) continue;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = 32 * wave + 8 * (i / 4) + 4 * half + (i % 4);
      const int n = 32 * c + l32;
      g[(int64_t)m * D + n] = acc[c][i];
      g[(int64_t)n * D + m] = acc[c][i];
    }
  }
}

constexpr int kEigThreads = 256;
constexpr int kEigWaves = kEigThreads / kWave;

// DPP move of a double within its 16-lane row (both 32-bit halves take the
// same lane pattern; the patterns used have a source for every lane).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

// The fp64 D x D matrices of the next two kernels live in registers, cyclic
// over a grid of GR x GC threads: thread (ry, cx) holds the elements
// (GR a + ry, GC b + cx).  Per elimination step a thread then needs D / GR row
// and D / GC column entries of the published vectors (a whole row a thread
// would need D / 2 of each), and a block of finished rows or columns drops out
// of every thread's loops at once, so the updates shrink with the trailing
// matrix and stay balanced.  A step's column block is a template argument
// (phase_loop), which keeps all register indices static.
template <int KB, int NB, typename F>
__device__ __forceinline__ void phase_loop(F&& f) {
  if constexpr (KB < NB) {
    f(std::integral_constant<int, KB>{});
    phase_loop<KB + 1, NB>(f);
  }
}

// 1 / x: the hardware reciprocal (4.5e-8 relative) and two Newton steps.
__device__ __forceinline__ double rcp_f64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// Sum over 8 adjacent lanes, the same bits in each of them.
__device__ __forceinline__ double sum8(double v) {
  v += dpp_f64<0xB1>(v);          // lane ^ 1
  v += dpp_f64<0x4E>(v);          // lane ^ 2
  return v + dpp_f64<0x141>(v);   // the mirrored lane of the 8, in the other quad
}

// Right-looking Cholesky of G_K = L L^T.  Step k: the owners of row k publish
// it (by symmetry also column k), every thread scales its row entries by 1 /
// pivot and updates its elements right of and below the pivot.  An element is
// final once its column is eliminated, so column k of the lower triangle ends
// as L[:, k] * L[k][k] in the owners' registers; the scaling and the stores
// come after the last step (stores inside the loop would be drained at every
// barrier: 140 us for 112 groups of width 128 that way, 42 this way).  A pivot
// <= 0 (W_K of lower rank than d_head, up to rounding) zeroes its column, which
// keeps L L^T equal to G_K on the range of W_K.
template <int D>
__global__ __launch_bounds__(kEigThreads) void chol_kernel(ClassifyArgs a) {
  constexpr int NB = D / 16;
  __shared__ double rowbuf[2][D], pivot[D], rdiag[D];
  const int n_heads = a.Hq + a.Hkv;
  const int grp = blockIdx.x % a.Hkv;
  const int layer = blockIdx.x / a.Hkv;
  const float* g = a.gram + ((int64_t)layer * n_heads + a.Hq + grp) * D * D;
  double* out = a.chol + ((int64_t)layer * a.Hkv + grp) * D * D;
  const int t = threadIdx.x;
  const int ry = t >> 4, cx = t & 15;
  double m[NB][NB];
#pragma unroll
  for (int r = 0; r < NB; ++r)
#pragma unroll
    for (int c = 0; c < NB; ++c) m[r][c] = (double)g[(int64_t)(16 * r + ry) * D + 16 * c + cx];
  phase_loop<0, NB>([&](auto kb) {
    constexpr int KB = decltype(kb)::value;
#pragma unroll 1
    for (int kk = 0; kk < 16; ++kk) {
      double* rb = rowbuf[kk & 1];
      if (ry == kk)
#pragma unroll
        for (int c = KB; c < NB; ++c) rb[16 * c + cx] = m[KB][c];
      __syncthreads();
      const double piv = rb[16 * KB + kk];
      if (t == 0) pivot[16 * KB + kk] = piv;
      const double inv = piv > 0.0 ? rcp_f64(piv) : 0.0;
      double s[NB], x[NB];
#pragma unroll
      for (int r = KB; r < NB; ++r) {
        s[r] = rb[16 * r + ry] * inv;
        x[r] = rb[16 * r + cx];
      }
      s[KB] = ry > kk ? s[KB] : 0.0;
      x[KB] = cx > kk ? x[KB] : 0.0;
#pragma unroll
      for (int r = KB; r < NB; ++r)
#pragma unroll
        for (int c = KB; c < NB; ++c) m[r][c] = fma(-s[r], x[c], m[r][c]);
    }
  });
  __syncthreads();
  if (t < D) rdiag[t] = pivot[t] > 0.0 ? 1.0 / sqrt(pivot[t]) : 0.0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NB; ++r)
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int i = 16 * r + ry, j = 16 * c + cx;
      out[(int64_t)i * D + j] = j <= i ? m[r][c] * rdiag[j] : 0.0;
    }
}

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

// D += A B for A 16 x 4, B 4 x 16 in fp64: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; register r of the result holds row 4r + l / 16, column
// l % 16, which is the B operand of a product whose k index runs over the rows
// 4r .. 4r + 3.
__device__ __forceinline__ f64x4 mfma_f64(double x, double y, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}

// Per (layer, query head): B = L^T (QQ L) and its tridiagonal form.  The
// diagonal d[0..D) and the off-diagonal e[0..D-1) replace the head's QQ in the
// workspace, which no one else reads.
//
// Products: wave w computes column tiles of 16.  T = QQ L needs k >= the
// tile's first column only (L is lower triangular) and stays in the wave's
// registers as the B operand of L^T T, whose row tiles at or below the
// diagonal are computed (B is symmetric); chunks of 64 columns go through LDS
// to their owners.
//
// Householder tridiagonalisation (Golub and Van Loan, Alg. 8.3.1): step k
// takes x = column k below the diagonal, v = x - alpha e_1 with |alpha| = |x|,
// p = beta A v, K = beta p.v / 2, and A <- A - v p^T - (p - 2 K v) v^T on rows
// and columns k+1...  The 8 lanes of a grid row hold all of v and p over their
// columns, so every one derives alpha, beta and K itself (with the same bits);
// v and p cross LDS once each.  A grid of 32 x 8 (4 x 16 elements a thread at
// width 128) keeps the sums over a row of the grid short: D / 32 of them over
// three lane exchanges.  Bound: fp64 issue, 3 (D - k)^2 / 256 fused
// multiply-adds a thread and about 200 other instructions a step, and the
// step's serial chain (two barriers, a square root, a reciprocal); two
// workgroups a CU overlap theirs.  784 heads of width 128: 350 us with the
// products (405 on a 16 x 16 grid).
template <int D>
__global__ __launch_bounds__(kEigThreads, 2) void tridiag_kernel(ClassifyArgs a) {
  constexpr int NT = D / 16;           // 16 x 16 tiles of the products
  constexpr int JC = 64;               // columns per chunk of the products: one tile a wave
  constexpr int NJ = D / JC;
  constexpr int GR = 32, GC = 8;
  constexpr int NR = D / GR, NC = D / GC;
  __shared__ double buf[D][JC + 1];
  __shared__ double xbuf[2][D], pbuf[D], dd[D], ee[D];

  const int n_heads = a.Hq + a.Hkv;
  const int h = blockIdx.x % a.Hq;
  const int layer = blockIdx.x / a.Hq;
  const int grp = h / a.gs;
  float* qq = a.gram + ((int64_t)layer * n_heads + h) * D * D;
  const double* L = a.chol + ((int64_t)layer * a.Hkv + grp) * D * D;
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int l16 = lane & 15, lr = lane >> 4;
  const int ry = t / GC, cx = t % GC;

  double m[NR][NC];
#pragma unroll
  for (int J = 0; J < NJ; ++J) {
    const int jt = (JC / 16) * J + wave;  // this wave's column tile
    f64x4 T[NT];
#pragma unroll
    for (int I = 0; I < NT; ++I) T[I] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int k0 = 16 * jt; k0 < D; k0 += 8) {
      double y[2];
      float x[2][NT];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = k0 + 4 * u + lr;
        y[u] = L[(int64_t)k * D + 16 * jt + l16];
#pragma unroll
        for (int I = 0; I < NT; ++I) x[u][I] = qq[(int64_t)k * D + 16 * I + l16];  // QQ is exactly symmetric
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int I = 0; I < NT; ++I) T[I] = mfma_f64((double)x[u][I], y[u], T[I]);
    }
    phase_loop<0, NT>([&](auto rb) {
      constexpr int I = decltype(rb)::value;
      if (I < jt) return;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kb = I; kb < NT; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma_f64(L[(int64_t)(16 * kb + 4 * r + lr) * D + 16 * I + l16], T[kb][r], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[16 * I + 4 * r + lr][16 * wave + l16] = acc[r];
    });
    __syncthreads();
    // element (i, j) is in the chunk of the lesser of the two tile indices,
    // i's or j's; within a diagonal tile both triangles were computed
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int i = GR * r + ry, j = GC * c + cx;
        if (i / 16 >= j / 16) {
          if (j / JC == J) m[r][c] = buf[i][j % JC];
        } else {
          if (i / JC == J) m[r][c] = buf[j][i % JC];
        }
      }
    __syncthreads();
  }

  phase_loop<0, NC>([&](auto kb) {
    constexpr int KB = decltype(kb)::value;       // column block of step k
    constexpr int KR = KB * GC / GR;              // and its row block
    constexpr int NK = KB == NC - 1 ? GC - 2 : GC;  // steps 0 .. D - 3
    constexpr int KB1 = KB + 1 < NC ? KB + 1 : KB, KR1 = (KB + 1) * GC / GR < NR ? (KB + 1) * GC / GR : KR;
#pragma unroll 1
    for (int kk = 0; kk < NK; ++kk) {
      const int k = GC * KB + kk;
      double* xb = xbuf[kk & 1];
      if (cx == kk)
#pragma unroll
        for (int r = KR; r < NR; ++r) xb[GR * r + ry] = m[r][KB];
      __syncthreads();
      double vc[NC], vr[NR];
#pragma unroll
      for (int c = KB; c < NC; ++c) vc[c] = xb[GC * c + cx];
#pragma unroll
      for (int r = KR; r < NR; ++r) vr[r] = xb[GR * r + ry];
      const double x0 = xb[k + 1];
      if (t == 0) dd[k] = xb[k];
      // x beyond its first entry; entries at or left of it lie in block KB
      // (the first of the next block when k is a block's last column)
      const bool last = kk == GC - 1;
      vc[KB] = cx > kk + 1 ? vc[KB] : 0.0;
      if (KB1 != KB) vc[KB1] = last && cx == 0 ? 0.0 : vc[KB1];
      double part = 0.0;
#pragma unroll
      for (int c = KB; c < NC; ++c) part = fma(vc[c], vc[c], part);
      const double xn2 = sum8(part);
      // Entries of B are at least 1e-90 in scale (fp32 Gram matrices), so a
      // square below 1e-290 is rounding noise.
      if (xn2 < 1e-290) {
        if (t == 0) ee[k] = x0;
        continue;
      }
      // |x| = s2 * rsqrt(s2), the hardware estimate (1e-7) refined twice
      const double s2 = fma(x0, x0, xn2);
      double rs = __builtin_amdgcn_rsq(s2);
      rs = fma(rs, fma(-0.5 * s2 * rs, rs, 0.5), rs);
      rs = fma(rs, fma(-0.5 * s2 * rs, rs, 0.5), rs);
      double nx = s2 * rs;
      nx = fma(0.5 * rs, fma(-nx, nx, s2), nx);
      const double alpha = x0 > 0.0 ? -nx : nx;
      const double v0 = x0 - alpha;
      const double beta = 2.0 * rcp_f64(fma(v0, v0, xn2));
      if (t == 0) ee[k] = alpha;
      vc[KB] = cx == kk + 1 ? v0 : vc[KB];
      if (KB1 != KB) vc[KB1] = last && cx == 0 ? v0 : vc[KB1];
      const int row = ry + GR * KR;  // rows of the first block
      vr[KR] = row > k + 1 ? vr[KR] : (row == k + 1 ? v0 : 0.0);
      if (KR1 != KR) vr[KR1] = ry + GR * KR1 == k + 1 ? v0 : vr[KR1];
      double pr[NR], pc[NC];
#pragma unroll
      for (int r = KR; r < NR; ++r) {
        double q0 = 0.0, q1 = 0.0;
#pragma unroll
        for (int c = KB; c < NC; ++c) (c & 1 ? q1 : q0) = fma(m[r][c], vc[c], c & 1 ? q1 : q0);
        pr[r] = beta * sum8(q0 + q1);
      }
      if (cx == 0)
#pragma unroll
        for (int r = KR; r < NR; ++r) pbuf[GR * r + ry] = pr[r];
      __syncthreads();
      double pv = 0.0;
#pragma unroll
      for (int c = KB; c < NC; ++c) {
        pc[c] = pbuf[GC * c + cx];
        pv = fma(pc[c], vc[c], pv);
      }
      const double K2 = -beta * sum8(pv);  // -2 K
#pragma unroll
      for (int r = KR; r < NR; ++r) {
        const double w = fma(K2, vr[r], pr[r]);
#pragma unroll
        for (int c = KB; c < NC; ++c) m[r][c] = fma(-vr[r], pc[c], fma(-w, vc[c], m[r][c]));
      }
    }
  });
  if (ry == GR - 2 && cx == GC - 2) dd[D - 2] = m[NR - 1][NC - 1];
  if (ry == GR - 2 && cx == GC - 1) ee[D - 2] = m[NR - 1][NC - 1];
  if (ry == GR - 1 && cx == GC - 1) {
    dd[D - 1] = m[NR - 1][NC - 1];
    ee[D - 1] = 0.0;
  }
  __syncthreads();
  double* tri = reinterpret_cast<double*>(qq);
  if (t < D) {
    tri[t] = dd[t];
    tri[D + t] = ee[t];
  }
}

// Number of eigenvalues of the symmetric tridiagonal matrix below x: the sign
// changes of its leading principal minors p_i = (d_i - x) p_{i-1} - e_{i-1}^2
// p_{i-2}, which a step of three fp64 operations and one shift into a sign
// mask follows (the pivots p_i / p_{i-1} would need a reciprocal each).  The
// matrix is scaled to a norm in [1/2, 1) and e^2 >= 2^-120, so eight steps move
// the larger of two neighbours by less than 2^980 down and 2^13 up: both are
// rescaled by a power of two after that many.  p_i = 0 needs no care, its
// neighbours then have opposite signs.  Each p_i is exact for d and e^2 changed
// by a few ulps (Wilkinson, The Algebraic Eigenvalue Problem, 5.39-40).
// de[i] = (d_i, e_{i-1}^2).
__device__ __forceinline__ uint32_t hi32(double v) { return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32); }

template <int D>
__device__ __forceinline__ int sturm_count(const double2* de, double x) {
  double pp = 0.0, p = 1.0;
  uint32_t last = 0;
  int n = 0;
#pragma unroll 1
  for (int i0 = 0; i0 < D; i0 += 32) {
    uint32_t signs = 0;
#pragma unroll
    for (int j0 = 0; j0 < 32; j0 += 8) {
#pragma unroll
      for (int j = j0; j < j0 + 8; ++j) {
        const double2 v = de[i0 + j];
        const double q = fma(v.x - x, p, -(v.y * pp));
        pp = p;
        p = q;
        signs = __builtin_amdgcn_alignbit(signs, hi32(q), 31);
      }
      // 2^-exponent of the larger, from its exponent bits
      const uint32_t top = max(hi32(p) & 0x7ff00000u, hi32(pp) & 0x7ff00000u);
      const double sc = __builtin_bit_cast(double, (uint64_t)(0x7fe00000u - top) << 32);
      p *= sc;
      pp *= sc;
    }
    n += __builtin_popcount(signs ^ __builtin_amdgcn_alignbit(last, signs, 1));
    last = signs;
  }
  return n;
}

// Per (layer, query head): bisection on the tridiagonal matrix, sigma =
// sqrt(max(lambda, 0)) and eff_rank (Eq. 4).  One thread an eigenvalue, 256 / D
// heads a workgroup: its four wavefronts land on the four SIMDs of a CU (with
// one wavefront a workgroup several shared a SIMD: 238 us for 784 heads of
// width 128 against 189).  Bound: fp64 issue, 47 counts of D steps of four
// instructions an eigenvalue; 154 us for 784 heads of width 128.
template <int D>
__global__ __launch_bounds__(kEigThreads) void spectrum_kernel(ClassifyArgs a) {
  constexpr int NH = kEigThreads / D, NW = D / kWave;  // heads a workgroup, wavefronts a head
  __shared__ double2 de_s[NH][D];
  __shared__ double ebuf[NH][D + 1], red[2][NH][NW];
  __shared__ int cnt_s[NH][D];
  const int n_heads = a.Hq + a.Hkv;
  const int slot = threadIdx.x / D, t = threadIdx.x % D;
  const bool live = blockIdx.x * NH + slot < a.L * a.Hq;
  const int item = live ? blockIdx.x * NH + slot : a.L * a.Hq - 1;
  const int h = item % a.Hq;
  const int layer = item / a.Hq;
  const double* tri = reinterpret_cast<const double*>(a.gram + ((int64_t)layer * n_heads + h) * D * D);
  const int wave = t >> 6, lane = t & 63;
  double2* de = de_s[slot];
  int* cnt = cnt_s[slot];
  const double d = tri[t], e = tri[D + t];  // e[D - 1] = 0
  ebuf[slot][t + 1] = e;
  if (t == 0) ebuf[slot][0] = 0.0;
  __syncthreads();
  const double e_prev = ebuf[slot][t];

  // Gershgorin interval of the whole matrix
  const double rad = fabs(e_prev) + fabs(e);
  double lo = d - rad, hi = d + rad;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, kWave));
    hi = fmax(hi, __shfl_xor(hi, o, kWave));
  }
  if (lane == 0) {
    red[0][slot][wave] = lo;
    red[1][slot][wave] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    lo = fmin(lo, red[0][slot][w]);
    hi = fmax(hi, red[1][slot][w]);
  }
  // Scaled by a power of two to a norm in [1/2, 1): exact, and p = sigma /
  // sum(sigma) does not see it.
  const double norm = fmax(fabs(lo), fabs(hi));
  const int ex = -__builtin_amdgcn_frexp_exp(norm);
  const double es = __builtin_amdgcn_ldexp(e_prev, ex);
  de[t] = double2{__builtin_amdgcn_ldexp(d, ex), fmax(es * es, 0x1p-120)};
  const double tnorm = __builtin_amdgcn_ldexp(norm, ex);
  const double atol = 2.220446049250313e-16 * tnorm;
  const double l0 = __builtin_amdgcn_ldexp(lo, ex) - 2.0 * atol;
  const double h0 = __builtin_amdgcn_ldexp(hi, ex) + 2.0 * atol;
  __syncthreads();

  // Eigenvalue t (ascending) is bracketed by count(blo) <= t < count(bhi).
  // First the D threads count at D interior points for all of them, then each
  // halves its own interval until the width is below atol; every eigenvalue
  // takes the same number of rounds.
  const double step = (h0 - l0) / (D + 1);
  cnt[t] = sturm_count<D>(de, l0 + step * (t + 1));
  __syncthreads();
  int below = 0, above = D + 1;  // interior points 1 .. D; counts <= t at `below`, > t at `above`
  while (above - below > 1) {
    const int mid = (above + below) / 2;
    if (cnt[mid - 1] <= t) below = mid;
    else above = mid;
  }
  double blo = below > 0 ? l0 + step * below : l0;
  double bhi = above <= D ? l0 + step * above : h0;
  double w = step;
  for (int it = 0; it < 64 && w > atol; ++it, w *= 0.5) {
    const double mid = 0.5 * (blo + bhi);
    if (sturm_count<D>(de, mid) <= t) blo = mid;
    else bhi = mid;
  }

  // eigenvalues at or below the rounding floor of the reduction are zero
  // (a rank-deficient W_Q or W_K leaves only such values), so they add no
  // term to the entropy; for the zero matrix every eigenvalue is zero
  const double lam = 0.5 * (blo + bhi);
  const double sigma = (tnorm > 0.0 && lam > D * atol) ? sqrt(lam) : 0.0;

  // eff_rank = exp(-sum p log p), p = sigma / sum sigma over sigma > 0
  double s = wave_sum_f64(sigma);
  if (lane == 0) red[0][slot][wave] = s;
  __syncthreads();
  double ssum = 0.0;
#pragma unroll
  for (int w2 = 0; w2 < NW; ++w2) ssum += red[0][slot][w2];
  double term = 0.0;
  if (sigma > 0.0 && ssum > 0.0) {
    const double p = sigma / ssum;
    term = p * log(p);
  }
  s = wave_sum_f64(term);
  if (lane == 0) red[1][slot][wave] = s;
  __syncthreads();
  if (t == 0 && live) {
    double hsum = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) hsum += red[1][slot][w2];
    a.head_rank[(int64_t)layer * a.Hq + h] = exp(-hsum);
  }
}

// Group score = mean eff_rank of the group's query heads; the n_retrieval
// lowest scores are retrieval groups (0), the rest streaming (1).
__global__ __launch_bounds__(kWave) void select_kernel(ClassifyArgs a) {
  __shared__ double sc[kMaxKvHeads];
  const int layer = blockIdx.x;
  const int g = threadIdx.x;
  double s = 0.0;
  if (g < a.Hkv) {
    const double* hr = a.head_rank + (int64_t)layer * a.Hq + g * a.gs;
    for (int j = 0; j < a.gs; ++j) s += hr[j];
    s /= a.gs;
    sc[g] = s;
  }
  __syncthreads();
  if (g < a.Hkv) {
    int rank = 0;
    for (int o = 0; o < a.Hkv; ++o) rank += (sc[o] < s) || (sc[o] == s && o < g);
    a.group_score[(int64_t)layer * a.Hkv + g] = s;
    a.head_is_streaming[(int64_t)layer * a.Hkv + g] = rank >= a.n_retrieval ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------
// Cross-layer head similarity of H2Share (Eq. sim, by the trace identities of
// the trace-reduction appendix): for anchor layer l and reuse layer l',
//   <M_h, M_h'>_F = tr(W_Q^h W_Q'^h'^T . W_K'^g' W_K^g^T)
//                 = sum_ab (W_Q^h W_Q'^h'^T)[a][b] (W_K^g W_K'^g'^T)[a][b],
//   |M_h|_F^2     = sum_ab (W_Q W_Q^T)[a][b] (W_K W_K^T)[a][b]  (symmetric Grams).

// C = A B^T for a d x d_model slice A of one weight and a slice B of another
// (bf16 MFMA, fp32 accumulation), the slab of 64 columns of both staged in
// LDS.  Wave w computes the 32-row block w against all column blocks.
// STORE: C goes to kx[(g * Hkv + g') * D * D]; otherwise the tile is multiplied
// elementwise with kx of the heads' groups and summed into num[h][h'].
template <int D, bool STORE>
__global__ __launch_bounds__(64 * (D / 32)) void cross_kernel(SimilarityArgs a) {
  constexpr int NRB = D / 32;
  __shared__ __align__(16) bf16 stage[2][2][D][kGramRowPad];
  __shared__ double red[NRB];
  const int n = STORE ? a.Hkv : a.Hq;
  const int u = blockIdx.x / n, v = blockIdx.x % n;  // (anchor unit, reuse unit)
  const bf16* wa = STORE ? static_cast<const bf16*>(a.wk_a) + (int64_t)u * D * a.wk_a_sr
                         : static_cast<const bf16*>(a.wq_a) + (int64_t)u * D * a.wq_a_sr;
  const bf16* wb = STORE ? static_cast<const bf16*>(a.wk_r) + (int64_t)v * D * a.wk_r_sr
                         : static_cast<const bf16*>(a.wq_r) + (int64_t)v * D * a.wq_r_sr;
  const int64_t rsa = STORE ? a.wk_a_sr : a.wq_a_sr, rsb = STORE ? a.wk_r_sr : a.wq_r_sr;
  const int t = threadIdx.x;
  const int wave = t >> 6, lane = t & 63, l32 = lane & 31, half = lane >> 5;
  const int lrow = t >> 1, lcol = (t & 1) * 32;
  const bf16* srca = wa + (int64_t)lrow * rsa + lcol;
  const bf16* srcb = wb + (int64_t)lrow * rsb + lcol;

  f32x16 acc[NRB];
#pragma unroll
  for (int c = 0; c < NRB; ++c) acc[c] = f32x16{};
  u32x4 la[4], lb[4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      la[s2] = ld16(srca + k0 + 8 * s2);
      lb[s2] = ld16(srcb + k0 + 8 * s2);
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      st16(&stage[buf][0][lrow][lcol + 8 * s2], la[s2]);
      st16(&stage[buf][1][lrow][lcol + 8 * s2], lb[s2]);
    }
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      const bf16x8 xa = as_bf16x8(*reinterpret_cast<const u32x4*>(&stage[buf][0][32 * wave + l32][32 * half + 8 * s2]));
#pragma unroll
      for (int c = 0; c < NRB; ++c) {
        const bf16x8 xb = as_bf16x8(*reinterpret_cast<const u32x4*>(&stage[buf][1][32 * c + l32][32 * half + 8 * s2]));
        acc[c] = mfma32(xa, xb, acc[c]);
      }
    }
  };
  gload(0);
  lstore(0);
  __syncthreads();
  const int n_it = a.d_model / kGramBK;
  for (int it = 0; it < n_it; ++it) {
    const int cur = it & 1;
    const bool more = it + 1 < n_it;
    if (more) gload((it + 1) * kGramBK);
    compute(cur);
    if (more) lstore(cur ^ 1);
    __syncthreads();
  }

  if (STORE) {
    float* out = a.kx + (int64_t)(u * a.Hkv + v) * D * D;
#pragma unroll
    for (int c = 0; c < NRB; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = 32 * wave + 8 * (i / 4) + 4 * half + (i % 4);
        out[(int64_t)m * D + 32 * c + l32] = acc[c][i];
      }
  } else {
    const float* kx = a.kx + (int64_t)((u / a.gs) * a.Hkv + v / a.gs) * D * D;
    double sum = 0.0;
#pragma unroll
    for (int c = 0; c < NRB; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = 32 * wave + 8 * (i / 4) + 4 * half + (i % 4);
        sum += (double)acc[c][i] * (double)kx[(int64_t)m * D + 32 * c + l32];
      }
    sum = wave_sum_f64(sum);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (t == 0) {
      double tot = 0.0;
#pragma unroll
      for (int w = 0; w < NRB; ++w) tot += red[w];
      a.num[(int64_t)u * a.Hq + v] = tot;
    }
  }
}

// |M_h|_F^2 of every query head of both layers from the Grams:
// blockIdx.x = layer * Hq + h.
template <int D>
__global__ __launch_bounds__(kEigThreads) void norm_kernel(SimilarityArgs a) {
  __shared__ double red[kEigWaves];
  const int layer = blockIdx.x / a.Hq, h = blockIdx.x % a.Hq;
  const int n_heads = a.Hq + a.Hkv;
  const float* qq = a.gram + ((int64_t)layer * n_heads + h) * D * D;
  const float* kk = a.gram + ((int64_t)layer * n_heads + a.Hq + h / a.gs) * D * D;
  double sum = 0.0;
  for (int e = threadIdx.x; e < D * D; e += kEigThreads) sum += (double)qq[e] * (double)kk[e];
  sum = wave_sum_f64(sum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < kEigWaves; ++w) tot += red[w];
    a.n2[blockIdx.x] = tot;
  }
}

// Normalisation, group means and the mapping (one workgroup).
__global__ __launch_bounds__(kEigThreads) void mapping_kernel(SimilarityArgs a) {
  const int hq = a.Hq, hkv = a.Hkv, gs = a.gs;
  const double* n2 = a.n2;  // [2][Hq] squared norms
  for (int e = threadIdx.x; e < hq * hq; e += kEigThreads) {
    const int h = e / hq, h2 = e % hq;
    a.head_sim[e] = a.num[e] / (sqrt(n2[h]) * sqrt(n2[hq + h2]));
  }
  __syncthreads();
  for (int e = threadIdx.x; e < hkv * hkv; e += kEigThreads) {
    const int g = e / hkv, g2 = e % hkv;
    double sum = 0.0;
    for (int i = 0; i < gs; ++i)
      for (int j = 0; j < gs; ++j) sum += a.head_sim[(int64_t)(g * gs + i) * hq + g2 * gs + j];
    a.group_sim[e] = sum / (gs * gs);
  }
  __syncthreads();
  const int g2 = threadIdx.x;
  if (g2 < hkv) {
    int best = -1, rank = -1, r = 0;
    if (!((a.reuse_streaming >> g2) & 1ull)) {
      for (int g = 0; g < hkv; ++g) {
        if ((a.anchor_streaming >> g) & 1ull) continue;
        if (best < 0 || a.group_sim[g * hkv + g2] > a.group_sim[best * hkv + g2]) {
          best = g;
          rank = r;
        }
        ++r;
      }
    }
    a.mapping[g2] = rank;
  }
}

template <int D>
hipError_t launch_similarity_d(const SimilarityArgs& a, hipStream_t s) {
  // Grams of both layers (the classifier's kernel, one layer each)
  for (int layer = 0; layer < 2; ++layer) {
    ClassifyArgs c;
    __builtin_memset(&c, 0, sizeof(c));
    c.wq = layer ? a.wq_r : a.wq_a;
    c.wk = layer ? a.wk_r : a.wk_a;
    c.wq_sr = layer ? a.wq_r_sr : a.wq_a_sr;
    c.wk_sr = layer ? a.wk_r_sr : a.wk_a_sr;
    c.L = 1; c.Hq = a.Hq; c.Hkv = a.Hkv; c.gs = a.gs; c.d_model = a.d_model;
    c.gram = a.gram + (int64_t)layer * (a.Hq + a.Hkv) * D * D;
    hipLaunchKernelGGL(gram_kernel<D>, dim3(a.Hq + a.Hkv), dim3(64 * (D / 32)), 0, s, c);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((cross_kernel<D, true>), dim3(a.Hkv * a.Hkv), dim3(64 * (D / 32)), 0, s, a);
  hipLaunchKernelGGL((cross_kernel<D, false>), dim3(a.Hq * a.Hq), dim3(64 * (D / 32)), 0, s, a);
  hipLaunchKernelGGL(norm_kernel<D>, dim3(2 * a.Hq), dim3(kEigThreads), 0, s, a);
  hipLaunchKernelGGL(mapping_kernel, dim3(1), dim3(kEigThreads), 0, s, a);
  return hipGetLastError();
}

template <int D>
hipError_t launch_classify_d(const ClassifyArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(gram_kernel<D>, dim3(a.L * (a.Hq + a.Hkv)), dim3(64 * (D / 32)), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chol_kernel<D>, dim3(a.L * a.Hkv), dim3(kEigThreads), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(tridiag_kernel<D>, dim3(a.L * a.Hq), dim3(kEigThreads), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  constexpr int kHeads = kEigThreads / D;  // heads a workgroup
  hipLaunchKernelGGL(spectrum_kernel<D>, dim3((a.L * a.Hq + kHeads - 1) / kHeads), dim3(kEigThreads), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(select_kernel, dim3(a.L), dim3(kWave), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_classify(const ClassifyArgs& a, int d, hipStream_t s) {
  return d == 128 ? launch_classify_d<128>(a, s) : launch_classify_d<64>(a, s);
}

hipError_t launch_similarity(const SimilarityArgs& a, int d, hipStream_t s) {
  return d == 128 ? launch_similarity_d<128>(a, s) : launch_similarity_d<64>(a, s);
}

}  // namespace aoh
