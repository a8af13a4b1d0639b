// Complex FP64 GEMMs of the KB projectors and of P_c = 1 - Psi Psi^H on the
// gfx950 FP64 matrix cores (v_mfma_f64_16x16x4f64).
//
// A complex product is split into real MFMAs without any cross-lane traffic:
// each lane loads two consecutive complex elements (32 bytes) of its row and
// feeds their four real parts to four successive MFMAs, so the four lane
// groups of a wavefront cover eight complex k per MFMA quadruple. Because the
// k order inside a reduction is free, the A and B fragments only have to agree
// on which k each lane group carries.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kernels.hpp"
#include "stern.h"

namespace stern {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kGemmThreads = 256;  // 4 waves, 2 x 2 arrangement of 32 x 32 wave tiles

// C[n][m] (partial over the K range of this split) = sum_k conj(A[m][k]) X[xidx[n]][k]
// for one operand, or two with rows X of their own (blocks of 64 rows m from mb0 on belong to the second)
__global__ __launch_bounds__(kGemmThreads) void k_zgemm_reduce(ZRows s0, ZRows s1, int mb0, int ldx,
                                                               const int* __restrict__ xidx, int ncols, int K,
                                                               int kchunk) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const bool second = (int)blockIdx.x >= mb0;
  const Z64* __restrict__ A = second ? s1.A : s0.A;
  const Z64* __restrict__ X = second ? s1.X : s0.X;
  Z64* __restrict__ cpart = second ? s1.part : s0.part;
  const int M_pad = second ? s1.M_pad : s0.M_pad, M = second ? s1.M : s0.M;
  const int m0 = ((int)blockIdx.x - (second ? mb0 : 0)) * 64 + (wave & 1) * 32;
  const int n0 = blockIdx.y * 64 + (wave >> 1) * 32;
  if (m0 >= M || n0 >= ncols) return;  // padding only (no barrier, no LDS)
  const int split = blockIdx.z;
  const int kb = split * kchunk;
  const int ke = min(K, kb + kchunk);
  const Z64* ar[2];
  const Z64* xr[2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi) ar[bi] = A + (size_t)(m0 + 16 * bi + l16) * K;
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    const int n = n0 + 16 * bj + l16;
    const int row = n < ncols ? (xidx ? xidx[n] : n) : (xidx ? xidx[0] : 0);
    xr[bj] = X + (size_t)row * ldx;
  }
  v4d cre[2][2], cim[2][2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      cre[bi][bj] = v4d{0.0, 0.0, 0.0, 0.0};
      cim[bi][bj] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  // The next step's fragments are loaded before this step's products (every load unconditional:
  // columns past ncols read row 0, whose products are never stored), so they arrive while the
  // products of this step run. A last block of 16 columns or fewer runs half the products.
  Z64 na0[2], na1[2], nx0[2], nx1[2];
  auto steps = [&](auto nb) {
    constexpr int NB = decltype(nb)::value;
    auto load = [&](int kc) {
      const int k = kc + 2 * g;
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) {
        na0[bi] = ar[bi][k];
        na1[bi] = ar[bi][k + 1];
      }
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        nx0[bj] = xr[bj][k];
        nx1[bj] = xr[bj][k + 1];
      }
    };
    if (kb < ke) load(kb);
    for (int kc = kb; kc < ke; kc += 8) {
      Z64 a0[2], a1[2], x0[2], x1[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a0[u] = na0[u];
        a1[u] = na1[u];
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        x0[u] = nx0[u];
        x1[u] = nx1[u];
      }
      load(min(kc + 8, ke - 8));  // the last step reloads itself, unused
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
          // Re conj(a) x = a.re x.re + a.im x.im ; Im conj(a) x = a.re x.im - a.im x.re
          cre[bi][bj] = mfma(a0[bi].re, x0[bj].re, cre[bi][bj]);
          cre[bi][bj] = mfma(a0[bi].im, x0[bj].im, cre[bi][bj]);
          cre[bi][bj] = mfma(a1[bi].re, x1[bj].re, cre[bi][bj]);
          cre[bi][bj] = mfma(a1[bi].im, x1[bj].im, cre[bi][bj]);
          cim[bi][bj] = mfma(a0[bi].re, x0[bj].im, cim[bi][bj]);
          cim[bi][bj] = mfma(a0[bi].im, -x0[bj].re, cim[bi][bj]);
          cim[bi][bj] = mfma(a1[bi].re, x1[bj].im, cim[bi][bj]);
          cim[bi][bj] = mfma(a1[bi].im, -x1[bj].re, cim[bi][bj]);
        }
    }
  };
  if (n0 + 16 < ncols)
    steps(std::integral_constant<int, 2>{});
  else
    steps(std::integral_constant<int, 1>{});
  // D[i][j] of a 16x16 block: column j = lane % 16, row i = lane / 16 + 4 r in accumulator element r
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    const int n = n0 + 16 * bj + l16;
    if (n >= ncols) continue;
    Z64* dst = cpart + ((size_t)split * ncols + n) * M_pad;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
#pragma unroll
      for (int r = 0; r < 4; ++r) dst[m0 + 16 * bi + g + 4 * r] = zmk(cre[bi][bj][r], cim[bi][bj][r]);
    }
  }
}

// The reduce for few columns (the convergence tail, single rows, small cells): a wave takes 16 rows and
// 16 BJ columns, so that 16 BJ columns cost the matrix cores what they hold and not the 64 of the tile
// above, and K is split much finer, as one wave's chain over a long chunk is what such a reduce waits for
// (64 cycles a product, 8 BJ products and one load latency a step). The loads of a step are issued two
// steps ahead. M = 16 (64 with padding), up to 16 columns, K = 576: 48 -> 5.6 us; M = 128, up to 16 columns,
// K = 16,896: 48 -> 11.4 us, both averages over a solve.
template <int BJ>
__global__ __launch_bounds__(kGemmThreads) void k_zgemm_reduce_cols(ZRows s0, ZRows s1, int mb0, int ldx,
                                                                    const int* __restrict__ xidx, int ncols, int K,
                                                                    int kchunk) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const bool second = (int)blockIdx.x >= mb0;
  const Z64* __restrict__ A = second ? s1.A : s0.A;
  const Z64* __restrict__ X = second ? s1.X : s0.X;
  Z64* __restrict__ cpart = second ? s1.part : s0.part;
  const int M_pad = second ? s1.M_pad : s0.M_pad, M = second ? s1.M : s0.M;
  const int m0 = ((int)blockIdx.x - (second ? mb0 : 0)) * 64 + wave * 16;
  const int split = blockIdx.z;
  const int kb = split * kchunk, ke = min(K, kb + kchunk);  // a multiple of 16 apart
  if (m0 >= M) return;  // padding only (no barrier, no LDS)
  const Z64* ar = A + (size_t)(m0 + l16) * K + 2 * g;
  const Z64* xr[BJ];
#pragma unroll
  for (int bj = 0; bj < BJ; ++bj) {
    const int n = min(16 * bj + l16, ncols - 1);  // columns past ncols repeat the last one and are not stored
    xr[bj] = X + (size_t)(xidx ? xidx[n] : n) * ldx + 2 * g;
  }
  v4d cre[BJ], cim[BJ];
#pragma unroll
  for (int bj = 0; bj < BJ; ++bj) cre[bj] = cim[bj] = v4d{0.0, 0.0, 0.0, 0.0};
  Z64 a[2][2], x[2][BJ][2];
  auto load = [&](int b, int k) {
    a[b][0] = ar[k];
    a[b][1] = ar[k + 1];
#pragma unroll
    for (int bj = 0; bj < BJ; ++bj) {
      x[b][bj][0] = xr[bj][k];
      x[b][bj][1] = xr[bj][k + 1];
    }
  };
  if (kb < ke) {
    load(0, kb);
    load(1, kb + 8);
  }
  for (int kc = kb; kc < ke; kc += 16) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const Z64 a0 = a[b][0], a1 = a[b][1];
      Z64 x0[BJ], x1[BJ];
#pragma unroll
      for (int bj = 0; bj < BJ; ++bj) {
        x0[bj] = x[b][bj][0];
        x1[bj] = x[b][bj][1];
      }
      load(b, min(kc + 16, ke - 16) + 8 * b);  // the last round reloads itself, unused
#pragma unroll
      for (int bj = 0; bj < BJ; ++bj) {
        cre[bj] = mfma(a0.re, x0[bj].re, cre[bj]);
        cim[bj] = mfma(a0.re, x0[bj].im, cim[bj]);
        cre[bj] = mfma(a0.im, x0[bj].im, cre[bj]);
        cim[bj] = mfma(a0.im, -x0[bj].re, cim[bj]);
        cre[bj] = mfma(a1.re, x1[bj].re, cre[bj]);
        cim[bj] = mfma(a1.re, x1[bj].im, cim[bj]);
        cre[bj] = mfma(a1.im, x1[bj].im, cre[bj]);
        cim[bj] = mfma(a1.im, -x1[bj].re, cim[bj]);
      }
    }
  }
#pragma unroll
  for (int bj = 0; bj < BJ; ++bj) {
    const int n = 16 * bj + l16;
    if (n >= ncols) continue;
    Z64* dst = cpart + ((size_t)split * ncols + n) * M_pad + m0 + g;
#pragma unroll
    for (int r = 0; r < 4; ++r) dst[4 * r] = zmk(cre[bj][r], cim[bj][r]);
  }
}

// C[n][m] = scale * sum over the splits, m < M. P threads to an output (1, or 8 where there are at least as
// many splits, so that a few outputs of many splits are still read by many threads): each sums every P-th
// split and the parts are added in order. M = 128 at K = 16,896, average over an FP64 solve:
// 18 -> 10 us.
template <int P>
__global__ __launch_bounds__(256) void k_sum_parts(ZRows s0, ZRows s1, int nb0, int nsplit, int ncols) {
  constexpr int O = 256 / P;  // outputs per workgroup; workgroups from nb0 on belong to the second operand
  __shared__ Z64 part[P > 1 ? P : 1][P > 1 ? O : 1];
  const bool second = (int)blockIdx.x >= nb0;
  const Z64* __restrict__ cpart = second ? s1.part : s0.part;
  Z64* __restrict__ C = second ? s1.C : s0.C;
  const int M_pad = second ? s1.M_pad : s0.M_pad, M = ((second ? s1.M : s0.M) + 7) / 8 * 8;
  const double scale = second ? s1.scale : s0.scale;
  const int o = threadIdx.x % O, q = threadIdx.x / O;
  const int i = ((int)blockIdx.x - (second ? nb0 : 0)) * O + o;
  const bool live = i < ncols * M;
  const size_t at = live ? (size_t)(i / M) * M_pad + i % M : 0, total = (size_t)ncols * M_pad;
  double re = 0.0, im = 0.0;
  if (live)
    for (int s = q; s < nsplit; s += P) {
      const Z64 v = cpart[s * total + at];
      re += v.re;
      im += v.im;
    }
  if constexpr (P > 1) {
    part[q][o] = zmk(re, im);
    __syncthreads();
    if (q != 0) return;
#pragma unroll
    for (int p = 1; p < P; ++p) {
      re += part[p][o].re;
      im += part[p][o].im;
    }
  }
  if (live) C[at] = zmk(scale * re, scale * im);
}

// Y[yidx[n]][k] += sum_m A[m][k] C[n][m], over the rows of one operand or of two. PUPD: Y is left as it is and the
// sum goes into the search direction, P[s] = (Y[s] + A C) + beta[s] P[s] (s = yidx[n]). Bounded to 4 waves per
// SIMD: the compiler then keeps the accumulators in VGPRs instead of 104 VGPRs + 64 AGPRs at 3 waves; 59 -> 70
// TFLOP/s at M = 1,024, 4,096 columns, K = 91,072.
__device__ __forceinline__ void put_row(Z64* y, Z64* p, double b, double re, double im) {
  const Z64 old = *y, t = zmk(old.re + re, old.im + im);
  if (p) {
    const Z64 q = *p;
    *p = zmk(t.re + b * q.re, t.im + b * q.im);
  } else {
    *y = t;
  }
}
template <bool PUPD>
__global__ __launch_bounds__(kGemmThreads, 4) void k_zgemm_expand(ZRows s0, ZRows s1, int K, Z64* __restrict__ Y,
                                                               int ldy, const int* __restrict__ yidx, int ncols,
                                                               Z64* __restrict__ P, const double* __restrict__ beta) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const int k0 = blockIdx.x * 64 + (wave & 1) * 32;
  const int n0 = blockIdx.y * 64 + (wave >> 1) * 32;
  if (n0 >= ncols) return;  // padding only (no barrier, no LDS)
  int nn[2];
  bool nv[2];
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    nn[bj] = n0 + 16 * bj + l16;
    nv[bj] = nn[bj] < ncols;
  }
  v4d dre[2][2], dim_[2][2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      dre[bi][bj] = v4d{0.0, 0.0, 0.0, 0.0};
      dim_[bi][bj] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  // next step's fragments loaded before this step's products; columns past ncols read column 0; a last block
  // of 16 columns or fewer runs half the products
  Z64 na0[2], na1[2], nc0[2], nc1[2];
  auto steps = [&](auto nb) {
    constexpr int NB = decltype(nb)::value;
    for (int seg = 0; seg < 2; ++seg) {
      const Z64* __restrict__ A = seg ? s1.A : s0.A;
      const Z64* __restrict__ C = seg ? s1.C : s0.C;
      const int M_pad = seg ? s1.M_pad : s0.M_pad, M = ((seg ? s1.M : s0.M) + 7) / 8 * 8;
      if (M == 0) continue;
      auto load = [&](int m) {
        const int mm = m + 2 * g;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi) {
          const int kk = k0 + 16 * bi + l16;
          na0[bi] = A[(size_t)mm * K + kk];
          na1[bi] = A[(size_t)(mm + 1) * K + kk];
        }
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
          const size_t o = (size_t)(nv[bj] ? nn[bj] : 0) * M_pad + mm;
          nc0[bj] = C[o];
          nc1[bj] = C[o + 1];
        }
      };
      load(0);
      for (int m = 0; m < M; m += 8) {
        Z64 a0[2], a1[2], c0[2], c1[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          a0[u] = na0[u];
          a1[u] = na1[u];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          c0[u] = nc0[u];
          c1[u] = nc1[u];
        }
        load(min(m + 8, M - 8));  // the last step reloads itself, unused
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
          for (int bj = 0; bj < NB; ++bj) {
            // Re a c = a.re c.re - a.im c.im ; Im a c = a.re c.im + a.im c.re
            dre[bi][bj] = mfma(a0[bi].re, c0[bj].re, dre[bi][bj]);
            dre[bi][bj] = mfma(a0[bi].im, -c0[bj].im, dre[bi][bj]);
            dre[bi][bj] = mfma(a1[bi].re, c1[bj].re, dre[bi][bj]);
            dre[bi][bj] = mfma(a1[bi].im, -c1[bj].im, dre[bi][bj]);
            dim_[bi][bj] = mfma(a0[bi].re, c0[bj].im, dim_[bi][bj]);
            dim_[bi][bj] = mfma(a0[bi].im, c0[bj].re, dim_[bi][bj]);
            dim_[bi][bj] = mfma(a1[bi].re, c1[bj].im, dim_[bi][bj]);
            dim_[bi][bj] = mfma(a1[bi].im, c1[bj].re, dim_[bi][bj]);
          }
      }
    }
  };
  if (n0 + 16 < ncols)
    steps(std::integral_constant<int, 2>{});
  else
    steps(std::integral_constant<int, 1>{});
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    if (!nv[bj]) continue;
    const int row = yidx ? yidx[nn[bj]] : nn[bj];
    Z64* y = Y + (size_t)row * ldy;
    const double bt = PUPD ? beta[row] : 0.0;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + 16 * bi + g + 4 * r;
        put_row(y + k, PUPD ? P + (size_t)row * ldy + k : nullptr, bt, dre[bi][bj][r], dim_[bi][bj][r]);
      }
    }
  }
}

// The expand for few columns: a wave takes 16 k and 16 BJ columns (see k_zgemm_reduce_cols), the loads of a
// step two steps ahead. Up to 16 columns, averages over a solve: M = 16, K = 576: 12 -> 4.3 us;
// M = 128, K = 16,896: 43 -> 15 us.
template <int BJ, bool PUPD>
__global__ __launch_bounds__(kGemmThreads) void k_zgemm_expand_cols(ZRows s0, ZRows s1, int K, Z64* __restrict__ Y,
                                                                    int ldy, const int* __restrict__ yidx, int ncols,
                                                                    Z64* __restrict__ P,
                                                                    const double* __restrict__ beta) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const int k0 = blockIdx.x * 64 + wave * 16;
  v4d dre[BJ], dim_[BJ];
#pragma unroll
  for (int bj = 0; bj < BJ; ++bj) dre[bj] = dim_[bj] = v4d{0.0, 0.0, 0.0, 0.0};
  Z64 a[2][2], c[2][BJ][2];
  for (int seg = 0; seg < 2; ++seg) {
    const int M_pad = seg ? s1.M_pad : s0.M_pad, M = ((seg ? s1.M : s0.M) + 7) / 8 * 8;
    if (M == 0) continue;
    const Z64* __restrict__ ar = (seg ? s1.A : s0.A) + (size_t)(2 * g) * K + k0 + l16;
    const Z64* __restrict__ C = seg ? s1.C : s0.C;
    const Z64* cr[BJ];
#pragma unroll
    for (int bj = 0; bj < BJ; ++bj) cr[bj] = C + (size_t)min(16 * bj + l16, ncols - 1) * M_pad + 2 * g;
    auto load = [&](int b, int m) {
      const int mm = min(m, M - 8);  // steps past the end read the last one, unused
      a[b][0] = ar[(size_t)mm * K];
      a[b][1] = ar[(size_t)(mm + 1) * K];
#pragma unroll
      for (int bj = 0; bj < BJ; ++bj) {
        c[b][bj][0] = cr[bj][mm];
        c[b][bj][1] = cr[bj][mm + 1];
      }
    };
    auto step = [&](int b, int m) {
      const Z64 a0 = a[b][0], a1 = a[b][1];
      Z64 c0[BJ], c1[BJ];
#pragma unroll
      for (int bj = 0; bj < BJ; ++bj) {
        c0[bj] = c[b][bj][0];
        c1[bj] = c[b][bj][1];
      }
      load(b, m + 16);
#pragma unroll
      for (int bj = 0; bj < BJ; ++bj) {
        dre[bj] = mfma(a0.re, c0[bj].re, dre[bj]);
        dim_[bj] = mfma(a0.re, c0[bj].im, dim_[bj]);
        dre[bj] = mfma(a0.im, -c0[bj].im, dre[bj]);
        dim_[bj] = mfma(a0.im, c0[bj].re, dim_[bj]);
        dre[bj] = mfma(a1.re, c1[bj].re, dre[bj]);
        dim_[bj] = mfma(a1.re, c1[bj].im, dim_[bj]);
        dre[bj] = mfma(a1.im, -c1[bj].im, dre[bj]);
        dim_[bj] = mfma(a1.im, c1[bj].re, dim_[bj]);
      }
    };
    load(0, 0);
    load(1, 8);
    int m = 0;
    for (; m + 16 <= M; m += 16) {
      step(0, m);
      step(1, m + 8);
    }
    if (m < M) step(0, m);
  }
#pragma unroll
  for (int bj = 0; bj < BJ; ++bj) {
    const int n = 16 * bj + l16;
    if (n >= ncols) continue;
    const int row = yidx ? yidx[n] : n;
    const size_t o = (size_t)row * ldy + k0 + g;
    const double bt = PUPD ? beta[row] : 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      put_row(Y + o + 4 * r, PUPD ? P + o + 4 * r : nullptr, bt, dre[bj][r], dim_[bj][r]);
  }
}

}  // namespace

constexpr int kGemm64TargetGroups = 2048;  // workgroups a split-K reduce aims for by default
// Columns up to which the kernels for few columns run: beyond three blocks of 16 the 64-column tile wastes
// at most a quarter of its products and reads A once for more columns per load.
constexpr int kFewCols = 48, kFewColsGroups = 512;

int nsplit_bound(int M_pad, int ncols, int K, int target) {
  if (target <= 0) target = kGemm64TargetGroups;
  const int base = (M_pad / 64) * ((ncols + 63) / 64);
  int ns = (target + base - 1) / base;
  const int maxs = K / 256 > 0 ? K / 256 : 1;
  if (ns > maxs) ns = maxs;
  if (ns < 1) ns = 1;
  return ns;
}

// A split-K reduce's workgroups all take the same time, and kGemm64PerCu of them run at once on a CU (4 waves
// per SIMD), 1,024 on 256 CUs: a factor that leaves the last round nearly empty wastes it. 517 columns of M = 1,024, K = 91,072 in 15
// splits are 2,160 workgroups, three rounds for 2.1; in 14 they are 2,016, two: 8.3 -> 7.6 ms (7.2 ms with the last block of columns
// at half its products).
constexpr int kGemm64PerCu = 4;

int choose_nsplit(int M_pad, int ncols, int K, int target, int n_cu) {
  const int bound = nsplit_bound(M_pad, ncols, K, target);
  if (ncols > kFewCols) {
    const int base = (M_pad / 64) * ((ncols + 63) / 64);
    int best = bound;
    double fill = 0.0;
    for (int ns = bound; 2 * ns > bound; --ns) {
      const double rounds = (double)base * ns / (kGemm64PerCu * n_cu), f = rounds / std::ceil(rounds);
      if (f > fill + 0.02) {
        fill = f;
        best = ns;
      }
    }
    return best;
  }
  // few columns: chunks of 64 k or more, and a count of workgroups of their own: a target is set for, or found on, many
  // columns (M = 1,024, K = 91,072, 16 columns: P_c 712 us, with a target of 4,096 774)
  const int base = M_pad / 64;
  int ns = std::min((kFewColsGroups + base - 1) / base, K / 64);
  if (ns < 1) ns = 1;
  // within the fixed area of the allocation-free entry point wherever it takes the call
  auto fits = [&](int splits) { return 16.0 * ncols * (K + (splits + 1.0) * M_pad) <= (double)STERN_NOALLOC_SCRATCH_BYTES; };
  if (ns > bound && !fits(ns) && fits(bound)) ns = bound;
  return ns;
}

void launch_zgemm_reduce2(const ZRows& s0, const ZRows& s1, int ldx, const int* xidx, int ncols, int K, int nsplit,
                          hipStream_t st) {
  if (ncols <= 0) return;
  int kchunk = (K + nsplit - 1) / nsplit;
  kchunk = (kchunk + 15) / 16 * 16;
  const int mb0 = (s0.M + 63) / 64, mb = mb0 + (s1.M + 63) / 64;
  if (ncols <= kFewCols) {
    const dim3 grid(mb, 1, nsplit);
    if (ncols <= 16)
      k_zgemm_reduce_cols<1><<<grid, kGemmThreads, 0, st>>>(s0, s1, mb0, ldx, xidx, ncols, K, kchunk);
    else if (ncols <= 32)
      k_zgemm_reduce_cols<2><<<grid, kGemmThreads, 0, st>>>(s0, s1, mb0, ldx, xidx, ncols, K, kchunk);
    else
      k_zgemm_reduce_cols<3><<<grid, kGemmThreads, 0, st>>>(s0, s1, mb0, ldx, xidx, ncols, K, kchunk);
    return;
  }
  k_zgemm_reduce<<<dim3(mb, (ncols + 63) / 64, nsplit), kGemmThreads, 0, st>>>(s0, s1, mb0, ldx, xidx, ncols, K,
                                                                              kchunk);
}

void launch_sum_parts2(const ZRows& s0, const ZRows& s1, int nsplit, int ncols, hipStream_t st) {
  const int t0 = ncols * ((s0.M + 7) / 8 * 8), t1 = ncols * ((s1.M + 7) / 8 * 8);
  if (t0 + t1 <= 0) return;
  const int O = nsplit >= 8 ? 32 : 256, nb0 = (t0 + O - 1) / O, nb = nb0 + (t1 + O - 1) / O;
  if (nsplit >= 8)
    k_sum_parts<8><<<nb, 256, 0, st>>>(s0, s1, nb0, nsplit, ncols);
  else
    k_sum_parts<1><<<nb, 256, 0, st>>>(s0, s1, nb0, nsplit, ncols);
}

namespace {
template <bool PUPD>
void expand2(const ZRows& s0, const ZRows& s1, Z64* Y, int ldy, const int* yidx, int ncols, int K, hipStream_t st,
             Z64* P, const double* beta) {
  if (ncols <= 16)
    k_zgemm_expand_cols<1, PUPD><<<K / 64, kGemmThreads, 0, st>>>(s0, s1, K, Y, ldy, yidx, ncols, P, beta);
  else if (ncols <= 32)
    k_zgemm_expand_cols<2, PUPD><<<K / 64, kGemmThreads, 0, st>>>(s0, s1, K, Y, ldy, yidx, ncols, P, beta);
  else if (ncols <= kFewCols)
    k_zgemm_expand_cols<3, PUPD><<<K / 64, kGemmThreads, 0, st>>>(s0, s1, K, Y, ldy, yidx, ncols, P, beta);
  else
    k_zgemm_expand<PUPD><<<dim3(K / 64, (ncols + 63) / 64), kGemmThreads, 0, st>>>(s0, s1, K, Y, ldy, yidx, ncols, P,
                                                                                  beta);
}
}  // namespace
void launch_zgemm_expand2(const ZRows& s0, const ZRows& s1, Z64* Y, int ldy, const int* yidx, int ncols, int K,
                          hipStream_t st, Z64* P, const double* beta) {
  if (ncols <= 0) return;
  if (P)
    expand2<true>(s0, s1, Y, ldy, yidx, ncols, K, st, P, beta);
  else
    expand2<false>(s0, s1, Y, ldy, yidx, ncols, K, st, P, beta);
}

void launch_zgemm_reduce(const Z64* A, int M_pad, const Z64* X, int ldx, const int* xidx, int ncols, int K,
                         Z64* cpart, int nsplit, hipStream_t st, int M) {
  launch_zgemm_reduce2(ZRows{A, X, cpart, nullptr, M_pad, M, 0.0}, ZRows{}, ldx, xidx, ncols, K, nsplit, st);
}
void launch_sum_parts(const Z64* cpart, int nsplit, int ncols, int M_pad, double scale, Z64* C, hipStream_t st,
                      int M) {
  launch_sum_parts2(ZRows{nullptr, nullptr, const_cast<Z64*>(cpart), C, M_pad, M, scale}, ZRows{}, nsplit, ncols, st);
}
void launch_zgemm_expand(const Z64* A, int M_pad, const Z64* C, Z64* Y, int ldy, const int* yidx, int ncols, int K,
                         hipStream_t st, int M) {
  launch_zgemm_expand2(ZRows{A, nullptr, nullptr, const_cast<Z64*>(C), M_pad, M, 0.0}, ZRows{}, Y, ldy, yidx, ncols,
                       K, st, nullptr, nullptr);
}

}  // namespace stern
