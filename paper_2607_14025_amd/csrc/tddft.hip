// Grid kernels of the TDDFT Liouville apply (Tamm-Dancoff; Sec. II.C.1, eq. bse_tddft): the
// band-summed transition densities rho_e = sum_v conj(psi_v) a_{e,v}, the Coulomb factor on the
// 4 Ecut sphere, the products V_e psi_v, and for the bare-exchange direct term the occupied pair
// densities conj(psi_w) psi_v whose potentials are the integrals tau_{wv} of eq. tau_u and the
// sums sum_w tau_{wv} a_{e,w}. All of it is streaming work on
// full N^3 grids (one read and one write per point and band), so the kernels are plain
// grid-stride loops with coalesced complex FP64 accesses; the FFTs between them are the
// library's pencil and plane kernels.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace stern {

namespace {

constexpr int kGridThreads = 256;

// rho[e][j] = scale sum_v conj(psi_r[v][j]) a_r[e nb + v][j], bands summed in order
__global__ __launch_bounds__(kGridThreads) void k_band_density(const Z64* __restrict__ psi_r,
                                                               const Z64* __restrict__ a_r, int nb, size_t n3,
                                                               double scale, Z64* __restrict__ rho) {
  const int e = blockIdx.y;
  const Z64* ae = a_r + (size_t)e * nb * n3;
  for (size_t j = (size_t)blockIdx.x * kGridThreads + threadIdx.x; j < n3; j += (size_t)gridDim.x * kGridThreads) {
    double re = 0.0, im = 0.0;
    for (int v = 0; v < nb; ++v) {
      const Z64 p = psi_r[(size_t)v * n3 + j], a = ae[(size_t)v * n3 + j];
      re += p.re * a.re + p.im * a.im;
      im += p.re * a.im - p.im * a.re;
    }
    rho[(size_t)e * n3 + j] = zmk(scale * re, scale * im);
  }
}

// c[i] *= fac / g2h[i mod K]; zero where g2h = 0 (G = 0 and the padding, whatever they held)
__global__ __launch_bounds__(kGridThreads) void k_coulomb(Z64* __restrict__ c, const double* __restrict__ g2h, int K,
                                                          size_t total, double fac) {
  for (size_t i = (size_t)blockIdx.x * kGridThreads + threadIdx.x; i < total; i += (size_t)gridDim.x * kGridThreads) {
    const double h = g2h[i % K];
    const Z64 v = c[i];
    c[i] = h > 0.0 ? zmk(fac / h * v.re, fac / h * v.im) : zmk(0.0, 0.0);
  }
}

// out[e nb + v][j] = v_r[e][j] psi_r[v][j] (- alpha acc[e nb + v][j] when acc is given)
__global__ __launch_bounds__(kGridThreads) void k_grid_mul(const Z64* __restrict__ v_r, const Z64* __restrict__ psi_r,
                                                           int nb, size_t n3, const Z64* __restrict__ acc,
                                                           double alpha, Z64* __restrict__ out) {
  const int row = blockIdx.y, e = row / nb, v = row - e * nb;
  const Z64* ve = v_r + (size_t)e * n3;
  const Z64* pv = psi_r + (size_t)v * n3;
  const Z64* ac = acc ? acc + (size_t)row * n3 : nullptr;
  Z64* o = out + (size_t)row * n3;
  for (size_t j = (size_t)blockIdx.x * kGridThreads + threadIdx.x; j < n3; j += (size_t)gridDim.x * kGridThreads) {
    const Z64 a = ve[j], p = pv[j];
    Z64 r = zmk(a.re * p.re - a.im * p.im, a.re * p.im + a.im * p.re);
    if (ac) {
      const Z64 c = ac[j];
      r = zmk(r.re - alpha * c.re, r.im - alpha * c.im);
    }
    o[j] = r;
  }
}

// The direct term of a block of bands v in [v0, v0 + nv), nv <= VB, from the potentials of the pairs w <= v
// only: tau_{vw} = conj(tau_{wv}), so pair (w, v) adds tau a_w to band v and conj(tau) a_v to band w:
//   acc[e nb + v][j] += sum_{w <= v} tau_{wv}[j] a_r[e nb + w][j],   acc[e nb + w][j] += conj(tau_{wv}[j]) a_r[e nb + v][j], w < v,
// tau rows in the order of pair_of. Streaming: a thread keeps one grid point, the block's a_v and sums of EB
// excitations in registers and walks w, so a_w and acc_w pass once per VB bands and tau once per EB excitations.
// NS > 0: tau is still without its screening sum_a w[a][j] pc[pair][a] (n <= NS), added here in registers.
// 50 bands, 48^3, 3 excitations, 12 potentials: 13 launches of 212 us, against 50 of 65 (the products) and
// 50 of 52 (the screening) with one band at a time and every pair formed twice.
template <int VB, int EB, int NS>
__global__ __launch_bounds__(kGridThreads) void k_exch_block(const Z64* __restrict__ tau, const Z64* __restrict__ a_r,
                                                             int n_exc, int nb, int v0, int nv, size_t n3,
                                                             const double* __restrict__ scr,
                                                             const Z64* __restrict__ pc, int n, Z64* __restrict__ acc) {
  const int e0 = blockIdx.y * EB;
  const size_t j = (size_t)blockIdx.x * kGridThreads + threadIdx.x;
  if (j >= n3) return;
  const Z64 zero = zmk(0.0, 0.0);
  Z64 av[VB][EB], sv[VB][EB];
#pragma unroll
  for (int q = 0; q < VB; ++q)
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      av[q][e] = sv[q][e] = zero;
      if (q < nv && e0 + e < n_exc) av[q][e] = a_r[((size_t)(e0 + e) * nb + v0 + q) * n3 + j];
    }
  double f[NS > 0 ? NS : 1];
  if constexpr (NS > 0) {
#pragma unroll
    for (int a = 0; a < NS; ++a) f[a] = a < n ? scr[(size_t)a * n3 + j] : 0.0;
  }
  for (int w = 0; w < v0 + nv; ++w) {
    Z64 t[VB], aw[EB], cw[EB];
#pragma unroll
    for (int q = 0; q < VB; ++q) {  // pair (w, v0 + q): row q v0 + q (q + 1) / 2 + w
      const bool on = q < nv && w <= v0 + q;
      const size_t row = (size_t)q * v0 + q * (q + 1) / 2 + w;
      t[q] = zero;
      if (on) t[q] = tau[row * n3 + j];
      if constexpr (NS > 0) {
        if (on) {
          const Z64* p = pc + row * n;
#pragma unroll
          for (int a = 0; a < NS; ++a)
            if (a < n) {
              t[q].re += f[a] * p[a].re;
              t[q].im += f[a] * p[a].im;
            }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      aw[e] = cw[e] = zero;
      if (e0 + e < n_exc) aw[e] = a_r[((size_t)(e0 + e) * nb + w) * n3 + j];
    }
#pragma unroll
    for (int q = 0; q < VB; ++q)
#pragma unroll
      for (int e = 0; e < EB; ++e) {
        sv[q][e].re += t[q].re * aw[e].re - t[q].im * aw[e].im;
        sv[q][e].im += t[q].re * aw[e].im + t[q].im * aw[e].re;
        if (w < v0 + q) {
          cw[e].re += t[q].re * av[q][e].re + t[q].im * av[q][e].im;
          cw[e].im += t[q].re * av[q][e].im - t[q].im * av[q][e].re;
        }
      }
#pragma unroll
    for (int e = 0; e < EB; ++e)
      if (e0 + e < n_exc) {
        Z64* o = acc + ((size_t)(e0 + e) * nb + w) * n3 + j;
        Z64 c = *o;
        c = zmk(c.re + cw[e].re, c.im + cw[e].im);
#pragma unroll
        for (int q = 0; q < VB; ++q)  // the band's own sum is complete once w has reached it
          if (w == v0 + q) c = zmk(c.re + sv[q][e].re, c.im + sv[q][e].im);
        *o = c;
      }
  }
}

// parts[s][pair][a] = sum over the s-th stretch of the grid of w[a][j] conj(psi_w[j]) psi_v[j], the pairs (w, v) of a
// block of bands as in k_exch_block. A workgroup takes one w, the block's VB bands and AT potentials, so the VB AT
// products a point share its 1 + VB orbital and AT potential values.
constexpr int kProjA = 8;
template <int VB>
__global__ __launch_bounds__(kGridThreads) void k_scr_proj(const Z64* __restrict__ psi_r, const double* __restrict__ scr,
                                                           int n, int v0, int nv, size_t n3, size_t stretch,
                                                           int npairs, Z64* __restrict__ parts) {
  constexpr int AT = kProjA;
  __shared__ Z64 sh[kGridThreads / 64][VB * AT];
  const int w = blockIdx.x, a0 = blockIdx.z * AT;
  const size_t j0 = blockIdx.y * stretch, j1 = min(n3, j0 + stretch);
  Z64 s[VB][AT];
#pragma unroll
  for (int q = 0; q < VB; ++q)
#pragma unroll
    for (int a = 0; a < AT; ++a) s[q][a] = zmk(0.0, 0.0);
  const Z64* pw = psi_r + (size_t)w * n3;
  for (size_t j = j0 + threadIdx.x; j < j1; j += kGridThreads) {
    const Z64 x = pw[j];
    double f[AT];
#pragma unroll
    for (int a = 0; a < AT; ++a) f[a] = scr[(size_t)min(a0 + a, n - 1) * n3 + j];
#pragma unroll
    for (int q = 0; q < VB; ++q) {
      const Z64 y = psi_r[(size_t)(v0 + min(q, nv - 1)) * n3 + j];
      const double re = x.re * y.re + x.im * y.im, im = x.re * y.im - x.im * y.re;
#pragma unroll
      for (int a = 0; a < AT; ++a) {
        s[q][a].re += f[a] * re;
        s[q][a].im += f[a] * im;
      }
    }
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < VB; ++q)
#pragma unroll
    for (int a = 0; a < AT; ++a) {
      double re = s[q][a].re, im = s[q][a].im;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o);
        im += __shfl_xor(im, o);
      }
      if (lane == 0) sh[wave][q * AT + a] = zmk(re, im);
    }
  __syncthreads();
  const int q = threadIdx.x / AT, a = threadIdx.x % AT;
  if (q >= nv || a0 + a >= n || w > v0 + q) return;
  Z64 t = zmk(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < kGridThreads / 64; ++k) t = t + sh[k][q * AT + a];
  const size_t row = (size_t)q * v0 + q * (q + 1) / 2 + w;
  parts[((size_t)blockIdx.y * npairs + row) * n + a0 + a] = t;
}

// pc[i] = scale c[i mod n] sum_s parts[s][i], s in order
__global__ void k_scr_sum(const Z64* __restrict__ parts, int ns, int total, int n, const double* __restrict__ c,
                          double scale, Z64* __restrict__ pc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  Z64 t = zmk(0.0, 0.0);
  for (int s = 0; s < ns; ++s) t = t + parts[(size_t)s * total + i];
  pc[i] = zscale(t, scale * c[i % n]);
}

// y[i] += x[i]
__global__ __launch_bounds__(kGridThreads) void k_add(Z64* __restrict__ y, const Z64* __restrict__ x, size_t n) {
  for (size_t i = (size_t)blockIdx.x * kGridThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kGridThreads) {
    const Z64 a = y[i], b = x[i];
    y[i] = zmk(a.re + b.re, a.im + b.im);
  }
}

// tau[r][j] += sum_a w[a][j] pc[r][a] (more potentials than k_exch_block holds in registers)
__global__ __launch_bounds__(kGridThreads) void k_scr_add(Z64* __restrict__ tau, const double* __restrict__ w,
                                                          const Z64* __restrict__ pc, int n, size_t n3) {
  const int r = blockIdx.y;
  Z64* t = tau + (size_t)r * n3;
  const Z64* p = pc + (size_t)r * n;
  for (size_t j = (size_t)blockIdx.x * kGridThreads + threadIdx.x; j < n3; j += (size_t)gridDim.x * kGridThreads) {
    double re = 0.0, im = 0.0;
    for (int a = 0; a < n; ++a) {
      const double f = w[(size_t)a * n3 + j];
      re += f * p[a].re;
      im += f * p[a].im;
    }
    const Z64 v = t[j];
    t[j] = zmk(v.re + re, v.im + im);
  }
}

unsigned grid_blocks(size_t n, int per_row_rows) {
  // enough workgroups to fill the chip several times over, fewer when a launch has many rows
  const size_t want = std::max<size_t>(1, 2048 / (size_t)std::max(1, per_row_rows));
  return (unsigned)std::max<size_t>(1, std::min<size_t>((n + kGridThreads - 1) / kGridThreads, want));
}

}  // namespace

void launch_band_density(const Z64* psi_r, const Z64* a_r, int n_exc, int nb, size_t n3, double scale, Z64* rho,
                         hipStream_t st) {
  if (n_exc <= 0 || nb <= 0) return;
  dim3 grid(grid_blocks(n3, n_exc), n_exc);
  k_band_density<<<grid, kGridThreads, 0, st>>>(psi_r, a_r, nb, n3, scale, rho);
}

void launch_coulomb(Z64* c, const double* g2h, int K, int nvec, double fac, hipStream_t st) {
  const size_t total = (size_t)K * nvec;
  if (total == 0) return;
  k_coulomb<<<grid_blocks(total, 1), kGridThreads, 0, st>>>(c, g2h, K, total, fac);
}

void launch_grid_mul(const Z64* v_r, const Z64* psi_r, int n_exc, int nb, size_t n3, const Z64* acc, double alpha,
                     Z64* out, hipStream_t st) {
  if (n_exc <= 0 || nb <= 0) return;
  dim3 grid(grid_blocks(n3, n_exc * nb), n_exc * nb);
  k_grid_mul<<<grid, kGridThreads, 0, st>>>(v_r, psi_r, nb, n3, acc, alpha, out);
}

void launch_exch_block(const Z64* tau, const Z64* a_r, int n_exc, int nb, int v0, int nv, size_t n3,
                       const double* scr, const Z64* pc, int n, Z64* acc, hipStream_t st) {
  if (n_exc <= 0 || nv <= 0) return;
  const unsigned gx = (unsigned)((n3 + kGridThreads - 1) / kGridThreads);
  auto go = [&](auto eb, auto ns) {
    constexpr int EB = decltype(eb)::value, NS = decltype(ns)::value;
    k_exch_block<kExchBands, EB, NS><<<dim3(gx, (n_exc + EB - 1) / EB), kGridThreads, 0, st>>>(
        tau, a_r, n_exc, nb, v0, nv, n3, scr, pc, n, acc);
  };
  auto with = [&](auto ns) {  // excitations in registers: as few passes over tau as 4 allow, evenly filled
    const int passes = (n_exc + 3) / 4, eb = (n_exc + passes - 1) / passes;
    if (eb == 1) go(std::integral_constant<int, 1>{}, ns);
    else if (eb == 2) go(std::integral_constant<int, 2>{}, ns);
    else if (eb == 3) go(std::integral_constant<int, 3>{}, ns);
    else go(std::integral_constant<int, 4>{}, ns);
  };
  if (n > 0) with(std::integral_constant<int, kExchScr>{});
  else with(std::integral_constant<int, 0>{});
}

int scr_proj_stretches(int v0, int nv, int n, size_t n3, int n_cu) {
  const int groups = (v0 + nv) * ((n + kProjA - 1) / kProjA);  // about 4 workgroups per CU, 4 points a thread or more
  const size_t want = std::max(1, 4 * n_cu / std::max(1, groups));
  return (int)std::max<size_t>(1, std::min(want, n3 / (4 * kGridThreads)));
}
void launch_scr_proj(const Z64* psi_r, const double* scr, const double* c, int n, int v0, int nv, size_t n3, int n_cu,
                     double scale, Z64* parts, Z64* pc, hipStream_t st) {
  if (n <= 0 || nv <= 0) return;
  const int ns = scr_proj_stretches(v0, nv, n, n3, n_cu), npairs = nv * v0 + nv * (nv + 1) / 2, total = npairs * n;
  const size_t stretch = (n3 + ns - 1) / ns;
  k_scr_proj<kExchBands><<<dim3(v0 + nv, ns, (n + kProjA - 1) / kProjA), kGridThreads, 0, st>>>(
      psi_r, scr, n, v0, nv, n3, stretch, npairs, parts);
  k_scr_sum<<<(total + 255) / 256, 256, 0, st>>>(parts, ns, total, n, c, scale / (double)n3, pc);
}

void launch_add(Z64* y, const Z64* x, size_t n, hipStream_t st) {
  if (n == 0) return;
  k_add<<<grid_blocks(n, 1), kGridThreads, 0, st>>>(y, x, n);
}

void launch_scr_add(Z64* tau, const double* w, const Z64* pc, int n, int nrows, size_t n3, hipStream_t st) {
  if (n <= 0 || nrows <= 0) return;
  k_scr_add<<<dim3(grid_blocks(n3, nrows), nrows), kGridThreads, 0, st>>>(tau, w, pc, n, n3);
}

}  // namespace stern
