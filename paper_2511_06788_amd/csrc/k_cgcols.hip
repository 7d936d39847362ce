// Step 1's conjugate gradients for small grids: one work-group runs the whole
// CG of one column on chip.
//
// The N source problems H y_j = u_j are independent (Section 4.1, Step 1), so
// on a grid that fits one compute unit a column needs no other work-group: its
// search direction p lives in LDS (with one zero word that stands for every
// neighbour outside the grid), r and y live in registers, and an iteration is
// three barriers instead of the four dependent launches of the sweeps.  The
// arithmetic is that of the sweeps (k_stencil.hip) column by column, with the
// same stopping rule; only the order of the dot products' sums differs.
//
// Bound by the LDS reads of the stencil (seven values per point and iteration)
// and, on the smallest grids, by the latency of the two reductions.  The launch
// path pays 15 to 30 us of dependent launches per iteration however small the
// problem.  Measured, one FP64 step with the sweeps and with this kernel: 32 x 32,
// N = 8 735 -> 165 us; 128 x 128, N = 15 3378 -> 1212 us, N = 128 8030 -> 1917 us;
// 24^3, N = 16 796 -> 456 us; 25 x 25 x 26, N = 512 11.5 -> 8.1 ms.  Faster at
// every width from 1 to 512, so the limit is what one compute unit holds.
//
// Columns are point-major, so a work-group reads one value of every row; the
// XCD-contiguous mapping lets the columns of one cache line meet in one L2.
#include <algorithm>

#include "ope_internal.h"

namespace {

// Sum over the work-group in a fixed order, the result in every thread.  `red`
// holds one value per wave; calls in a row need two arrays.
template <int TH>
__device__ __forceinline__ double wg_sum_all(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < TH / 64; ++w) s += red[w];
  return s;
}

// Ends a group of points of an unrolled loop: nothing moves across, and what is
// formed from the thread's index and neighbour bits is formed anew, so that a
// thread does not hold the addresses of all its points at once.
__device__ __forceinline__ void pace(uint32_t& tid, uint32_t& nb) {
  asm volatile("" : "+v"(tid), "+v"(nb));
  __builtin_amdgcn_sched_barrier(0);
}

// TH threads with PPT points each (thread t: points t, t + TH, ...), GP of them
// at a time.
template <typename T, int PPT, int TH, int GP>
__global__ __launch_bounds__(TH) void k_cg_cols(const T* __restrict__ R, T* __restrict__ Y,
                                                const T* __restrict__ diag, OpeGrid g, uint32_t n, uint32_t N,
                                                int32_t max_iter, const double* __restrict__ rho0,
                                                const double* __restrict__ target, int32_t* __restrict__ active,
                                                OpeScalars* __restrict__ sc) {
  extern __shared__ __align__(16) char cg_lds[];
  T* const p = reinterpret_cast<T*>(cg_lds);                 // n values, then the zero word
  __shared__ double red[2][TH / 64];
  const uint32_t col = xcd_remap(blockIdx.x, gridDim.x);
  if (active[col] == 0) return;                              // uniform over the work-group
  const uint32_t m0 = g.m0, s2 = g.m0 * g.m1;
  T r[PPT], y[PPT];
  uint32_t nb[(PPT + 3) / 4];                                // per point: which neighbours exist (bits x-, x+, y-, ...)
  uint32_t tid = threadIdx.x;
#pragma unroll
  for (int k = 0; k < (PPT + 3) / 4; ++k) nb[k] = 0;
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    // a slot past the grid is point n, the zero word: no neighbours, r = y = 0
    const uint32_t i = min(tid + (uint32_t)k * TH, n), ic = min(i, n - 1u);
    const T rv = R[(uint64_t)ic * N + col], yv = Y[(uint64_t)ic * N + col];
    r[k] = i < n ? rv : T(0);
    y[k] = i < n ? yv : T(0);
    const uint32_t x = ic % m0, q = ic / m0, yy = q % g.m1, z = q / g.m1;
    const uint32_t b = (x > 0 ? 1u : 0u) | (x + 1 < m0 ? 2u : 0u) | (yy > 0 ? 4u : 0u) | (yy + 1 < g.m1 ? 8u : 0u) |
                       (z > 0 ? 16u : 0u) | (z + 1 < g.m2 ? 32u : 0u);
    nb[k / 4] |= (i < n ? b : 0u) << (8 * (k % 4));
    p[i] = r[k];
    if (k % 4 == 3) {
      asm volatile("" : "+v"(r[k]), "+v"(y[k]));
      pace(tid, nb[k / 4]);
    }
  }
  if (threadIdx.x == 0) p[n] = T(0);                         // every thread that writes it writes zero
  const T cx = (T)g.cx, cy = (T)g.cy, cz = (T)g.cz;
  const double tgt = target[col];
  double rho = rho0[col];
  bool act = true;
  int32_t err = 0;
  int32_t it = 0;
  const bool flat = g.m2 == 1;                               // 2D: no z neighbours anywhere
  for (; act && it < max_iter; ++it) {
    __syncthreads();                                         // p is complete
#pragma unroll
    for (int k = 0; k < (PPT + 3) / 4; ++k) pace(tid, nb[k]);
    T h[PPT];
    double s = 0.0;
    // the diagonal comes from L2: its values one group of points ahead
    T dn[GP];
#pragma unroll
    for (int u = 0; u < GP; ++u) dn[u] = diag[min(tid + (uint32_t)u * TH, n - 1u)];
#pragma unroll
    for (int k0 = 0; k0 < PPT; k0 += GP) {
      T d[GP];
#pragma unroll
      for (int u = 0; u < GP; ++u) {
        d[u] = dn[u];
        if (k0 + GP < PPT) dn[u] = diag[min(tid + (uint32_t)(k0 + GP + u) * TH, n - 1u)];
      }
#pragma unroll
      for (int u = 0; u < GP; ++u) {
        const int k = k0 + u;
        const uint32_t i = min(tid + (uint32_t)k * TH, n);
        const uint32_t b = nb[k / 4] >> (8 * (k % 4));
        const T xm = p[b & 1u ? i - 1u : n], xp = p[b & 2u ? i + 1u : n];
        const T ym = p[b & 4u ? i - m0 : n], yp = p[b & 8u ? i + m0 : n];
        T zs = T(0);
        if (!flat) zs = p[b & 16u ? i - s2 : n] + p[b & 32u ? i + s2 : n];
        const T pc = p[i];
        h[k] = d[u] * pc - (cx * (xm + xp) + cy * (ym + yp) + cz * zs);
        s += (double)pc * (double)h[k];
      }
#pragma unroll
      for (int u = 0; u < GP; ++u) asm volatile("" : "+v"(h[k0 + u]));
      asm volatile("" : "+v"(s));
      pace(tid, nb[k0 / 4]);                                 // GP points in flight, not all PPT
    }
    const double ph = wg_sum_all<TH>(s, red[0]);
    if (!isfinite(ph)) err = OPE_ENONFINITE;
    const double alpha = (ph > 0.0 && isfinite(ph)) ? rho / ph : 0.0;
    const T a = (T)alpha;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      r[k] = r[k] - a * h[k];
      y[k] = y[k] + a * p[min(tid + (uint32_t)k * TH, n)];
      s += (double)r[k] * (double)r[k];
      if (k % 2 == 1) {
        asm volatile("" : "+v"(y[k - 1]), "+v"(y[k]), "+v"(s));
        pace(tid, nb[k / 4]);
      }
    }
    const double rr = wg_sum_all<TH>(s, red[1]);             // its barrier also ends every read of p
    if (!isfinite(rr)) {
      err = OPE_ENONFINITE;
      act = false;
      continue;
    }
    const T b = (T)(rr / rho);
    rho = rr;
    act = rr > tgt;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const uint32_t i = tid + (uint32_t)k * TH;
      if (i < n) p[i] = r[k] + b * p[i];
      if (k % 4 == 3) pace(tid, nb[k / 4]);
    }
  }
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const uint32_t i = tid + (uint32_t)k * TH;
    if (i < n) Y[(uint64_t)i * N + col] = y[k];
  }
  if (threadIdx.x == 0) {
    active[col] = act ? 1 : 0;
    atomicMax(&sc->cg_iters, it);
    if (err) sc->err = err;
  }
}

template <typename T, int PPT, int TH, int GP>
void go(ope_ctx* c, void* y, int32_t max_iter, const T* diag) {
  const uint32_t n = (uint32_t)c->n, N = (uint32_t)c->N;
  hipLaunchKernelGGL((k_cg_cols<T, PPT, TH, GP>), dim3(N), dim3(TH), (size_t)(n + 1) * sizeof(T), c->stream,
                     (const T*)c->Rb[0], (T*)y, diag, c->g, n, N, max_iter, c->rho, c->target, c->active, c->sc);
}

template <typename T>
void pick(ope_ctx* c, void* y, int32_t max_iter, const T* diag) {
  if (c->n <= 1024) go<T, 4, 256, 4>(c, y, max_iter, diag);
  else if (c->n <= 4096) go<T, 4, 1024, 4>(c, y, max_iter, diag);
  else if (c->n <= 8192) go<T, 8, 1024, 2>(c, y, max_iter, diag);
  else go<T, 32, 512, 2>(c, y, max_iter, diag);
}

}  // namespace

// The grid fits one work-group (pick: at most 512 threads of 32 points, p in at
// most 128 KiB of LDS), the CG runs without the preconditioner, and the launch is
// bounded: nothing on the host can stop it before max_iter iterations of 8 to 20 us
// each, about a second at CGC_MAX_ITER; a caller who allows more gets the sweeps,
// whose launches end after an iteration.  While a kernel of the CG sweeps is being
// timed the sweeps run, so that there is something to time.
constexpr int32_t CGC_MAX_ITER = 1 << 16;

bool cg_cols_fits(const ope_ctx* c, int32_t max_iter) {
  const bool timed = c->prof_kernel == OPE_KERNEL_CG_SWEEP_A || c->prof_kernel == OPE_KERNEL_CG_SWEEP_B ||
                     c->prof_kernel == OPE_KERNEL_CG_SWEEP_B_Y || c->prof_kernel == OPE_KERNEL_CG_REDUCE;
  return !c->mg_on && !timed && c->n <= 16384 && max_iter <= CGC_MAX_ITER;
}

hipError_t launch_cg_cols(ope_ctx* c, void* y, int32_t max_iter) {
  if (c->prec == OPE_FP64) pick<double>(c, y, max_iter, c->diag);
  else pick<float>(c, y, max_iter, c->diag32);
  return hipGetLastError();
}
