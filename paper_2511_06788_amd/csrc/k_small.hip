// FP64 kernels on N x N matrices: the small solve of
// Steps 2-3 (Section 4.1), the warm-start inverse Lam^{-1}, the per-step
// scalars, and the Ritz values (Householder tridiagonalisation and bisection).
//
// For N <= 128 one work-group of 16 waves holds an N x N matrix in registers, in
// 16 x 16 blocks in the layout of the FP64 matrix instruction's accumulator, and
// inverts it by block Gauss-Jordan elimination without pivoting; larger N use
// the Newton-Schulz pieces below.  No
// pivoting is needed: the Step-2 matrix has symmetric part >= I (Lemma 3.1 and
// its generalisation to an inexact GU), and Lam = U^T H U is SPD, so every
// pivot of either is positive.
#include <type_traits>

#include "ope_internal.h"

namespace {

constexpr int SW = 1024;      // threads of the small kernels

// Deterministic work-group sum (fixed tree order).
__device__ double wg_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = SW / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  const double out = red[0];
  __syncthreads();
  return out;
}

// Blocks of an N x N matrix over the 16 waves: a wave holds CB neighbouring blocks
// of one block row (four waves to a block row for CB = 1, else two), element
// (kr + 4 r, ci) of a block in register r of lane 16 kr + ci.
typedef double v4d __attribute__((ext_vector_type(4)));

template <int CB>
struct Blocks {
  uint32_t kr, ci, br, bc0, nb;
  __device__ explicit Blocks(uint32_t N) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    kr = lane >> 4;
    ci = lane & 15u;
    br = CB == 1 ? wave >> 2 : wave >> 1;
    bc0 = CB == 1 ? wave & 3u : (wave & 1u) * CB;
    nb = (N + 15u) / 16u;
  }
  __device__ bool has(int b) const { return br < nb && bc0 + b < nb; }        // uniform over the wave
  __device__ uint32_t row(int r) const { return 16u * br + kr + 4u * (uint32_t)r; }
  __device__ uint32_t col(int b) const { return 16u * (bc0 + b) + ci; }
};

__device__ __forceinline__ v4d mma64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int LDF = 17, LDX = 144;                     // row strides without bank conflicts
constexpr int MKC = 32, LDA = 33;                      // contraction indices per chunk of a product

union SmallLds {
  struct {                                             // of the inversion
    double F[2][128 * LDF];
    double R[16 * LDX], X[16 * LDX];
    double P[16 * LDF];
  } inv;
  struct {                                             // of a product: MKC rows of B (and of A, transposed)
    double A[MKC * LDX], B[MKC * LDX];
  } mm;
};
static_assert(128 * LDA <= MKC * LDX, "A by columns fits where it does by rows");

// acc += op(A) B for the wave's blocks, op the transpose when TA; EYE: A - I.
// Chunks of MKC contraction indices staged in LDS, the next chunk's loads in
// flight; zero outside the N x N matrices.  Called by the whole work-group; L must
// be free, and is when it returns.
template <int CB, bool TA, bool EYE>
__device__ void blk_mm(const double* A, const double* B, uint32_t N, const Blocks<CB>& o, SmallLds& lds,
                       v4d (&acc)[CB]) {
  auto& L = lds.mm;
  constexpr int PT = MKC * 128 / SW;                   // values of a chunk per thread
  double ga[PT], gb[PT];
  const bool same = TA && A == B;
  auto load = [&](uint32_t k0) {
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const uint32_t e = threadIdx.x + (uint32_t)SW * u;
      const uint32_t kb = k0 + e / 128u, j = e % 128u;                         // by rows
      gb[u] = kb < N && j < N ? B[kb * N + j] : 0.0;
      if (TA) {
        ga[u] = !same && kb < N && j < N ? A[kb * N + j] : 0.0;
      } else {
        const uint32_t i = e / MKC, k = k0 + e % MKC;                          // by columns
        ga[u] = i < N && k < N ? A[i * N + k] - (EYE && i == k ? 1.0 : 0.0) : 0.0;
      }
    }
  };
  const double* const pa = same ? L.B : L.A;
  load(0);
  for (uint32_t k0 = 0; k0 < N; k0 += MKC) {
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const uint32_t e = threadIdx.x + (uint32_t)SW * u;
      L.B[e / 128u * LDX + e % 128u] = gb[u];
      if (TA) {
        if (!same) L.A[e / 128u * LDX + e % 128u] = ga[u];
      } else {
        L.A[e / MKC * LDA + e % MKC] = ga[u];
      }
    }
    __syncthreads();
    if (k0 + MKC < N) load(k0 + MKC);
    if (o.has(0)) {
#pragma unroll 2
      for (uint32_t k = o.kr; k < MKC; k += 4) {
        const double a = TA ? pa[k * LDX + 16 * o.br + o.ci] : L.A[(16 * o.br + o.ci) * LDA + k];
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[b] = mma64(a, L.B[k * LDX + o.col(b)], acc[b]);
      }
    }
    __syncthreads();
  }
}

// Gauss-Jordan inversion of one 16 x 16 block by one wave, a pivot at a time; row
// P is register P / 4 of the lanes 16 (P % 4) ...  The next pivot's element is
// updated ahead of the others, by the same operations, and divided while they
// follow, so the division (the longest chain of a pivot) is hidden.  Returns
// whether a pivot was not a finite number above 1e-300.
__device__ __forceinline__ double inv16_recip(double piv, bool* bad) {
  const bool ok = isfinite(piv) && piv > 1e-300;
  *bad |= !ok;
  double q = 1.0 / piv;
  asm volatile("" : "+v"(q));                          // no branch around the division
  return ok ? q : 0.0;
}

template <int P>
__device__ __forceinline__ void inv16_pivot(v4d& w, double pinv, uint32_t kr, uint32_t ci, bool* bad) {
  constexpr int R = P >> 2, G = P & 3;
  double x = __shfl(w[R], (int)(16u * G + ci));        // row P at the lane's column
  double next = 0.0;
  if constexpr (P < 15) {
    constexpr int R1 = (P + 1) >> 2, G1 = (P + 1) & 3;
    const double a01 = lane_value(w[R], 16u * G + P + 1), a10 = lane_value(w[R1], 16u * G1 + P);
    const double a11 = lane_value(w[R1], 16u * G1 + P + 1);
    next = inv16_recip(fma(-a10, a01 * pinv, a11), bad);
  }
  const bool pc = ci == (uint32_t)P;
  x = (pc ? 1.0 : x) * pinv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double f = dpp_move<0x150 + P>(w[r]);        // column P at the lane's row
    const double v = fma(-f, x, pc ? 0.0 : w[r]);
    w[r] = (r == R && kr == (uint32_t)G) ? x : v;
  }
  if constexpr (P < 15) inv16_pivot<P + 1>(w, next, kr, ci, bad);
}

__device__ __forceinline__ bool inv16(v4d& w, uint32_t kr, uint32_t ci) {
  bool bad = false;
  const double pinv = inv16_recip(lane_value(w[0], 0u), &bad);
  inv16_pivot<0>(w, pinv, kr, ci, &bad);
  return bad;
}

// In-place inversion of the matrix in w (padded to whole blocks with the unit
// matrix), one block of 16 pivots per step.  With K the pivot indices, P = W[K,K]
// and X = P^{-1} [W[K,:] with W[K,K] replaced by I],
//   rows not in K:  W[i,:] <- W'[i,:] - W[i,K] X   (W' = W with columns K zeroed)
//   rows in K:      W[K,:] <- X.
// The wave that holds the next pivot block updates it first and inverts it while
// the others work, so a step has two barriers: after the pivot row, column and
// P^{-1} are published (R, F, P), and after X.  The serial chain of 16 pivots
// bounds a step: 4900 of 7000 clocks at N = 64, and 7900 of 11400 at N = 128, where
// the matrix instructions of the wave's neighbours delay it.  lds must be free; *bad is valid after the next barrier.
template <int CB>
__device__ void blk_invert(v4d (&w)[CB], const Blocks<CB>& o, SmallLds& lds, int* bad) {
  auto& L = lds.inv;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (uint32_t K = 0;; ++K) {
    // the update of step K - 1, then pivot block K
    double f[4];
    if (K > 0 && o.br < o.nb) {
#pragma unroll
      for (int s = 0; s < 4; ++s) f[s] = -L.F[~K & 1u][(16 * o.br + o.ci) * LDF + o.kr + 4 * s];
    }
    auto update = [&](int b) {
      if (o.br + 1 == K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) w[b][r] = L.X[(o.kr + 4 * r) * LDX + o.col(b)];
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) w[b] = mma64(f[s], L.X[(o.kr + 4 * s) * LDX + o.col(b)], w[b]);
      }
      __builtin_amdgcn_sched_barrier(0);               // one block's operands in registers at a time
    };
    const bool own = K < o.nb && o.br == K && o.bc0 <= K && K < o.bc0 + CB;
    if (own) {
      __builtin_amdgcn_s_setprio(3);                   // the others wait for this one
      v4d p;
#pragma unroll
      for (int b = 0; b < CB; ++b)
        if (o.bc0 + b == K) {
          if (K > 0) update(b);
          p = w[b];
        }
      if (inv16(p, o.kr, o.ci)) *bad = 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) L.P[(o.kr + 4 * r) * LDF + o.ci] = p[r];
      __builtin_amdgcn_s_setprio(0);
    }
    if (K > 0) {
#pragma unroll
      for (int b = 0; b < CB; ++b)
        if (o.has(b) && !(own && o.bc0 + b == K)) update(b);
    }
    if (K == o.nb) break;
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      if (o.br == K && o.has(b))
#pragma unroll
        for (int r = 0; r < 4; ++r) L.R[(o.kr + 4 * r) * LDX + o.col(b)] = w[b][r];
      if (o.br < o.nb && o.bc0 + b == K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          L.F[K & 1u][o.row(r) * LDF + o.ci] = w[b][r];
          w[b][r] = 0.0;
        }
      }
    }
    __syncthreads();
    if (wave < o.nb) {                                 // X, one block column per wave
      v4d x = {0.0, 0.0, 0.0, 0.0};
      if (wave == K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = L.P[(o.kr + 4 * r) * LDF + o.ci];
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
          x = mma64(L.P[o.ci * LDF + o.kr + 4 * s], L.R[(o.kr + 4 * s) * LDX + 16 * wave + o.ci], x);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) L.X[(o.kr + 4 * r) * LDX + 16 * wave + o.ci] = x[r];
    }
    __syncthreads();
  }
  __syncthreads();
}

// For the one-work-group kernels: the blocks per wave for N (see Blocks); fewer
// leave fewer waves idle (both kernels of a step at N = 96: 100 us with 3, about
// 125 with 4).
template <typename Go>
void with_blocks(uint32_t N, Go&& go) {
  if (N <= 64) go(std::integral_constant<int, 1>{});
  else if (N <= 96) go(std::integral_constant<int, 3>{});
  else go(std::integral_constant<int, 4>{});
}

// Energy, drift, |Lam|_F, column norms, and Lam^{-1} for the warm start.  N = 128:
// 55 us (109 with four pivots per step on the vector units).
template <int CB>
__global__ __launch_bounds__(SW) void k_prep_small(const double* __restrict__ C, const double* __restrict__ Lam,
                                                   double* __restrict__ Linv, double* __restrict__ cnorm2,
                                                   uint32_t N, OpeScalars* __restrict__ sc, float* __restrict__ Lam32,
                                                   float* __restrict__ Linv32) {
  __shared__ double red[3][16];
  __shared__ __align__(16) SmallLds lds;
  __shared__ int bad;
  const Blocks<CB> o(N);
  if (threadIdx.x == 0) bad = 0;
  v4d w[CB];
  double e = 0.0, lf = 0.0, dr = 0.0;
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      w[b][r] = i == j ? 1.0 : 0.0;
      if (i < N && j < N) {
        const double lij = Lam[i * N + j], lji = Lam[j * N + i], cij = C[i * N + j], d = cij - w[b][r];
        if (i == j) {
          e += lij;
          cnorm2[i] = cij;
        }
        w[b][r] = 0.5 * (lij + lji);
        if (Lam32) Lam32[i * N + j] = (float)lij;
        lf += lij * lij;
        dr += d * d;
      }
    }
  e = wave_sum(e);
  lf = wave_sum(lf);
  dr = wave_sum(dr);
  if ((threadIdx.x & 63u) == 0) {
    red[0][threadIdx.x >> 6] = e;
    red[1][threadIdx.x >> 6] = lf;
    red[2][threadIdx.x >> 6] = dr;
  }
  __syncthreads();
  blk_invert<CB>(w, o, lds, &bad);
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      if (i < N && j < N) {
        Linv[i * N + j] = w[b][r];
        if (Linv32) Linv32[i * N + j] = (float)w[b][r];
      }
    }
  if (threadIdx.x == 0) {
    e = lf = dr = 0.0;
    for (int u = 0; u < 16; ++u) {
      e += red[0][u];
      lf += red[1][u];
      dr += red[2][u];
    }
    sc->energy = 0.5 * e;
    sc->lam_fro = sqrt(lf);
    sc->drift = sqrt(dr);
    int err = 0;
    if (!isfinite(e) || !isfinite(lf) || !isfinite(dr)) err = OPE_ENONFINITE;
    else if (bad) err = OPE_EPIVOT;
    sc->err = err;                 // first writer of the step: resets earlier errors
  }
}

// Outer residual, inner tolerance and CG start state (one step of Algorithm 1).
__global__ __launch_bounds__(SW) void k_cg_setup(const double* __restrict__ rcol, const double* __restrict__ rho0,
                                                 const double* __restrict__ cnorm2, double eta_rel, double eta_floor,
                                                 uint32_t N, double* __restrict__ rho, double* __restrict__ target,
                                                 double* __restrict__ alpha, double* __restrict__ beta,
                                                 int32_t* __restrict__ active, OpeScalars* __restrict__ sc) {
  __shared__ double red[SW];
  double s = 0.0;
  for (uint32_t j = threadIdx.x; j < N; j += SW) s += rcol[j];
  s = wg_sum(s, red);
  const double res = sqrt(s) / sc->lam_fro;
  double eta = eta_rel * res;
  if (!(eta > eta_floor)) eta = eta_floor;
  for (uint32_t j = threadIdx.x; j < N; j += SW) {
    const double t = eta * eta * cnorm2[j];
    target[j] = t;
    rho[j] = rho0[j];
    alpha[j] = 0.0;
    alpha[N + j] = 0.0;        // both iteration-parity halves
    beta[j] = 0.0;
    active[j] = rho0[j] > t ? 1 : 0;
  }
  if (threadIdx.x == 0) {
    sc->cg_iters = 0;
    sc->residual = res;
    sc->eta = eta;
    if (!isfinite(res) && sc->err == 0) sc->err = OPE_ENONFINITE;
  }
}

// Stand-alone Step 1: tolerance relative to the column norms of U.
__global__ __launch_bounds__(SW) void k_solve_setup(const double* __restrict__ rho0, const double* __restrict__ unorm2,
                                                    double tol, uint32_t N, double* __restrict__ rho,
                                                    double* __restrict__ target, double* __restrict__ alpha,
                                                    double* __restrict__ beta, int32_t* __restrict__ active,
                                                    OpeScalars* __restrict__ sc) {
  for (uint32_t j = threadIdx.x; j < N; j += SW) {
    const double t = tol * tol * unorm2[j];
    target[j] = t;
    rho[j] = rho0[j];
    alpha[j] = 0.0;
    alpha[N + j] = 0.0;        // both iteration-parity halves
    beta[j] = 0.0;
    active[j] = rho0[j] > t ? 1 : 0;
  }
  if (threadIdx.x == 0) {
    sc->err = 0;
    sc->cg_iters = 0;
  }
}

// Steps 2-3: M = I + tau/2 (S_a - S_b) + tau^2/4 (T - S_a S_b), S_a = S_b^T,
// B = M^{-1}, A = 2/tau (I - B) + S_b B, Z = [I - tau A ; tau B].
//
// On one compute unit the FP64 matrix instructions take 14 us for each of the two
// products and for the inversion at N = 128; the rest is the inversion's pivots
// (about 300 clocks each, 128 of them in a row).  N = 128: 117 us, against 212 for
// four pivots at a time on the vector units and products read from LDS value by
// value; N = 17 15 against 32.
template <int CB>
__global__ __launch_bounds__(SW) void k_small_solve(const double* __restrict__ Sb, const double* __restrict__ T,
                                                    double tau, uint32_t N, double* Bws, double* __restrict__ Z,
                                                    double* __restrict__ Aout, OpeScalars* __restrict__ sc) {
  __shared__ __align__(16) SmallLds lds;
  __shared__ int bad;
  const Blocks<CB> o(N);
  if (threadIdx.x == 0) bad = 0;
  v4d w[CB], acc[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) acc[b] = v4d{0.0, 0.0, 0.0, 0.0};
  blk_mm<CB, true, false>(Sb, Sb, N, o, lds, acc);          // S_a S_b
  const double ht = 0.5 * tau, qt = 0.25 * tau * tau;
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      w[b][r] = i == j ? 1.0 : 0.0;
      if (i < N && j < N) w[b][r] += ht * (Sb[j * N + i] - Sb[i * N + j]) + qt * (T[i * N + j] - acc[b][r]);
      acc[b][r] = 0.0;
    }
  __syncthreads();
  blk_invert<CB>(w, o, lds, &bad);
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (o.row(r) < N && o.col(b) < N) Bws[o.row(r) * N + o.col(b)] = w[b][r];          // B
  __syncthreads();
  blk_mm<CB, false, false>(Sb, Bws, N, o, lds, acc);        // S_b B
  const double it = 2.0 / tau;
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      if (i < N && j < N) {
        const double bij = Bws[i * N + j];             // not kept in registers over the product
        const double dij = i == j ? 1.0 : 0.0, a = it * (dij - bij) + acc[b][r];
        Z[i * N + j] = dij - tau * a;
        Z[(N + i) * N + j] = tau * bij;
        if (Aout) Aout[i * N + j] = a;
      }
    }
  if (threadIdx.x == 0 && bad && sc->err == 0) sc->err = OPE_EPIVOT;
}

// Mixed-precision Steps 2-3 in delta form.  With P = Y - U S_b and
// C = <U,U>, T - S_a S_b = P^T P - S_b^T (C - I) S_b, so the Step-2 matrix is
// M = I + tau/2 (S_a - S_b) + tau^2/4 (P^T P - S_b^T (C - I) S_b), B = M^{-1},
// and Step 4 is U' = U + U Z1 + P Z2 with Z1 = -2 (I - B), Z2 = tau B: the
// same map as the FP64 step for any U, written so that both products vanish
// at a fixed point (their BF16 rounding vanishes with them).  The
// S_b^T (C - I) S_b term keeps the step orthogonality-preserving when the
// FP32 iterate has drifted; without it the drift is amplified at large tau.
// Z is written in FP32 (2N x N) for the BF16 product; Wsm is N x N scratch.
// N = 128: 112 us (294 before, as k_small_solve).
template <int CB>
__global__ __launch_bounds__(SW) void k_small_solve_delta(const double* __restrict__ Sb,
                                                          const double* __restrict__ Tp,
                                                          const double* __restrict__ C, double tau, uint32_t N,
                                                          double* Wsm, float* __restrict__ Z32,
                                                          OpeScalars* __restrict__ sc) {
  __shared__ __align__(16) SmallLds lds;
  __shared__ int bad;
  const Blocks<CB> o(N);
  if (threadIdx.x == 0) bad = 0;
  v4d w[CB], acc[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) acc[b] = v4d{0.0, 0.0, 0.0, 0.0};
  blk_mm<CB, false, true>(C, Sb, N, o, lds, acc);           // (C - I) S_b
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (o.row(r) < N && o.col(b) < N) Wsm[o.row(r) * N + o.col(b)] = acc[b][r];
      acc[b][r] = 0.0;
    }
  __syncthreads();
  blk_mm<CB, true, false>(Sb, Wsm, N, o, lds, acc);         // S_b^T (C - I) S_b
  const double ht = 0.5 * tau, qt = 0.25 * tau * tau;
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      w[b][r] = i == j ? 1.0 : 0.0;
      if (i < N && j < N) w[b][r] += ht * (Sb[j * N + i] - Sb[i * N + j]) + qt * (Tp[i * N + j] - acc[b][r]);
    }
  __syncthreads();
  blk_invert<CB>(w, o, lds, &bad);
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t i = o.row(r), j = o.col(b);
      if (i < N && j < N) {
        const double dij = i == j ? 1.0 : 0.0;
        Z32[i * N + j] = (float)(-2.0 * (dij - w[b][r]));
        Z32[(N + i) * N + j] = (float)(tau * w[b][r]);
      }
    }
  if (threadIdx.x == 0 && bad && sc->err == 0) sc->err = OPE_EPIVOT;
}

__global__ void k_to_f32(const double* __restrict__ src, float* __restrict__ dst, uint64_t count) {
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < count; e += (uint64_t)gridDim.x * blockDim.x)
    dst[e] = (float)src[e];
}

__global__ void k_to_f64(const float* __restrict__ src, double* __restrict__ dst, uint64_t count) {
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < count; e += (uint64_t)gridDim.x * blockDim.x)
    dst[e] = (double)src[e];
}

// ---------------------------------------------------------------------------
// Ritz values: eigenvalues of a symmetric N x N matrix (N <= 512) by a
// Householder tridiagonalisation in one work-group (Golub and Van Loan,
// "Matrix Computations", section 8.3.1: A <- A - v w^T - w v^T per column) and
// bisection on Sturm counts, one wave per eigenvalue.  Both are backward
// stable: every eigenvalue is within a small multiple of eps |A| of exact.
// The tridiagonalisation is a serial chain of N - 2 column steps, a few
// microseconds each.  Up to 128 columns the matrix stays in registers, bound by
// the instructions of a step; wider matrices stay in global memory (L2), two or
// more threads to a column, bound by one compute unit's L2 bandwidth.  Measured
// with the bisection (56 us at N = 128), ope_residual as a whole, against the
// parallel cyclic Jacobi iteration this replaces: 64^3, N = 128 4.5 to 12.0 (by its sweeps) -> 1.26 ms;
// N = 512 on 32^3 28 ms, where the Jacobi iteration alone took 1300 ms.
// ---------------------------------------------------------------------------

// Householder vector of x (entries k + 1 .. N - 1): v = x with the entry k + 1
// replaced by v0, beta = 2 / v^T v; e is the off-diagonal it leaves.  sigma: the
// sum of squares past the entry k + 1.  Up to tiny (house_tiny) those entries
// count as zero and x as already reduced (beta = 0): the squares of smaller ones
// lose their digits to the exponent range, and beta its finiteness.
struct House {
  double v0, beta, e;
  __device__ House(double alpha, double sigma, double tiny) {
    if (sigma <= tiny) {
      v0 = 0.0;
      beta = 0.0;
      e = alpha;
      return;
    }
    const double mu = sqrt(alpha * alpha + sigma);
    v0 = alpha >= 0.0 ? alpha + mu : alpha - mu;
    e = alpha >= 0.0 ? -mu : mu;
    beta = 1.0 / (mu * (mu + fabs(alpha)));
  }
};

// The line for a matrix A of Frobenius norm fro: what is dropped of a column moves
// the eigenvalues by at most 1e-22 |A|, far below a backward-stable method's
// eps |A| (or by 1e-145, where |A|^2 itself is that small).
__device__ __forceinline__ double house_tiny(double fro) { return fmax(1e-44 * fro * fro, 1e-290); }

// N <= 128, the matrix in the registers of four waves (thread t: column t % 128,
// rows t / 128 + 2 r; one wave per SIMD, since what every wave repeats below
// grows with their number: 16 waves of 16 rows took 462 us at N = 128).  Every
// wave holds all of v and w (lane l: entries l and l + 64), so forming them
// needs no barrier, and takes the entries of its rows (the same for all its
// lanes) from the lanes that hold them.
constexpr int TW = 256;       // threads
constexpr int TR = 64;        // rows per thread
constexpr int TB = 8;         // rows skipped together once they are reduced

__global__ __launch_bounds__(TW) void k_tridiag_reg(const double* __restrict__ Asrc, uint32_t N, const double* __restrict__ fro,
                                                    double* __restrict__ dg, double* __restrict__ od) {
  __shared__ double x[2][128];
  __shared__ double part[2][128];
  __shared__ double ds[128], es[128];             // written out at the end: a barrier waits for global stores
  const uint32_t lane = threadIdx.x & 63u, j = threadIdx.x & 127u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t q = wave >> 1;                   // row group
  const bool upper = (wave & 1u) != 0;            // the wave's columns: 64 + lane
  const double tiny = house_tiny(*fro);
  double w[TR];
#pragma unroll
  for (int r = 0; r < TR; ++r) {
    const uint32_t i = q + 2u * (uint32_t)r;
    w[r] = (i < N && j < N) ? 0.5 * (Asrc[(uint64_t)i * N + j] + Asrc[(uint64_t)j * N + i]) : 0.0;
  }
  for (uint32_t k = 0; k + 2 < N; ++k) {
    double* xk = x[k & 1u];
    // column k from the diagonal down
    if (j == k) {
#pragma unroll
      for (int r = 0; r < TR; ++r) {
        const uint32_t i = q + 2u * (uint32_t)r;
        xk[i] = i >= k ? w[r] : 0.0;
      }
    }
    __syncthreads();
    double va = xk[lane], vb = xk[lane + 64u];
    const double alpha = xk[k + 1u];
    if (threadIdx.x == 0) ds[k] = xk[k];
    const double sigma = wave_sum((lane > k + 1u ? va * va : 0.0) + (lane + 64u > k + 1u ? vb * vb : 0.0));
    const House h(alpha, sigma, tiny);
    if (threadIdx.x == 0) es[k] = h.e;
    if (h.beta == 0.0) continue;                  // uniform: every wave formed the same sums
    if (lane <= k + 1u) va = lane == k + 1u ? h.v0 : 0.0;
    if (lane + 64u <= k + 1u) vb = lane + 64u == k + 1u ? h.v0 : 0.0;
    // the thread's part of A v (columns by symmetry), v being zero up to row k
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < TR / TB; ++b) {
      if (q + 2u * (uint32_t)(TB * b + TB - 1) <= k) continue;
#pragma unroll
      for (int r = TB * b; r < TB * b + TB; ++r)
        s[r & 3] = fma(w[r], lane_value(r < 32 ? va : vb, q + 2u * (uint32_t)(r & 31)), s[r & 3]);
    }
    part[q][j] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    const double pa = h.beta * (part[0][lane] + part[1][lane]);
    const double pb = h.beta * (part[0][lane + 64u] + part[1][lane + 64u]);
    const double K = 0.5 * h.beta * wave_sum(pa * va + pb * vb);
    const double wa = pa - K * va, wb = pb - K * vb;
    const double vj = upper ? vb : va, wj = upper ? wb : wa;
#pragma unroll
    for (int b = 0; b < TR / TB; ++b) {
      if (q + 2u * (uint32_t)(TB * b + TB - 1) <= k) continue;
#pragma unroll
      for (int r = TB * b; r < TB * b + TB; ++r) {
        const uint32_t l = q + 2u * (uint32_t)(r & 31);
        w[r] -= lane_value(r < 32 ? va : vb, l) * wj + lane_value(r < 32 ? wa : wb, l) * vj;
      }
    }
    // `part` is rewritten only after the next barrier
  }
  // the last 2 x 2 block
#pragma unroll
  for (int r = 0; r < TR; ++r) {
    const uint32_t i = q + 2u * (uint32_t)r;
    if (i >= N) continue;
    if (i == j && i + 2 >= N) ds[i] = w[r];
    if (N >= 2 && i == N - 1 && j == N - 2) es[N - 2] = w[r];
  }
  __syncthreads();
  if (threadIdx.x < N) dg[threadIdx.x] = ds[threadIdx.x];
  if (threadIdx.x + 1 < N) od[threadIdx.x] = es[threadIdx.x];
}

// 128 < N <= 512, the matrix in global memory W: thread t owns the rows
// gi, gi + G, ... of column j (G groups of NC = N rounded up to 64 threads).
__global__ __launch_bounds__(SW) void k_tridiag(const double* __restrict__ Asrc, double* __restrict__ W, uint32_t N,
                                                const double* __restrict__ fro, double* __restrict__ dg,
                                                double* __restrict__ od) {
  __shared__ double x[2][512], ws[512], part[SW];
  __shared__ double ds[512], es[512];             // written out at the end
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t NC = (N + 63u) & ~63u, G = SW / NC;
  const uint32_t j = threadIdx.x % NC, gi = threadIdx.x / NC;
  const bool own = gi < G && j < N;
  const double tiny = house_tiny(*fro);
  if (own)
    for (uint32_t i = gi; i < N; i += G)
      W[(uint64_t)i * N + j] = 0.5 * (Asrc[(uint64_t)i * N + j] + Asrc[(uint64_t)j * N + i]);
  // column 0 (= row 0)
  if (own && gi == 0) x[0][j] = W[j];
  for (uint32_t k = 0; k + 2 < N; ++k) {
    double* xk = x[k & 1u];
    double* xn = x[(k + 1u) & 1u];
    __syncthreads();
    double sg = 0.0;
    for (uint32_t i = lane; i < N; i += 64u) sg += i > k + 1u ? xk[i] * xk[i] : 0.0;
    const double sigma = wave_sum(sg);
    const House h(xk[k + 1u], sigma, tiny);
    if (threadIdx.x == 0) {
      ds[k] = xk[k];
      es[k] = h.e;
    }
    auto v_at = [&](uint32_t i) -> double { return i == k + 1u ? h.v0 : (i > k ? xk[i] : 0.0); };
    // rows of this thread below k
    const uint32_t i0 = k + 1u + (gi + G - (k + 1u) % G) % G;
    if (h.beta != 0.0) {
      double s = 0.0;
      if (own && j > k) {
#pragma unroll 8
        for (uint32_t i = i0; i < N; i += G) s = fma(W[(uint64_t)i * N + j], v_at(i), s);
      }
      part[threadIdx.x] = s;
      __syncthreads();
      double pv = 0.0;
      for (uint32_t i = lane; i < N; i += 64u) {
        double t = 0.0;
        for (uint32_t g = 0; g < G; ++g) t += part[g * NC + i];
        pv += t * v_at(i);
      }
      const double K = 0.5 * h.beta * h.beta * wave_sum(pv);
      if (threadIdx.x < N) {
        double t = 0.0;
        for (uint32_t g = 0; g < G; ++g) t += part[g * NC + threadIdx.x];
        ws[threadIdx.x] = threadIdx.x > k ? h.beta * t - K * v_at(threadIdx.x) : 0.0;
      }
      __syncthreads();
      if (own && j > k) {
        const double vj = v_at(j), wj = ws[j];
#pragma unroll 8
        for (uint32_t i = i0; i < N; i += G) {
          const double t = W[(uint64_t)i * N + j] - (v_at(i) * wj + ws[i] * vj);
          W[(uint64_t)i * N + j] = t;
          if (i == k + 1u) xn[j] = t;
        }
      }
    } else if (own && j > k && i0 == k + 1u) {
      xn[j] = W[(uint64_t)(k + 1u) * N + j];
    }
  }
  // the last 2 x 2 block
  if (own)
    for (uint32_t i = gi; i < N; i += G) {
      if (i == j && i + 2 >= N) ds[i] = W[(uint64_t)i * N + i];
      if (i == N - 1 && j == N - 2) es[N - 2] = W[(uint64_t)i * N + j];
    }
  __syncthreads();
  if (threadIdx.x < N) dg[threadIdx.x] = ds[threadIdx.x];
  if (threadIdx.x + 1 < N) od[threadIdx.x] = es[threadIdx.x];
}

// Eigenvalue blockIdx.x (ascending) of the tridiagonal matrix (dg, od): the wave
// counts the eigenvalues below 64 points of the current interval at once
// (negative pivots of T - x I), so an interval shrinks 65-fold per round.  Twelve
// rounds reach neighbouring doubles from any interval up to 65^12 ulp wide.
__global__ __launch_bounds__(64) void k_bisect(const double* __restrict__ dg, const double* __restrict__ od, uint32_t N,
                                               double* __restrict__ evals) {
  __shared__ double d[512], e2[512];
  const uint32_t lane = threadIdx.x, k = blockIdx.x;
  double lo = INFINITY, hi = -INFINITY, em = 0.0;
  for (uint32_t i = lane; i < N; i += 64u) {
    const double di = dg[i], el = i > 0 ? od[i - 1] : 0.0, er = i + 1 < N ? od[i] : 0.0;
    d[i] = di;
    e2[i] = el * el;
    em = fmax(em, el * el);
    lo = fmin(lo, di - fabs(el) - fabs(er));
    hi = fmax(hi, di + fabs(el) + fabs(er));
  }
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, m));
    hi = fmax(hi, __shfl_xor(hi, m));
    em = fmax(em, __shfl_xor(em, m));
  }
  __syncthreads();
  // pivots smaller than this count as negative; e2 / pmin stays finite
  const double pmin = em * 1e-60 + 1e-200;
  const double slack = 4e-16 * fmax(fabs(lo), fabs(hi)) + pmin;
  lo -= slack;
  hi += slack;
  for (int round = 0; round < 12; ++round) {
    const double t = lo + (hi - lo) * ((double)(lane + 1u) * (1.0 / 65.0));
    uint32_t cnt = 0;
    double q = 1.0, r = 1.0;
    for (uint32_t i = 0; i < N; ++i) {
      q = (d[i] - t) - e2[i] * r;
      if (fabs(q) < pmin) q = -pmin;
      cnt += q < 0.0 ? 1u : 0u;
      r = __builtin_amdgcn_rcp(q);                // refined to within an ulp or so
      r = fma(r, fma(-q, r, 1.0), r);
      r = fma(r, fma(-q, r, 1.0), r);
    }
    // points with at most k eigenvalues below them lie at or left of eigenvalue k
    const uint64_t left = __ballot(cnt <= k);
    const int c = __popcll(left);                 // a prefix of the lanes, up to rounding
    const double a = c > 0 ? __shfl(t, c - 1) : lo, b = c < 64 ? __shfl(t, c) : hi;
    if (a == lo && b == hi) break;                // no point left inside
    lo = a;
    hi = b;
  }
  if (lane == 0) evals[k] = 0.5 * (lo + hi);
}

// ---------------------------------------------------------------------------
// N > 128: the same small phase from multi-work-group pieces.  Inverses by
// Newton-Schulz, X <- X (2I - M X), on the FP64 matrix cores (k_sqmm): it
// converges quadratically from X0 = M^T / (|M|_1 |M|_inf) for any
// non-singular M, and from X0 = I / |M|_inf for SPD M (Lam); the Step-2
// matrix has symmetric part >= I and Lam is SPD, so both are well
// conditioned.  A device-side state stops the iteration once
// |I - M X_k|_F <= 1e-10 (one more update then squares the error).
// ---------------------------------------------------------------------------

// one work-group: energy, |Lam|_F, drift, column norms, sym(Lam) into Ls,
// X0 = I / |Ls|_inf, and the Newton-Schulz state reset
__global__ __launch_bounds__(SW) void k_big_prep(const double* __restrict__ C, const double* __restrict__ Lam,
                                                 double* __restrict__ Ls, double* __restrict__ X0,
                                                 double* __restrict__ cnorm2, uint32_t N,
                                                 OpeScalars* __restrict__ sc, float* __restrict__ Lam32,
                                                 NsState* __restrict__ ns) {
  __shared__ double red[SW];
  double e = 0.0, lf = 0.0, dr = 0.0, rmax = 0.0;
  for (uint32_t i = threadIdx.x; i < N; i += SW) {
    double rs = 0.0;
    for (uint32_t j = 0; j < N; ++j) {
      const double lij = Lam[(uint64_t)i * N + j], lji = Lam[(uint64_t)j * N + i];
      const double ls = 0.5 * (lij + lji);
      Ls[(uint64_t)i * N + j] = ls;
      if (Lam32) Lam32[(uint64_t)i * N + j] = (float)lij;
      const double cij = C[(uint64_t)i * N + j] - (i == j ? 1.0 : 0.0);
      lf += lij * lij;
      dr += cij * cij;
      rs += fabs(ls);
    }
    e += Lam[(uint64_t)i * N + i];
    cnorm2[i] = C[(uint64_t)i * N + i];
    rmax = rs > rmax ? rs : rmax;
  }
  e = wg_sum(e, red);
  lf = wg_sum(lf, red);
  dr = wg_sum(dr, red);
  red[threadIdx.x] = rmax;
  __syncthreads();
  for (int s = SW / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  const double scale = red[0] > 0.0 ? 1.0 / red[0] : 0.0;
  for (uint32_t q = threadIdx.x; q < N * N; q += SW) X0[q] = (q % (N + 1) == 0) ? scale : 0.0;
  if (threadIdx.x == 0) {
    sc->energy = 0.5 * e;
    sc->lam_fro = sqrt(lf);
    sc->drift = sqrt(dr);
    int err = 0;
    if (!isfinite(e) || !isfinite(lf) || !isfinite(dr) || !(scale > 0.0)) err = OPE_ENONFINITE;
    sc->err = err;                 // first writer of the step: resets earlier errors
    ns->done = 0;
    ns->cur = 0;
    ns->upd_skip = 0;
    ns->iters = 0;
  }
}

// M = I + tau/2 (S_b^T - S_b) + tau^2/4 (T - P) (N^2 threads); with the
// transpose X0 = M^T / (|M|_1 |M|_inf) written by k_big_init.
__global__ void k_big_form_m(const double* __restrict__ Sb, const double* __restrict__ T,
                             const double* __restrict__ P, double tau, uint32_t N, double* __restrict__ M) {
  const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (uint64_t)N * N) return;
  const uint32_t i = (uint32_t)(q / N), j = (uint32_t)(q % N);
  M[q] = (i == j ? 1.0 : 0.0) + 0.5 * tau * (Sb[(uint64_t)j * N + i] - Sb[q]) + 0.25 * tau * tau * (T[q] - P[q]);
}

// one work-group: X0 = M^T / (|M|_1 |M|_inf), Newton-Schulz state reset
__global__ __launch_bounds__(SW) void k_big_init(const double* __restrict__ M, uint32_t N, double* __restrict__ X0,
                                                 NsState* __restrict__ ns, OpeScalars* __restrict__ sc) {
  __shared__ double red[SW];
  double rmax = 0.0, cmax = 0.0;
  for (uint32_t i = threadIdx.x; i < N; i += SW) {
    double rs = 0.0, cs = 0.0;
    for (uint32_t j = 0; j < N; ++j) {
      rs += fabs(M[(uint64_t)i * N + j]);
      cs += fabs(M[(uint64_t)j * N + i]);
    }
    rmax = rs > rmax ? rs : rmax;
    cmax = cs > cmax ? cs : cmax;
  }
  red[threadIdx.x] = rmax;
  __syncthreads();
  for (int s = SW / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  const double ninf = red[0];
  __syncthreads();
  red[threadIdx.x] = cmax;
  __syncthreads();
  for (int s = SW / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  const double n1 = red[0];
  const double a = (ninf > 0.0 && n1 > 0.0 && isfinite(ninf * n1)) ? 1.0 / (ninf * n1) : 0.0;
  for (uint32_t q = threadIdx.x; q < N * N; q += SW) {
    const uint32_t i = q / N, j = q % N;
    X0[q] = a * M[(uint64_t)j * N + i];
  }
  if (threadIdx.x == 0) {
    ns->done = 0;
    ns->cur = 0;
    ns->upd_skip = 0;
    ns->iters = 0;
    if (!(a > 0.0) && sc->err == 0) sc->err = OPE_EPIVOT;
  }
}

// after G = M X_k with its residual partials: |I - G|_F, the stop decision,
// and which buffer the update of iteration k writes
__global__ __launch_bounds__(256) void k_ns_check(const double* __restrict__ part, uint32_t nparts, uint32_t k,
                                                  NsState* __restrict__ ns) {
  __shared__ double red[256];
  if (ns->done) {
    if (threadIdx.x == 0) ns->upd_skip = 1;
    return;
  }
  double s = 0.0;
  for (uint32_t q = threadIdx.x; q < nparts; q += 256) s += part[q];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double r = sqrt(red[0]);
    ns->res = r;
    ns->iters = (int32_t)k + 1;
    ns->upd_skip = 0;
    ns->cur = (int32_t)((k + 1) & 1u);
    if (!isfinite(r)) {
      ns->done = 2;              // failed: no further iterations
      ns->upd_skip = 1;
      ns->cur = (int32_t)(k & 1u);
    } else if (r <= 1e-10) {
      ns->done = 1;              // this iteration's update is the last
    }
  }
}

// the inverse into Dst from the buffer holding it; sets EPIVOT if the
// iteration did not converge
__global__ void k_ns_take(const double* __restrict__ X0, const double* __restrict__ X1, uint32_t N,
                          const NsState* __restrict__ ns, double* __restrict__ Dst, float* __restrict__ Dst32,
                          OpeScalars* __restrict__ sc) {
  const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double* X = ns->cur ? X1 : X0;
  if (q < (uint64_t)N * N) {
    Dst[q] = X[q];
    if (Dst32) Dst32[q] = (float)X[q];
  }
  if (q == 0 && ns->done != 1 && sc->err == 0) sc->err = OPE_EPIVOT;
}

// Z = [I - tau A ; tau B] (FP64) or, for the delta form, Z32 = [-2 (I - B) ; tau B]
__global__ void k_big_z(const double* __restrict__ A, const double* __restrict__ B, double tau, uint32_t N,
                        double* __restrict__ Z, float* __restrict__ Z32) {
  const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (uint64_t)N * N) return;
  const uint32_t i = (uint32_t)(q / N), j = (uint32_t)(q % N);
  const double d = i == j ? 1.0 : 0.0;
  if (Z) {
    Z[q] = d - tau * A[q];
    Z[(uint64_t)N * N + q] = tau * B[q];
  } else {
    Z32[q] = (float)(-2.0 * (d - B[q]));
    Z32[(uint64_t)N * N + q] = (float)(tau * B[q]);
  }
}

// Z = (I - C) / 2, the correction of U <- U + U Z = U (3I - C) / 2
__global__ void k_renorm(const double* __restrict__ C, uint32_t N, float* __restrict__ Z) {
  const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (uint64_t)N * N) return;
  const uint32_t i = (uint32_t)(q / N), j = (uint32_t)(q % N);
  Z[q] = (float)(0.5 * ((i == j ? 1.0 : 0.0) - C[q]));
}

// Drift check after a mixed-precision update: drift = |C - I|_F of the new
// iterate (C = U^T U accumulated in FP64); above thr the next predicated
// product applies U <- U + U (I - C) / 2 = U (3 I - C) / 2, one Newton-Schulz
// step toward the nearest orthonormal block (drift E -> O(E^2)).  Z receives
// the correction (I - C) / 2: formed as U + U Z, its small terms are summed
// among themselves before U is added; as U (3I - C)/2 in FP32 they would be
// absorbed one by one into an accumulator of the size of U.
__global__ __launch_bounds__(SW) void k_drift_check(const double* __restrict__ C, uint32_t N, double thr,
                                                    float* __restrict__ Z, OpeScalars* __restrict__ sc) {
  __shared__ double red[SW];
  double s = 0.0;
  const uint64_t nn = (uint64_t)N * N;
  for (uint64_t q = threadIdx.x; q < nn; q += SW) {
    const uint32_t i = (uint32_t)(q / N), j = (uint32_t)(q % N);
    const double d = C[q] - (i == j ? 1.0 : 0.0);
    s += d * d;
    Z[q] = (float)(-0.5 * d);
  }
  s = wg_sum(s, red);
  if (threadIdx.x == 0) {
    const double drift = sqrt(s);
    sc->drift_after = drift;
    const int on = drift > thr && sc->err == 0 && isfinite(drift);
    sc->renorm = on;
    sc->renorms += on;
  }
}

__global__ void k_copy_pred(const void* __restrict__ src, void* __restrict__ dst, uint64_t words,
                            const OpeScalars* __restrict__ sc, int pred) {
  if ((pred & ROWMM_IF_OK) && sc->err != 0) return;
  if ((pred & ROWMM_IF_RENORM) && sc->renorm == 0) return;
  const uint64_t* s = (const uint64_t*)src;
  uint64_t* d = (uint64_t*)dst;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < words; e += (uint64_t)gridDim.x * blockDim.x)
    d[e] = s[e];
}

}  // namespace

// Newton-Schulz iterations on M (from X0 in ns_x[0]) in chunks of 8 with a
// host check of the device state between chunks; the inverse goes to Dst.
static hipError_t ns_invert(ope_ctx* c, const double* M, double* Dst, float* Dst32) {
  const uint32_t N = (uint32_t)c->N;
  const uint32_t t = (N + 63) / 64;
  hipError_t e;
  for (int k = 0; k < 96; ++k) {
    double* X = c->ns_x[k & 1];
    double* Xn = c->ns_x[(k + 1) & 1];
    if ((e = launch_sqmm(c, M, 0, X, 0, nullptr, 1.0, 0.0, 0.0, c->ns_g, N, &c->ns->done, c->ns_part)) != hipSuccess)
      return e;
    hipLaunchKernelGGL(k_ns_check, dim3(1), dim3(256), 0, c->stream, c->ns_part, t * t, (uint32_t)k, c->ns);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // X_{k+1} = 2 X_k - X_k G
    if ((e = launch_sqmm(c, X, 0, c->ns_g, 0, X, -1.0, 2.0, 0.0, Xn, N, &c->ns->upd_skip, nullptr)) != hipSuccess)
      return e;
    if (k % 8 == 7) {
      if ((e = hipMemcpyAsync(c->hns, c->ns, sizeof(NsState), hipMemcpyDeviceToHost, c->stream)) != hipSuccess)
        return e;
      if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return e;
      if (c->hns->done) break;
    }
  }
  const uint64_t nn = (uint64_t)N * N;
  hipLaunchKernelGGL(k_ns_take, dim3((uint32_t)((nn + 255) / 256)), dim3(256), 0, c->stream, c->ns_x[0], c->ns_x[1],
                     N, c->ns, Dst, Dst32, c->sc);
  return hipGetLastError();
}

static hipError_t big_prep(ope_ctx* c) {
  const uint32_t N = (uint32_t)c->N;
  hipLaunchKernelGGL(k_big_prep, dim3(1), dim3(SW), 0, c->stream, c->C, c->Lam, c->ns_m, c->ns_x[0], c->cnorm2, N,
                     c->sc, c->Lam32, c->ns);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return ns_invert(c, c->ns_m, c->Linv, c->Linv32);
}

// B = M^{-1} for M = I + tau/2 (S_b^T - S_b) + tau^2/4 (T' - P), P in ns_p
static hipError_t big_form_and_invert(ope_ctx* c, const double* Sb, const double* Tp, double tau, double* B) {
  const uint32_t N = (uint32_t)c->N;
  const uint64_t nn = (uint64_t)N * N;
  hipLaunchKernelGGL(k_big_form_m, dim3((uint32_t)((nn + 255) / 256)), dim3(256), 0, c->stream, Sb, Tp, c->ns_p, tau,
                     N, c->ns_m);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_big_init, dim3(1), dim3(SW), 0, c->stream, c->ns_m, N, c->ns_x[0], c->ns, c->sc);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return ns_invert(c, c->ns_m, B, nullptr);
}

static hipError_t big_small_solve(ope_ctx* c, const double* Sb, const double* T, double tau, double* Z, double* A,
                                  double* B) {
  const uint32_t N = (uint32_t)c->N;
  const uint64_t nn = (uint64_t)N * N;
  hipError_t e;
  // P = S_a S_b = S_b^T S_b
  if ((e = launch_sqmm(c, Sb, 1, Sb, 0, nullptr, 1.0, 0.0, 0.0, c->ns_p, N, nullptr, nullptr)) != hipSuccess) return e;
  if ((e = big_form_and_invert(c, Sb, T, tau, B)) != hipSuccess) return e;
  // A = 2/tau (I - B) + S_b B
  double* Aw = A ? A : c->A;
  if ((e = launch_sqmm(c, Sb, 0, B, 0, B, 1.0, -2.0 / tau, 2.0 / tau, Aw, N, nullptr, nullptr)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_big_z, dim3((uint32_t)((nn + 255) / 256)), dim3(256), 0, c->stream, Aw, B, tau, N, Z,
                     (float*)nullptr);
  return hipGetLastError();
}

static hipError_t big_small_solve_delta(ope_ctx* c, const double* Sb, const double* Tp, double tau) {
  const uint32_t N = (uint32_t)c->N;
  const uint64_t nn = (uint64_t)N * N;
  hipError_t e;
  // Wsm = (C - I) S_b = C S_b - S_b ; P = S_b^T Wsm
  if ((e = launch_sqmm(c, c->C, 0, Sb, 0, Sb, 1.0, -1.0, 0.0, c->Wsm, N, nullptr, nullptr)) != hipSuccess) return e;
  if ((e = launch_sqmm(c, Sb, 1, c->Wsm, 0, nullptr, 1.0, 0.0, 0.0, c->ns_p, N, nullptr, nullptr)) != hipSuccess)
    return e;
  if ((e = big_form_and_invert(c, Sb, Tp, tau, c->B)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_big_z, dim3((uint32_t)((nn + 255) / 256)), dim3(256), 0, c->stream, (const double*)nullptr,
                     c->B, tau, N, (double*)nullptr, c->Z32);
  return hipGetLastError();
}

hipError_t launch_renorm_matrix(ope_ctx* c, const double* C, float* Z32) {
  const uint64_t nn = (uint64_t)c->N * c->N;
  hipLaunchKernelGGL(k_renorm, dim3((uint32_t)((nn + 255) / 256)), dim3(256), 0, c->stream, C, (uint32_t)c->N, Z32);
  return hipGetLastError();
}

hipError_t launch_copy_pred(ope_ctx* c, const void* src, void* dst, uint64_t bytes, int pred) {
  uint64_t words = bytes / 8;
  uint64_t grid = (words + 255) / 256;
  if (grid > 8192) grid = 8192;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_copy_pred, dim3((uint32_t)grid), dim3(256), 0, c->stream, src, dst, words, c->sc, pred);
  return hipGetLastError();
}

hipError_t launch_drift_check(ope_ctx* c, const double* C, float* Z32, double thr) {
  hipLaunchKernelGGL(k_drift_check, dim3(1), dim3(SW), 0, c->stream, C, (uint32_t)c->N, thr, Z32, c->sc);
  return hipGetLastError();
}

hipError_t launch_prep_small(ope_ctx* c) {
  if (c->N > OPE_MAX_N_ONE_WG) return big_prep(c);
  ProfScope ps(c, OPE_KERNEL_SMALL);
  with_blocks((uint32_t)c->N, [&](auto cb) {
    hipLaunchKernelGGL((k_prep_small<decltype(cb)::value>), dim3(1), dim3(SW), 0, c->stream, c->C, c->Lam, c->Linv,
                       c->cnorm2, (uint32_t)c->N, c->sc, c->Lam32, c->Linv32);
  });
  return hipGetLastError();
}

hipError_t launch_small_solve_delta(ope_ctx* c, const double* Sb, const double* Tperp, double tau) {
  if (c->N > OPE_MAX_N_ONE_WG) return big_small_solve_delta(c, Sb, Tperp, tau);
  ProfScope ps(c, OPE_KERNEL_SMALL);
  with_blocks((uint32_t)c->N, [&](auto cb) {
    hipLaunchKernelGGL((k_small_solve_delta<decltype(cb)::value>), dim3(1), dim3(SW), 0, c->stream, Sb, Tperp, c->C,
                       tau, (uint32_t)c->N, c->Wsm, c->Z32, c->sc);
  });
  return hipGetLastError();
}

hipError_t launch_small_to_f32(ope_ctx* c, const double* src, float* dst, int64_t count) {
  hipLaunchKernelGGL(k_to_f32, dim3(64), dim3(256), 0, c->stream, src, dst, (uint64_t)count);
  return hipGetLastError();
}

hipError_t launch_convert(ope_ctx* c, const void* src, void* dst, int64_t count, int to_double) {
  const uint64_t n = (uint64_t)count;
  uint64_t grid = (n + 255) / 256;
  if (grid > 8192) grid = 8192;
  if (grid < 1) grid = 1;
  if (to_double)
    hipLaunchKernelGGL(k_to_f64, dim3((uint32_t)grid), dim3(256), 0, c->stream, (const float*)src, (double*)dst, n);
  else
    hipLaunchKernelGGL(k_to_f32, dim3((uint32_t)grid), dim3(256), 0, c->stream, (const double*)src, (float*)dst, n);
  return hipGetLastError();
}

hipError_t launch_cg_setup(ope_ctx* c, const double* rho0, const double* rcol) {
  hipLaunchKernelGGL(k_cg_setup, dim3(1), dim3(SW), 0, c->stream, rcol, rho0, c->cnorm2, c->eta_rel, c->eta_floor,
                     (uint32_t)c->N, c->rho, c->target, c->alpha, c->beta, c->active, c->sc);
  return hipGetLastError();
}

hipError_t launch_solve_setup(ope_ctx* c, const double* rho0, double tol) {
  hipLaunchKernelGGL(k_solve_setup, dim3(1), dim3(SW), 0, c->stream, rho0, c->cnorm2, tol, (uint32_t)c->N, c->rho,
                     c->target, c->alpha, c->beta, c->active, c->sc);
  return hipGetLastError();
}

hipError_t launch_small_solve(ope_ctx* c, const double* Sb, const double* T, double tau, double* Z, double* A,
                              double* B) {
  if (c->N > OPE_MAX_N_ONE_WG) return big_small_solve(c, Sb, T, tau, Z, A, B ? B : c->B);
  ProfScope ps(c, OPE_KERNEL_SMALL);
  with_blocks((uint32_t)c->N, [&](auto cb) {
    hipLaunchKernelGGL((k_small_solve<decltype(cb)::value>), dim3(1), dim3(SW), 0, c->stream, Sb, T, tau,
                       (uint32_t)c->N, B ? B : c->B, Z, A, c->sc);
  });
  return hipGetLastError();
}

hipError_t launch_lam_eig(ope_ctx* c, double* evals) {
  const uint32_t N = (uint32_t)c->N;
  double *dg = c->B, *od = c->B + N;               // scratch between steps; 2 N - 1 values (N = 1: one)
  if (N <= OPE_MAX_N_ONE_WG)
    hipLaunchKernelGGL(k_tridiag_reg, dim3(1), dim3(TW), 0, c->stream, c->Lam, N, &c->sc->lam_fro, dg, od);
  else
    hipLaunchKernelGGL(k_tridiag, dim3(1), dim3(SW), 0, c->stream, c->Lam, c->Wsm, N, &c->sc->lam_fro, dg, od);
  hipLaunchKernelGGL(k_bisect, dim3(N), dim3(64), 0, c->stream, dg, od, N, evals);
  return hipGetLastError();
}
