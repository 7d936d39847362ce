// Multigrid V-cycle: the preconditioner of Step 1's preconditioned CG
// (ope_set_multigrid).  Step 1 of the scheme (Section 4.1) solves the N source
// problems H y_j = u_j; the paper leaves the solver open.  One symmetric
// V-cycle per CG iteration takes the iteration count of the warm-started
// Step 1 at 64^3 from about seventy to about five.
//
// Hierarchy (built on the host at set-up): level k+1 halves every axis with
// more than one node (m' = ceil(m / 2); coarse node I is the parent of fine
// nodes 2I and 2I + 1), doubles its spacing (c_a' = c_a / 4), and takes as
// potential the mean of V + shift over the existing children; the first level
// k >= 1 with at most 64 nodes is solved exactly with a dense inverse
// (Cholesky on the host).  Transfers per coarsened axis: prolongation
// 3/4 e_I + 1/4 e_J (J = I - 1 for even fine nodes, I + 1 for odd ones,
// missing J = 0), restriction R = P^T / 2^d.  V-cycle, damped Jacobi
// (omega = 0.8) once on each side of the coarse correction:
//   x0 = omega b / d;  r1 = b - H x0;  e = B_{k+1}(R r1);  x1 = x0 + P e;
//   z = x1 + omega (b - H x1) / d.
// Kernels, per level: k_mg_tstencil (r1, one stencil over x0 formed on the
// fly from b), k_mg_zrestrict (R r1), k_mg_tpost (x1 = x0 + P e and z, one
// stencil over x1; on level 0 also the per-column partial sums of r^T z and
// r^T r that the PCG needs); from the first level of at most MC_MAX nodes down
// (as many levels as MC_LEVELS and MC_LDS hold), all in one launch (k_mg_coarse).  The
// stencil and transfer kernels march along z (see zmarch_shape, tshape); the
// smoother's factors omega / d are precomputed per level.
// Layout: every block is n x N row-major (a grid point's N values
// contiguous), x fastest, as everywhere in the library; a thread owns one
// 16-byte chunk (VW elements) or one element of a point's row, FP64, or
// FP32 for mixed-precision contexts (dot products accumulated in FP64).  Columns
// whose CG has converged are skipped, and keep what the last V-cycle that ran them
// left, which the first one of every CG has for all columns (pcg_begin).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "ope_internal.h"

namespace {

constexpr double MG_OMEGA = 0.8;
constexpr int64_t MG_COARSEST_MAX = 64;
constexpr uint32_t MG_WG = 256;

struct MgGeom {
  uint32_t m0, m1, m2;
  double cx, cy, cz;
};

// VW consecutive elements of a point's row (16 bytes or less), loaded and
// stored as one access.
template <typename T, int VW>
struct alignas(sizeof(T) * VW) Chunk {
  T v[VW];
};

template <typename T, int VW>
__device__ __forceinline__ void ldr(const T* __restrict__ a, uint64_t row, uint32_t N, uint32_t v, T (&o)[VW]) {
  const Chunk<T, VW> t = *reinterpret_cast<const Chunk<T, VW>*>(a + row * N + (uint64_t)VW * v);
#pragma unroll
  for (int k = 0; k < VW; ++k) o[k] = t.v[k];
}

template <typename T, int VW>
__device__ __forceinline__ void str(T* __restrict__ a, uint64_t row, uint32_t N, uint32_t v, const T (&o)[VW]) {
  Chunk<T, VW> t;
#pragma unroll
  for (int k = 0; k < VW; ++k) t.v[k] = o[k];
  *reinterpret_cast<Chunk<T, VW>*>(a + row * N + (uint64_t)VW * v) = t;
}

template <typename T, int VW>
__device__ __forceinline__ void zero(T (&a)[VW]) {
#pragma unroll
  for (int k = 0; k < VW; ++k) a[k] = T(0);
}

template <int VW>
__device__ __forceinline__ bool vec_active(const int32_t* __restrict__ active, uint32_t v) {
  if (!active) return true;
  bool a = false;
#pragma unroll
  for (int k = 0; k < VW; ++k) a |= active[v * VW + k] != 0;
  return a;
}

// VW elements at a lane's byte offset `o` into a plane whose pointer is the same
// for the whole wave.  A lane's columns do not change over a march along z, so
// its offsets are formed once and a plane costs one scalar addition instead of a
// 64-bit multiplication per access.  O is 32 bits wide where a plane of every
// array is smaller than 4 GiB (narrow_planes), else 64.
template <typename T, int VW, typename O>
__device__ __forceinline__ void ldo(const T* __restrict__ plane, O o, T (&v)[VW]) {
  const Chunk<T, VW> t = *reinterpret_cast<const Chunk<T, VW>*>(reinterpret_cast<const char*>(plane) + o);
#pragma unroll
  for (int k = 0; k < VW; ++k) v[k] = t.v[k];
}

template <typename T, int VW, typename O>
__device__ __forceinline__ void sto(T* __restrict__ plane, O o, const T (&v)[VW]) {
  Chunk<T, VW> t;
#pragma unroll
  for (int k = 0; k < VW; ++k) t.v[k] = v[k];
  *reinterpret_cast<Chunk<T, VW>*>(reinterpret_cast<char*>(plane) + o) = t;
}

// Fine nodes and weights of coarse node I along one axis: always four taps
// (2I - 1, 2I, 2I + 1, 2I + 2 with weights 1/8, 3/8, 3/8, 1/8, the factor 1/2
// of R = P^T / 2^d included), a missing node clamped into the grid with weight
// zero; an axis that is not coarsened has the one tap I with weight 1.  The
// fixed count lets every load of a gather be issued before the first is used.
__device__ __forceinline__ void restrict_taps(uint32_t I, uint32_t mf, uint32_t (&f)[4], double (&w)[4]) {
  const bool one = mf == 1;                       // uniform: selects, no branch
  const uint32_t c = one ? I : 2 * I;
  f[0] = I > 0 ? c - 1 : c;
  f[1] = c;
  f[2] = c + 1 < mf ? c + 1 : c;
  f[3] = c + 2 < mf ? c + 2 : c;
  w[0] = I > 0 ? 0.125 : 0.0;
  w[1] = one ? 1.0 : 0.375;
  w[2] = c + 1 < mf ? 0.375 : 0.0;
  w[3] = c + 2 < mf ? 0.125 : 0.0;
}

// Coarse nodes and weights of fine node f along one axis: always two taps,
// the parent f / 2 with 3/4 and the other neighbour (f / 2 - 1 for even f,
// f / 2 + 1 for odd f) with 1/4, or weight zero (clamped to the parent) when
// it is missing; an axis that is not coarsened has the tap f with weight 1.
__device__ __forceinline__ void prolong_taps(uint32_t f, uint32_t mf, uint32_t mc, uint32_t (&I)[2], double (&w)[2]) {
  const bool one = mf == 1;                       // uniform: selects, no branch
  const uint32_t h = f / 2;                       // (0 on an axis that is not coarsened)
  const bool odd = (f & 1u) != 0;
  const bool in = odd ? h + 1 < mc : h > 0;
  I[0] = h;
  I[1] = in ? (odd ? h + 1 : h - 1) : h;
  w[0] = one ? 1.0 : 0.75;
  w[1] = in ? 0.25 : 0.0;
}

// ---------------------------------------------------------------------------
// The coarse end of a V-cycle in one launch.  From the first level of at most
// MC_MAX nodes down, one work-group takes one column through every level: the
// field being smoothed and each level's right-hand side and correction stay in
// LDS, the coarsest level is a product with the dense inverse.  The levels'
// own launches (three per level) move next to nothing and cost a launch's 4-5 us
// each, one after the other: at 64^3, N = 17, the four launches from the 8^3
// level down took 23 us, this one 7.5 us (8.3 at N = 128).  Bound by the
// instructions of one compute unit per column (about 2000 per thread with two
// levels), which is why the line is not drawn higher: with the 16^3 level in it,
// it took 27 us, against 16 us for that level's three launches.
// ---------------------------------------------------------------------------
constexpr uint32_t MC_MAX = 2048;                 // nodes of the first fused level
constexpr uint32_t MC_WG = 512;
constexpr uint32_t MC_PPT = MC_MAX / MC_WG;       // nodes per thread
constexpr int MC_LEVELS = 8;                      // levels fused (at most)
constexpr size_t MC_LDS = 131072;                 // LDS bytes of the fused levels (at most)

struct McLevel {
  uint32_t m0, m1, m2, n;
  uint32_t mag0, mag1;                            // ceil(2^32 / m) of m0 and m1 (0 for m = 1), for divisions of i < 2^16
  uint32_t b, e, wd, dg;                          // LDS offsets below the first level: right-hand side, correction,
                                                  // omega / diagonal, diagonal
  double cx, cy, cz;
};
struct McArgs {
  int32_t nl;                                     // levels, the last one solved with inv
  uint32_t cst, ncst;                             // LDS offset and length of the lower levels' constants
  const double *diag0, *wd0;                      // the first level's diagonal and omega / diagonal
  const double* cdat;                             // the lower levels' (the order of the LDS offsets)
  const double* inv;
  McLevel lv[MC_LEVELS];
};

struct McNode {
  uint32_t x, y, z;
};
__device__ __forceinline__ McNode mc_node(const McLevel& L, uint32_t i) {
  McNode q;
  const uint32_t r = L.mag0 ? __umulhi(i, L.mag0) : i;
  q.x = i - r * L.m0;
  q.z = L.mag1 ? __umulhi(r, L.mag1) : r;
  q.y = r - q.z * L.m1;
  return q;
}

// (H f)_i for the level's field f in LDS, d its diagonal there; f[n] is the zero
// that stands for every neighbour outside the grid
template <typename T>
__device__ __forceinline__ T mc_apply(const McLevel& L, const T* f, uint32_t i, T d) {
  const McNode q = mc_node(L, i);
  const uint32_t s1 = L.m0, s2 = L.m0 * L.m1;
  const T xs = f[q.x > 0 ? i - 1 : L.n] + f[q.x + 1 < L.m0 ? i + 1 : L.n];
  const T ys = f[q.y > 0 ? i - s1 : L.n] + f[q.y + 1 < L.m1 ? i + s1 : L.n];
  const T zs = f[q.z > 0 ? i - s2 : L.n] + f[q.z + 1 < L.m2 ? i + s2 : L.n];
  return d * f[i] - ((T)L.cx * xs + (T)L.cy * ys + (T)L.cz * zs);
}

// (R f)_i of the finer level L's field f at node i of the coarser level C
template <typename T>
__device__ __forceinline__ T mc_restrict(const McLevel& L, const McLevel& C, const T* f, uint32_t i) {
  const McNode q = mc_node(C, i);
  uint32_t fx[4], fy[4], fz[4];
  double wx[4], wy[4], wz[4];
  restrict_taps(q.x, L.m0, fx, wx);
  restrict_taps(q.y, L.m1, fy, wy);
  restrict_taps(q.z, L.m2, fz, wz);
  T o = T(0);
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {
    T az = T(0);
#pragma unroll
    for (int bb = 0; bb < 4; ++bb) {
      const T* row = f + (fz[cc] * L.m1 + fy[bb]) * L.m0;
      T ax = T(0);
#pragma unroll
      for (int aa = 0; aa < 4; ++aa) ax += (T)wx[aa] * row[fx[aa]];
      az += (T)wy[bb] * ax;
    }
    o += (T)wz[cc] * az;
  }
  return o;
}

// (P e)_i at node i of the finer level L from the coarser level C's e
template <typename T>
__device__ __forceinline__ T mc_prolong(const McLevel& L, const McLevel& C, const T* e, uint32_t i) {
  const McNode q = mc_node(L, i);
  uint32_t Ix[2], Iy[2], Iz[2];
  double wx[2], wy[2], wz[2];
  prolong_taps(q.x, L.m0, C.m0, Ix, wx);
  prolong_taps(q.y, L.m1, C.m1, Iy, wy);
  prolong_taps(q.z, L.m2, C.m2, Iz, wz);
  T o = T(0);
#pragma unroll
  for (int cc = 0; cc < 2; ++cc) {
    T az = T(0);
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      const T* row = e + (Iz[cc] * C.m1 + Iy[bb]) * C.m0;
      az += (T)wy[bb] * ((T)wx[0] * row[Ix[0]] + (T)wx[1] * row[Ix[1]]);
    }
    o += (T)wz[cc] * az;
  }
  return o;
}

// Every global load is issued before the first phase (the first level's values
// and the inverse's rows into registers, the lower levels' constants into LDS):
// a load inside a phase would put an L2 latency between two barriers.
template <typename T>
__global__ __launch_bounds__(MC_WG, 4) void k_mg_coarse(const T* __restrict__ B, T* __restrict__ E, McArgs a,
                                                     const int32_t* __restrict__ active, uint32_t N) {
  extern __shared__ __align__(16) char mc_lds[];
  T* const s = reinterpret_cast<T*>(mc_lds);
  T* const f = s;                                 // the field: n values of the level at hand and the zero
  const uint32_t t = threadIdx.x;
  const uint32_t col = xcd_remap(blockIdx.x, gridDim.x);
  if (active && active[col] == 0) return;         // uniform over the work-group
  const McLevel& L0 = a.lv[0];
  const McLevel& LC = a.lv[a.nl - 1];
  T b0[MC_PPT], w0[MC_PPT], d0[MC_PPT], iv[8];    // iv: entries p + 8 u of row t / 8 of the inverse
#pragma unroll
  for (uint32_t u = 0; u < MC_PPT; ++u) b0[u] = B[(uint64_t)min(t + u * MC_WG, L0.n - 1) * N + col];
#pragma unroll
  for (uint32_t u = 0; u < MC_PPT; ++u) {
    const uint32_t i = min(t + u * MC_WG, L0.n - 1);
    w0[u] = (T)a.wd0[i];
    d0[u] = (T)a.diag0[i];
  }
  const uint32_t ri = t / 8u, rp = t % 8u;
#pragma unroll
  for (uint32_t u = 0; u < 8; ++u)
    iv[u] = (ri < LC.n && rp + 8 * u < LC.n) ? (T)a.inv[ri * LC.n + rp + 8 * u] : T(0);
  for (uint32_t i = t; i < a.ncst; i += MC_WG) s[a.cst + i] = (T)a.cdat[i];
  if (a.nl == 1) {
    // the coarsest level alone
#pragma unroll
    for (uint32_t u = 0; u < MC_PPT; ++u)
      if (t + u * MC_WG < L0.n) f[t + u * MC_WG] = b0[u];
  } else {
    // first level, down
#pragma unroll
    for (uint32_t u = 0; u < MC_PPT; ++u)
      if (t + u * MC_WG < L0.n) f[t + u * MC_WG] = w0[u] * b0[u];
    if (t == 0) f[L0.n] = T(0);
    __syncthreads();
    T r[MC_PPT];                                  // r1 = b - H x0 replaces x0 once every thread has read it
#pragma unroll
    for (uint32_t u = 0; u < MC_PPT; ++u) {
      const uint32_t i = t + u * MC_WG;
      r[u] = i < L0.n ? b0[u] - mc_apply(L0, f, i, d0[u]) : T(0);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < MC_PPT; ++u)
      if (t + u * MC_WG < L0.n) f[t + u * MC_WG] = r[u];
    __syncthreads();
    for (uint32_t i = t; i < a.lv[1].n; i += MC_WG) s[a.lv[1].b + i] = mc_restrict(L0, a.lv[1], f, i);
  }
  __syncthreads();
  for (int k = 1; k + 1 < a.nl; ++k) {            // the lower levels, down
    const McLevel& L = a.lv[k];
    const McLevel& C = a.lv[k + 1];
    const T *b = s + L.b, *wd = s + L.wd, *dg = s + L.dg;
    T* e = s + L.e;                               // r1 until the correction takes its place
    for (uint32_t i = t; i < L.n; i += MC_WG) f[i] = wd[i] * b[i];
    if (t == 0) f[L.n] = T(0);
    __syncthreads();
    for (uint32_t i = t; i < L.n; i += MC_WG) e[i] = b[i] - mc_apply(L, f, i, dg[i]);
    __syncthreads();
    for (uint32_t i = t; i < C.n; i += MC_WG) s[C.b + i] = mc_restrict(L, C, e, i);
    __syncthreads();
  }
  {
    // e = A^{-1} b on the coarsest level: eight threads to a row
    const T* b = a.nl == 1 ? f : s + LC.b;
    T v = T(0);
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u)
      if (rp + 8 * u < LC.n) v += iv[u] * b[rp + 8 * u];
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    if (ri < LC.n && rp == 0) {
      if (a.nl == 1) E[(uint64_t)ri * N + col] = v;
      else s[LC.e + ri] = v;
    }
    if (a.nl == 1) return;
    __syncthreads();
  }
  for (int k = a.nl - 2; k >= 1; --k) {           // the lower levels, up
    const McLevel& L = a.lv[k];
    const McLevel& C = a.lv[k + 1];
    const T *b = s + L.b, *wd = s + L.wd, *dg = s + L.dg;
    for (uint32_t i = t; i < L.n; i += MC_WG) f[i] = wd[i] * b[i] + mc_prolong(L, C, s + C.e, i);
    if (t == 0) f[L.n] = T(0);
    __syncthreads();
    for (uint32_t i = t; i < L.n; i += MC_WG) s[L.e + i] = f[i] + wd[i] * (b[i] - mc_apply(L, f, i, dg[i]));
    __syncthreads();
  }
  // first level, up
#pragma unroll
  for (uint32_t u = 0; u < MC_PPT; ++u) {
    const uint32_t i = t + u * MC_WG;
    if (i < L0.n) f[i] = w0[u] * b0[u] + mc_prolong(L0, a.lv[1], s + a.lv[1].e, i);
  }
  if (t == 0) f[L0.n] = T(0);
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < MC_PPT; ++u) {
    const uint32_t i = t + u * MC_WG;
    if (i < L0.n) E[(uint64_t)i * N + col] = f[i] + w0[u] * (b0[u] - mc_apply(L0, f, i, d0[u]));
  }
}

// z-march decomposition of a level: a work-group owns PL = 256 / NV
// consecutive x nodes (thread t: vector t % NV of node t / NV) of one y row
// over ZC consecutive z planes, keeping the field of the planes below, at and
// above the current one in registers; work-groups are numbered x segment
// fastest, then y, then z range, and spread XCD-contiguously, so one XCD
// streams neighbouring rows of the same planes (their y neighbours hit L2).
struct ZMarch {
  uint32_t PL, nxs, nzc, ZC;
};

ZMarch zmarch_shape(uint32_t m0, uint32_t m1, uint32_t m2, uint32_t NV) {
  ZMarch s;
  s.PL = MG_WG / NV;
  s.nxs = (m0 + s.PL - 1) / s.PL;
  const uint64_t cols = (uint64_t)s.nxs * m1;
  uint64_t nzc = (2048 + cols - 1) / cols;          // at least 2048 work-groups when the grid allows
  if (nzc > m2) nzc = m2;
  if (nzc < 1) nzc = 1;
  s.ZC = (uint32_t)((m2 + nzc - 1) / nzc);
  s.nzc = (m2 + s.ZC - 1) / s.ZC;
  return s;
}

struct ZPos {
  uint32_t x, y, z0, z1, v;
  bool ok;
};

template <int VW>
__device__ __forceinline__ ZPos zpos(const MgGeom& g, const ZMarch& zs, const int32_t* __restrict__ active,
                                     uint32_t NV) {
  ZPos q;
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t xs = L % zs.nxs, r = L / zs.nxs;
  q.y = r % g.m1;
  const uint32_t zc = r / g.m1;
  const uint32_t t = threadIdx.x;
  const bool lane_ok = t < zs.PL * NV;
  q.v = lane_ok ? t % NV : 0;
  q.x = xs * zs.PL + (lane_ok ? t / NV : 0);
  q.z0 = zc * zs.ZC;
  q.z1 = q.z0 + zs.ZC < g.m2 ? q.z0 + zs.ZC : g.m2;
  q.ok = lane_ok && q.x < g.m0 && vec_active<VW>(active, q.v);
  return q;
}

// x-y tiled form of the stencil sweeps: a work-group of TX TY NVS threads
// owns a TX x TY tile of grid columns over ZC planes, for one slice of NVS
// consecutive vector groups (of the NV = N / VW of a row; thread t: group
// t % NVS of the slice, column t / NVS).  At each plane the tile's field
// values and those of the one-column ring around it go to LDS, so the x and y
// neighbours come from LDS (each ring value is loaded once per work-group
// instead of by every neighbouring thread), and the z neighbours stay in
// registers.  Slicing the row lets the tile grow (the ring costs 2(TX + TY) + 4
// extra columns per TX TY) within the same threads and LDS.
struct TShape {
  uint32_t TX, TY, nxt, nyt, nzc, ZC, NS, NVS;
};

constexpr uint32_t MG_TWG = 1024;                 // threads of a tiled work-group (at most)
constexpr uint32_t MG_TLDS_BYTES = 36864;         // LDS of one plane's tile and ring

// Slices of a row: halved as long as that keeps a slice at least 8 vector groups
// wide (a 128-byte run of FP64 pairs) and divides NV.  Where that leaves more than
// MG_SLICE of a row of more than two such, slices of equal width and a shorter last
// one: a whole row of an odd NV leaves a tile of so few columns that its ring is
// several times as large (V-cycles of one step at 64^3, FP64: N = 250, NV = 125,
// 12.6 -> 3.5 ms, N = 130 4.3 -> 2.4, N = 200 3.7 -> 3.2; 45x38x51, N = 45 0.75 ->
// 0.69; but NV = 25 in two slices, N = 50 at 48^3, 0.56 -> 0.60).
constexpr uint32_t MG_SLICE = 16;
uint32_t tslices(uint32_t NV) {
  uint32_t ns = 1;
  while (NV % (2 * ns) == 0 && NV / (2 * ns) >= 8) ns *= 2;
  if (NV > 2 * MG_SLICE && NV / ns > MG_SLICE) ns = (NV + MG_SLICE - 1) / MG_SLICE;
  return ns;
}

TShape tshape(uint32_t m0, uint32_t m1, uint32_t m2, uint32_t NV, uint32_t N, uint32_t esz) {
  TShape s;
  s.NS = tslices(NV);
  s.NVS = (NV + s.NS - 1) / s.NS;
  // columns per work-group: as many as MG_TWG threads hold (measured at 64^3,
  // N = 128: 1024 threads on 16 x 8 tiles beat 512 on 8 x 8 and 256 on 8 x 4,
  // whose rings cost more than the extra work-groups per compute unit gain)
  const uint32_t P = std::max(1u, MG_TWG / s.NVS);
  const uint64_t rowb = (uint64_t)s.NVS * (N / NV) * esz;      // LDS bytes of one column's slice
  uint32_t tx = 1;
  while ((tx * 2) * (tx * 2) <= P) tx *= 2;       // a square tile of powers of two, x side first
  if (tx * tx * 2 <= P) tx *= 2;
  s.TX = std::min(tx, m0);
  s.TY = std::max(1u, std::min(P / s.TX, m1));
  // fit the tile and its ring in the LDS array (a 1 x 1 tile always fits:
  // 9 columns of at most 4 KB)
  while ((uint64_t)(s.TX + 2) * (s.TY + 2) * rowb > MG_TLDS_BYTES && s.TX * s.TY > 1) {
    if (s.TY > 1) --s.TY;
    else --s.TX;
  }
  s.nxt = (m0 + s.TX - 1) / s.TX;
  s.nyt = (m1 + s.TY - 1) / s.TY;
  // z ranges: one work-group of this size fits a compute unit, two of at most half
  // of it (256 or 512 places), so a launch runs in rounds of as many, each as long as
  // a range and about two planes of set-up; the count with the shortest total (64^3,
  // N = 17, 80 tiles: 480 work-groups of 11 planes in 2 rounds, against 560 of 10 in
  // 3).  A few tiles of a long thin grid fill one round with more than 64 ranges
  // each (V-cycle, us, at least 512 work-groups in all / 64 ranges at most in rounds
  // of 256 / this rule: 16 x 16 x 1000, N = 4 86 / 99 / 76, 8 x 8 x 4000, N = 8 158 /
  // 225 / 105, 4 x 4 x 8000, N = 16 205 / 333 / 114).
  const uint64_t tiles = (uint64_t)s.nxt * s.nyt * s.NS;
  const uint64_t places = s.TX * s.TY * s.NVS > MG_TWG / 2 ? 256 : 512;
  const uint64_t most = std::min<uint64_t>(m2, std::max<uint64_t>(64, places / tiles));
  uint64_t best = UINT64_MAX;
  for (uint32_t nzc = 1; nzc <= most; ++nzc) {
    const uint32_t ZC = (m2 + nzc - 1) / nzc, nr = (m2 + ZC - 1) / ZC;
    const uint64_t cost = ((tiles * nr + places - 1) / places) * (ZC + 2);
    if (cost < best) {
      best = cost;
      s.ZC = ZC;
    }
  }
  s.nzc = (m2 + s.ZC - 1) / s.ZC;
  return s;
}

// Ring columns per thread of a tiled sweep: ceil(2 (TX + TY) / (TX TY)) <= 4,
// as 1, 2 or 4.
int ring_per_thread(const TShape& ts) {
  const uint32_t P = ts.TX * ts.TY, need = (2 * (ts.TX + ts.TY) + P - 1) / P;
  return need <= 1 ? 1 : need <= 2 ? 2 : 4;
}

// Work-group L of a tiled sweep: tile (xt, yt), z chunk zc, slice sl; `row` is
// its partial-sum row (the tile and chunk; the slices of one tile share it).
struct TPos {
  uint32_t xt, yt, zc, sl, row;
};

__device__ __forceinline__ TPos tpos(const TShape& ts, uint32_t L) {
  TPos q;
  q.sl = L % ts.NS;                               // first: neighbouring slices share 128-byte lines
  uint32_t r = L / ts.NS;
  q.xt = r % ts.nxt;
  r /= ts.nxt;
  q.yt = r % ts.nyt;
  q.zc = r / ts.nyt;
  q.row = (q.zc * ts.nyt + q.yt) * ts.nxt + q.xt;
  return q;
}

// Ring column j of a tiled work-group (k = pt + j P, k < 2 (TX + TY): bottom
// row, top row, left column, right column): its grid column (when inside
// the grid) and its LDS slot.
struct RingCol {
  uint32_t x, y;
  uint32_t slot;
  bool ok, in;
};

__device__ __forceinline__ RingCol ring_col(const MgGeom& g, const TShape& ts, uint32_t x0, uint32_t y0, uint32_t k,
                                            uint32_t NVS, uint32_t vl, uint32_t VW, bool act) {
  RingCol rc;
  const uint32_t RING = 2 * (ts.TX + ts.TY), W = ts.TX + 2;
  rc.ok = k < RING;
  rc.in = false;
  rc.x = rc.y = 0;
  rc.slot = 0;
  if (!rc.ok) return rc;
  int64_t hx, hy;
  uint32_t cx, cy;
  if (k < ts.TX) {
    hx = (int64_t)x0 + k; hy = (int64_t)y0 - 1; cx = k + 1; cy = 0;
  } else if (k < 2 * ts.TX) {
    hx = (int64_t)x0 + (k - ts.TX); hy = (int64_t)y0 + ts.TY; cx = k - ts.TX + 1; cy = ts.TY + 1;
  } else if (k < 2 * ts.TX + ts.TY) {
    hx = (int64_t)x0 - 1; hy = (int64_t)y0 + (k - 2 * ts.TX); cx = 0; cy = k - 2 * ts.TX + 1;
  } else {
    hx = (int64_t)x0 + ts.TX; hy = (int64_t)y0 + (k - 2 * ts.TX - ts.TY); cx = ts.TX + 1;
    cy = k - 2 * ts.TX - ts.TY + 1;
  }
  rc.slot = ((cy * W + cx) * NVS + vl) * VW;
  rc.in = act && hx >= 0 && hx < (int64_t)g.m0 && hy >= 0 && hy < (int64_t)g.m1;
  if (rc.in) {
    rc.x = (uint32_t)hx;
    rc.y = (uint32_t)hy;
  }
  return rc;
}

// Pre-smoothing residual r1 = b - H x0 with x0 = omega b / d formed on the fly,
// as an x-y tiled sweep (see TShape).  The loads are issued one plane ahead
// (the ring's b and omega/d of the next plane, the own column's two planes
// ahead), so a plane's wait finds them arrived; the two tile buffers
// alternate, one barrier per plane.
template <typename T, int VW, int R, typename O>
__global__ __launch_bounds__(MG_TWG) void k_mg_tstencil(const T* __restrict__ b, T* __restrict__ out, MgGeom g,
                                                       const double* __restrict__ diag, const double* __restrict__ wd,
                                                       const int32_t* __restrict__ active, uint32_t N, TShape ts) {
  __shared__ __align__(16) T tiles[2][MG_TLDS_BYTES / sizeof(T)];
  const uint32_t t = threadIdx.x;
  const uint32_t NVS = ts.NVS;
  const uint32_t vl = t % NVS, pt = t / NVS;
  const uint32_t tx = pt % ts.TX, ty = pt / ts.TX;
  const TPos wp = tpos(ts, xcd_remap(blockIdx.x, gridDim.x));
  const uint32_t v = wp.sl * NVS + vl;
  const uint32_t x0 = wp.xt * ts.TX, y0 = wp.yt * ts.TY;
  const uint32_t x = x0 + tx, y = y0 + ty;
  const bool inb = x < g.m0 && y < g.m1;
  const bool act = v < N / VW && vec_active<VW>(active, v);    // (the last slice may be short)
  if (!__syncthreads_or(act ? 1 : 0)) return;     // every column of the slice has stopped
  const bool own = inb && act;
  const uint32_t z0 = wp.zc * ts.ZC, z1 = z0 + ts.ZC < g.m2 ? z0 + ts.ZC : g.m2;
  const uint64_t s2 = (uint64_t)g.m0 * g.m1, s2N = s2 * N;       // points and elements of a plane
  const uint32_t W = ts.TX + 2, P = ts.TX * ts.TY;
  auto slot = [&](uint32_t cx, uint32_t cy) -> uint32_t { return ((cy * W + cx) * NVS + vl) * VW; };
  auto field_off = [&](uint32_t cx, uint32_t cy) -> O {
    return (((O)cy * g.m0 + cx) * N + (O)VW * v) * (O)sizeof(T);
  };
  auto coef_off = [&](uint32_t cx, uint32_t cy) -> O { return ((O)cy * g.m0 + cx) * (O)sizeof(double); };
  RingCol rc[R];
  O ro[R], rwo[R];
  T rb[R][VW], rw[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    rc[j] = ring_col(g, ts, x0, y0, pt + (uint32_t)j * P, NVS, vl, VW, act);
    ro[j] = field_off(rc[j].x, rc[j].y);
    rwo[j] = coef_off(rc[j].x, rc[j].y);
  }
  const O oo = own ? field_off(x, y) : 0, owo = own ? coef_off(x, y) : 0;
  auto coef = [&](const double* plane, O o) -> T {
    return (T)*reinterpret_cast<const double*>(reinterpret_cast<const char*>(plane) + o);
  };
  auto ring_load = [&](uint32_t z) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      zero(rb[j]);
      rw[j] = T(0);
      if (rc[j].in) {
        ldo<T, VW, O>(b + z * s2N, ro[j], rb[j]);
        rw[j] = coef(wd + z * s2, rwo[j]);
      }
    }
  };
  // own column: x0 at z - 1 and z, b and d at z, the raw b and omega/d of z + 1
  T fm[VW], fc[VW], bc[VW], bn[VW];
  T wn = T(0), dc = T(0);
  zero(fm);
  zero(fc);
  zero(bc);
  zero(bn);
  if (own) {
    if (z0 > 0) {
      ldo<T, VW, O>(b + (z0 - 1) * s2N, oo, fm);
      const T wm = coef(wd + (z0 - 1) * s2, owo);
#pragma unroll
      for (int k = 0; k < VW; ++k) fm[k] = wm * fm[k];
    }
    ldo<T, VW, O>(b + z0 * s2N, oo, bc);
    const T w0 = coef(wd + z0 * s2, owo);
#pragma unroll
    for (int k = 0; k < VW; ++k) fc[k] = w0 * bc[k];
    dc = coef(diag + z0 * s2, owo);
    if (z0 + 1 < g.m2) {
      ldo<T, VW, O>(b + (z0 + 1) * s2N, oo, bn);
      wn = coef(wd + (z0 + 1) * s2, owo);
    }
  }
  ring_load(z0);
  for (uint32_t z = z0; z < z1; ++z) {
    T* tile = tiles[z & 1];
#pragma unroll
    for (int k = 0; k < VW; ++k) tile[slot(tx + 1, ty + 1) + k] = fc[k];
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (rc[j].ok) {
#pragma unroll
        for (int k = 0; k < VW; ++k) tile[rc[j].slot + k] = rw[j] * rb[j][k];
      }
    // the next plane's ring and the own column two planes ahead
    if (z + 1 < z1) ring_load(z + 1);
    T fp[VW], b2[VW];
    T w2 = T(0), d2 = T(0);
#pragma unroll
    for (int k = 0; k < VW; ++k) fp[k] = wn * bn[k];
    zero(b2);
    if (own && z + 1 < z1) {
      if (z + 2 < g.m2) {
        ldo<T, VW, O>(b + (z + 2) * s2N, oo, b2);
        w2 = coef(wd + (z + 2) * s2, owo);
      }
      d2 = coef(diag + (z + 1) * s2, owo);
    }
    __syncthreads();
    if (own) {
      T o[VW];
      const uint32_t sxm = slot(tx, ty + 1), sxp = slot(tx + 2, ty + 1), sym = slot(tx + 1, ty),
                     syp = slot(tx + 1, ty + 2);
#pragma unroll
      for (int k = 0; k < VW; ++k) {
        const T hxv = dc * fc[k] - ((T)g.cx * (tile[sxm + k] + tile[sxp + k]) +
                                    (T)g.cy * (tile[sym + k] + tile[syp + k]) + (T)g.cz * (fm[k] + fp[k]));
        o[k] = bc[k] - hxv;
      }
      sto<T, VW, O>(out + z * s2N, oo, o);
    }
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      fm[k] = fc[k];
      fc[k] = fp[k];
      bc[k] = bn[k];
      bn[k] = b2[k];
    }
    wn = w2;
    dc = d2;
  }
}

// The prolongation P e along one fine column, marched plane by plane: the
// x-y interpolations of the coarse planes K - 1, K, K + 1 around the current
// plane's parent K = z / 2 stay in registers (each coarse plane read once,
// through four offsets fixed over the march).
template <typename T, int VW, typename O>
struct PeMarch {
  O off[2][2];                                    // [y tap][x tap]
  T wx[2], wy[2];
  T lo[VW], mid[VW], hi[VW];

  // x-y interpolation of the coarse plane at `plane`
  __device__ __forceinline__ void interp(const T* __restrict__ plane, T (&o)[VW]) const {
    T e[2][2][VW];
#pragma unroll
    for (int bb = 0; bb < 2; ++bb)
#pragma unroll
      for (int a = 0; a < 2; ++a) ldo<T, VW, O>(plane, off[bb][a], e[bb][a]);
#pragma unroll
    for (int k = 0; k < VW; ++k)
      o[k] = wy[0] * (wx[0] * e[0][0][k] + wx[1] * e[0][1][k]) + wy[1] * (wx[0] * e[1][0][k] + wx[1] * e[1][1][k]);
  }
  // planes around z (flat: no z axis, the one coarse plane 0); csN: elements of a coarse plane
  __device__ __forceinline__ void init(const T* __restrict__ E, const MgGeom& fg, const MgGeom& cg, uint64_t csN,
                                       uint32_t fx, uint32_t fy, uint32_t z, uint32_t N, uint32_t v) {
    uint32_t Ix[2], Iy[2];
    double dx[2], dy[2];
    prolong_taps(fx, fg.m0, cg.m0, Ix, dx);
    prolong_taps(fy, fg.m1, cg.m1, Iy, dy);
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      wx[bb] = (T)dx[bb];
      wy[bb] = (T)dy[bb];
#pragma unroll
      for (int a = 0; a < 2; ++a) off[bb][a] = (((O)Iy[bb] * cg.m0 + Ix[a]) * N + (O)VW * v) * (O)sizeof(T);
    }
    zero(lo);
    zero(hi);
    const uint32_t K = fg.m2 == 1 ? 0 : z / 2;
    interp(E + K * csN, mid);
    if (fg.m2 > 1) {
      if (K >= 1) interp(E + (K - 1) * csN, lo);
      if (K + 1 < cg.m2) interp(E + (K + 1) * csN, hi);
    }
  }
  // move to plane z (the plane after the current one)
  __device__ __forceinline__ void step(const T* __restrict__ E, const MgGeom& cg, uint64_t csN, uint32_t z) {
    if (z % 2 != 0) return;
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      lo[k] = mid[k];
      mid[k] = hi[k];
    }
    zero(hi);
    if (z / 2 + 1 < cg.m2) interp(E + (z / 2 + 1) * csN, hi);
  }
  __device__ __forceinline__ void value(uint32_t z, bool flat, T (&pe)[VW]) const {
#pragma unroll
    for (int k = 0; k < VW; ++k) pe[k] = flat ? mid[k] : T(0.75) * mid[k] + T(0.25) * (z % 2 == 0 ? lo[k] : hi[k]);
  }
};

// Prolongation and post-smoothing in one x-y tiled sweep (as k_mg_tstencil):
// x1 = omega b / d + P e is formed on the fly for the tile's columns and its
// ring, then z = x1 + omega (b - H x1) / d; with DOTS also the per-column
// sums of b z and b b (row `wp.row` of part).  The ring columns are spread
// over the threads, each with its own P e march; b and the coefficients are
// loaded one plane ahead (the own column's two).  Bound by one work-group's
// progress per compute unit (its registers and threads leave room for no
// second): instructions and the barrier of every plane.  Offsets fixed over the
// march, the loads a plane ahead and rounds without a short last one (tshape)
// took it from 60 to 40 us at 64^3, N = 17 (its bytes alone take 16 us), 193 to
// 163 us at N = 128 (121 us) and 110 to 95 us in FP32.
template <typename T, int VW, bool DOTS, int R, typename O>
__global__ __launch_bounds__(MG_TWG) void k_mg_tpost(const T* __restrict__ b, const T* __restrict__ E,
                                                    T* __restrict__ out, MgGeom g, MgGeom cg,
                                                    const double* __restrict__ diag, const double* __restrict__ wd,
                                                    const int32_t* __restrict__ active, uint32_t N, TShape ts,
                                                    double* __restrict__ part) {
  // two tile buffers (planes alternate), so one barrier per plane suffices
  __shared__ __align__(16) T tiles[2][MG_TLDS_BYTES / sizeof(T)];
  const uint32_t t = threadIdx.x;
  const uint32_t NVS = ts.NVS;
  const uint32_t vl = t % NVS, pt = t / NVS;
  const uint32_t tx = pt % ts.TX, ty = pt / ts.TX;
  const TPos wp = tpos(ts, xcd_remap(blockIdx.x, gridDim.x));
  const uint32_t v = wp.sl * NVS + vl;
  const uint32_t x0 = wp.xt * ts.TX, y0 = wp.yt * ts.TY;
  const uint32_t x = x0 + tx, y = y0 + ty;
  const bool inb = x < g.m0 && y < g.m1;
  const bool act = v < N / VW && vec_active<VW>(active, v);    // (the last slice may be short)
  if (!__syncthreads_or(act ? 1 : 0)) {          // every column of the slice has stopped
    if constexpr (DOTS) {
      const uint32_t SC = ts.NVS * VW, c0 = wp.sl * SC;
      for (uint32_t c = t; c < SC && c0 + c < N; c += blockDim.x) {
        part[(uint64_t)wp.row * 2 * N + c0 + c] = 0.0;
        part[(uint64_t)wp.row * 2 * N + N + c0 + c] = 0.0;
      }
    }
    return;
  }
  const bool own = inb && act;
  const uint32_t z0 = wp.zc * ts.ZC, z1 = z0 + ts.ZC < g.m2 ? z0 + ts.ZC : g.m2;
  const uint64_t s2 = (uint64_t)g.m0 * g.m1, s2N = s2 * N;       // points and elements of a plane
  const uint64_t csN = (uint64_t)cg.m0 * cg.m1 * N;              // elements of a coarse plane
  const bool flat = g.m2 == 1;
  const uint32_t W = ts.TX + 2, P = ts.TX * ts.TY;
  auto slot = [&](uint32_t cx, uint32_t cy) -> uint32_t { return ((cy * W + cx) * NVS + vl) * VW; };
  auto field_off = [&](uint32_t cx, uint32_t cy) -> O {
    return (((O)cy * g.m0 + cx) * N + (O)VW * v) * (O)sizeof(T);
  };
  auto coef_off = [&](uint32_t cx, uint32_t cy) -> O { return ((O)cy * g.m0 + cx) * (O)sizeof(double); };
  auto coef = [&](const double* plane, O o) -> T {
    return (T)*reinterpret_cast<const double*>(reinterpret_cast<const char*>(plane) + o);
  };
  // ring columns of this thread: k = pt + j P, j < R (R P at least the ring's
  // 2 (TX + TY) columns); b and omega/d of the current plane
  RingCol rc[R];
  O ro[R], rwo[R];
  T rb[R][VW], rw[R];
  PeMarch<T, VW, O> rm[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    rc[j] = ring_col(g, ts, x0, y0, pt + (uint32_t)j * P, NVS, vl, VW, act);
    ro[j] = field_off(rc[j].x, rc[j].y);
    rwo[j] = coef_off(rc[j].x, rc[j].y);
    if (rc[j].in) rm[j].init(E, g, cg, csN, rc[j].x, rc[j].y, z0, N, v);
  }
  auto ring_load = [&](uint32_t z) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      zero(rb[j]);
      rw[j] = T(0);
      if (rc[j].in) {
        ldo<T, VW, O>(b + z * s2N, ro[j], rb[j]);
        rw[j] = coef(wd + z * s2, rwo[j]);
      }
    }
  };
  // own column: x1 at z - 1 and z; b, omega/d and d at z; b and omega/d at z + 1
  PeMarch<T, VW, O> om;
  T fm[VW], fc[VW], bc[VW], bn[VW], pe[VW];
  T wc = T(0), wn = T(0), dc = T(0);
  zero(fm);
  zero(fc);
  zero(bc);
  zero(bn);
  const O oo = own ? field_off(x, y) : 0, owo = own ? coef_off(x, y) : 0;
  if (own) {
    if (z0 > 0) {                                 // the march starts one plane below
      om.init(E, g, cg, csN, x, y, z0 - 1, N, v);
      om.value(z0 - 1, flat, pe);
      ldo<T, VW, O>(b + (z0 - 1) * s2N, oo, fm);
      const T wm = coef(wd + (z0 - 1) * s2, owo);
#pragma unroll
      for (int k = 0; k < VW; ++k) fm[k] = wm * fm[k] + pe[k];
      om.step(E, cg, csN, z0);
    } else {
      om.init(E, g, cg, csN, x, y, z0, N, v);
    }
    om.value(z0, flat, pe);
    ldo<T, VW, O>(b + z0 * s2N, oo, bc);
    wc = coef(wd + z0 * s2, owo);
    dc = coef(diag + z0 * s2, owo);
#pragma unroll
    for (int k = 0; k < VW; ++k) fc[k] = wc * bc[k] + pe[k];
    if (z0 + 1 < g.m2) {
      ldo<T, VW, O>(b + (z0 + 1) * s2N, oo, bn);
      wn = coef(wd + (z0 + 1) * s2, owo);
    }
  }
  ring_load(z0);
  double srz[VW], srr[VW];
  zero(srz);
  zero(srr);
  for (uint32_t z = z0; z < z1; ++z) {
    T* tile = tiles[z & 1];
#pragma unroll
    for (int k = 0; k < VW; ++k) tile[slot(tx + 1, ty + 1) + k] = fc[k];
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (rc[j].ok) {
        T hv[VW];
        zero(hv);
        if (rc[j].in) {
          rm[j].value(z, flat, hv);
#pragma unroll
          for (int k = 0; k < VW; ++k) hv[k] = rw[j] * rb[j][k] + hv[k];
        }
#pragma unroll
        for (int k = 0; k < VW; ++k) tile[rc[j].slot + k] = hv[k];
      }
    // the next plane's ring, the own column two planes ahead
    if (z + 1 < z1) {
      ring_load(z + 1);
#pragma unroll
      for (int j = 0; j < R; ++j)
        if (rc[j].in) rm[j].step(E, cg, csN, z + 1);
    }
    T fp[VW], b2[VW];
    T w2 = T(0), d2 = T(0);
    zero(fp);
    zero(b2);
    if (own) {
      if (z + 1 < z1) {
        if (z + 2 < g.m2) {
          ldo<T, VW, O>(b + (z + 2) * s2N, oo, b2);
          w2 = coef(wd + (z + 2) * s2, owo);
        }
        d2 = coef(diag + (z + 1) * s2, owo);
      }
      if (z + 1 < g.m2) {
        om.step(E, cg, csN, z + 1);
        om.value(z + 1, flat, pe);
#pragma unroll
        for (int k = 0; k < VW; ++k) fp[k] = wn * bn[k] + pe[k];
      }
    }
    __syncthreads();
    if (own) {
      T o[VW];
      const uint32_t sxm = slot(tx, ty + 1), sxp = slot(tx + 2, ty + 1), sym = slot(tx + 1, ty),
                     syp = slot(tx + 1, ty + 2);
#pragma unroll
      for (int k = 0; k < VW; ++k) {
        const T hxv = dc * fc[k] - ((T)g.cx * (tile[sxm + k] + tile[sxp + k]) +
                                    (T)g.cy * (tile[sym + k] + tile[syp + k]) + (T)g.cz * (fm[k] + fp[k]));
        o[k] = fc[k] + wc * (bc[k] - hxv);
      }
      sto<T, VW, O>(out + z * s2N, oo, o);
      if constexpr (DOTS) {
#pragma unroll
        for (int k = 0; k < VW; ++k) {
          srz[k] += (double)bc[k] * (double)o[k];
          srr[k] += (double)bc[k] * (double)bc[k];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      fm[k] = fc[k];
      fc[k] = fp[k];
      bc[k] = bn[k];
      bn[k] = b2[k];
    }
    wc = wn;
    wn = w2;
    dc = d2;
  }
  if constexpr (DOTS) {
    // per-column sums over the tile's columns in order, b z then b b (LDS
    // reused, one quantity at a time)
    double* red = reinterpret_cast<double*>(&tiles[0][0]);
    const uint32_t SC = NVS * VW, c0 = wp.sl * SC;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      __syncthreads();            // the last plane's (or the previous pass's) reads are done
#pragma unroll
      for (int k = 0; k < VW; ++k) red[t * VW + k] = q == 0 ? srz[k] : srr[k];
      __syncthreads();
      for (uint32_t c = t; c < SC && c0 + c < N; c += blockDim.x) {
        const uint32_t cv = c / VW, ck = c % VW;
        double a = 0.0;
        for (uint32_t l = 0; l < P; ++l) a += red[(l * NVS + cv) * VW + ck];
        part[(uint64_t)wp.row * 2 * N + (uint64_t)q * N + c0 + c] = a;
      }
    }
  }
}

// coarse B = R T, z-marched over the coarse planes of a coarse (I, J) column:
// the x-y restriction of each fine plane is formed once and added to the two
// coarse planes it feeds.
template <typename T, int VW>
__global__ __launch_bounds__(MG_WG) void k_mg_zrestrict(const T* __restrict__ R1, T* __restrict__ B,
                                                       MgGeom fg, MgGeom cg, const int32_t* __restrict__ active,
                                                       uint32_t N, uint32_t NV, ZMarch zs) {
  const ZPos q = zpos<VW>(cg, zs, active, NV);
  if (!q.ok) return;
  const uint32_t v = q.v;
  uint32_t fx[4], fy[4];
  double wx[4], wy[4];
  restrict_taps(q.x, fg.m0, fx, wx);
  restrict_taps(q.y, fg.m1, fy, wy);
  auto rxy = [&](uint32_t z, T(&o)[VW]) {
    zero(o);
#pragma unroll
    for (int bb = 0; bb < 4; ++bb) {
      T ax[VW];
      zero(ax);
      const uint64_t row = ((uint64_t)z * fg.m1 + fy[bb]) * fg.m0;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        T t[VW];
        ldr<T, VW>(R1, row + fx[a], N, v, t);
#pragma unroll
        for (int k = 0; k < VW; ++k) ax[k] += (T)wx[a] * t[k];
      }
#pragma unroll
      for (int k = 0; k < VW; ++k) o[k] += (T)wy[bb] * ax[k];
    }
  };
  const uint64_t cs2 = (uint64_t)cg.m0 * cg.m1;
  uint64_t P = ((uint64_t)q.z0 * cg.m1 + q.y) * cg.m0 + q.x;
  if (fg.m2 == 1) {                 // no z axis
    T o[VW];
    rxy(0, o);
    str<T, VW>(B, P, N, v, o);
    return;
  }
  // fine planes 2K - 1, 2K, 2K + 1, 2K + 2 with weights 1/8, 3/8, 3/8, 1/8;
  // the last two are the first two of coarse plane K + 1
  T ra[VW], rb[VW];
  zero(ra);
  zero(rb);
  if (q.z0 >= 1) rxy(2 * q.z0 - 1, ra);
  rxy(2 * q.z0, rb);
  for (uint32_t K = q.z0; K < q.z1; ++K, P += cs2) {
    T rc[VW], rd[VW], o[VW];
    zero(rc);
    zero(rd);
    if (2 * K + 1 < fg.m2) rxy(2 * K + 1, rc);
    if (2 * K + 2 < fg.m2) rxy(2 * K + 2, rd);
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      o[k] = T(0.125) * ra[k] + T(0.375) * rb[k] + T(0.375) * rc[k] + T(0.125) * rd[k];
      ra[k] = rc[k];
      rb[k] = rd[k];
    }
    str<T, VW>(B, P, N, v, o);
  }
}

// The PCG's scalars from the (partial or stage) rows of r^T z and r^T r, in one
// work-group: column sums in a fixed order (thread t: column t % 2N, rows
// t / 2N, t / 2N + G, ...; 8 running sums, then the G groups in order), then
//   START: rho = r^T z (the CG set-up has already set the targets and the
//          convergence flags from |r|^2);
//   else:  for a running column beta = r^T z / rho, rho = r^T z, and it keeps
//          running while |r|^2 > target (a non-positive r^T z, which an SPD
//          preconditioner cannot give, stops it); flags (nullable, pinned host
//          memory) receives a copy of the flags.
// One launch instead of three (two reduction stages and the scalars) while the
// partial values are few, as in 3D (a tile's slices share a row); more than PS_MAX of
// them (2D, where the rows are the tiles of the whole plane) go through a first stage
// over the chip.  One launch / with the stage, us: 64^3 N = 17 (240 x 34 values) 6.3
// / 9.7, N = 128 FP32 (64 x 256) 7.6 / 10.0, 300^2 N = 16 (722 x 32) 8.9 / 9.4, 100^3
// N = 64 (182 x 128) 11.4 / 10.7, 48^3 N = 250 (144 x 500) 19.6 / 11.6, 200^2 N = 65
// (575 x 130) 16.1 / 10.1, 500^2 N = 128 (2016 x 256) 94 / 14.5, 1000^2 N = 128 (7875
// x 256) 374 / 23.
constexpr uint32_t PS_WG = 1024;
constexpr int64_t PS_MAX = (int64_t)1 << 15;

template <bool START>
__global__ __launch_bounds__(PS_WG) void k_pcg_scalars(const double* __restrict__ part, uint32_t nrows, uint32_t N,
                                                      double* __restrict__ rho, double* __restrict__ beta,
                                                      const double* __restrict__ target,
                                                      int32_t* __restrict__ active, OpeScalars* __restrict__ sc,
                                                      int32_t* __restrict__ flags) {
  __shared__ double red[PS_WG], dots[PS_WG];
  const uint32_t nc = 2 * N, G = PS_WG / nc;                   // 2N <= 1024 (N <= 512)
  const uint32_t col = threadIdx.x % nc, gi = threadIdx.x / nc;
  double a = 0.0;
  if (gi < G) {
    double q[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    uint32_t w = gi;
    for (; w + 7 * G < nrows; w += 8 * G) {
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) q[u] += part[(uint64_t)(w + u * G) * nc + col];
    }
    for (; w < nrows; w += G) q[0] += part[(uint64_t)w * nc + col];
    a = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
  }
  red[threadIdx.x] = a;
  __syncthreads();
  if (gi == 0) {
    double t = 0.0;
    for (uint32_t k = 0; k < G; ++k) t += red[k * nc + col];
    dots[col] = t;
  }
  __syncthreads();
  const uint32_t j = threadIdx.x;
  if (j >= N) return;
  const double rz = dots[j], rr = dots[N + j];
  if (START) {
    rho[j] = rz;
    return;
  }
  int32_t act = 0;
  double b = 0.0;
  if (active[j]) {
    if (!isfinite(rz) || !isfinite(rr)) {
      if (sc->err == 0) sc->err = OPE_ENONFINITE;
    } else {
      b = rz / rho[j];
      rho[j] = rz;
      act = (rr > target[j] && rz > 0.0) ? 1 : 0;
    }
  }
  beta[j] = b;
  active[j] = act;
  if (flags) flags[j] = act;
}

// The fused levels' geometry and LDS layout: the field of the first (and its
// zero), the lower levels' constants (omega / diagonal and diagonal, level by
// level, as mg_build lays them out in mg_cdat), then each lower level's
// right-hand side and correction.  *values: the LDS needed.
McArgs coarse_args(const MgLevel* lv, int nl, int k0, size_t* values) {
  McArgs a{};
  a.nl = nl - k0;
  auto magic = [](uint32_t m) -> uint32_t { return m > 1 ? (uint32_t)((((uint64_t)1 << 32) + m - 1) / m) : 0u; };
  uint32_t off = (uint32_t)lv[k0].n + 1;
  a.cst = off;
  for (int k = 0; k < a.nl; ++k) {
    const MgLevel& g = lv[k0 + k];
    McLevel& L = a.lv[k];
    L.m0 = g.m0;
    L.m1 = g.m1;
    L.m2 = g.m2;
    L.n = (uint32_t)g.n;
    L.mag0 = magic(g.m0);
    L.mag1 = magic(g.m1);
    L.cx = g.cx;
    L.cy = g.cy;
    L.cz = g.cz;
    if (k == 0) continue;
    L.wd = off;
    L.dg = off + L.n;
    off += 2 * L.n;
  }
  a.ncst = off - a.cst;
  for (int k = 1; k < a.nl; ++k) {
    McLevel& L = a.lv[k];
    L.b = off;
    L.e = off + L.n;
    off += 2 * L.n;
  }
  *values = off;
  return a;
}

inline MgGeom geom(const MgLevel& L) { return MgGeom{L.m0, L.m1, L.m2, L.cx, L.cy, L.cz}; }

// Storage type of the blocks (the context's: FP64, or FP32 for OPE_MIXED) and
// elements per thread (16 bytes when N allows).
inline uint32_t mg_esz(const ope_ctx* c) { return c->prec == OPE_FP64 ? 8u : 4u; }
inline uint32_t mg_vw(const ope_ctx* c) {
  if (c->prec == OPE_FP64) return c->N % 2 == 0 ? 2u : 1u;
  return c->N % 4 == 0 ? 4u : (c->N % 2 == 0 ? 2u : 1u);
}

// Dense inverse of an SPD matrix (row-major, n x n) by Cholesky: A = L L^T,
// A^{-1} = L^{-T} L^{-1}.  False if A is not positive definite.
bool spd_inverse(std::vector<double>& A, int n) {
  std::vector<double> L((size_t)n * n, 0.0);
  for (int j = 0; j < n; ++j) {
    double s = A[(size_t)j * n + j];
    for (int k = 0; k < j; ++k) s -= L[(size_t)j * n + k] * L[(size_t)j * n + k];
    if (!(s > 0.0)) return false;
    const double ljj = std::sqrt(s);
    L[(size_t)j * n + j] = ljj;
    for (int i = j + 1; i < n; ++i) {
      double t = A[(size_t)i * n + j];
      for (int k = 0; k < j; ++k) t -= L[(size_t)i * n + k] * L[(size_t)j * n + k];
      L[(size_t)i * n + j] = t / ljj;
    }
  }
  // Li = L^{-1} (lower triangular), by forward substitution per column
  std::vector<double> Li((size_t)n * n, 0.0);
  for (int c = 0; c < n; ++c) {
    for (int i = c; i < n; ++i) {
      double t = (i == c) ? 1.0 : 0.0;
      for (int k = c; k < i; ++k) t -= L[(size_t)i * n + k] * Li[(size_t)k * n + c];
      Li[(size_t)i * n + c] = t / L[(size_t)i * n + i];
    }
  }
  // A^{-1} = Li^T Li
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) {
      double t = 0.0;
      for (int k = i; k < n; ++k) t += Li[(size_t)k * n + i] * Li[(size_t)k * n + j];
      A[(size_t)i * n + j] = t;
      A[(size_t)j * n + i] = t;
    }
  return true;
}

}  // namespace

void mg_free(ope_ctx* c) {
  for (int k = 0; k < c->mg_levels; ++k) {
    if (k > 0 && c->mg[k].diag) (void)hipFree(c->mg[k].diag);
    if (c->mg[k].wd) (void)hipFree(c->mg[k].wd);
  }
  if (c->mg_mem) (void)hipFree(c->mg_mem);
  if (c->mg_inv) (void)hipFree(c->mg_inv);
  if (c->mg_cdat) (void)hipFree(c->mg_cdat);
  if (c->mg_part) (void)hipFree(c->mg_part);
  c->mg_mem = nullptr;
  c->mg_inv = nullptr;
  c->mg_cdat = nullptr;
  c->mg_part = nullptr;
  c->mg_Z = nullptr;
  for (int k = 0; k < OPE_MG_MAX_LEVELS; ++k) c->mg[k] = MgLevel{};
  c->mg_levels = 0;
  c->mg_k0 = 0;
  c->mg_on = 0;
}

ope_status mg_build(ope_ctx* c) {
  mg_free(c);
  const int64_t N = c->N;
  // level 0: the operator; its potential W = diag - 2 (cx + cy + cz)
  std::vector<double> W((size_t)c->n);
  if (hipMemcpy(W.data(), c->diag, sizeof(double) * c->n, hipMemcpyDeviceToHost) != hipSuccess) return OPE_EHIP;
  std::vector<std::vector<double>> diags;       // the diagonal of every level (level 0: the context's)
  diags.push_back(W);
  const double dsum0 = 2.0 * (c->g.cx + c->g.cy + c->g.cz);
  for (auto& w : W) w -= dsum0;
  MgLevel L0{};
  L0.m0 = c->g.m0;
  L0.m1 = c->g.m1;
  L0.m2 = c->g.m2;
  L0.cx = c->g.cx;
  L0.cy = c->g.cy;
  L0.cz = c->g.cz;
  L0.n = c->n;
  L0.diag = c->diag;
  MgLevel lv[OPE_MG_MAX_LEVELS];
  lv[0] = L0;
  int nl = 1;
  std::vector<double> Wc;
  while (nl == 1 || lv[nl - 1].n > MG_COARSEST_MAX) {
    const MgLevel& f = lv[nl - 1];
    MgLevel q{};
    q.m0 = f.m0 > 1 ? (f.m0 + 1) / 2 : 1;
    q.m1 = f.m1 > 1 ? (f.m1 + 1) / 2 : 1;
    q.m2 = f.m2 > 1 ? (f.m2 + 1) / 2 : 1;
    if (q.m0 == f.m0 && q.m1 == f.m1 && q.m2 == f.m2) break;
    if (nl == OPE_MG_MAX_LEVELS) return OPE_EUNSUPPORTED;
    q.cx = f.m0 > 1 ? f.cx / 4.0 : f.cx;
    q.cy = f.m1 > 1 ? f.cy / 4.0 : f.cy;
    q.cz = f.m2 > 1 ? f.cz / 4.0 : f.cz;
    q.n = (int64_t)q.m0 * q.m1 * q.m2;
    // coarse potential: mean over the existing children
    Wc.assign((size_t)q.n, 0.0);
    for (uint32_t K = 0; K < q.m2; ++K)
      for (uint32_t J = 0; J < q.m1; ++J)
        for (uint32_t I = 0; I < q.m0; ++I) {
          double s = 0.0;
          int cnt = 0;
          const uint32_t zs = f.m2 > 1 ? 2 * K : K, ze = f.m2 > 1 ? std::min(2 * K + 2, f.m2) : K + 1;
          const uint32_t ys = f.m1 > 1 ? 2 * J : J, ye = f.m1 > 1 ? std::min(2 * J + 2, f.m1) : J + 1;
          const uint32_t xs = f.m0 > 1 ? 2 * I : I, xe = f.m0 > 1 ? std::min(2 * I + 2, f.m0) : I + 1;
          for (uint32_t z = zs; z < ze; ++z)
            for (uint32_t y = ys; y < ye; ++y)
              for (uint32_t x = xs; x < xe; ++x) {
                s += W[((size_t)z * f.m1 + y) * f.m0 + x];
                ++cnt;
              }
          Wc[((size_t)K * q.m1 + J) * q.m0 + I] = s / cnt;
        }
    W.swap(Wc);
    std::vector<double> d((size_t)q.n);
    const double dsum = 2.0 * (q.cx + q.cy + q.cz);
    for (int64_t p = 0; p < q.n; ++p) d[(size_t)p] = W[(size_t)p] + dsum;
    diags.push_back(d);
    lv[nl++] = q;
  }
  if (nl < 2) return OPE_EUNSUPPORTED;
  // coarsest operator, dense, and its inverse
  const MgLevel& cl = lv[nl - 1];
  const int nc = (int)cl.n;
  std::vector<double> A((size_t)nc * nc, 0.0);
  const std::vector<double>& dc = diags[(size_t)nl - 1];
  for (uint32_t z = 0; z < cl.m2; ++z)
    for (uint32_t y = 0; y < cl.m1; ++y)
      for (uint32_t x = 0; x < cl.m0; ++x) {
        const size_t p = ((size_t)z * cl.m1 + y) * cl.m0 + x;
        A[p * nc + p] = dc[p];
        if (x > 0) A[p * nc + p - 1] = -cl.cx;
        if (x + 1 < cl.m0) A[p * nc + p + 1] = -cl.cx;
        if (y > 0) A[p * nc + p - cl.m0] = -cl.cy;
        if (y + 1 < cl.m1) A[p * nc + p + cl.m0] = -cl.cy;
        if (z > 0) A[p * nc + p - (size_t)cl.m0 * cl.m1] = -cl.cz;
        if (z + 1 < cl.m2) A[p * nc + p + (size_t)cl.m0 * cl.m1] = -cl.cz;
      }
  if (!spd_inverse(A, nc)) return OPE_ENOTSPD;
  // device memory: level diagonals, blocks (level 0: T and Z; others: B, E, T)
  // (levels 1 .. k0 - 1: B, E and T; level k0: B and E; the fused levels below
  // it live in LDS)
  int k0 = nl - 1;                                // first fused level
  while (k0 > 1 && lv[k0 - 1].n <= MC_MAX && nl - (k0 - 1) <= MC_LEVELS) {
    size_t values = 0;
    (void)coarse_args(lv, nl, k0 - 1, &values);
    if (values * sizeof(double) > MC_LDS) break;  // levels that shrink along one axis only
    --k0;
  }
  std::vector<double> cdat;                       // constants of the levels below k0
  for (int k = k0 + 1; k < nl; ++k) {
    for (const double d : diags[(size_t)k]) cdat.push_back(MG_OMEGA / d);
    cdat.insert(cdat.end(), diags[(size_t)k].begin(), diags[(size_t)k].end());
  }
  int64_t elems = 2 * c->n * N;
  for (int k = 1; k <= k0; ++k) elems += (k < k0 ? 3 : 2) * lv[k].n * N;
  const uint32_t esz = mg_esz(c);
  {
    const uint32_t NV = (uint32_t)N / mg_vw(c);
    const TShape ts = tshape(lv[0].m0, lv[0].m1, lv[0].m2, NV, (uint32_t)N, esz);
    c->mg_rows = (int64_t)ts.nxt * ts.nyt * ts.nzc;        // partial rows of the level-0 post-smoothing
  }
  bool ok = hipMalloc(&c->mg_mem, (size_t)esz * (size_t)elems) == hipSuccess;
  ok = ok && hipMalloc((void**)&c->mg_inv, sizeof(double) * (size_t)nc * nc) == hipSuccess;
  ok = ok && hipMalloc((void**)&c->mg_cdat, sizeof(double) * std::max<size_t>(cdat.size(), 1)) == hipSuccess;
  ok = ok && hipMalloc((void**)&c->mg_part, sizeof(double) * (size_t)c->mg_rows * 2 * N) == hipSuccess;
  for (int k = 1; k < nl && ok; ++k) ok = hipMalloc((void**)&lv[k].diag, sizeof(double) * lv[k].n) == hipSuccess;
  for (int k = 0; k < nl && ok; ++k) ok = hipMalloc((void**)&lv[k].wd, sizeof(double) * lv[k].n) == hipSuccess;
  c->mg_levels = nl;
  for (int k = 0; k < nl; ++k) c->mg[k] = lv[k];
  if (!ok) {
    mg_free(c);
    return OPE_ENOMEM;
  }
  char* mem = (char*)c->mg_mem;
  c->mg[0].T = mem;
  mem += (size_t)esz * c->n * N;
  c->mg_Z = mem;
  mem += (size_t)esz * c->n * N;
  for (int k = 1; k <= k0; ++k) {
    c->mg[k].B = mem;
    mem += (size_t)esz * c->mg[k].n * N;
    c->mg[k].E = mem;
    mem += (size_t)esz * c->mg[k].n * N;
    if (k == k0) break;
    c->mg[k].T = mem;
    mem += (size_t)esz * c->mg[k].n * N;
  }
  c->mg_k0 = k0;
  ok = hipMemcpy(c->mg_inv, A.data(), sizeof(double) * (size_t)nc * nc, hipMemcpyHostToDevice) == hipSuccess;
  if (!cdat.empty())
    ok = ok && hipMemcpy(c->mg_cdat, cdat.data(), sizeof(double) * cdat.size(), hipMemcpyHostToDevice) == hipSuccess;
  for (int k = 1; k < nl && ok; ++k)
    ok = hipMemcpy(c->mg[k].diag, diags[(size_t)k].data(), sizeof(double) * c->mg[k].n, hipMemcpyHostToDevice) ==
         hipSuccess;
  for (int k = 0; k < nl && ok; ++k) {
    std::vector<double> w(diags[(size_t)k].size());
    for (size_t p = 0; p < w.size(); ++p) w[p] = MG_OMEGA / diags[(size_t)k][p];
    ok = hipMemcpy(c->mg[k].wd, w.data(), sizeof(double) * c->mg[k].n, hipMemcpyHostToDevice) == hipSuccess;
  }
  if (!ok) {
    mg_free(c);
    return OPE_EHIP;
  }
  return OPE_OK;
}

template <typename T, int VW, typename O>
static hipError_t vcycle_t(ope_ctx* c, const T* r, T* z, const int32_t* active, bool dots) {
  const uint32_t N = (uint32_t)c->N, NV = N / VW;
  const int k0 = c->mg_k0;                        // first fused level, at least 1
  hipStream_t s = c->stream;
  for (int k = 0; k < k0; ++k) {
    const MgLevel& f = c->mg[k];
    const MgLevel& q = c->mg[k + 1];
    const T* in = k == 0 ? r : (const T*)f.B;
    const TShape ts = tshape(f.m0, f.m1, f.m2, NV, N, sizeof(T));
    const ZMarch zq = zmarch_shape(q.m0, q.m1, q.m2, NV);
    const dim3 sgrid(ts.nxt * ts.nyt * ts.nzc * ts.NS), sblock(ts.TX * ts.TY * ts.NVS);
    switch (ring_per_thread(ts)) {
      case 1:
        hipLaunchKernelGGL((k_mg_tstencil<T, VW, 1, O>), sgrid, sblock, 0, s, in, (T*)f.T, geom(f), f.diag, f.wd, active,
                           N, ts);
        break;
      case 2:
        hipLaunchKernelGGL((k_mg_tstencil<T, VW, 2, O>), sgrid, sblock, 0, s, in, (T*)f.T, geom(f), f.diag, f.wd, active,
                           N, ts);
        break;
      default:
        hipLaunchKernelGGL((k_mg_tstencil<T, VW, 4, O>), sgrid, sblock, 0, s, in, (T*)f.T, geom(f), f.diag, f.wd, active,
                           N, ts);
    }
    hipLaunchKernelGGL((k_mg_zrestrict<T, VW>), dim3(zq.nxs * q.m1 * zq.nzc), dim3(MG_WG), 0, s, (const T*)f.T,
                       (T*)q.B, geom(f), geom(q), active, N, NV, zq);
  }
  size_t values = 0;
  McArgs ma = coarse_args(c->mg, c->mg_levels, k0, &values);
  ma.diag0 = c->mg[k0].diag;
  ma.wd0 = c->mg[k0].wd;
  ma.cdat = c->mg_cdat;
  ma.inv = c->mg_inv;
  hipLaunchKernelGGL((k_mg_coarse<T>), dim3(N), dim3(MC_WG), values * sizeof(T), s, (const T*)c->mg[k0].B, (T*)c->mg[k0].E, ma, active,
                     N);
  for (int k = k0 - 1; k >= 0; --k) {
    const MgLevel& f = c->mg[k];
    const MgLevel& q = c->mg[k + 1];
    const T* in = k == 0 ? r : (const T*)f.B;
    T* out = k == 0 ? z : (T*)f.E;
    const T* qe = (const T*)q.E;
    const TShape ts = tshape(f.m0, f.m1, f.m2, NV, N, sizeof(T));
    const uint32_t rows = ts.nxt * ts.nyt * ts.nzc;
    const uint32_t P = ts.TX * ts.TY;
    const int R = ring_per_thread(ts);
    const dim3 grid(rows * ts.NS), block(P * ts.NVS);
    const bool d = k == 0 && dots;
    double* part = d ? c->mg_part : nullptr;
    auto post = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, block, 0, s, in, qe, out, geom(f), geom(q), f.diag, f.wd, active, N, ts, part);
    };
    {
      ProfScope ps(c, d ? OPE_KERNEL_MG_POST : OPE_KERNEL_COUNT);   // only the finest level is timed
      if (d) {
        if (R == 1) post(k_mg_tpost<T, VW, true, 1, O>);
        else if (R == 2) post(k_mg_tpost<T, VW, true, 2, O>);
        else post(k_mg_tpost<T, VW, true, 4, O>);
        c->mg_rows_used = rows;
      } else {
        if (R == 1) post(k_mg_tpost<T, VW, false, 1, O>);
        else if (R == 2) post(k_mg_tpost<T, VW, false, 2, O>);
        else post(k_mg_tpost<T, VW, false, 4, O>);
      }
    }
  }
  return hipGetLastError();
}

// Whether a plane of the finest level's blocks (and of its coefficients, at most
// 8 bytes a point) stays below 4 GiB: always in 3D (checked when the context is
// created), in 2D, where the one plane is the whole block, up to 2^29 FP64 values.
static bool narrow_planes(const ope_ctx* c) {
  return (uint64_t)c->mg[0].m0 * c->mg[0].m1 * (uint64_t)c->N * 8u < ((uint64_t)1 << 32);
}

template <typename T, int VW>
static hipError_t vcycle(ope_ctx* c, const void* r, void* z, const int32_t* active, bool dots) {
  return narrow_planes(c) ? vcycle_t<T, VW, uint32_t>(c, (const T*)r, (T*)z, active, dots)
                          : vcycle_t<T, VW, uint64_t>(c, (const T*)r, (T*)z, active, dots);
}

hipError_t mg_vcycle(ope_ctx* c, const void* r, void* z, const int32_t* active, bool dots) {
  ProfScope ps(c, OPE_KERNEL_MG);
  if (c->prec == OPE_FP64) {
    if (mg_vw(c) == 2) return vcycle<double, 2>(c, r, z, active, dots);
    return vcycle<double, 1>(c, r, z, active, dots);
  }
  switch (mg_vw(c)) {
    case 4: return vcycle<float, 4>(c, r, z, active, dots);
    case 2: return vcycle<float, 2>(c, r, z, active, dots);
    default: return vcycle<float, 1>(c, r, z, active, dots);
  }
}

template <bool START>
static hipError_t launch_pcg_scalars(ope_ctx* c, int32_t* flags) {
  const double* part = c->mg_part;
  int64_t rows = c->mg_rows_used;
  if (rows * 2 * c->N > PS_MAX) {
    const hipError_t e = launch_reduce_stage(c, &part, &rows, 2 * c->N);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_pcg_scalars<START>, dim3(1), dim3(PS_WG), 0, c->stream, part, (uint32_t)rows, (uint32_t)c->N,
                     c->rho, c->beta, c->target, c->active, c->sc, flags);
  return hipGetLastError();
}

hipError_t launch_pcg_start(ope_ctx* c) { return launch_pcg_scalars<true>(c, nullptr); }

hipError_t launch_pcg_beta(ope_ctx* c, int32_t* flags) {
  ProfScope ps(c, OPE_KERNEL_CG_REDUCE);
  return launch_pcg_scalars<false>(c, flags);
}
