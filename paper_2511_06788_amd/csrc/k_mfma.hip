// Dense tall-skinny contractions of the step on the gfx950 matrix cores.
//
//  * Inner matrices <X, Y> = X^T Y over the n grid rows (the Grams
//    <U,U>, <U,HU>, <U,GU>, <GU,GU> used by Steps 2-3 of Section 4.1).
//  * Row-block products Out = cbeta C + ascale (X0 M0 + X1 M1) with small N x N
//    matrices (the residual HU - U Lam, the warm start U Lam^{-1}, Step 4's
//    update, and in mixed precision the projection Y - U <U,Y>).
//
// Three arithmetic kinds, chosen per call:
//   MK_F64   v_mfma_f64_16x16x4f64 on FP64 (inputs FP64, or FP32 widened)
//   MK_F32   v_mfma_f32_16x16x4f32 on FP32 inputs, FP32 accumulation
//   MK_BF16  v_mfma_f32_16x16x32_bf16: FP32 inputs rounded to BF16, FP32 accumulation
// Operand layout for lane l (checked on the device): the A operand supplies
// A[l % 16][k] and the B operand B[k][l % 16], with k = l / 16 (16x16x4) or
// k = 8 (l / 16) + e, e = 0..7 (16x16x32).  The 16 x 16 accumulator holds
// D[l / 16 + 4 r][l % 16] in element r for the FP64 instruction and
// D[4 (l / 16) + r][l % 16] for the FP32 and BF16 instructions.
//
// For the Gram the contraction index is the grid row, so a lane reads
// X[row0 + k][i0 + l%16]: rows of 16 consecutive orbitals.  Split-K over rows
// writes one partial per split (in FP64); a fixed-order column reduction
// follows, so results are bitwise reproducible.
//
// Kernels by shape.  Grams: straight from global memory into registers
// (k_gram_rows), except wide aligned products of two FP32 blocks and wide BF16
// ones, which stage panels in LDS with 128 x 128 work-group tiles (k_gram_lds).
// Row products: k_rowmm_strip (M in LDS, 16 rows per
// wave from global memory) for FP64 up to 112 columns or of any unaligned rows
// and for FP32 up to 80; wide aligned rows k_rowmm_lds (both panels in LDS); of
// the rest (BF16, and the FP32 widths that the strip is slower at) up to 32
// columns k_rowmm_narrow and above k_rowmm.
#include <algorithm>
#include <type_traits>

#include "ope_internal.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int KIND> struct Mk;
template <> struct Mk<MK_F64> {
  using acc_t = v4d;
  static constexpr int KSTEP = 4;       // contraction length per instruction
  static constexpr int KPL = 1;         // contraction elements per lane
  __device__ static uint32_t drow(uint32_t kr, int r) { return kr + 4u * (uint32_t)r; }
};
template <> struct Mk<MK_F32> {
  using acc_t = v4f;
  static constexpr int KSTEP = 4;
  static constexpr int KPL = 1;
  __device__ static uint32_t drow(uint32_t kr, int r) { return 4u * kr + (uint32_t)r; }
};
template <> struct Mk<MK_BF16> {
  using acc_t = v4f;
  static constexpr int KSTEP = 32;
  static constexpr int KPL = 8;
  __device__ static uint32_t drow(uint32_t kr, int r) { return 4u * kr + (uint32_t)r; }
};

// Contraction indices per LDS panel of the staged kernels: at least 16, and a
// whole MFMA contraction step.
template <int KIND> struct PanelRows { static constexpr int KC = Mk<KIND>::KSTEP < 16 ? 16 : Mk<KIND>::KSTEP; };

// One MFMA with operands given as KPL values per lane (in the input type).
template <int KIND, typename TI>
__device__ __forceinline__ typename Mk<KIND>::acc_t mma(const TI (&a)[Mk<KIND>::KPL], const TI (&b)[Mk<KIND>::KPL],
                                                        typename Mk<KIND>::acc_t c) {
  if constexpr (KIND == MK_F64) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[0], (double)b[0], c, 0, 0, 0);
  } else if constexpr (KIND == MK_F32) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32((float)a[0], (float)b[0], c, 0, 0, 0);
  } else {
    v8bf av, bv;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      av[e] = (__bf16)(float)a[e];
      bv[e] = (__bf16)(float)b[e];
    }
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
  }
}

template <typename V>
__device__ __forceinline__ V zero_acc() {
  V z;
#pragma unroll
  for (int r = 0; r < 4; ++r) z[r] = 0;
  return z;
}

constexpr int GT2 = 128;    // tile edge and wave tile edge of the Grams from LDS
constexpr int GW2 = 64;

// Grams straight from global memory (k_gram_rows).  The four waves of a
// work-group take the contraction steps w, w + 4, ... of its rows, and every
// wave holds all the 16 x 16 blocks of the output tile: a value is loaded once
// per wave and feeds a whole row or column of blocks from its register (for
// A^T A as both operands), with no LDS and no barrier in the loop.  The loads of
// the next groups of U steps are in flight while one is multiplied.  The waves' tiles
// are summed in LDS in wave order at the end.  Bound by memory up to about 64
// columns of FP64 and by the matrix cores above; the kernels before it loaded
// every value once per block that used it, computed both triangles and reduced
// twice as many partials in two launches.  A^T A at 48^3, FP64 (us, before ->
// after, with the sum of the partials): N = 17 19 -> 14, 45 41 -> 20, 96 120 -> 33,
// 128 69 -> 57, 161 272 -> 115, 256 292 -> 176, 512 984 -> 652; two blocks 96
// 119 -> 47.
//   G_SAME   A^T A, the NB (NB + 1) / 2 blocks on and above the block diagonal
//   G_UPPER  A^T B known to be symmetric, the same blocks
//   G_FULL   any A^T B in NB x NB tiles
// Loads have a uniform base and a fixed 32-bit offset per lane and block (O; 64
// bits where 32 rows may span 2^31 bytes).  Columns past the edge read the last
// column: their values reach only output that is not stored.
enum { G_SAME = 0, G_UPPER = 1, G_FULL = 2 };

// Split and tile of a work-group (grid: splits x tiles, the tiles all of them or
// those on and above the diagonal).  With the splits a multiple of 8 the tiles of
// one split run on one XCD (work-groups a multiple of 8 apart), whose L2 then
// serves the rows they share.
__device__ __forceinline__ void gram_place(uint32_t ntj, int upper, uint32_t* ks, uint32_t* ti, uint32_t* tj) {
  const uint32_t nt = gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
  uint32_t t = blockIdx.y;
  *ks = blockIdx.x;
  if (nt > 1 && gridDim.x % 8u == 0) {
    *ks = lin / (8u * nt) * 8u + lin % 8u;
    t = lin / 8u % nt;
  }
  if (!upper) {
    *ti = t / ntj;
    *tj = t % ntj;
    return;
  }
  uint32_t a = 0;
  while (t >= ntj - a) t -= ntj - a++;
  *ti = a;
  *tj = a + t;
}

template <typename TI, int KIND, int NB, int MODE>
struct GramTile {
  static constexpr int KPL = Mk<KIND>::KPL;
  static constexpr int NBLK = MODE == G_FULL ? NB * NB : NB * (NB + 1) / 2;
  static constexpr int LB = MODE == G_SAME ? NB : 2 * NB;                     // values of a step per lane and row
  static constexpr int SB = LB * KPL * (int)sizeof(TI);                       // its bytes
  static constexpr int ACC = NBLK * (KIND == MK_F64 ? 8 : 4);                 // accumulator registers
  // steps per group: 128 bytes per lane, at most four; where the accumulators
  // leave one wave per SIMD, one step per group and more groups in flight instead
  static constexpr int U0 = SB >= 128 ? 1 : (128 + SB - 1) / SB > 4 ? 4 : (128 + SB - 1) / SB;
  static constexpr int OCC = ACC + U0 * SB / 2 <= 200 ? 2 : 1;                // work-groups per compute unit
  static constexpr int U = OCC == 2 ? U0 : 1;
  // (36 FP64 blocks do not fit the 256 accumulation registers: four of them move
  // in and out by every step, 104 us for A^T A at 64^3, N = 128, of 61 for the
  // matrix instructions alone)
  static constexpr int FIT = (352 - ACC) / (SB / 4);
  static constexpr int DEPTH = OCC == 2 || FIT < 2 ? 2 : FIT > 4 ? 4 : FIT;   // groups in registers
  static_assert(MODE != G_FULL || NB > 4 || OCC == 2, "gram_t plans two tiles per compute unit");
  // blocks of tile row a: columns first(a) .. NB - 1, numbered from at(a, first(a))
  static __device__ constexpr int first(int a) { return MODE == G_FULL ? 0 : a; }
  static __device__ constexpr int at(int a, int b) { return MODE == G_FULL ? a * NB + b : a * NB - a * (a - 1) / 2 + b - a; }
};

template <typename TI, int KIND, int NB, int MODE, typename O>
__global__ __launch_bounds__(256, (GramTile<TI, KIND, NB, MODE>::OCC)) void k_gram_rows(
    const TI* __restrict__ A, uint64_t lda, uint32_t na, const TI* __restrict__ B, uint64_t ldb, uint32_t nb,
    uint32_t rows, uint32_t rows_per_split, uint32_t ntj, int upper, double* __restrict__ part) {
  using M = Mk<KIND>;
  using T = GramTile<TI, KIND, NB, MODE>;
  using acc_t = typename M::acc_t;
  constexpr int KPL = M::KPL, U = T::U, NBLK = T::NBLK;
  constexpr bool TWO = MODE != G_SAME;
  __shared__ double red[4][NB][4][64];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  uint32_t ks, ti, tj;
  gram_place(ntj, upper, &ks, &ti, &tj);
  const uint32_t i0 = ti * (16u * NB), j0 = tj * (16u * NB);
  const uint32_t r0 = (uint32_t)min((uint64_t)rows, (uint64_t)ks * rows_per_split);
  const uint32_t r1 = r0 + min(rows - r0, rows_per_split);
  O ao[NB], bo[TWO ? NB : 1];
#pragma unroll
  for (int x = 0; x < NB; ++x) ao[x] = min(i0 + 16u * x + ci, na - 1u);
  if constexpr (TWO) {
#pragma unroll
    for (int x = 0; x < NB; ++x) bo[x] = min(j0 + 16u * x + ci, nb - 1u);
  }
  acc_t acc[NBLK];
#pragma unroll
  for (int q = 0; q < NBLK; ++q) acc[q] = zero_acc<acc_t>();
  struct Vals {
    TI a[U][NB][KPL], b[U][TWO ? NB : 1][KPL];
  };
  const uint64_t sa = (uint64_t)kr * KPL * lda, sb = (uint64_t)kr * KPL * ldb;
  auto load = [&](auto tail, uint32_t g, Vals& v) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t st = ((g * U + u) * 4u + wave) * M::KSTEP, p = r0 + st;  // uniform
#pragma unroll
      for (int e = 0; e < KPL; ++e) {
        uint64_t ra = sa, rb = sb;
        bool ok = true;
        const TI *pa = A + (uint64_t)(p + e) * lda, *pb = B + (uint64_t)(p + e) * ldb;
        if constexpr (decltype(tail)::value) {
          ok = st + kr * KPL + e < r1 - r0;
          if (!ok) {                                  // any row of the split, and zero instead of its value
            pa = A + (uint64_t)r0 * lda;
            pb = B + (uint64_t)r0 * ldb;
            ra = rb = 0;
          }
        }
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          const TI t = pa[(O)ra + ao[x]];
          v.a[u][x][e] = ok ? t : TI(0);
        }
        if constexpr (TWO) {
#pragma unroll
          for (int x = 0; x < NB; ++x) {
            const TI t = pb[(O)rb + bo[x]];
            v.b[u][x][e] = ok ? t : TI(0);
          }
        }
      }
    }
  };
  auto mul = [&](const Vals& v) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = T::first(i); j < NB; ++j) {
          if constexpr (TWO) acc[T::at(i, j)] = mma<KIND, TI>(v.a[u][i], v.b[u][j], acc[T::at(i, j)]);
          else acc[T::at(i, j)] = mma<KIND, TI>(v.a[u][i], v.a[u][j], acc[T::at(i, j)]);
        }
  };
  // groups of 4 U steps (U per wave); the last one may end before its last row
  constexpr uint32_t GR = 4u * U * M::KSTEP;
  const uint32_t ng = (r1 - r0) / GR;
  // a group's registers are loaded again as soon as it is multiplied; with two
  // groups only, that form spills and the other group is loaded before
  constexpr uint32_t D = T::DEPTH;
  constexpr bool BEFORE = T::OCC == 1 && D == 2;
  Vals v[D];
  if constexpr (BEFORE) {
    if (ng > 0) load(std::false_type{}, 0, v[0]);
    for (uint32_t g = 0; g < ng; g += 2) {
      if (g + 1 < ng) load(std::false_type{}, g + 1, v[1]);
      __builtin_amdgcn_sched_barrier(0);
      mul(v[0]);
      if (g + 1 < ng) {
        if (g + 2 < ng) load(std::false_type{}, g + 2, v[0]);
        __builtin_amdgcn_sched_barrier(0);
        mul(v[1]);
      }
    }
  } else {
#pragma unroll
    for (uint32_t d = 0; d < D; ++d)
      if (d < ng) load(std::false_type{}, d, v[d]);
    for (uint32_t g = 0; g < ng; g += D) {
#pragma unroll
      for (uint32_t d = 0; d < D; ++d) {
        if (g + d >= ng) break;                       // uniform, as the next
        __builtin_amdgcn_sched_barrier(0);
        mul(v[d]);
        __builtin_amdgcn_sched_barrier(0);
        if (g + d + D < ng) load(std::false_type{}, g + d + D, v[d]);
      }
    }
  }
  if (r0 + ng * GR < r1) {
    load(std::true_type{}, ng, v[0]);
    mul(v[0]);
  }
  double* out = part + (uint64_t)ks * na * nb;
#pragma unroll
  for (int a = 0; a < NB; ++a) {                      // the blocks of tile row a over the four waves
    if (a > 0) __syncthreads();
#pragma unroll
    for (int b = T::first(a); b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][b][r][lane] = (double)acc[T::at(a, b)][r];
    __syncthreads();
    const uint32_t i = i0 + 16u * a + M::drow(kr, (int)wave);
#pragma unroll
    for (int b = T::first(a); b < NB; ++b) {
      const uint32_t j = j0 + 16u * b + ci;
      const double v = red[0][b][wave][lane] + red[1][b][wave][lane] + red[2][b][wave][lane] + red[3][b][wave][lane];
      if (i < na && j < nb) out[(uint64_t)i * nb + j] = v;
    }
  }
}

// Sum of the ks partial Grams, 64 entries (four rows of one 16 x 16 block) per
// work-group of 16 waves that split the partials, added in a fixed order.  UPPER:
// the blocks on and above the block diagonal hold values; the others mirror them.
// A launch of few loads in flight is bound by their latency, so each thread keeps
// eight.
template <bool UPPER>
__global__ __launch_bounds__(1024) void k_gram_sum(const double* __restrict__ part, uint32_t ks, uint32_t na,
                                                   uint32_t nb, double* __restrict__ out) {
  __shared__ double red[16][64];
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t nbj = (nb + 15u) / 16u;
  uint32_t a = 0, b = blockIdx.x >> 2;
  if constexpr (UPPER) {
    while (b >= nbj - a) b -= nbj - a++;
    b += a;
  } else {
    a = b / nbj;
    b %= nbj;
  }
  const uint32_t i = 16u * a + 4u * (blockIdx.x & 3u) + (lane >> 4), j = 16u * b + (lane & 15u);
  const bool ok = i < na && j < nb;
  const uint64_t o = (uint64_t)i * nb + j, sz = (uint64_t)na * nb;
  double s = 0.0;
  if (ok) {
    const uint32_t n = ks > w ? (ks - w + 15u) / 16u : 0u;      // partials w, w + 16, ...
    const double* p = part + w * sz + o;
    uint32_t k = 0;
    for (; k + 8 <= n; k += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(uint64_t)(k + u) * 16u * sz];
      s += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    for (; k < n; ++k) s += p[(uint64_t)k * 16u * sz];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w != 0 || !ok) return;
  double t = red[0][lane];
#pragma unroll
  for (int u = 1; u < 16; ++u) t += red[u][lane];
  out[o] = t;
  if (UPPER && a != b) out[(uint64_t)j * nb + i] = t;
}

// Row-block products Out = cbeta Cm + ascale (X0 M0 + X1 M1).  Work-group =
// 4 waves, 2 (rows) x 2 (columns); a wave owns 32 rows x 64 columns (2 x 4
// MFMA blocks), the work-group 64 x 128.  TI is the type of X, M, Cm and Out.
// Predication of the row-block products (bits of `predicated`): ROWMM_IF_OK
// skips the launch when the step's device error flag is set (a failed small
// solve leaves the block untouched), ROWMM_IF_RENORM unless the drift check
// asked for a re-normalisation.
__device__ __forceinline__ bool rowmm_skip(int predicated, const OpeScalars* __restrict__ sc) {
  return ((predicated & ROWMM_IF_OK) && sc->err != 0) || ((predicated & ROWMM_IF_RENORM) && sc->renorm == 0);
}

constexpr int RT = 64;      // rows per work-group tile
constexpr int CT = 128;     // columns per work-group tile

template <typename TI, int KIND, int NSRC>
__global__ __launch_bounds__(256) void k_rowmm(const TI* X0, const TI* __restrict__ M0, const TI* X1,
                                               const TI* __restrict__ M1, const TI* Cm, double cbeta, double ascale,
                                               TI* Out, uint32_t n, uint32_t N, int want_colsq, int predicated,
                                               const OpeScalars* __restrict__ sc, double* __restrict__ part) {
  using MK = Mk<KIND>;
  using acc_t = typename MK::acc_t;
  __shared__ double colsq[2][CT];
  if (rowmm_skip(predicated, sc)) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t wr = wave >> 1, wc = wave & 1u;
  const uint32_t row_base = blockIdx.x * RT + wr * 32;
  const uint32_t col_base = blockIdx.y * CT + wc * 64;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  acc_t acc[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = zero_acc<acc_t>();

#pragma unroll
  for (int s = 0; s < NSRC; ++s) {
    const TI* X = s == 0 ? X0 : X1;
    const TI* M = s == 0 ? M0 : M1;
    for (uint32_t k = 0; k < N; k += MK::KSTEP) {
      TI av[2][MK::KPL], bv[4][MK::KPL];
#pragma unroll
      for (int e = 0; e < MK::KPL; ++e) {
        const uint32_t kk = k + kr * MK::KPL + e;   // contraction index held by this lane
        const bool kok = kk < N;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const uint32_t row = row_base + a * 16 + ci;
          av[a][e] = (kok && row < n) ? X[(uint64_t)row * N + kk] : TI(0);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const uint32_t col = col_base + b * 16 + ci;
          bv[b][e] = (kok && col < N) ? M[(uint64_t)kk * N + col] : TI(0);
        }
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mma<KIND, TI>(av[a], bv[b], acc[a][b]);
    }
  }
  // Out may alias X0 (in-place Step 4): every wave of the tile has finished
  // reading its rows before any wave writes.
  __syncthreads();
  double sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t row = row_base + a * 16 + MK::drow(kr, r);
        const uint32_t col = col_base + b * 16 + ci;
        if (row < n && col < N) {
          const uint64_t o = (uint64_t)row * N + col;
          TI v = (TI)(ascale * (double)acc[a][b][r]);
          if (cbeta != 0.0) v += (TI)cbeta * Cm[o];
          Out[o] = v;
          sq[b] += (double)v * (double)v;
        }
      }
  if (!want_colsq) return;
  // per-column sums over the tile's rows: lanes l, l^16, l^32, l^48 share a column
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    sq[b] += __shfl_xor(sq[b], 16);
    sq[b] += __shfl_xor(sq[b], 32);
  }
  if (kr == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) colsq[wr][wc * 64 + b * 16 + ci] = sq[b];
  }
  __syncthreads();
  if (threadIdx.x < CT) {
    const uint32_t col = blockIdx.y * CT + threadIdx.x;
    if (col < N) part[(uint64_t)blockIdx.x * N + col] = colsq[0][threadIdx.x] + colsq[1][threadIdx.x];
  }
}

// Narrow row-block products (N <= 32): work-group tile 128 rows x N columns,
// each wave 32 rows x 32 columns (2 x 2 MFMA blocks).  The tile's rows of X,
// of Cm and of the result are contiguous in memory, so they pass through LDS
// and every global access is a run of whole rows (the MFMA operand pattern
// itself reads 16 rows x 4 values per instruction, 16 cache lines).  Sources
// are staged one after the other; the LDS row stride is odd, so the 16 rows of
// an operand read fall in distinct banks.
constexpr int RTN = 128;    // rows per work-group tile
constexpr int LDXN = 33;    // LDS row stride of the staged tile

template <typename TI, int KIND, int NSRC>
__global__ __launch_bounds__(256) void k_rowmm_narrow(const TI* X0, const TI* __restrict__ M0, const TI* X1,
                                                      const TI* __restrict__ M1, const TI* Cm, double cbeta,
                                                      double ascale, TI* Out, uint32_t n, uint32_t N, int want_colsq,
                                                      int predicated, const OpeScalars* __restrict__ sc,
                                                      double* __restrict__ part) {
  using MK = Mk<KIND>;
  using acc_t = typename MK::acc_t;
  __shared__ TI xs[RTN * LDXN];
  __shared__ TI ms[32 * 32];
  __shared__ double colsq[8][32];
  if (rowmm_skip(predicated, sc)) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  const uint32_t row0 = blockIdx.x * RTN;
  const uint32_t tc = threadIdx.x & 31u, tg = threadIdx.x >> 5;    // column and row group of the copies
  const uint32_t wr = wave * 32u;                                  // the wave's first row in the tile
  acc_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = zero_acc<acc_t>();
#pragma unroll
  for (int s = 0; s < NSRC; ++s) {
    const TI* X = s == 0 ? X0 : X1;
    const TI* M = s == 0 ? M0 : M1;
    if (s > 0) __syncthreads();                  // the previous source's operands are consumed
#pragma unroll 4
    for (uint32_t u = 0; u < RTN / 8; ++u) {
      const uint32_t r = tg + 8u * u, gr = row0 + r;
      xs[r * LDXN + tc] = (gr < n && tc < N) ? X[(uint64_t)gr * N + tc] : TI(0);
    }
    for (uint32_t e = threadIdx.x; e < 32u * 32u; e += 256u) {
      const uint32_t kk = e >> 5, col = e & 31u;
      ms[e] = (kk < N && col < N) ? M[(uint64_t)kk * N + col] : TI(0);
    }
    __syncthreads();
    // contraction over the zero-padded 32 indices, in whole MFMA steps
    for (uint32_t k = 0; k < N; k += MK::KSTEP) {
      TI av[2][MK::KPL], bv[2][MK::KPL];
#pragma unroll
      for (int e = 0; e < MK::KPL; ++e) {
        const uint32_t kk = k + kr * MK::KPL + e;
#pragma unroll
        for (int a = 0; a < 2; ++a) av[a][e] = xs[(wr + a * 16 + ci) * LDXN + kk];
#pragma unroll
        for (int b = 0; b < 2; ++b) bv[b][e] = ms[kk * 32 + b * 16 + ci];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = mma<KIND, TI>(av[a], bv[b], acc[a][b]);
    }
  }
  // every operand read of the tile is done before the result replaces it
  // (Out may alias X0: in-place Step 4)
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        xs[(wr + a * 16 + MK::drow(kr, r)) * LDXN + b * 16 + ci] = (TI)(ascale * (double)acc[a][b][r]);
  __syncthreads();
  double sq = 0.0;
#pragma unroll 4
  for (uint32_t u = 0; u < RTN / 8; ++u) {
    const uint32_t r = tg + 8u * u, gr = row0 + r;
    if (gr < n && tc < N) {
      const uint64_t o = (uint64_t)gr * N + tc;
      TI v = xs[r * LDXN + tc];
      if (cbeta != 0.0) v += (TI)cbeta * Cm[o];
      Out[o] = v;
      sq += (double)v * (double)v;
    }
  }
  if (!want_colsq) return;
  colsq[tg][tc] = sq;
  __syncthreads();
  if (threadIdx.x < N) {
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += colsq[g][threadIdx.x];
    part[(uint64_t)blockIdx.x * N + threadIdx.x] = t;
  }
}

// Row-block products from LDS (N a multiple of the 16-byte chunk, aligned
// blocks): work-group tile RTW rows x 128 columns, each wave RTW/2 x 64
// (RTW/32 x 4 MFMA blocks; RTW = 128, or 64 for the FP64 kind).  Panels of KC contraction indices are staged in LDS, double
// buffered: X's rows (read as 16-byte chunks) are stored transposed, Xt[k][row],
// so that the MFMA operand reads of both panels are contiguous across lanes,
// and the KC rows of M beside them.  M is read once per work-group instead of
// once per wave and 64-row tile.  At N = 128 the four products of an FP64 step
// move ten blocks of 64^3 rows (571 us at the copy rate) and measured 1030 us, 935
// with unconditional loads and the xor-ed layout below; at 96^3, N = 512 they are
// bound by the matrix cores (45.0 -> 42.7 ms, 54 of 73 TFLOP/s).
constexpr int RT2 = 128;    // rows per work-group tile
constexpr int RT2H = 64;    // rows per work-group tile of the FP64 kind

template <typename TI, int KIND, int NSRC, int RTW>
__global__ __launch_bounds__(256, RTW == RT2H ? 3 : 2) void k_rowmm_lds(const TI* X0, const TI* __restrict__ M0, const TI* X1,
                                                   const TI* __restrict__ M1, const TI* Cm, double cbeta,
                                                   double ascale, TI* Out, uint32_t n, uint32_t N, int want_colsq,
                                                   int predicated, const OpeScalars* __restrict__ sc,
                                                   double* __restrict__ part) {
  using MK = Mk<KIND>;
  using acc_t = typename MK::acc_t;
  constexpr int KC = PanelRows<KIND>::KC;
  constexpr int VPC = 16 / (int)sizeof(TI);
  constexpr int XC = KC / VPC;                        // chunks per X row and panel
  constexpr int XCT = RTW * XC / 256;                 // X chunks per thread
  constexpr int AR = RTW / 32;                        // 16-row MFMA blocks per wave (a wave spans RTW / 2 rows)
  constexpr int MCR = CT / VPC;                       // chunks per M panel row
  constexpr int MCT = KC * MCR / 256;                 // M chunks per thread
  static_assert(XCT * 256 == RTW * XC && MCT * 256 == KC * MCR, "panel chunks must divide the work-group");
  typedef unsigned int Chunk __attribute__((ext_vector_type(4)));
  union ChunkV {
    Chunk c;
    TI v[VPC];
  };
  __shared__ __align__(16) TI xt[2][KC][RTW];
  __shared__ __align__(16) TI mp[2][KC][CT];
  __shared__ double colsq[2][CT];
  if (rowmm_skip(predicated, sc)) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t wr = wave >> 1, wc = wave & 1u;
  const uint32_t row0 = blockIdx.x * RTW, col0 = blockIdx.y * CT;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  acc_t acc[AR][4];
#pragma unroll
  for (int a = 0; a < AR; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = zero_acc<acc_t>();
  const uint32_t kpan = (N + KC - 1) / KC;          // panels per source
  const uint32_t npan = NSRC * kpan;
  ChunkV cx[XCT], cm[MCT];
  const Chunk z = {0u, 0u, 0u, 0u};
  // Loads are unconditional (a branch or a select behind one would wait for it
  // before the matrix instructions): past the edge they take the last row, column
  // or contraction index.  Rows' and columns' values reach only output that is not
  // stored; contraction indices past N are zeroed on the way into LDS.
  uint32_t ox[XCT], om[MCT];
#pragma unroll
  for (int u = 0; u < XCT; ++u) ox[u] = min((threadIdx.x + 256u * u) / XC, n - 1u - row0) * N;
#pragma unroll
  for (int u = 0; u < MCT; ++u) om[u] = min((threadIdx.x + 256u * u) % MCR * VPC, N - VPC - col0);
  auto load = [&](uint32_t t) {
    const uint32_t k0 = (t < kpan ? t : t - kpan) * KC;
    const TI* X = (t < kpan ? X0 : X1) + (uint64_t)row0 * N + k0;
    const TI* M = (t < kpan ? M0 : M1) + (uint64_t)k0 * N + col0;
#pragma unroll
    for (int u = 0; u < XCT; ++u)
      cx[u].c = *reinterpret_cast<const Chunk*>(X + ox[u] + min((threadIdx.x + 256u * u) % XC * VPC, N - VPC - k0));
#pragma unroll
    for (int u = 0; u < MCT; ++u)
      cm[u].c = *reinterpret_cast<const Chunk*>(M + min((threadIdx.x + 256u * u) / MCR, N - 1u - k0) * N + om[u]);
    __builtin_amdgcn_sched_barrier(0);
  };
  // FP64: LDS columns are xor-ed with a few bits of the contraction index k, so that
  // the transposed stores of X and the four k of an operand read spread over the
  // banks (N = 128, four products at 48^3: 450 -> 425 us; FP32 lost 10% to the
  // addresses of its 4-byte stores, 361 -> 396)
  auto swz_x = [](uint32_t k) -> uint32_t { return KIND == MK_F64 ? ((k >> 1 & 3u) << 3) ^ ((k & 1u) << 4) : 0u; };
  auto swz_m = [](uint32_t k) -> uint32_t { return KIND == MK_F64 ? (k & 1u) << 4 : 0u; };
  auto store = [&](int buf, uint32_t t) {
    const uint32_t left = N - (t < kpan ? t : t - kpan) * KC;
    __builtin_amdgcn_sched_barrier(0);
    if (left < KC) {                                  // uniform
#pragma unroll
      for (int u = 0; u < XCT; ++u)
        if ((threadIdx.x + 256u * u) % XC * VPC >= left) cx[u].c = z;
#pragma unroll
      for (int u = 0; u < MCT; ++u)
        if ((threadIdx.x + 256u * u) / MCR >= left) cm[u].c = z;
    }
#pragma unroll
    for (int u = 0; u < XCT; ++u) {
      const uint32_t c = threadIdx.x + 256u * u;
      const uint32_t r = c / XC, kc = (c % XC) * VPC;
#pragma unroll
      for (int e = 0; e < VPC; ++e) xt[buf][kc + e][r ^ swz_x(kc + e)] = cx[u].v[e];
    }
#pragma unroll
    for (int u = 0; u < MCT; ++u) {
      const uint32_t c = threadIdx.x + 256u * u;
      const uint32_t kk = c / MCR, col = (c % MCR) * VPC;
      *reinterpret_cast<Chunk*>(&mp[buf][kk][col ^ swz_m(kk)]) = cm[u].c;
    }
  };
  // where that puts the columns 16 q + ci, q = 0, 1, for a lane's k = kr mod 4
  constexpr int NS = KIND == MK_F64 ? 2 : 1;
  uint32_t bx[NS], bm[NS];
#pragma unroll
  for (uint32_t q = 0; q < (uint32_t)NS; ++q) {
    bx[q] = (16u * q + ci) ^ (KIND == MK_F64 ? ((kr >> 1) << 3) ^ ((kr & 1u) << 4) : 0u);
    bm[q] = (16u * q + ci) ^ (KIND == MK_F64 ? (kr & 1u) << 4 : 0u);
  }
  load(0);
  store(0, 0);
  __syncthreads();
  for (uint32_t t = 0; t < npan; ++t) {
    const int buf = (int)(t & 1u);
    if (t + 1 < npan) load(t + 1);
#pragma unroll
    for (int kk = 0; kk < KC / MK::KSTEP; ++kk) {
      TI av[AR][MK::KPL], bv[4][MK::KPL];
#pragma unroll
      for (int e = 0; e < MK::KPL; ++e) {
        const uint32_t k = kk * MK::KSTEP + kr * MK::KPL + e;
#pragma unroll
        for (int a = 0; a < AR; ++a)
          av[a][e] = xt[buf][k][wr * (RTW / 2) + a / NS * (16 * NS) + bx[(a ^ kk) % NS]];
#pragma unroll
        for (int b = 0; b < 4; ++b) bv[b][e] = mp[buf][k][wc * 64 + b / NS * (16 * NS) + bm[b % NS]];
      }
#pragma unroll
      for (int a = 0; a < AR; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mma<KIND, TI>(av[a], bv[b], acc[a][b]);
    }
    if (t + 1 < npan) store(buf ^ 1, t + 1);
    __syncthreads();
  }
  // every wave has read all of its rows (the last panel is in LDS) before any
  // wave writes: Out may alias X0 (in-place Step 4)
  double sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < AR; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t row = row0 + wr * (RTW / 2) + a * 16 + MK::drow(kr, r);
        const uint32_t col = col0 + wc * 64 + b * 16 + ci;
        if (row < n && col < N) {
          const uint64_t o = (uint64_t)row * N + col;
          TI v = (TI)(ascale * (double)acc[a][b][r]);
          if (cbeta != 0.0) v += (TI)cbeta * Cm[o];
          Out[o] = v;
          sq[b] += (double)v * (double)v;
        }
      }
  if (!want_colsq) return;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    sq[b] += __shfl_xor(sq[b], 16);
    sq[b] += __shfl_xor(sq[b], 32);
  }
  if (kr == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) colsq[wr][wc * 64 + b * 16 + ci] = sq[b];
  }
  __syncthreads();
  if (threadIdx.x < CT) {
    const uint32_t col = col0 + threadIdx.x;
    if (col < N) part[(uint64_t)blockIdx.x * N + col] = colsq[0][threadIdx.x] + colsq[1][threadIdx.x];
  }
}

// Row-block products of the FP64 and FP32 kinds at any width (k_rowmm_strip).  A
// work-group of eight waves holds a chunk of M in LDS (KC contraction indices x
// 128 columns, two buffers) and walks over 128-row tiles; a wave takes 16 rows by
// all 128 columns, so no other wave reads its rows and their values go from
// global memory straight into the A operand.  The contraction order is free, so
// a lane takes 16 consecutive bytes of its row (VPC values) and the VPC
// instructions of a group use the k = VPC kr + e it then holds: 16 rows x 64
// contiguous bytes per load, against 16 x 8 values of one MFMA.
// With one source and N <= 2 KC both chunks of M stay in LDS for the whole
// launch, and the waves run on with no barrier, one wave's epilogue under
// another's matrix instructions; otherwise chunks stream through the two buffers
// (one barrier per chunk of 128 matrix instructions per wave).  The next chunk's
// loads are in flight while the current one is multiplied.
// Columns in blocks of 16 (NB of them, so that a narrow M costs no idle
// instructions).  VEC: rows split into whole aligned 16-byte chunks; else values
// are loaded one by one.
// Bound by memory up to about 64 columns and by the matrix cores above; what the
// kernels before it lost was a whole 128-column tile of instructions for any
// width above 32, rows re-read by the waves of the other column half, and a
// barrier per panel.  One step's four products at 48^3, FP64: N = 17 113 -> 81 us,
// 45 262 -> 146, 96 391 -> 324, 127 722 -> 538 (the full table is at the rule in
// rowmm_t).
template <typename TI>
struct Strip {
  static constexpr int VPC = 16 / (int)sizeof(TI);
  static constexpr int XG = 8;                        // 16-byte groups of a row per chunk and lane
  static constexpr int KC = XG * 4 * VPC;             // 64 (FP64) or 128 (FP32) contraction indices per chunk
  // row stride of M in LDS: the four kr rows of an operand read fall in distinct
  // banks (rows VPC apart: 2 * 136 * 2 words = 32 mod 64; 4 * 132 = 16 mod 64)
  static constexpr int LD = sizeof(TI) == 8 ? 136 : 132;
  static constexpr int BUF = KC * LD;                 // elements of a buffer
};
constexpr int ST_ROWS = 128;                          // rows per tile
constexpr int ST_WG = 512;

template <typename TI, int KIND, int NB, bool VEC>
__global__ __launch_bounds__(ST_WG, 2) void k_rowmm_strip(const TI* X0, const TI* __restrict__ M0, const TI* X1,
                                                          const TI* __restrict__ M1, const TI* Cm, double cbeta,
                                                          double ascale, TI* Out, uint32_t n, uint32_t N,
                                                          uint32_t ntiles, int want_colsq, int predicated,
                                                          const OpeScalars* __restrict__ sc,
                                                          double* __restrict__ part) {
  using MK = Mk<KIND>;
  using acc_t = typename MK::acc_t;
  using S = Strip<TI>;
  constexpr int VPC = S::VPC, XG = S::XG, KC = S::KC, LD = S::LD;
  constexpr int MR = 128 / VPC;                       // 16-byte chunks per row of M
  constexpr int MT = KC * MR / ST_WG;                 // of them per thread
  static_assert(MT * ST_WG == KC * MR, "M chunks must divide the work-group");
  typedef unsigned int Chunk __attribute__((ext_vector_type(4)));
  union ChunkV {
    Chunk c;
    TI v[VPC];
  };
  extern __shared__ __align__(16) char strip_lds[];
  TI* const ml = reinterpret_cast<TI*>(strip_lds);    // one or two buffers, then the column sums
  if (rowmm_skip(predicated, sc)) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  const uint32_t col0 = blockIdx.y * 128u;
  const uint32_t kc = (N + KC - 1) / KC;              // chunks per source
  const uint32_t nch = X1 ? 2 * kc : kc;
  const bool resident = nch <= 2;
  auto load_x = [&](uint32_t tile, uint32_t c, ChunkV(&x)[XG]) {
    const TI* X = c < kc ? X0 : X1;
    const uint32_t kb = (c < kc ? c : c - kc) * KC, k0 = kb + VPC * kr;
    const uint32_t row = tile * ST_ROWS + wave * 16u + ci;
    const TI* p = X + (uint64_t)row * N + k0;
    const bool rok = tile < ntiles && row < n;
#pragma unroll
    for (int t = 0; t < XG; ++t) {
      if (kb + 4 * VPC * t >= N) break;               // uniform: nothing is left of the contraction
      if constexpr (VEC) {
        x[t].c = (rok && k0 + 4 * VPC * t < N) ? *reinterpret_cast<const Chunk*>(p + 4 * VPC * t) : Chunk{0u, 0u, 0u, 0u};
      } else {
#pragma unroll
        for (int e = 0; e < VPC; ++e) x[t].v[e] = (rok && k0 + 4 * VPC * t + e < N) ? p[4 * VPC * t + e] : TI(0);
      }
    }
  };
  ChunkV mc[MT];
  auto load_m = [&](uint32_t c) {
    const TI* M = c < kc ? M0 : M1;
    const uint32_t k0 = (c < kc ? c : c - kc) * KC;
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      const uint32_t q = threadIdx.x + (uint32_t)ST_WG * u;
      const uint32_t k = k0 + q / MR, col = col0 + (q % MR) * VPC;
      const TI* p = M + (uint64_t)k * N + col;
      if constexpr (VEC) {
        mc[u].c = (k < N && col < N) ? *reinterpret_cast<const Chunk*>(p) : Chunk{0u, 0u, 0u, 0u};
      } else {
#pragma unroll
        for (int e = 0; e < VPC; ++e) mc[u].v[e] = (k < N && col + e < N) ? p[e] : TI(0);
      }
    }
  };
  auto store_m = [&](uint32_t buf) {
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      const uint32_t q = threadIdx.x + (uint32_t)ST_WG * u;
      *reinterpret_cast<Chunk*>(ml + buf * S::BUF + (q / MR) * LD + (q % MR) * VPC) = mc[u].c;
    }
  };
  double sq[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) sq[b] = 0.0;
  ChunkV xc[XG], xn[XG];
  load_x(blockIdx.x, 0, xn);
  load_m(0);
  store_m(0);
  if (resident && nch == 2) {
    load_m(1);
    store_m(1);
  }
  __syncthreads();
  uint32_t step = 0;                                  // streamed chunks so far
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    acc_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = zero_acc<acc_t>();
    for (uint32_t c = 0; c < nch; ++c, ++step) {
      const bool last = c + 1 == nch;
      const uint32_t nt = last ? tile + gridDim.x : tile, ncx = last ? 0 : c + 1;    // the next chunk
#pragma unroll
      for (int t = 0; t < XG; ++t) xc[t] = xn[t];
      load_x(nt, ncx, xn);
      const bool more = !resident && nt < ntiles;     // uniform
      if (more) load_m(ncx);
      const TI* mb = ml + (resident ? c : (step & 1u)) * S::BUF + VPC * kr * LD + ci;
      const uint32_t left = N - (c < kc ? c : c - kc) * KC;
#pragma unroll
      for (int t = 0; t < XG; ++t) {
        if (4u * VPC * t >= left) break;              // uniform
#pragma unroll
        for (int e = 0; e < VPC; ++e) {
          const TI av[1] = {xc[t].v[e]};
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const TI bv[1] = {mb[(4 * VPC * t + e) * LD + 16 * b]};
            acc[b] = mma<KIND, TI>(av, bv, acc[b]);
          }
        }
      }
      if (more) store_m((step + 1) & 1u);             // its last readers passed the previous barrier
      if (!resident) __syncthreads();
    }
    // every read of this wave's rows is done: Out may alias X0 (in-place Step 4)
    const uint32_t r0 = tile * ST_ROWS + wave * 16u;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t row = r0 + MK::drow(kr, r), col = col0 + 16u * b + ci;
        if (row < n && col < N) {
          const uint64_t o = (uint64_t)row * N + col;
          TI v = (TI)(ascale * (double)acc[b][r]);
          if (cbeta != 0.0) v += (TI)cbeta * Cm[o];
          Out[o] = v;
          sq[b] += (double)v * (double)v;
        }
      }
  }
  if (!want_colsq) return;
  // per-column sums over the work-group's rows: lanes l, l^16, l^32, l^48 share a
  // column, then the waves in order
  double* red = reinterpret_cast<double*>(strip_lds);
  __syncthreads();                                    // M is no longer read
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    sq[b] += __shfl_xor(sq[b], 16);
    sq[b] += __shfl_xor(sq[b], 32);
    if (kr == 0) red[wave * 128u + 16u * b + ci] = sq[b];
  }
  __syncthreads();
  if (threadIdx.x < 16u * NB && col0 + threadIdx.x < N) {
    double t = 0.0;
#pragma unroll
    for (uint32_t w = 0; w < ST_WG / 64; ++w) t += red[w * 128u + threadIdx.x];
    part[(uint64_t)blockIdx.x * N + col0 + threadIdx.x] = t;
  }
}

// The start of a step in one pass over the block (at most 128 columns): with U, HU,
// Lam and Lam^{-1},
//   R = HU - U Lam  (its column sums of squares only: the outer residual),
//   Y = U Lam^{-1}, r = -R Lam^{-1} and its column sums of squares.
// As three row products this reads and writes seven blocks; here two are read and
// two written, and R stays in registers.  A wave takes 16 rows and multiplies
// transposed, (M^T X^T), so that an accumulator (a lane has one row and columns
// 16 b + 4 kr + 0..3 of block b) is the next product's operand as it stands: the
// contraction takes the columns in that order.  Where the accumulator's rows are
// kr + 4 r (FP64) the columns of M are read in the order 4 (m % 4) + m / 4 instead.
// M in LDS in chunks of 32 columns, all of them resident up to 80 columns (waves
// then run free of each other); above, two buffers, one barrier per chunk.
// Bound by memory up to about 64 columns and by the matrix cores above (353 us of
// FP64 at 64^3, N = 128).  Against three row products and their two reductions:
// 64^3, N = 128 632 -> 516 us, mixed 327 -> 264, N = 17 101 -> 36; all products of
// a step at 48^3: N = 45 146 -> 91 us, 64 192 -> 125, 96 324 -> 280, 112 402 -> 357,
// 127 538 -> 475, 128 425 -> 406; mixed 64 187 -> 135, 128 358 -> 328.
template <typename TI, int NB>
struct StartTile {
  static constexpr int KR = 16 * NB;                  // rows of a chunk
  static constexpr int S = 36;                        // its row stride: rows 4 apart in distinct banks
  static constexpr int NCH = (NB + 1) / 2;            // chunks per matrix
  static constexpr int BUF = KR * S;
  static constexpr bool RESIDENT = NB <= 5;
  static constexpr int LDS = (RESIDENT ? 2 * NCH : 2) * BUF * (int)sizeof(TI);
  static constexpr int OCC = NB <= (sizeof(TI) == 8 ? 3 : 5) ? 2 : 1;         // work-groups per compute unit
};

// Sums over the 16 lanes of a row: lane ci gets that of v[ci % 8].
__device__ __forceinline__ double scatter_sum8(double (&v)[8], uint32_t ci) {
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] += dpp_move<0x140>(v[i]);                  // lane 15 - ci
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = ci & 4u ? v[i + 4] : v[i], send = ci & 4u ? v[i] : v[i + 4];
    v[i] = keep + dpp_move<0x141>(send);                                      // lane 7 - ci of eight
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = ci & 2u ? v[i + 2] : v[i], send = ci & 2u ? v[i] : v[i + 2];
    v[i] = keep + dpp_move<0x4E>(send);                                       // lane ci ^ 2
  }
  const double keep = ci & 1u ? v[1] : v[0], send = ci & 1u ? v[0] : v[1];
  return keep + dpp_move<0xB1>(send);                                         // lane ci ^ 1
}

template <typename TI, int KIND, int NB, bool VEC>
__global__ __launch_bounds__(ST_WG, (2 * StartTile<TI, NB>::OCC)) void k_start(
    const TI* __restrict__ U, const TI* __restrict__ HU, const TI* __restrict__ Lam, const TI* __restrict__ Linv,
    TI* __restrict__ Y, TI* __restrict__ R0, uint32_t n, uint32_t N, uint32_t ntiles, double* __restrict__ part) {
  using MK = Mk<KIND>;
  using acc_t = typename MK::acc_t;
  using T = StartTile<TI, NB>;
  constexpr int VPC = 16 / (int)sizeof(TI), NCH = T::NCH, S = T::S;
  constexpr int PR = 32 / VPC, PT = (T::KR * PR + ST_WG - 1) / ST_WG;
  typedef unsigned int Chunk __attribute__((ext_vector_type(4)));
  union Quad {                                        // four consecutive columns of a row
    Chunk c[4 / VPC];
    TI v[4];
  };
  union ChunkV {
    Chunk c;
    TI v[VPC];
  };
  extern __shared__ __align__(16) char strip_lds[];
  TI* const ml = reinterpret_cast<TI*>(strip_lds);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  const uint32_t mc = KIND == MK_F64 ? 4u * (ci & 3u) + (ci >> 2) : ci;       // the accumulator row's column of M
  ChunkV mv[PT];
  // Loads are unconditional: past the edge they take the last row or column, whose
  // values meet zeros of M in LDS or reach only output that is not stored.
  auto m_at = [&](uint32_t tid, int u, uint32_t s, int e, bool* in) -> uint32_t {    // value e of 16-byte group u
    const uint32_t q = tid + (uint32_t)ST_WG * u;
    const uint32_t k = q / PR, col = 32u * (s < NCH ? s : s - NCH) + (q % PR) * VPC + (uint32_t)e;
    *in = k < N && col < N;
    return min(k, N - 1u) * N + min(col, N - (VEC ? (uint32_t)VPC : 1u));
  };
  auto load_m = [&](uint32_t s) {                     // chunk s of Lam, then of Lam^{-1}
    const TI* M = s < NCH ? Lam : Linv;
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                     // every chunk's offsets kept over the tiles would spill
    bool in;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      if constexpr (VEC) {
        mv[u].c = *reinterpret_cast<const Chunk*>(M + m_at(tid, u, s, 0, &in));
      } else {
#pragma unroll
        for (int e = 0; e < VPC; ++e) mv[u].v[e] = M[m_at(tid, u, s, e, &in)];
      }
    }
  };
  auto store_m = [&](uint32_t s, uint32_t buf) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const uint32_t q = tid + (uint32_t)ST_WG * u;
      ChunkV v;
#pragma unroll
      for (int e = 0; e < VPC; ++e) {
        bool in;
        (void)m_at(tid, u, s, e, &in);
        v.v[e] = in ? mv[u].v[e] : TI(0);
      }
      if (PT * ST_WG == T::KR * PR || q < (uint32_t)(T::KR * PR))
        *reinterpret_cast<Chunk*>(ml + buf * T::BUF + q / PR * S + (q % PR) * VPC) = v.c;
    }
  };
  uint32_t row = 0;
  bool rok = false;
  // columns 16 b + 4 kr .. of the lane's row; p: that row's column 4 kr
  auto load_quad = [&](const TI* p, int b) {
    Quad v;
    const uint32_t left = N - 16u * b - (VEC ? (uint32_t)VPC : 1u);           // the block's last group or column
#pragma unroll
    for (int e = 0; e < 4; e += VEC ? VPC : 1) {
      const uint32_t at = b + 1 < NB ? 4u * kr + e : min(4u * kr + e, left);
      const TI* q = p + 16 * b + (b + 1 < NB ? (int64_t)e : (int64_t)at - 4 * kr);
      if constexpr (VEC) v.c[e / VPC] = *reinterpret_cast<const Chunk*>(q);
      else v.v[e] = *q;
    }
    return v;
  };
  auto store_quad = [&](TI* p, int b, const Quad& v) {
#pragma unroll
    for (int e = 0; e < 4; e += VEC ? VPC : 1)
      if (rok && (b + 1 < NB || 16u * b + 4u * kr + e < N)) {
        if constexpr (VEC) *reinterpret_cast<Chunk*>(p + 16 * b + e) = v.c[e / VPC];
        else p[16 * b + e] = v.v[e];
      }
  };
  // the operands of M for half a block of the contraction: two steps of two column blocks
  struct Ops {
    TI v[2][2];
  };
  auto ops = [&](const TI* m, int t, bool two) {
    Ops o;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = 16 * (t >> 1) + 2 * (t & 1) + r;
      o.v[r][0] = m[k * S];
      o.v[r][1] = two ? m[k * S + 16] : TI(0);
    }
    return o;
  };
  load_m(0);
  store_m(0, 0);
  if constexpr (T::RESIDENT) {
    for (uint32_t s = 1; s < 2u * NCH; ++s) {
      load_m(s);
      store_m(s, s);
    }
  }
  __syncthreads();
  uint32_t step = 0;                                  // chunks so far (streamed)
  auto begin = [&](uint32_t s) -> const TI* {         // chunk s of this tile; the next one's loads start
    __builtin_amdgcn_sched_barrier(0);                // a chunk's operands in registers at a time
    if constexpr (T::RESIDENT) return ml + s * T::BUF;
    load_m(s + 1 < 2u * NCH ? s + 1 : 0u);
    __builtin_amdgcn_sched_barrier(0);
    return ml + (step & 1u) * T::BUF;
  };
  auto end = [&](uint32_t s) {
    if constexpr (!T::RESIDENT) {
      __builtin_amdgcn_sched_barrier(0);
      store_m(s + 1 < 2u * NCH ? s + 1 : 0u, ~step & 1u);    // its last readers passed the previous barrier
      ++step;
      __syncthreads();
    }
  };
  double sqr[NCH], sq0[NCH];
#pragma unroll
  for (int j = 0; j < NCH; ++j) sqr[j] = sq0[j] = 0.0;
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    row = tile * ST_ROWS + wave * 16u + ci;
    rok = row < n;
    const uint64_t at = (uint64_t)min(row, n - 1u) * N + 4u * kr;
    Quad u[NB], res[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) u[b] = load_quad(U + at, b);
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const bool two = 2 * j + 1 < NB;                // static
      const TI* m = begin(j) + 4u * kr * S + mc;
      Quad h[2];
      h[0] = load_quad(HU + at, 2 * j);
      if (two) h[1] = load_quad(HU + at, 2 * j + 1);
      acc_t acc[2] = {zero_acc<acc_t>(), zero_acc<acc_t>()};
      Ops o[2];
      o[0] = ops(m, 0, two);
#pragma unroll
      for (int t = 0; t < 2 * NB; ++t) {
        if (t + 1 < 2 * NB) o[(t + 1) & 1] = ops(m, t + 1, two);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const TI a0[1] = {o[t & 1].v[r][0]}, a1[1] = {o[t & 1].v[r][1]}, xv[1] = {u[t >> 1].v[2 * (t & 1) + r]};
          acc[0] = mma<KIND, TI>(a0, xv, acc[0]);
          if (two) acc[1] = mma<KIND, TI>(a1, xv, acc[1]);
        }
      }
      double v[8];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[4 * q + r] = 0.0;
          if (2 * j + q < NB) {
            const TI x = h[q].v[r] - (TI)acc[q][r];
            res[2 * j + q].v[r] = x;
            v[4 * q + r] = rok ? (double)x * (double)x : 0.0;
          }
        }
      sqr[j] += scatter_sum8(v, ci);
      end(j);
    }
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const bool two = 2 * j + 1 < NB;
      const TI* m = begin(NCH + j) + 4u * kr * S + mc;
      acc_t ay[2] = {zero_acc<acc_t>(), zero_acc<acc_t>()}, ar[2] = {zero_acc<acc_t>(), zero_acc<acc_t>()};
      Ops o[2];
      o[0] = ops(m, 0, two);
#pragma unroll
      for (int t = 0; t < 2 * NB; ++t) {
        if (t + 1 < 2 * NB) o[(t + 1) & 1] = ops(m, t + 1, two);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const TI a0[1] = {o[t & 1].v[r][0]}, a1[1] = {o[t & 1].v[r][1]};
          const TI xv[1] = {u[t >> 1].v[2 * (t & 1) + r]}, rv[1] = {res[t >> 1].v[2 * (t & 1) + r]};
          ay[0] = mma<KIND, TI>(a0, xv, ay[0]);
          ar[0] = mma<KIND, TI>(a0, rv, ar[0]);
          if (two) {
            ay[1] = mma<KIND, TI>(a1, xv, ay[1]);
            ar[1] = mma<KIND, TI>(a1, rv, ar[1]);
          }
        }
      }
      double v[8];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        Quad yv, rv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          yv.v[r] = (TI)ay[q][r];
          rv.v[r] = (TI)-ar[q][r];
          v[4 * q + r] = rok && 2 * j + q < NB ? (double)rv.v[r] * (double)rv.v[r] : 0.0;
        }
        if (2 * j + q < NB) {
          store_quad(Y + at, 2 * j + q, yv);
          store_quad(R0 + at, 2 * j + q, rv);
        }
      }
      sq0[j] += scatter_sum8(v, ci);
      end(NCH + j);
    }
  }
  // a lane's sums belong to column 32 j + 16 (ci % 8 / 4) + 4 kr + ci % 4; then the waves in order
  double* red = reinterpret_cast<double*>(strip_lds);
  __syncthreads();                                    // M is no longer read
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const uint32_t col = 32u * j + 16u * (ci >> 2 & 1u) + 4u * kr + (ci & 3u);
    if (ci < 8u) {
      red[wave * 256u + col] = sq0[j];
      red[wave * 256u + 128u + col] = sqr[j];
    }
  }
  __syncthreads();
  for (uint32_t c = threadIdx.x; c < 2u * N; c += ST_WG) {
    const uint32_t at = c < N ? c : 128u + c - N;
    double t = 0.0;
#pragma unroll
    for (uint32_t w = 0; w < ST_WG / 64; ++w) t += red[w * 256u + at];
    part[(uint64_t)blockIdx.x * 2u * N + c] = t;
  }
}

// Square FP64 products of N x N matrices (the small solves for large N):
// D = alpha op(A) op(B) + beta C + gamma I, op = transpose when ta / tb is
// set.  Work-group tile 64 x 64 (4 waves of 32 x 32), operands straight from
// global memory (the matrices are L2-resident).  When res is given, the
// work-group adds sum over its tile of (delta_ij - D_ij)^2 into res[block]
// (the Newton-Schulz residual |I - M X|_F^2).  A non-zero *skip makes the
// launch a no-op (device-side convergence of an iteration).
__global__ __launch_bounds__(256) void k_sqmm(const double* __restrict__ A, int ta, const double* __restrict__ B,
                                              int tb, const double* __restrict__ C, double alpha, double beta,
                                              double gamma, double* __restrict__ D, uint32_t N,
                                              const int32_t* __restrict__ skip, double* __restrict__ res) {
  using MK = Mk<MK_F64>;
  __shared__ double red[256];
  if (skip && *skip) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t i_base = blockIdx.y * 64 + (wave >> 1) * 32;
  const uint32_t j_base = blockIdx.x * 64 + (wave & 1u) * 32;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  v4d acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = zero_acc<v4d>();
  for (uint32_t k0 = 0; k0 < N; k0 += 4) {
    const uint32_t k = k0 + kr;
    double av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const uint32_t i = i_base + a * 16 + ci;
      av[a] = (k < N && i < N) ? (ta ? A[(uint64_t)k * N + i] : A[(uint64_t)i * N + k]) : 0.0;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t j = j_base + b * 16 + ci;
      bv[b] = (k < N && j < N) ? (tb ? B[(uint64_t)j * N + k] : B[(uint64_t)k * N + j]) : 0.0;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
  }
  double rs = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t i = i_base + a * 16 + MK::drow(kr, r);
        const uint32_t j = j_base + b * 16 + ci;
        if (i < N && j < N) {
          const uint64_t o = (uint64_t)i * N + j;
          double v = alpha * acc[a][b][r];
          if (beta != 0.0) v += beta * C[o];
          if (i == j) v += gamma;
          D[o] = v;
          const double e = (i == j ? 1.0 : 0.0) - v;
          rs += e * e;
        }
      }
  if (!res) return;
  red[threadIdx.x] = rs;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) res[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// Wide FP32 and BF16 Grams from LDS (both sides >= 128 columns, 16-byte aligned
// rows): work-group tile 128 x 128, each wave a 64 x 64 sub-tile (4 x 4 MFMA
// blocks).  The work-group stages KC-row panels of both operands in LDS (double
// buffered; the next panel's 16-byte loads are in flight while the current one
// is consumed), so each operand element crosses L2 once per work-group
// instead of once per wave: at these instructions' rate smaller tiles need more
// L1-to-L2 traffic than the chip sustains.

// Panel staging: the 16-byte chunks of KC rows
// starting at row p of columns c0 .. c0 + 127 of X (zero outside the rows
// [.., r1) and the columns [.., nc)).
template <typename TI, int KC>
struct PanelChunks {
  static constexpr int VPC = 16 / (int)sizeof(TI);      // values per 16-byte chunk
  static constexpr int CPR = GT2 / VPC;                  // chunks per panel row
  static constexpr int CPT = KC * CPR / 256;             // chunks per thread
  static_assert(CPT * 256 == KC * CPR, "panel chunks must divide the work-group");
  typedef unsigned int Chunk __attribute__((ext_vector_type(4)));
  Chunk ch[CPT];
  __device__ void load(const TI* __restrict__ X, uint64_t ld, uint32_t nc, uint32_t c0, uint32_t p, uint32_t r1) {
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const uint32_t c = threadIdx.x + 256u * u;
      const uint32_t row = c / CPR, col = (c % CPR) * VPC;
      const uint32_t gr = p + row;
      const Chunk z = {0u, 0u, 0u, 0u};
      ch[u] = (gr < r1 && c0 + col < nc) ? *reinterpret_cast<const Chunk*>(X + (uint64_t)gr * ld + c0 + col) : z;
    }
  }
  __device__ void store(TI (*panel)[GT2]) const {
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const uint32_t c = threadIdx.x + 256u * u;
      const uint32_t row = c / CPR, col = (c % CPR) * VPC;
      *reinterpret_cast<Chunk*>(&panel[row][col]) = ch[u];
    }
  }
};

template <typename TI, int KIND>
__global__ __launch_bounds__(256) void k_gram_lds(const TI* __restrict__ A, uint64_t lda, uint32_t na,
                                                  const TI* __restrict__ B, uint64_t ldb, uint32_t nb,
                                                  uint32_t rows, uint32_t rows_per_split, uint32_t ntj, int upper,
                                                  double* __restrict__ part) {
  using M = Mk<KIND>;
  using acc_t = typename M::acc_t;
  constexpr int KC = PanelRows<KIND>::KC;
  __shared__ __align__(16) TI pa[2][KC][GT2];
  __shared__ __align__(16) TI pb[2][KC][GT2];
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t wi = (wave >> 1) * GW2, wj = (wave & 1u) * GW2;     // the wave's sub-tile in the tile
  uint32_t ks, ti, tj;
  gram_place(ntj, upper, &ks, &ti, &tj);
  const uint32_t i0 = ti * GT2, j0 = tj * GT2;
  const uint32_t kr = lane >> 4, ci = lane & 15u;
  const uint32_t r0 = (uint32_t)min((uint64_t)rows, (uint64_t)ks * rows_per_split);
  const uint32_t r1 = r0 + min(rows - r0, rows_per_split);
  acc_t acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = zero_acc<acc_t>();
  PanelChunks<TI, KC> ca, cb;
  const uint32_t npan = (r1 > r0) ? (r1 - r0 + KC - 1) / KC : 0;
  if (npan > 0) {
    ca.load(A, lda, na, i0, r0, r1);
    cb.load(B, ldb, nb, j0, r0, r1);
    ca.store(pa[0]);
    cb.store(pb[0]);
  }
  __syncthreads();
  for (uint32_t t = 0; t < npan; ++t) {
    const int buf = (int)(t & 1u);
    if (t + 1 < npan) {
      ca.load(A, lda, na, i0, r0 + (t + 1) * KC, r1);
      cb.load(B, ldb, nb, j0, r0 + (t + 1) * KC, r1);
    }
#pragma unroll
    for (int kk = 0; kk < KC / M::KSTEP; ++kk) {
      TI av[4][M::KPL], bv[4][M::KPL];
#pragma unroll
      for (int e = 0; e < M::KPL; ++e) {
        const uint32_t row = kk * M::KSTEP + kr * M::KPL + e;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          av[a][e] = pa[buf][row][wi + a * 16 + ci];
          bv[a][e] = pb[buf][row][wj + a * 16 + ci];
        }
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mma<KIND, TI>(av[a], bv[b], acc[a][b]);
    }
    if (t + 1 < npan) {
      ca.store(pa[buf ^ 1]);
      cb.store(pb[buf ^ 1]);
    }
    __syncthreads();
  }
  double* out = part + (uint64_t)ks * na * nb;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t i = i0 + wi + a * 16 + M::drow(kr, r);
        const uint32_t j = j0 + wj + b * 16 + ci;
        if (i < na && j < nb) out[(uint64_t)i * nb + j] = (double)acc[a][b][r];
      }
}

// Splits of the rows over a Gram's work-groups (nt tiles, occ of them per compute
// unit at a time).  One tile: one work-group per place.  Several: a multiple of 8
// (see gram_place), the k per XCD for which whole rounds of its 32 occ places
// lose least; cost is the time relative to a tile's work of one round.  Returns
// the splits, at most max_ks.
int64_t gram_splits(int64_t nt, int64_t occ, int64_t max_ks, double* cost) {
  int64_t best = std::min<int64_t>(max_ks, std::max<int64_t>(1, 256 * occ / nt));
  *cost = (double)((nt * best + 256 * occ - 1) / (256 * occ) * occ) / (double)best;
  if (nt == 1) return best;
  double at = 0;
  for (int64_t k = 1; k <= 64 && 8 * k <= max_ks; ++k) {
    const double v = (double)((nt * k + 32 * occ - 1) / (32 * occ) * occ) / (double)(8 * k);
    if (k == 1 || v < 0.98 * at) best = 8 * k, *cost = at = v;
  }
  return best;
}

template <typename TI, int KIND>
hipError_t gram_t(ope_ctx* c, const TI* A, int64_t lda, int na, const TI* B, int64_t ldb, int nb, int64_t rows,
                  double* out, bool symmetric = false) {
  constexpr int64_t VPC = 16 / (int64_t)sizeof(TI);
  // A^T A (or a product known to be symmetric): the blocks on and above the diagonal
  const bool same = A == B && lda == ldb && na == nb;
  const bool upper = na == nb && (same || symmetric);
  const int64_t max_ks = c->part_cap / ((int64_t)na * nb);
  if (max_ks < 1) return hipErrorInvalidValue;
  auto tiles = [&](int edge, uint32_t* tj) {
    const uint32_t ti = (uint32_t)((na + edge - 1) / edge);
    *tj = (uint32_t)((nb + edge - 1) / edge);
    return upper ? *tj * (*tj + 1) / 2 : ti * *tj;
  };
  uint32_t tj = 1;
  // Tiles of 128 staged in LDS, or smaller ones from registers.  From registers
  // each tile loads its own columns through L2 (about 7 TB/s of it at 64 x 64
  // tiles), which FP64 instructions leave time for and faster ones do not.
  // Products at 48^3, LDS / registers, us:
  //   FP64 two blocks N = 128 93/75, 256 309/290, 512 1021/981; A^T A 256 258/176,
  //   512 919/652 (ten tiles fill the chip badly): registers at every width.
  //   FP32 two blocks 128 57/78, 192 140/84, 256 148/176, 320 297/289, 512 508/706,
  //   so by the tiles each needs (a 128 tile costs 1.6 times a 96 one); A^T A 192
  //   112/75, 256 138/129, 384 293/193, 512 502/380: registers.
  //   BF16 two blocks 128 39/59, 256 76/86; A^T A 128 46/23 (one tile), 256 62/63.
  const bool aligned = (reinterpret_cast<uintptr_t>(A) % 16) == 0 && (reinterpret_cast<uintptr_t>(B) % 16) == 0 &&
                       lda % VPC == 0 && ldb % VPC == 0 && na % VPC == 0 && nb % VPC == 0;
  const bool lds = KIND != MK_F64 && aligned && na >= GT2 && nb >= GT2 &&
                   (KIND == MK_F32 ? !upper && 8 * tiles(GT2, &tj) < 5 * tiles(96, &tj) : !(upper && na == GT2));
  int64_t ks = 1, rps = 0;
  auto split = [&](int64_t want, int64_t group) {     // into whole groups of rows
    rps = ((rows + want - 1) / want + group - 1) / group * group;
    const int64_t used = (rows + rps - 1) / rps;      // later splits would hold no rows
    rps = std::min<int64_t>(rps, 0xffffffff);
    ks = want % 8 == 0 ? std::min(want, (used + 7) / 8 * 8) : used;
  };
  {
    ProfScope ps(c, OPE_KERNEL_GRAM);
    double cost = 0;
    auto go = [&](auto nbt, auto modet, auto off) {
      constexpr int NB = decltype(nbt)::value, MODE = decltype(modet)::value;
      using T = GramTile<TI, KIND, NB, MODE>;
      const uint32_t nt = tiles(16 * NB, &tj);
      split(gram_splits(nt, T::OCC, max_ks, &cost), 4 * T::U * Mk<KIND>::KSTEP);
      hipLaunchKernelGGL((k_gram_rows<TI, KIND, NB, MODE, decltype(off)>), dim3((uint32_t)ks, nt), dim3(256), 0,
                         c->stream, A, (uint64_t)lda, (uint32_t)na, B, (uint64_t)ldb, (uint32_t)nb, (uint32_t)rows,
                         (uint32_t)rps, tj, upper, c->part);
    };
    auto at = [&](auto nbt, auto modet) { go(nbt, modet, uint32_t{}); };
    auto one_tile = [&](auto modet) {
      switch ((na + 15) / 16) {
        case 1: at(std::integral_constant<int, 1>{}, modet); break;
        case 2: at(std::integral_constant<int, 2>{}, modet); break;
        case 3: at(std::integral_constant<int, 3>{}, modet); break;
        case 4: at(std::integral_constant<int, 4>{}, modet); break;
        case 5: at(std::integral_constant<int, 5>{}, modet); break;
        case 6: at(std::integral_constant<int, 6>{}, modet); break;
        case 7: at(std::integral_constant<int, 7>{}, modet); break;
        default: at(std::integral_constant<int, 8>{}, modet); break;
      }
    };
    constexpr std::integral_constant<int, G_SAME> SAME{};
    constexpr std::integral_constant<int, G_UPPER> UPPER{};
    constexpr std::integral_constant<int, G_FULL> FULL{};
    if (lds) {
      if constexpr (KIND != MK_F64) {
        const uint32_t nt = tiles(GT2, &tj);
        split(gram_splits(nt, 2, max_ks, &cost), Mk<KIND>::KSTEP);
        hipLaunchKernelGGL((k_gram_lds<TI, KIND>), dim3((uint32_t)ks, nt), dim3(256), 0, c->stream, A, (uint64_t)lda,
                           (uint32_t)na, B, (uint64_t)ldb, (uint32_t)nb, (uint32_t)rows, (uint32_t)rps, tj, upper,
                           c->part);
      }
    } else if (std::max(lda, ldb) > (int64_t)1 << 22) {                       // 32-bit offsets do not reach 32 rows
      go(std::integral_constant<int, 4>{}, FULL, uint64_t{});
    } else if (same && na <= GT2) {
      one_tile(SAME);
    } else if (std::is_same<TI, double>::value && upper && na <= GT2) {
      if constexpr (std::is_same<TI, double>::value) one_tile(UPPER);
    } else {
      // the tile edge (in blocks) of the least work: t^2 instructions and 2 t
      // loads per step and wave, a load at about one FP64 or FP32 instruction, or
      // four BF16 ones (whose step is 32 rows).  Edge 6 for FP32 only: the FP64
      // accumulators of 36 blocks leave one wave per SIMD, too few loads in flight
      // (A^T A at 512 912 us against 597), and BF16 values are 8 per lane and load.
      int best = 0;
      double least = 0;
      for (int t : {KIND == MK_F32 ? 6 : 4, 4, 3, 2, 1}) {
        gram_splits(tiles(16 * t, &tj), t == 6 ? GramTile<TI, KIND, 6, G_FULL>::OCC : 2, max_ks, &cost);
        cost *= t * t + (KIND == MK_BF16 ? 8 : 2) * t;
        if (best == 0 || cost < least) best = t, least = cost;
      }
      switch (best) {
        case 1: at(std::integral_constant<int, 1>{}, FULL); break;
        case 2: at(std::integral_constant<int, 2>{}, FULL); break;
        case 3: at(std::integral_constant<int, 3>{}, FULL); break;
        case 4: at(std::integral_constant<int, 4>{}, FULL); break;
        default:
          if constexpr (KIND == MK_F32) at(std::integral_constant<int, 6>{}, FULL);
      }
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const uint32_t bi = (uint32_t)((na + 15) / 16), bj = (uint32_t)((nb + 15) / 16);
  if (upper)
    hipLaunchKernelGGL((k_gram_sum<true>), dim3(bi * (bi + 1) / 2 * 4), dim3(1024), 0, c->stream, c->part, (uint32_t)ks,
                       (uint32_t)na, (uint32_t)nb, out);
  else
    hipLaunchKernelGGL((k_gram_sum<false>), dim3(bi * bj * 4), dim3(1024), 0, c->stream, c->part, (uint32_t)ks,
                       (uint32_t)na, (uint32_t)nb, out);
  return hipGetLastError();
}

template <typename TI, int KIND>
hipError_t rowmm_t(ope_ctx* c, const TI* X0, const TI* M0, const TI* X1, const TI* M1, const TI* Cm, double cbeta,
                   double ascale, TI* Out, int want_colsq, int predicated, int64_t* nparts) {
  const uint32_t n = (uint32_t)c->n, N = (uint32_t)c->N;
  // LDS-staged panels when every operand row splits into whole, aligned 16-byte chunks
  constexpr uint32_t VPC = 16 / (uint32_t)sizeof(TI);
  auto al16 = [](const void* q) { return q == nullptr || (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  const bool aligned = N % VPC == 0 && al16(X0) && al16(M0) && al16(X1) && al16(M1);
  if constexpr (KIND != MK_BF16) {
    // Which widths the strip takes, from the products of one step at 48^3 (us,
    // strip / the kernel it would have had):
    //   FP64 N = 8: 60/90, 17: 81/113, 33: 126/209, 45: 146/262, 64: 192/284,
    //   96: 324/391, 112: 401/450, 127: 538/722, 128: 520/520, 192: 1274/1215,
    //   256: 1688/1561; so all but aligned rows of more than 112.
    //   FP32 N = 16: 75/84, 17: 111/88, 32: 105/100, 33: 151/165, 48: 142/183,
    //   64: 187/227, 80: 240/258, 96: 303/298, 127: 519/503, 128: 447/362; an FP32
    //   instruction takes half the time of an FP64 one, and the LDS reads of 16
    //   rows per wave (one value per instruction) bound the strip from there on.
    const bool strip = KIND == MK_F64 ? N <= 112 || !aligned : N <= 16 || (N > 32 && N <= 80);
    if (strip) {
      using S = Strip<TI>;
      const uint32_t gc = (N + 127) / 128, ntiles = (n + ST_ROWS - 1) / ST_ROWS;
      if (gc != 1 && (Out == X0 || Out == X1)) return hipErrorInvalidValue;   // in place needs one column tile
      const uint32_t nch = (X1 ? 2 : 1) * ((N + S::KC - 1) / S::KC);
      // one work-group per compute unit (two where one buffer of M suffices)
      uint32_t gx = std::max(1u, (nch == 1 ? 512u : 256u) / gc);
      if (gx > ntiles) gx = ntiles;
      if (want_colsq && (int64_t)gx * N > c->part_cap) return hipErrorInvalidValue;
      const size_t lds =
          std::max<size_t>((size_t)std::min(nch, 2u) * S::BUF * sizeof(TI), ST_WG / 64 * 128 * sizeof(double));
      ProfScope ps(c, OPE_KERNEL_ROWMM);
      auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(gx, gc), dim3(ST_WG), lds, c->stream, X0, M0, X1, M1, Cm, cbeta, ascale, Out, n,
                           N, ntiles, want_colsq, predicated, c->sc, c->part);
      };
      auto width = [&](auto v) {
        constexpr bool VEC = decltype(v)::value;
        switch (gc > 1 ? 8u : (N + 15) / 16) {
          case 1: go(k_rowmm_strip<TI, KIND, 1, VEC>); break;
          case 2: go(k_rowmm_strip<TI, KIND, 2, VEC>); break;
          case 3: go(k_rowmm_strip<TI, KIND, 3, VEC>); break;
          case 4: go(k_rowmm_strip<TI, KIND, 4, VEC>); break;
          case 5: go(k_rowmm_strip<TI, KIND, 5, VEC>); break;
          default:
            if constexpr (KIND == MK_F64) {                   // FP32 ends at 80 columns
              if (N <= 96) go(k_rowmm_strip<TI, KIND, 6, VEC>);
              else if (N <= 112) go(k_rowmm_strip<TI, KIND, 7, VEC>);
              else if constexpr (!VEC) go(k_rowmm_strip<TI, KIND, 8, VEC>);
            }
        }
      };
      if (aligned) width(std::true_type{});
      else width(std::false_type{});
      if (nparts) *nparts = gx;
      return hipGetLastError();
    }
  }
  const bool narrow = N <= 32;
  const bool lds = !narrow && aligned;
  // FP64: 64-row tiles (132 VGPRs, three work-groups per compute unit, whose
  // output stores overlap the others' matrix-core work) measured 4% faster than
  // 128-row tiles (219 VGPRs, two) at 64^3, N = 128
  const uint32_t rt = KIND == MK_F64 ? RT2H : narrow ? RTN : (lds ? RT2 : RT);
  const uint32_t gr = (n + rt - 1) / rt, gc = (N + CT - 1) / CT;
  if (gc != 1 && (Out == X0 || Out == X1)) return hipErrorInvalidValue;  // in place needs one column tile
  if (want_colsq && (int64_t)gr * N > c->part_cap) return hipErrorInvalidValue;
  ProfScope ps(c, OPE_KERNEL_ROWMM);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(gr, gc), dim3(256), 0, c->stream, X0, M0, X1, M1, Cm, cbeta, ascale, Out, n, N,
                       want_colsq, predicated, c->sc, c->part);
  };
  if constexpr (KIND == MK_F64) {                             // aligned and wider than 112
    if (X1) go(k_rowmm_lds<TI, KIND, 2, RT2H>);
    else go(k_rowmm_lds<TI, KIND, 1, RT2H>);
  } else if (narrow) {
    if (X1) go(k_rowmm_narrow<TI, KIND, 2>);
    else go(k_rowmm_narrow<TI, KIND, 1>);
  } else if (lds) {
    if (X1) go(k_rowmm_lds<TI, KIND, 2, RT2>);
    else go(k_rowmm_lds<TI, KIND, 1, RT2>);
  } else {
    if (X1) go(k_rowmm<TI, KIND, 2>);
    else go(k_rowmm<TI, KIND, 1>);
  }
  if (nparts) *nparts = gr;
  return hipGetLastError();
}

template <typename TI, int KIND>
hipError_t start_t(ope_ctx* c, const TI* U, const TI* HU, const TI* Lam, const TI* Linv, TI* Y, TI* R0,
                   int64_t* nparts) {
  const uint32_t n = (uint32_t)c->n, N = (uint32_t)c->N;
  constexpr uint32_t VPC = 16 / (uint32_t)sizeof(TI);
  auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  const bool aligned = N % VPC == 0 && al16(U) && al16(HU) && al16(Lam) && al16(Linv) && al16(Y) && al16(R0);
  const uint32_t ntiles = (n + ST_ROWS - 1) / ST_ROWS;
  uint32_t gx = 0;
  ProfScope ps(c, OPE_KERNEL_ROWMM);
  auto go = [&](auto nbt, auto vect) {
    constexpr int NB = decltype(nbt)::value;
    constexpr bool VEC = decltype(vect)::value;
    using T = StartTile<TI, NB>;
    gx = (uint32_t)std::min<int64_t>(std::min<int64_t>(ntiles, 256 * T::OCC), c->part_cap / (2 * (int64_t)N));
    if (gx < 1) return;
    hipLaunchKernelGGL((k_start<TI, KIND, NB, VEC>), dim3(gx), dim3(ST_WG),
                       std::max<size_t>(T::LDS, ST_WG / 64 * 256 * sizeof(double)), c->stream, U, HU, Lam, Linv, Y, R0,
                       n, N, ntiles, c->part);
  };
  auto width = [&](auto vect) {
    switch ((N + 15) / 16) {
      case 1: go(std::integral_constant<int, 1>{}, vect); break;
      case 2: go(std::integral_constant<int, 2>{}, vect); break;
      case 3: go(std::integral_constant<int, 3>{}, vect); break;
      case 4: go(std::integral_constant<int, 4>{}, vect); break;
      case 5: go(std::integral_constant<int, 5>{}, vect); break;
      case 6: go(std::integral_constant<int, 6>{}, vect); break;
      case 7: go(std::integral_constant<int, 7>{}, vect); break;
      default: go(std::integral_constant<int, 8>{}, vect); break;
    }
  };
  if (aligned) width(std::true_type{});
  else width(std::false_type{});
  if (gx < 1) return hipErrorInvalidValue;
  *nparts = gx;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gram(ope_ctx* c, const double* A, int64_t lda, int na, const double* B, int64_t ldb, int nb,
                       int64_t rows, double* out) {
  return gram_t<double, MK_F64>(c, A, lda, na, B, ldb, nb, rows, out);
}

hipError_t launch_gram_sym(ope_ctx* c, const double* A, int64_t lda, const double* B, int64_t ldb, int n,
                           int64_t rows, double* out) {
  return gram_t<double, MK_F64>(c, A, lda, n, B, ldb, n, rows, out, true);
}

hipError_t launch_gram_f32(ope_ctx* c, int kind, const float* A, int64_t lda, int na, const float* B, int64_t ldb,
                           int nb, int64_t rows, double* out) {
  switch (kind) {
    case MK_F64: return gram_t<float, MK_F64>(c, A, lda, na, B, ldb, nb, rows, out);
    case MK_F32: return gram_t<float, MK_F32>(c, A, lda, na, B, ldb, nb, rows, out);
    default: return gram_t<float, MK_BF16>(c, A, lda, na, B, ldb, nb, rows, out);
  }
}

hipError_t launch_rowmm(ope_ctx* c, const double* X0, const double* M0, const double* X1, const double* M1,
                        const double* Cm, double cbeta, double ascale, double* Out, int want_colsq, int predicated,
                        int64_t* nparts) {
  return rowmm_t<double, MK_F64>(c, X0, M0, X1, M1, Cm, cbeta, ascale, Out, want_colsq, predicated, nparts);
}

hipError_t launch_sqmm(ope_ctx* c, const double* A, int ta, const double* B, int tb, const double* C, double alpha,
                       double beta, double gamma, double* D, uint32_t N, const int32_t* skip, double* res) {
  const uint32_t t = (N + 63) / 64;
  ProfScope ps(c, OPE_KERNEL_SMALL);
  hipLaunchKernelGGL(k_sqmm, dim3(t, t), dim3(256), 0, c->stream, A, ta, B, tb, C, alpha, beta, gamma, D, N, skip,
                     res);
  return hipGetLastError();
}

hipError_t launch_rowmm_f32(ope_ctx* c, int kind, const float* X0, const float* M0, const float* X1, const float* M1,
                            const float* Cm, double cbeta, double ascale, float* Out, int want_colsq, int predicated,
                            int64_t* nparts) {
  if (kind == MK_BF16)
    return rowmm_t<float, MK_BF16>(c, X0, M0, X1, M1, Cm, cbeta, ascale, Out, want_colsq, predicated, nparts);
  return rowmm_t<float, MK_F32>(c, X0, M0, X1, M1, Cm, cbeta, ascale, Out, want_colsq, predicated, nparts);
}

hipError_t launch_start(ope_ctx* c, const void* U, void* Y, void* R0, int64_t* nparts) {
  if (c->prec == OPE_FP64)
    return start_t<double, MK_F64>(c, (const double*)U, (const double*)c->HU, c->Lam, c->Linv, (double*)Y, (double*)R0,
                                   nparts);
  return start_t<float, MK_F32>(c, (const float*)U, (const float*)c->HU, c->Lam32, c->Linv32, (float*)Y, (float*)R0,
                                nparts);
}
