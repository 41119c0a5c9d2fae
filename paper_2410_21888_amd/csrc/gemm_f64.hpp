// FP64 MFMA GEMM for gfx950 (CDNA4): C[m, n] = sum_k A(m, k) B(k, n).
//
// Every dense contraction of the RI-MP2 fragment kernel is one of these:
//   (ia|jb) slab   V[(k,a), (j,b)] = sum_P B[(k,a), P] B[(j,b), P]    (B K-contiguous)
//   Gamma          G[(k,a), P]     = sum_(j,b) T[(k,a), (j,b)] B[(j,b), P] (B N-contiguous)
//   P_ab           sum_(k,j,c) T(a, (k,j,c)) X(b, (k,j,c))                (B K-contiguous)
//   P_ij           sum_(k,a,b) T(i, (k,a,b)) X(j, (k,a,b))                (B K-contiguous)
//   Gamma, transposed blocks (symmetric pair path)
//                  G[(j,b), P]    += sum_(k,a) T[(k,a), (j,b)] B[(k,a), P]
//                                 (A M-contiguous, B N-contiguous)
// and the adjacent gradient steps: the AO back-transform of Gamma (A
// M-contiguous: transposed MO coefficients) and the L' / L'' terms.
// The slab operands store the reduction index in two levels (runs of kdiv
// contiguous elements, runs ks1 apart), which the loaders follow directly so
// no operand is ever copied or transposed in HBM.
//
// Tiling: 256 threads = 4 waves in a 2 x 2 grid; each wave owns a
// (BM/2) x (BN/2) block of 16 x 16 accumulators fed by
// v_mfma_f64_16x16x4f64.  Lane layout of that instruction on gfx950
// (measured): lane l supplies A[l%16][l/16] and B[l/16][l%16]; accumulator
// register r of lane l holds D[4r + l/16][l%16].  Operand tiles are staged
// k-major in LDS (double-buffered, one barrier per BK chunk).  Global loads
// are 16 bytes (two consecutive reduction indices, or two consecutive columns
// of an N-contiguous operand).  Two loaders: the general one (FAST = 0, 16-byte
// loads where VEC says that they are aligned) issues the next chunk's loads
// before the current chunk's MFMAs and stores them to LDS halfway through
// them, with masks on edge tiles; the fast one (FAST = 1, 2, 3; chosen by the
// host) keeps loads two chunks ahead without any branch around them (see
// gemm_tile).
//
// Triangular launches (TRI): for a symmetric result only tiles with
// tile_m <= tile_n are computed; every element m < n is written at (m, n) and
// (n, m), and elements m > n of diagonal tiles are not written, so the lower
// triangle is always the mirror of the upper one whatever the tile size.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"

namespace rimp2 {

typedef double dbl4 __attribute__((ext_vector_type(4)));

// Element (r, k) at base[r * rs + (k / kdiv) * ks1 + (k % kdiv)].
struct KOperand {
  const double* base;
  int64_t rs;
  int64_t kdiv;
  int64_t ks1;
};

// Element (k, n) at base[k * ld + n].
struct NOperand {
  const double* base;
  int64_t ld;
};

struct GemmParams {
  int64_t M, N, K;
  int64_t kchunk;       // reduction length per split (multiple of BK)
  int32_t tiles_m, tiles_n, splits, group_m;
  KOperand A;           // A when K-contiguous
  NOperand Am;          // A when M-contiguous: element (m, k) at Am.base[k * Am.ld + m]
  KOperand Bk;          // B when K-contiguous
  NOperand Bn;          // B when N-contiguous
  double* C;            // split z writes C + z * split_stride
  int64_t ldc;
  int64_t split_stride;
  int32_t accumulate;   // nonzero: C += A B instead of C = A B (no split-K)
  // batch > 1: that many products of the same sizes in one launch (splits is
  // 1); product z uses A + z batch_a, B + z batch_b and C + z split_stride
  int32_t batch;
  int64_t batch_a, batch_b;
  const int32_t* status;  // nonzero: do nothing
  // Optional pair screening of an (ia|jb) slab: row m belongs to occupied
  // orbital skip_k0 + m / skip_nvir, column n to skip_j0 + n / skip_nvir; a
  // tile whose pairs are all screened out is not computed.  A pair {k, j} is
  // screened out when skip[k * skip_nocc + j] or skip[j * skip_nocc + k] is
  // nonzero (the mask names unordered pairs).
  const uint8_t* skip;
  int32_t skip_nvir, skip_k0, skip_j0, skip_nocc;
  // pair_upper (same row/column to pair mapping): a tile all of whose pairs
  // have pair_lo <= j < k is not computed (their blocks are the transposes of
  // blocks the same launch computes); workgroups are launched for the tiles
  // that pair_cols_skipped keeps (pair_map: those are not all of them).  Never
  // with split-K.
  int32_t pair_upper, pair_lo, pair_map;
  // The first (ia|jb) launch of a small fragment (its status is null: V is
  // scratch) also checks the orbital energies, in one more workgroup that writes
  // gap_status for the kernels after it; null otherwise.
  int32_t* gap_status;
  const double *gap_eo, *gap_ev;
  int32_t gap_nocc, gap_nvir;
};

// True when the tile need not be computed (uniform): every occupied pair it
// touches is screened out, or (pair_upper) has pair_lo <= j < k.
template <int BM, int BN>
__device__ __forceinline__ bool tile_screened(const GemmParams& p, int tm, int tn) {
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  if (p.pair_upper && p.skip_j0 + (min(p.N, n0 + BN) - 1) / p.skip_nvir < p.skip_k0 + m0 / p.skip_nvir &&
      p.skip_j0 + n0 / p.skip_nvir >= p.pair_lo)
    return true;
  if (p.skip == nullptr) return false;
  const int64_t k_lo = m0 / p.skip_nvir, k_hi = (min(p.M, m0 + BM) - 1) / p.skip_nvir;
  const int64_t j_lo = n0 / p.skip_nvir, j_hi = (min(p.N, n0 + BN) - 1) / p.skip_nvir;
  for (int64_t k = k_lo; k <= k_hi; ++k)
    for (int64_t j = j_lo; j <= j_hi; ++j)
      if (p.skip[(p.skip_k0 + k) * p.skip_nocc + p.skip_j0 + j] == 0 &&
          p.skip[(p.skip_j0 + j) * p.skip_nocc + p.skip_k0 + k] == 0)
        return false;
  return true;
}

// Maps the hardware workgroup id to a logical id so that the workgroups one
// XCD runs (dispatch is round-robin over the 8 XCDs) get consecutive logical
// ids, and therefore neighbouring tiles that share operand rows in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int w, int G) {
  const int q = G >> 3, rem = G & 7, x = w & 7;
  return x * q + (x < rem ? x : rem) + (w >> 3);
}

// ROLE gives each contraction its own kernel symbol (profiler names);
// ROLE_GAMMA_T and ROLE_AO also select the M-contiguous A loader.
enum GemmRole { ROLE_INTS = 0, ROLE_GAMMA = 1, ROLE_PAB = 2, ROLE_PIJ = 3, ROLE_GAMMA_T = 4, ROLE_AO = 5,
                ROLE_LTERM = 6, ROLE_BATCH = 7 };
// Roles whose A operand is M-contiguous.
constexpr bool role_a_mcontig(int role) { return role == ROLE_GAMMA_T || role == ROLE_AO; }

// Column tiles that a pair_upper launch leaves out for a whole raster group:
// with k_lo the occupied orbital of the group's first row, the tiles
// [from, from + return) hold only pairs pair_lo <= j < k_lo.  Columns are j0 +
// n / nvir.  The rows of a group start at the same or a later orbital, so a
// tile left out here is one tile_screened would drop.
__host__ __device__ inline int64_t pair_cols_skipped(int64_t k_lo, int64_t j0, int64_t pair_lo, int64_t nvir,
                                                     int64_t bn, int64_t tiles_n, int64_t* from) {
  const int64_t below = (k_lo - j0) * nvir / bn;   // tiles whose last column has j < k_lo
  const int64_t lo = pair_lo > j0 ? ((pair_lo - j0) * nvir + bn - 1) / bn : 0;
  *from = lo;
  const int64_t n = (below < tiles_n ? below : tiles_n) - lo;
  return n > 0 ? n : 0;
}

// Tile t of a pair_upper launch, counted over the tiles its raster groups
// keep: one lane counts one group and a wave prefix sum finds t's group.  The
// launch then holds no workgroups for the skipped half of a whole-slab
// (ia|jb), whose tiles all lie in the later groups: with every tile launched
// and consecutive tiles going to one XCD (xcd_remap), the first XCDs held
// nearly all of the work and the last ones nearly none, and the product ran
// at half its rate.  MFMA-bound; energy of nocc = 100, nvir = 600, naux =
// 1800: 178 -> 99 ms (36.7 -> 66 TFLOP/s); nocc = 97, nvir = 485, naux =
// 1746: 107 -> 59 ms.  (A launch that keeps all of its tiles takes the plain raster:
// the map costs 1 us a workgroup, of 10 where the product is that small.)
__device__ __forceinline__ void decode_pair_tile(int64_t t, int64_t k0, int64_t j0, int64_t pair_lo,
                                                 int64_t nvir, int bm, int bn, int tiles_m, int tiles_n, int group_m,
                                                 int& tm, int& tn) {
  const int lane = threadIdx.x & 63, ngrp = (tiles_m + group_m - 1) / group_m;
  for (int base = 0;; base += 64) {
    const int grp = base + lane;
    int64_t from = 0, skipped = 0;
    int gm = 0;
    if (grp < ngrp) {
      gm = min(group_m, tiles_m - grp * group_m);
      skipped = pair_cols_skipped(k0 + (int64_t)grp * group_m * bm / nvir, j0, pair_lo, nvir, bn, tiles_n, &from);
    }
    const int64_t cnt = gm * (tiles_n - skipped);
    int64_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t v = __shfl_up(incl, d, 64);
      if (lane >= d) incl += v;
    }
    const unsigned long long past = __ballot(incl > t);
    if (past == 0 && base + 64 < ngrp) {
      t -= __shfl(incl, 63, 64);
      continue;
    }
    const int w = past ? __ffsll(past) - 1 : 0;
    const int64_t u = t - (__shfl(incl, w, 64) - __shfl(cnt, w, 64));
    const int g = __shfl(gm, w, 64);
    const int64_t c = u / g;
    const int64_t f = __shfl(from, w, 64), s = __shfl(skipped, w, 64);
    // the same in every lane; readfirstlane keeps the tile's addresses scalar
    tm = __builtin_amdgcn_readfirstlane((base + w) * group_m + (int)(u - c * g));
    tn = __builtin_amdgcn_readfirstlane((int)(c < f ? c : c + s));
    return;
  }
}

// Decodes logical tile index t (< tiles of one split) into (tm, tn):
// triangular order (TRI), the kept tiles of a pair_upper launch (pair_map), or groups of
// group_m m-tiles.
template <int BM, int BN, bool TRI>
__device__ __forceinline__ void decode_tile(const GemmParams& p, int t, int& tm, int& tn) {
  if (TRI) {
    tm = 0;
    while (t >= p.tiles_m - tm) { t -= p.tiles_m - tm; ++tm; }
    tn = tm + t;
  } else if (p.pair_map) {
    decode_pair_tile(t, p.skip_k0, p.skip_j0, p.pair_lo, p.skip_nvir, BM, BN, p.tiles_m, p.tiles_n, p.group_m, tm,
                     tn);
  } else {
    const int gsz = p.group_m * p.tiles_n;
    const int grp = t / gsz;
    const int first_m = grp * p.group_m;
    const int gm = min(p.group_m, p.tiles_m - first_m);
    const int tin = t - grp * gsz;
    tm = first_m + tin % gm;
    tn = tin / gm;
  }
}

// Workgroup barrier that orders LDS accesses only: global loads issued before
// it stay in flight across it (a full __syncthreads waits for them).
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int BM, int BN, int BK>
struct GemmLds {
  double a[2][BK * (BM + 2)];
  __attribute__((aligned(16))) double b[2][BK * (BN + 2)];
};

// One output tile (tm, tn) of split z.  Ends with a workgroup barrier, so the
// LDS can be reused by the next tile.
// A_MC: A is M-contiguous (p.Am) and is loaded like an N-contiguous B, two
// consecutive rows m per 16-byte load, into the same k-major LDS layout.
template <int BM, int BN, int BK, bool B_NCONTIG, bool VEC, bool TRI, int FAST, bool A_MC = false>
__device__ __forceinline__ void gemm_tile(const GemmParams& p, int tm, int tn, int z, GemmLds<BM, BN, BK>& lds) {
  static_assert(BM % 32 == 0 && BN % 32 == 0 && BK % 8 == 0, "tile shape");
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));   // a 16-byte load at any double

  constexpr int LDA = BM + 2, LDB = BN + 2;
  constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 16, NI = WTN / 16;
  constexpr int KP = BK / 2;                   // k pairs per row (K-contiguous loader)
  constexpr int RSTEP = 256 / KP;              // rows per pass
  static_assert(BM % RSTEP == 0 && BN % RSTEP == 0, "K loader shape");
  constexpr int AN = BM / RSTEP, BKN = BN / RSTEP;
  constexpr int NP = BN / 2;                   // column pairs per k row (N-contiguous loader)
  constexpr int NSTEP = 256 / NP;              // k rows per pass
  constexpr int BNN = B_NCONTIG ? BK / NSTEP : 1;
  static_assert(!B_NCONTIG || (256 % NP == 0 && BK % NSTEP == 0), "N loader shape");
  constexpr int BREG = B_NCONTIG ? BNN : BKN;
  constexpr int MP = BM / 2;                   // row pairs per k row (M-contiguous A loader)
  constexpr int MSTEP = 256 / MP;              // k rows per pass
  constexpr int AMN = A_MC ? BK / MSTEP : 1;
  static_assert(!A_MC || (256 % MP == 0 && BK % MSTEP == 0), "M loader shape");
  constexpr int AREG = A_MC ? AMN : AN;

  auto& As = lds.a;
  auto& Bs = lds.b;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  // FAST: the last tile along an M-contiguous A (N-contiguous B) starts early
  // enough to hold whole pairs only, and stores its own rows (columns) from
  // mlo (nlo) on; a matrix narrower than the tile is even (fast_level)
  const int64_t mlo = (int64_t)tm * BM, nlo = (int64_t)tn * BN;
  const int64_t m0 = FAST > 0 && A_MC ? max((int64_t)0, min(mlo, p.M - BM)) : mlo;
  const int64_t n0 = FAST > 0 && B_NCONTIG ? max((int64_t)0, min(nlo, p.N - BN)) : nlo;

  const int64_t kbeg = (int64_t)z * p.kchunk;
  const int64_t kend = min(p.K, kbeg + p.kchunk);
  const int nchunks = (int)((kend - kbeg + BK - 1) / BK);

  // K-contiguous loaders: thread -> rows r0 + s*RSTEP, reduction pair (kk, kk+1)
  const int kk = 2 * (tid % KP), r0 = tid / KP;
  int64_t aq = 0, ar = 0, bq = 0, br = 0;
  if (!A_MC) { const int64_t k = kbeg + kk; aq = k / p.A.kdiv; ar = k - aq * p.A.kdiv; }
  if (!B_NCONTIG) { const int64_t k = kbeg + kk; bq = k / p.Bk.kdiv; br = k - bq * p.Bk.kdiv; }
  // N-contiguous loader: thread -> column pair nn, k rows kn0 + s*NSTEP
  const int nn = 2 * (tid % NP), kn0 = tid / NP;
  // M-contiguous A loader: thread -> row pair mm, k rows km0 + s*MSTEP
  const int mm = 2 * (tid % MP), km0 = tid / MP;
  const bool fullA = (m0 + BM <= p.M), fullB = (n0 + BN <= p.N);

  d2 ra[AREG], rb[BREG];

  // One K-contiguous operand tile: element (row, k) = base[row*rs + (k/kdiv)*ks1 + k%kdiv].
  // (q, r) is this thread's position for k = kc + kk.  With VEC the host has
  // checked that every pair (kk, kk+1) lies in one run and is 16-byte aligned.
  // The masked path steps (q, r) to kk+1 without division.
#define RIMP2_KLOAD(OP, ROW0, NROWS, FULLROWS, Q, R, DST, CNT)                                        \
  {                                                                                                 \
    if (VEC && (FULLROWS) && fullk) {                                                               \
      const double* src = OP.base + ((ROW0) + r0) * OP.rs + (Q) * OP.ks1 + (R);                     \
      const int64_t st = (int64_t)RSTEP * OP.rs;                                                    \
      _Pragma("unroll") for (int s = 0; s < CNT; ++s) DST[s] = *(const d2*)(src + s * st);          \
    } else {                                                                                        \
      const int64_t k0 = kc + kk;                                                                   \
      const int64_t off0 = (Q) * OP.ks1 + (R);                                                      \
      const int64_t off1 = ((R) + 1 < OP.kdiv) ? off0 + 1 : ((Q) + 1) * OP.ks1;                     \
      _Pragma("unroll") for (int s = 0; s < CNT; ++s) {                                             \
        const int64_t row = (ROW0) + r0 + s * RSTEP;                                                \
        const int64_t rb0 = min(row, (NROWS) - 1) * OP.rs;                                          \
        const bool rv = row < (NROWS);                                                              \
        const double v0 = (rv && k0 < kend) ? OP.base[rb0 + off0] : 0.0;                            \
        const double v1 = (rv && k0 + 1 < kend) ? OP.base[rb0 + off1] : 0.0;                        \
        DST[s][0] = v0;                                                                             \
        DST[s][1] = v1;                                                                             \
      }                                                                                             \
    }                                                                                               \
  }
  auto load_chunk = [&](int c) {
    const int64_t kc = kbeg + (int64_t)c * BK;
    const bool fullk = (kc + BK <= kend);
    if constexpr (!A_MC) {
      RIMP2_KLOAD(p.A, m0, p.M, fullA, aq, ar, ra, AN)
    } else {
      const int64_t m = m0 + mm;
      if (VEC && fullA && fullk) {
        const double* src = p.Am.base + (kc + km0) * p.Am.ld + m;
        const int64_t st = (int64_t)MSTEP * p.Am.ld;
#pragma unroll
        for (int s = 0; s < AMN; ++s) ra[s] = *(const d2*)(src + s * st);
      } else {
#pragma unroll
        for (int s = 0; s < AMN; ++s) {
          const int64_t k = kc + km0 + s * MSTEP;
          const double* row = p.Am.base + min(k, kend - 1) * p.Am.ld;
          const double x0 = (k < kend && m < p.M) ? row[m] : 0.0;
          const double x1 = (k < kend && m + 1 < p.M) ? row[m + 1] : 0.0;
          ra[s][0] = x0;
          ra[s][1] = x1;
        }
      }
    }
    if (!B_NCONTIG) {
      RIMP2_KLOAD(p.Bk, n0, p.N, fullB, bq, br, rb, BKN)
    } else {
      const int64_t n = n0 + nn;
      if (VEC && fullB && fullk) {
        const double* src = p.Bn.base + (kc + kn0) * p.Bn.ld + n;
        const int64_t st = (int64_t)NSTEP * p.Bn.ld;
#pragma unroll
        for (int s = 0; s < BNN; ++s) rb[s] = *(const d2*)(src + s * st);
      } else {
#pragma unroll
        for (int s = 0; s < BNN; ++s) {
          const int64_t k = kc + kn0 + s * NSTEP;
          const double* row = p.Bn.base + min(k, kend - 1) * p.Bn.ld;
          const double x0 = (k < kend && n < p.N) ? row[n] : 0.0;
          const double x1 = (k < kend && n + 1 < p.N) ? row[n + 1] : 0.0;
          rb[s][0] = x0;
          rb[s][1] = x1;
        }
      }
    }
    if (!A_MC) {
      ar += BK;
      while (ar >= p.A.kdiv) { ar -= p.A.kdiv; ++aq; }
    }
    if (!B_NCONTIG) {
      br += BK;
      while (br >= p.Bk.kdiv) { br -= p.Bk.kdiv; ++bq; }
    }
  };
#undef RIMP2_KLOAD
  auto store_from = [&](int buf, const d2 (&sa)[AREG], const d2 (&sb)[BREG]) {
    if (!A_MC) {
#pragma unroll
      for (int s = 0; s < AREG; ++s) {
        As[buf][kk * LDA + r0 + s * RSTEP] = sa[s][0];
        As[buf][(kk + 1) * LDA + r0 + s * RSTEP] = sa[s][1];
      }
    } else {
#pragma unroll
      for (int s = 0; s < AREG; ++s) *(d2*)&As[buf][(km0 + s * MSTEP) * LDA + mm] = sa[s];
    }
    if (!B_NCONTIG) {
#pragma unroll
      for (int s = 0; s < BKN; ++s) {
        Bs[buf][kk * LDB + r0 + s * RSTEP] = sb[s][0];
        Bs[buf][(kk + 1) * LDB + r0 + s * RSTEP] = sb[s][1];
      }
    } else {
#pragma unroll
      for (int s = 0; s < BNN; ++s) *(d2*)&Bs[buf][(kn0 + s * NSTEP) * LDB + nn] = sb[s];
    }
  };
  auto store_chunk = [&](int buf) { store_from(buf, ra, rb); };
  // MFMA fragments of k-step ks (4 reduction indices) from LDS buffer buf
  auto read_frag = [&](int buf, int ks, double* a, double* b) {
    const int kr = 4 * ks + (lane >> 4);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = As[buf][kr * LDA + wm * WTM + i * 16 + (lane & 15)];
#pragma unroll
    for (int j = 0; j < NI; ++j) b[j] = Bs[buf][kr * LDB + wn * WTN + j * 16 + (lane & 15)];
  };

  dbl4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};

  // FAST > 0 (chosen by the host: runs of the K operands at least one chunk
  // long, and M- or N-contiguous operands that hold whole pairs): the
  // split's full chunks go through a branch-free loader that issues each
  // chunk's global loads two chunks ahead into two register sets.  Rows (and
  // N-contiguous column pairs) past the edge of the matrix read the last valid
  // ones, which only reach accumulators that are never stored.  The loads are
  // unconditional (after the last full chunk it is loaded again), so the
  // compiler's wait counts stay exact, and the barriers order LDS only, so the
  // loads stay in flight across them.  A pair of doubles is one 16-byte load
  // at any 8-byte address: an odd row stride costs a second cache line per
  // 128-byte run, which the loads' two-chunk lead covers (measured against the
  // general loader's 8-byte loads: see fast_level).  Chunk starts advance by
  // uniform run steps; with FAST = 2 (even runs shorter than the reduction and
  // not a multiple of the chunk) a thread whose pair lies in the next run adds
  // one run step, and with FAST = 3 (odd runs, so that a pair can lie in two)
  // each element of a pair is loaded by itself with its own step.  A ragged
  // last chunk is then loaded with per-element masks and run on its own.
  // Every path sums each output element in the same order.
  if constexpr (FAST > 0) {
    const int nfull = (int)((kend - kbeg) / BK);
    if (nfull > 0) {
      d2 xa[2][AREG], xb[2][BREG];
      // start of the next chunk to load (uniform): offset of each K operand
      // and its position in the current run
      int64_t oa = 0, pa = 0, ob = 0, pb = 0;
      if (!A_MC) { const int64_t q = kbeg / p.A.kdiv; pa = kbeg - q * p.A.kdiv; oa = q * p.A.ks1 + pa; }
      else { oa = kbeg * p.Am.ld; }
      if (!B_NCONTIG) { const int64_t q = kbeg / p.Bk.kdiv; pb = kbeg - q * p.Bk.kdiv; ob = q * p.Bk.ks1 + pb; }
      else { ob = kbeg * p.Bn.ld; }
      int nload = 0;
      const double* ap[AREG];
      if (!A_MC) {
#pragma unroll
        for (int s = 0; s < AREG; ++s) ap[s] = p.A.base + min(m0 + r0 + s * RSTEP, p.M - 1) * p.A.rs + kk;
      } else {
        const int64_t m = min(m0 + mm, p.M - 2);
#pragma unroll
        for (int s = 0; s < AREG; ++s) ap[s] = p.Am.base + (int64_t)(km0 + s * MSTEP) * p.Am.ld + m;
      }
      const double* bp[BREG];
      if (!B_NCONTIG) {
#pragma unroll
        for (int s = 0; s < BREG; ++s) bp[s] = p.Bk.base + min(n0 + r0 + s * RSTEP, p.N - 1) * p.Bk.rs + kk;
      } else {
        const int64_t n = min(n0 + nn, p.N - 2);
#pragma unroll
        for (int s = 0; s < BREG; ++s) bp[s] = p.Bn.base + (int64_t)(kn0 + s * NSTEP) * p.Bn.ld + n;
      }
      // extra offset of element kk + d of this thread when it lies in the run after the chunk start's
      auto wrap = [&](const KOperand& o, int64_t pos, int d) -> int64_t {
        return (FAST >= 2 && pos + kk + d >= o.kdiv) ? o.ks1 - o.kdiv : 0;
      };
      auto fload = [&](d2 (&da)[AREG], d2 (&db)[BREG]) {
        if (!A_MC && FAST == 3) {
          const int64_t x0 = oa + wrap(p.A, pa, 0), x1 = oa + wrap(p.A, pa, 1) + 1;
#pragma unroll
          for (int s = 0; s < AREG; ++s) da[s] = d2{ap[s][x0], ap[s][x1]};
        } else {
          const int64_t xa_ = A_MC ? oa : oa + wrap(p.A, pa, 0);
#pragma unroll
          for (int s = 0; s < AREG; ++s) da[s] = *(const d2u*)(ap[s] + xa_);
        }
        if (!B_NCONTIG && FAST == 3) {
          const int64_t x0 = ob + wrap(p.Bk, pb, 0), x1 = ob + wrap(p.Bk, pb, 1) + 1;
#pragma unroll
          for (int s = 0; s < BREG; ++s) db[s] = d2{bp[s][x0], bp[s][x1]};
        } else {
          const int64_t xb_ = B_NCONTIG ? ob : ob + wrap(p.Bk, pb, 0);
#pragma unroll
          for (int s = 0; s < BREG; ++s) db[s] = *(const d2u*)(bp[s] + xb_);
        }
        if (++nload < nfull) {
          if (A_MC) {
            oa += (int64_t)BK * p.Am.ld;
          } else {
            oa += BK; pa += BK;
            if (pa >= p.A.kdiv) { pa -= p.A.kdiv; oa += p.A.ks1 - p.A.kdiv; }
          }
          if (B_NCONTIG) {
            ob += (int64_t)BK * p.Bn.ld;
          } else {
            ob += BK; pb += BK;
            if (pb >= p.Bk.kdiv) { pb -= p.Bk.kdiv; ob += p.Bk.ks1 - p.Bk.kdiv; }
          }
        }
      };
      fload(xa[0], xb[0]);
      fload(xa[1], xb[1]);
      store_from(0, xa[0], xb[0]);
      lds_sync();
      // chunk c (c % 2 == S) from LDS buffer S; chunk c+1 waits in register set S^1
      auto step = [&](int c, auto set) {
        constexpr int S = decltype(set)::value;
        const bool more = c + 1 < nfull;
        fload(xa[S], xb[S]);
#pragma unroll
        for (int ks = 0; ks < BK / 4; ++ks) {
          if (ks == BK / 8 && more) store_from(S ^ 1, xa[S ^ 1], xb[S ^ 1]);
          double a[MI], b[NI];
          read_frag(S, ks, a, b);
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        lds_sync();
      };
      int c = 0;
      for (; c + 1 < nfull; c += 2) {
        step(c, std::integral_constant<int, 0>{});
        step(c + 1, std::integral_constant<int, 1>{});
      }
      if (c < nfull) step(c, std::integral_constant<int, 0>{});
    }
    if (nfull < nchunks) {
      // the ragged last chunk: per-element masks
      const int64_t kt = kbeg + (int64_t)nfull * BK;
      const d2 zero = {0.0, 0.0};
      // elements k and k + 1 of the row at `row`, 0 past the end of the
      // reduction: without runs one load of the last whole pair, shifted
      const int64_t k = kt + kk;
      auto kpair = [&](const KOperand& o, const double* row) {
        d2 v = zero;
        if (FAST == 1 && o.kdiv >= p.K && p.K >= 2) {
          const d2 x = *(const d2u*)(row + min(k, kend - 2));
          v[0] = k + 1 < kend ? x[0] : k < kend ? x[1] : 0.0;
          v[1] = k + 1 < kend ? x[1] : 0.0;
        } else if (k < kend) {
          const int64_t q = k / o.kdiv, r = k - q * o.kdiv;
          v[0] = row[q * o.ks1 + r];
          if (k + 1 < kend) v[1] = row[r + 1 < o.kdiv ? q * o.ks1 + r + 1 : (q + 1) * o.ks1];
        }
        return v;
      };
      if (!A_MC) {
#pragma unroll
        for (int s = 0; s < AREG; ++s) ra[s] = kpair(p.A, p.A.base + min(m0 + r0 + s * RSTEP, p.M - 1) * p.A.rs);
      } else {
        const int64_t m = min(m0 + mm, p.M - 2);
#pragma unroll
        for (int s = 0; s < AREG; ++s) {
          const int64_t k = kt + km0 + s * MSTEP;
          ra[s] = k < kend ? (d2)*(const d2u*)(p.Am.base + k * p.Am.ld + m) : zero;
        }
      }
      if (!B_NCONTIG) {
#pragma unroll
        for (int s = 0; s < BREG; ++s) rb[s] = kpair(p.Bk, p.Bk.base + min(n0 + r0 + s * RSTEP, p.N - 1) * p.Bk.rs);
      } else {
        const int64_t n = min(n0 + nn, p.N - 2);
#pragma unroll
        for (int s = 0; s < BREG; ++s) {
          const int64_t k = kt + kn0 + s * NSTEP;
          rb[s] = k < kend ? (d2)*(const d2u*)(p.Bn.base + k * p.Bn.ld + n) : zero;
        }
      }
      store_chunk(0);
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < BK / 4; ++ks) {
        double a[MI], b[NI];
        read_frag(0, ks, a, b);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  } else if (nchunks > 0) {
    load_chunk(0);
    store_chunk(0);
    __syncthreads();
    for (int c = 0; c < nchunks; ++c) {
      const int buf = c & 1;
      const bool more = c + 1 < nchunks;
      if (more) load_chunk(c + 1);
#pragma unroll
      for (int ks = 0; ks < BK / 4; ++ks) {
        if (ks == BK / 8 && more) store_chunk(buf ^ 1);
        double a[MI], b[NI];
        read_frag(buf, ks, a, b);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }

  double* C = p.C + (int64_t)z * p.split_stride;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm * WTM + i * 16 + 4 * r + (lane >> 4);
        const int64_t n = n0 + wn * WTN + j * 16 + (lane & 15);
        if (m < p.M && n < p.N && (!(FAST > 0 && A_MC) || m >= mlo) && (!(FAST > 0 && B_NCONTIG) || n >= nlo)) {
          if (!TRI) {
            if (p.accumulate) C[m * p.ldc + n] += acc[i][j][r];
            else C[m * p.ldc + n] = acc[i][j][r];
          } else if (m <= n) {   // every lower element is the mirror of an upper one
            C[m * p.ldc + n] = acc[i][j][r];
            if (m < n) C[n * p.ldc + m] = acc[i][j][r];
          }
        }
      }
}

// Roles launched as batches of products.
constexpr bool role_batched(int role) { return role == ROLE_AO || role == ROLE_BATCH; }
// One workgroup per (split, tile); the hardware id is remapped XCD-aware.
template <int BM, int BN, int BK, bool B_NCONTIG, int ROLE, bool VEC, bool TRI, int FAST = 0>
__global__ __launch_bounds__(256, 2) void gemm_f64_kernel(GemmParams p) {
  if (p.status != nullptr && *p.status != 0) return;
  __shared__ GemmLds<BM, BN, BK> lds;
  int nwg = gridDim.x;
  if (ROLE == ROLE_INTS && p.gap_status != nullptr) {
    --nwg;
    if ((int)blockIdx.x == nwg) {
      gap_check_block(p.gap_eo, p.gap_nocc, p.gap_ev, p.gap_nvir, p.gap_status);
      return;
    }
  }
  const int wl = xcd_remap(blockIdx.x, nwg);
  const int ntiles = TRI ? p.tiles_m * (p.tiles_m + 1) / 2 : p.tiles_m * p.tiles_n;
  int z = wl / ntiles;   // 0 in a pair_upper launch: at most ntiles workgroups
  int tm, tn;
  decode_tile<BM, BN, TRI>(p, wl - z * ntiles, tm, tn);
  if (role_batched(ROLE) && p.batch > 1) {
    if (role_a_mcontig(ROLE)) p.Am.base += z * p.batch_a; else p.A.base += z * p.batch_a;
    if (B_NCONTIG) p.Bn.base += z * p.batch_b; else p.Bk.base += z * p.batch_b;
    p.C += z * p.split_stride;
    z = 0;
  }
  if (tile_screened<BM, BN>(p, tm, tn)) return;
  gemm_tile<BM, BN, BK, B_NCONTIG, VEC, TRI, FAST, role_a_mcontig(ROLE)>(p, tm, tn, z, lds);
}

// Gamma, P_ab and P_ij of a fragment whose products are each too small to fill
// the chip, in one launch: workgroups [0, n_gam) take Gamma's tiles (64), the
// longest, then P_ab's (64) and P_ij's (32).  FW: the fast loader's level of P_ab
// and P_ij (2 or 3).  Every element is summed as in the separate launches.
// Latency-bound; one after another they took 25 us at nocc = 5, nvir = 25, naux =
// 90 and 126 us at 20/100/400, together 11 and 108.
struct TailParams {
  GemmParams gam, ab, ij;
  int32_t n_gam, n_ab;
};
template <int FW>
__global__ __launch_bounds__(256, 4) void gemm_f64_tail(TailParams t) {
  if (*t.gam.status != 0) return;
  __shared__ __attribute__((aligned(16))) char lds[sizeof(GemmLds<64, 64, 16>)];
  int w = blockIdx.x, tm, tn;
  if (w < t.n_gam) {
    const int n = t.gam.tiles_m * t.gam.tiles_n, z = w / n;
    decode_tile<64, 64, false>(t.gam, w - z * n, tm, tn);
    gemm_tile<64, 64, 16, true, true, false, 1>(t.gam, tm, tn, z, *(GemmLds<64, 64, 16>*)lds);
    return;
  }
  w -= t.n_gam;
  if (w < t.n_ab) {
    const int n = t.ab.tiles_m * (t.ab.tiles_m + 1) / 2, z = w / n;
    decode_tile<64, 64, true>(t.ab, w - z * n, tm, tn);
    gemm_tile<64, 64, 16, false, true, true, FW>(t.ab, tm, tn, z, *(GemmLds<64, 64, 16>*)lds);
    return;
  }
  w -= t.n_ab;
  const int n = t.ij.tiles_m * (t.ij.tiles_m + 1) / 2, z = w / n;
  decode_tile<32, 32, true>(t.ij, w - z * n, tm, tn);
  gemm_tile<32, 32, 16, false, true, true, FW>(t.ij, tm, tn, z, *(GemmLds<32, 32, 16>*)lds);
}

// Grouped launch over many independent GEMMs (one per fragment): problem f owns
// work items [prefix[f], prefix[f+1]) = its tiles x splits, problems ordered
// largest first, one workgroup per item.  Workgroups are dispatched round-robin
// over the 8 XCDs; blocks of `block` consecutive items go to one XCD in turn, so
// that its workgroups share operand panels in its L2.  (Persistent workgroups
// that took items from counters fetched an item across the fabric before each
// tile, and their loop left the 128 x 128 tiles short of registers.)
template <class P>
struct Grouped {
  const P* probs;
  const int64_t* prefix;   // [nprob + 1]
  int32_t nprob, block;
};
// The workgroup's problem and item within it; false: past the last item.
template <class P>
__device__ __forceinline__ bool grouped_item(const Grouped<P>& G, int& f, int& u) {
  const int n = blockIdx.x >> 3, q = n / G.block;
  const int64_t t = ((int64_t)q * 8 + (blockIdx.x & 7)) * G.block + (n - q * G.block);
  if (t >= G.prefix[G.nprob]) return false;
  int lo = 0, hi = G.nprob - 1;   // last f with prefix[f] <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (G.prefix[mid] <= t) lo = mid; else hi = mid - 1;
  }
  f = lo;
  u = (int)(t - G.prefix[lo]);
  return true;
}

template <int BM, int BN, int BK, bool B_NCONTIG, int ROLE, bool VEC, bool TRI, int FAST = 0>
__global__ __launch_bounds__(256, 2) void gemm_f64_grouped(Grouped<GemmParams> G) {
  __shared__ GemmLds<BM, BN, BK> lds;
  int f, u;
  if (!grouped_item(G, f, u)) return;
  const GemmParams p = G.probs[f];
  if (p.status != nullptr && *p.status != 0) return;
  const int ntiles = TRI ? p.tiles_m * (p.tiles_m + 1) / 2 : p.tiles_m * p.tiles_n;
  const int z = u / ntiles;
  int tm, tn;
  decode_tile<BM, BN, TRI>(p, u - z * ntiles, tm, tn);
  if (tile_screened<BM, BN>(p, tm, tn)) return;
  gemm_tile<BM, BN, BK, B_NCONTIG, VEC, TRI, FAST>(p, tm, tn, z, lds);
}

}  // namespace rimp2
