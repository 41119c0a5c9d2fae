// Split-precision (Ozaki-style) products on gfx950 INT8 MFMA.
//
// A row (or column) x of an FP64 operand is scaled by 2^-e with
// e = ilogb(max |x|) + 1, so |x| 2^-e < 1, and written as S balanced base-128
// digits:  x = 2^e / 64 * sum_{s=1..S} d_s 128^(1-s),  |d_s| <= 64,  extracted
// exactly in FP64 with round-to-nearest (y = x 2^(6-e); d = rint(y);
// y = (y - d) * 128; ...).  The dropped remainder is at most 2^-7S relative
// to the row maximum.
//
// C = A B^T is then
//   C[m,n] = 2^(ea[m] + eb[n] - 12) * sum_{L=2..S+1} 128^(2-L) * sum_{s+t=L} D_s(A) D_t(B)^T
// (the products with s + t > S + 1 are below the digit truncation and are
// dropped: S(S+1)/2 integer products).  Each level is summed exactly in INT32
// by v_mfma_i32_16x16x64_i8; a launch reduces over at most kOzMaxK indices, so
// no level can overflow (7 * kOzMaxK * 64 * 64 < 2^31), and then combines the
// levels in FP64.
//
// MFMA lane layout (measured on gfx950): lane l supplies A[l%16][16(l/16)+b]
// and B[16(l/16)+b][l%16] for byte b; accumulator register r of lane l holds
// D[4(l/16)+r][l%16].  A and B digits are read with the same lane/byte -> k
// map, so the reduction index needs no particular order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rimp2 {

typedef int v4i __attribute__((ext_vector_type(4)));
constexpr int64_t kOzMaxK = 65536;

// Row-scaled digits of a K-contiguous FP64 matrix X[rows][K] (row stride ld):
// D[s][row][kp] (kp = K rounded up to 64, zero padded) and exps[row].
// One workgroup per row.
template <int S>
__device__ __forceinline__ void split_row(const double* X, int64_t rows, int64_t K, int64_t ld, int8_t* D,
                                          int64_t kp, int32_t* exps, int64_t row) {
  const double* x = X + row * ld;
  __shared__ double sm[256];
  double mx = 0.0;
  for (int64_t k = threadIdx.x; k < K; k += 256) mx = fmax(mx, fabs(x[k]));
  sm[threadIdx.x] = mx;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + w]);
    __syncthreads();
  }
  mx = sm[0];
  const int e = (mx > 0.0) ? ilogb(mx) + 1 : 0;
  if (threadIdx.x == 0) exps[row] = e;
  for (int64_t k = threadIdx.x; k < kp; k += 256) {
    double y = (k < K) ? ldexp(x[k], 6 - e) : 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double d = rint(y);
      D[((int64_t)s * rows + row) * kp + k] = (int8_t)d;
      y = (y - d) * 128.0;
    }
  }
}

template <int S>
__global__ __launch_bounds__(256) void split_rows_kernel(const double* X, int64_t rows, int64_t K, int64_t ld,
                                                         int8_t* D, int64_t kp, int32_t* exps, const int32_t* status) {
  if (status != nullptr && *status != 0) return;
  split_row<S>(X, rows, K, ld, D, kp, exps, blockIdx.x);
}

// Column maxima of X[K][N] (row stride ld) as IEEE bit patterns (non-negative
// doubles order like their bit patterns, so an integer max is exact and
// order-independent).  cmax must start at zero.
__device__ __forceinline__ void colmax_block(const double* X, int64_t K, int64_t N, int64_t ld,
                                             unsigned long long* cmax, int64_t bx, int64_t by) {
  const int64_t n = bx * 256 + threadIdx.x;
  if (n >= N) return;
  const int64_t k0 = by * 1024, k1 = min(K, k0 + 1024);
  double mx = 0.0;
  for (int64_t k = k0; k < k1; ++k) mx = fmax(mx, fabs(X[k * ld + n]));
  atomicMax(cmax + n, (unsigned long long)__double_as_longlong(mx));
}

__global__ __launch_bounds__(256) void colmax_kernel(const double* X, int64_t K, int64_t N, int64_t ld,
                                                     unsigned long long* cmax, const int32_t* status) {
  if (status != nullptr && *status != 0) return;
  colmax_block(X, K, N, ld, cmax, blockIdx.x, blockIdx.y);
}

// Column-scaled digits of X[K][N], written transposed: D[s][n][kp], exps[n].
// 32 x 32 tiles through LDS so both the read and the write are coalesced.
template <int S>
__device__ __forceinline__ void split_cols_tile(const double* X, int64_t K, int64_t N, int64_t ld,
                                                const unsigned long long* cmax, int8_t* D, int64_t kp,
                                                int32_t* exps, int64_t bx, int64_t by) {
  __shared__ double tile[32][33];
  const int64_t k0 = bx * 32, n0 = by * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 8 rows per pass
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t k = k0 + ty + 8 * r, n = n0 + tx;
    tile[ty + 8 * r][tx] = (k < K && n < N) ? X[k * ld + n] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t n = n0 + ty + 8 * r, k = k0 + tx;
    if (n >= N || k >= kp) continue;
    const double mx = __longlong_as_double((long long)cmax[n]);
    const int e = (mx > 0.0) ? ilogb(mx) + 1 : 0;
    if (k == 0) exps[n] = e;
    double y = ldexp(tile[tx][ty + 8 * r], 6 - e);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double d = rint(y);
      D[((int64_t)s * N + n) * kp + k] = (int8_t)d;
      y = (y - d) * 128.0;
    }
  }
}

template <int S>
__global__ __launch_bounds__(256) void split_cols_kernel(const double* X, int64_t K, int64_t N, int64_t ld,
                                                         const unsigned long long* cmax, int8_t* D, int64_t kp,
                                                         int32_t* exps, const int32_t* status) {
  if (status != nullptr && *status != 0) return;
  split_cols_tile<S>(X, K, N, ld, cmax, D, kp, exps, blockIdx.x, blockIdx.y);
}

struct OzParams {
  int64_t M, N, kp;            // kp: padded reduction length (multiple of 64), also the digit row stride
  int64_t k0, kc;              // this launch reduces over [k0, k0 + kc) (multiples of 64)
  int32_t accumulate;          // 0: C = the window's sum; 1: C += it
  const int8_t* A;             // digits [S][a_rows][kp]; output rows m use A row a_row0 + m
  int64_t a_slice, a_row0;
  const int8_t* B;             // digits [S][b_rows][kp]
  int64_t b_slice;
  const int32_t* ea;           // exponents of A rows (indexed like A rows)
  const int32_t* eb;
  double* C;
  int64_t ldc;
  int32_t tiles_m, tiles_n, group_m;
  // pair_nvir > 0: rows are (k, a) from orbital pair_k0 (a_row0 = pair_k0
  // pair_nvir), columns (j, b) from orbital pair_j0, and tiles that hold only
  // pairs pair_lo <= j < k are left out (oz8_tile_skipped, decode_pair_tile;
  // pair_map: the launch holds workgroups for fewer than all tiles)
  int32_t pair_nvir, pair_k0, pair_j0, pair_lo, pair_map;
  const int32_t* status;
};

// Tile shapes.  The waves form a WM x WN grid, each with MI x NI blocks of 16 x
// 16 outputs; the S digit slices of a 64-wide reduction step of both operands
// are staged in LDS (1 KB per slice and 16 rows), NBUF stages deep.  Within a
// 1 KB block lane l writes bytes [16 l, 16 l + 16), and it loads row r = l / 4,
// 16-byte chunk (l % 4) ^ oz8_swizzle(r): the 16-lane groups in which the LDS
// serves the fragment reads (lanes 0-3, 12-15, 20-27; 4-11, 16-19, 28-31; the
// same from 32 on) then meet no bank twice.  (With (r / 4) % 4 half of the
// LDS's active cycles were conflicts.)
// Bound by operand delivery under a power limit: random digits in registers
// alone reach 3.95 POP/s, a tile that stages from a warm L2 2.8, and the 7-digit
// (ia|jb) product of 40/900/3000 runs at 2.2.
//   OzSmall: 4 waves of 32 x 32, 64 x 64 outputs, two workgroups a CU.  NBUF = 2
//     double-buffers the stage; NBUF = 1 keeps one, copied after the step's
//     MFMAs, so that two workgroups share a CU at any S.
//   OzWide (S <= 5): 8 waves of 64 x 32, 128 x 128 outputs, one workgroup a CU
//     with two stages (S = 5: all 160 KB).  It stages half the bytes per
//     product: Gamma windows of 36000 x 3000 x 2816 at 5 digits 4.4 -> 3.7 ms
//     (2.1 -> 2.5 POP/s).  Reading the next stage's first fragments before the
//     barrier spilled registers and took 4.7.
struct OzSmall {
  static constexpr int WM = 2, WN = 2, MI = 2, NI = 2;
};
struct OzWide {
  static constexpr int WM = 2, WN = 4, MI = 4, NI = 2;
};
// 0, 2, 3, 1 for rows 0-3, 4-7, 8-11, 12-15 of a block.
__device__ __forceinline__ int oz8_swizzle(int r) { return (0x78 >> (2 * (r >> 2))) & 3; }
template <class T>
struct OzShape {
  static constexpr int BM = T::WM * T::MI * 16, BN = T::WN * T::NI * 16, THREADS = T::WM * T::WN * 64;
};
template <int S, class T = OzSmall>
struct OzLds {
  static constexpr int STAGE = S * (OzShape<T>::BM + OzShape<T>::BN) * 64;
};

// A tile whose pairs all have pair_lo <= j < k is skipped when p.pair_nvir >
// 0: the amplitude pass forms those blocks from their mirror.
__device__ __forceinline__ bool oz8_tile_skipped(const OzParams& p, int64_t m0, int64_t n0, int bn) {
  if (p.pair_nvir <= 0) return false;
  return p.pair_j0 + min(n0 + bn - 1, p.N - 1) / p.pair_nvir < p.pair_k0 + m0 / p.pair_nvir &&
         p.pair_j0 + n0 / p.pair_nvir >= p.pair_lo;
}

// Logical tile t of a launch: raster groups of group_m row tiles, of a pair
// launch the tiles they keep.
__device__ __forceinline__ void oz8_decode(const OzParams& p, int bm, int bn, int t, int& tm, int& tn) {
  if (p.pair_map) {
    decode_pair_tile(t, p.pair_k0, p.pair_j0, p.pair_lo, p.pair_nvir, bm, bn, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
  } else {
    const int gsz = p.group_m * p.tiles_n, grp = t / gsz, first_m = grp * p.group_m;
    const int gm = min(p.group_m, p.tiles_m - first_m), tin = t - grp * gsz;
    tm = first_m + tin % gm;
    tn = tin / gm;
  }
}

// One output tile at (m0, n0) over the reduction window [k0, k0 + kc).
template <int S, int NBUF, class T>
__device__ __forceinline__ void oz8_tile(const OzParams& p, int64_t m0, int64_t n0, int8_t (*lds)[OzLds<S, T>::STAGE]) {
  constexpr int MI = T::MI, NI = T::NI, RA = OzShape<T>::BM / 16, RB = OzShape<T>::BN / 16;   // row blocks of A, B
  constexpr int NW = T::WM * T::WN, CA = RA / NW, CB = RB / NW;   // row blocks each wave copies
  static_assert(RA % NW == 0 && RB % NW == 0, "row blocks per wave");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wv / T::WN, wn = wv % T::WN;

  // copy: rows past the end read the last row (their outputs are not stored);
  // a scalar base and a 32-bit lane offset per row block
  const int dr = lane >> 2, dc = (lane & 3) ^ oz8_swizzle(dr);
  const int8_t *tileA = p.A + (p.a_row0 + m0) * p.kp, *tileB = p.B + n0 * p.kp;
  uint32_t offA[CA], offB[CB];
#pragma unroll
  for (int c = 0; c < CA; ++c)
    offA[c] = (uint32_t)(min((int64_t)(16 * (wv + NW * c) + dr), p.M - 1 - m0) * p.kp + 16 * dc);
#pragma unroll
  for (int c = 0; c < CB; ++c)
    offB[c] = (uint32_t)(min((int64_t)(16 * (wv + NW * c) + dr), p.N - 1 - n0) * p.kp + 16 * dc);
  auto copy = [&](int buf, int64_t k) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int8_t *a = tileA + (s * p.a_slice + k), *b = tileB + (s * p.b_slice + k);
#pragma unroll
      for (int c = 0; c < CA; ++c)
        __builtin_amdgcn_global_load_lds((const void*)(a + offA[c]),
                                         (void*)(lds[buf] + (s * (RA + RB) + wv + NW * c) * 1024), 16, 0, 0);
#pragma unroll
      for (int c = 0; c < CB; ++c)
        __builtin_amdgcn_global_load_lds((const void*)(b + offB[c]),
                                         (void*)(lds[buf] + (s * (RA + RB) + RA + wv + NW * c) * 1024), 16, 0, 0);
    }
  };
  // fragment of lane (g, l16): row l16 of a row block, data chunk g
  const int fpos = (l16 * 4 + (g ^ oz8_swizzle(l16))) * 16;

  v4i acc[S][MI][NI];
#pragma unroll
  for (int L = 0; L < S; ++L)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[L][i][j] = v4i{0, 0, 0, 0};

  const int nsteps = (int)(p.kc / 64);
  auto frag_a = [&](const int8_t* L0, int s, v4i (&f)[MI]) {
#pragma unroll
    for (int i = 0; i < MI; ++i) f[i] = *(const v4i*)(L0 + (s * (RA + RB) + wm * MI + i) * 1024);
  };
  auto frag_b = [&](const int8_t* L0, int t, v4i (&f)[NI]) {
#pragma unroll
    for (int j = 0; j < NI; ++j) f[j] = *(const v4i*)(L0 + (t * (RA + RB) + RA + wn * NI + j) * 1024);
  };
  // LDS copies count in vmcnt: wait for this wave's (a barrier alone does not),
  // then the barrier makes every wave's visible and frees the stage they all read
  auto stage_barrier = [] {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };
  if (nsteps > 0) copy(0, p.k0);
  stage_barrier();
  for (int st = 0; st < nsteps; ++st) {
    const int b = NBUF == 2 ? st & 1 : 0;
    if (NBUF == 2 && st + 1 < nsteps) copy(b ^ 1, p.k0 + (int64_t)(st + 1) * 64);
    const int8_t* L0 = lds[b] + fpos;
    v4i fb[S][NI];
#pragma unroll
    for (int t = 0; t < S; ++t) frag_b(L0, t, fb[t]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      v4i fa[MI];
      frag_a(L0, s, fa);
#pragma unroll
      for (int t = 0; t < S - s; ++t)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[s + t][i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb[t][j], acc[s + t][i][j], 0, 0, 0);
    }
    if (st + 1 < nsteps) {
      stage_barrier();   // every wave is done reading the stage (and, of two, the next one is there)
      if (NBUF == 1) {
        copy(0, p.k0 + (int64_t)(st + 1) * 64);
        stage_barrier();
      }
    }
  }

  // the levels of each output are combined in FP64, scaled by the output's
  // exponents (a power of two: exact) and stored, or added to C
  // per row block i: the reads of exponents and C (clamped: always in bounds and
  // without a branch, so the loads go out together; what an out-of-range output
  // reads is never stored), then the stores
  int xb[NI];   // exponents of this lane's output columns
#pragma unroll
  for (int j = 0; j < NI; ++j) xb[j] = p.eb[min(n0 + (wn * NI + j) * 16 + l16, p.N - 1)];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    double w[NI][4];
    int xa[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) xa[r] = p.ea[p.a_row0 + min(m0 + (wm * MI + i) * 16 + 4 * g + r, p.M - 1)];
    if (p.accumulate) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t m = min(m0 + (wm * MI + i) * 16 + 4 * g + r, p.M - 1);
          const int64_t n = min(n0 + (wn * NI + j) * 16 + l16, p.N - 1);
          w[j][r] = p.C[m * p.ldc + n];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        double v = 0.0;
#pragma unroll
        for (int L = S - 1; L >= 0; --L) v = v * (1.0 / 128.0) + (double)acc[L][i][j][r];
        v = ldexp(v, xa[r] + xb[j] - 12);
        w[j][r] = p.accumulate ? v + w[j][r] : v;
      }
    }
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + (wm * MI + i) * 16 + 4 * g + r, n = n0 + (wn * NI + j) * 16 + l16;
        if (m < p.M && n < p.N) p.C[m * p.ldc + n] = w[j][r];
      }
  }
}

template <int S, int NBUF, class T>
__global__ __launch_bounds__(OzShape<T>::THREADS, 2) void gemm_oz8_kernel(OzParams p) {
  if (p.status != nullptr && *p.status != 0) return;
  __shared__ __attribute__((aligned(1024))) int8_t lds[NBUF][OzLds<S, T>::STAGE];
  constexpr int BM = OzShape<T>::BM, BN = OzShape<T>::BN;
  const int wl = xcd_remap(blockIdx.x, gridDim.x);
  int tm, tn;
  oz8_decode(p, BM, BN, wl, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  if (oz8_tile_skipped(p, m0, n0, BN)) return;
  oz8_tile<S, NBUF, T>(p, m0, n0, lds);
}

// Grouped launch over the split products of many fragments (see Grouped): it
// runs reduction window `window` of every problem (k0 = window * wlen, the first
// window stores and later ones add into C; the items of problems with fewer
// windows end at once).
template <int S, int NBUF, class T>
__global__ __launch_bounds__(OzShape<T>::THREADS, 2) void gemm_oz8_grouped(Grouped<OzParams> G, int64_t window,
                                                                         int64_t wlen) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[NBUF][OzLds<S, T>::STAGE];
  constexpr int BM = OzShape<T>::BM, BN = OzShape<T>::BN;
  int f, u;
  if (!grouped_item(G, f, u)) return;
  OzParams p = G.probs[f];
  if (p.status != nullptr && *p.status != 0) return;
  p.k0 = window * wlen;
  if (p.k0 >= p.kp && window > 0) return;
  p.kc = min(wlen, p.kp - p.k0);
  p.accumulate = window > 0;
  int tm, tn;
  oz8_decode(p, BM, BN, u, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  if (oz8_tile_skipped(p, m0, n0, BN)) return;
  oz8_tile<S, NBUF, T>(p, m0, n0, lds);
}

}  // namespace rimp2
