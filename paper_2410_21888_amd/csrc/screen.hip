// Learned pair screening for the RI-MP2 fragment kernel (gfx950): pair
// features, the rigorous pair bound, and the forward/backward/Adam kernels of
// the small FP64 network declared in include/rimp2_screen.h.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/rimp2.h"
#include "../../include/rimp2_screen.h"
#include "common.hpp"

using namespace rimp2;

namespace {

// a dispatch's grid size is a 32-bit count of work-items (the network's entry
// points refuse sample counts by it, as they always have, though their launches
// have at most 1024 workgroups)
constexpr int64_t kMaxItems = 0xffffffffLL;
constexpr int H = RIMP2_MLP_HIDDEN, NIN = RIMP2_MLP_IN, NP = RIMP2_MLP_PARAMS;
constexpr int OW1 = 0, OB1 = OW1 + H * NIN, OW2 = OB1 + H, OB2 = OW2 + H * H, OW3 = OB2 + H, OB3 = OW3 + H;

__device__ __forceinline__ double sigm(double z) { return 1.0 / (1.0 + exp(-z)); }
__device__ __forceinline__ double silu(double z) { return z * sigm(z); }
__device__ __forceinline__ double dsilu(double z) {
  const double s = sigm(z);
  return s * (1.0 + z * (1.0 - s));
}

// ---- features ---------------------------------------------------------------
// N[i][P] = ||B_i[:, P]||_2: a workgroup takes 64 columns P of one i, its four
// waves every fourth row a.  HBM-bound; with one workgroup per i, 100 of them
// read B (100/600/1800, 0.86 GB) in 1.9 ms, 0.15 ms now.
__global__ __launch_bounds__(256) void colnorm_kernel(const double* B, int nvir, int naux, double* N) {
  __shared__ double sh[4][64];
  const int np = (naux + 63) / 64, i = blockIdx.x / np, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int P = (blockIdx.x - i * np) * 64 + lane;
  const double* Bi = B + (int64_t)i * nvir * naux + min(P, naux - 1);
  double s = 0.0;
#pragma unroll 8
  for (int a = w; a < nvir; a += 4) {
    const double v = Bi[(int64_t)a * naux];
    s += v * v;
  }
  sh[w][lane] = s;
  __syncthreads();
  if (w == 0 && P < naux) N[(int64_t)i * naux + P] = sqrt(((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane]);
}
// nb[i] = ||B_i||_F from N, and evmin = min eps_vir (block 0 also)
__global__ __launch_bounds__(256) void rownorm_kernel(const double* N, int naux, double* nb, const double* ev,
                                                      int nvir, double* evmin) {
  __shared__ double sh[256];
  const int i = blockIdx.x;
  double s = 0.0;
  for (int P = threadIdx.x; P < naux; P += 256) {
    const double v = N[(int64_t)i * naux + P];
    s += v * v;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) nb[i] = sqrt(sh[0]);
  if (i == 0) {
    __syncthreads();
    double mn = INFINITY;
    for (int a = threadIdx.x; a < nvir; a += 256) mn = fmin(mn, ev[a]);
    sh[threadIdx.x] = mn;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) sh[threadIdx.x] = fmin(sh[threadIdx.x], sh[threadIdx.x + w]);
      __syncthreads();
    }
    if (threadIdx.x == 0) *evmin = sh[0];
  }
}
// One thread per pair (i, j), 16 x 16 pairs a workgroup; N's rows go through
// LDS in blocks of PB columns, summed in increasing P.
constexpr int PT = 16, PB = 32;
__global__ __launch_bounds__(PT * PT) void pair_kernel(int nocc, int naux, const double* N, const double* nb,
                                                       const double* eo, const double* r, const double* evmin,
                                                       double* feat, double* bound) {
  __shared__ double Ni[PT][PB + 1], Nj[PT][PB + 1];
  const int tj = threadIdx.x % PT, ti = threadIdx.x / PT;
  const int i0 = blockIdx.y * PT, j0 = blockIdx.x * PT, i = i0 + ti, j = j0 + tj;
  double s = 0.0;
  if (bound) {
    for (int P0 = 0; P0 < naux; P0 += PB) {
      for (int q = threadIdx.x; q < PT * PB; q += PT * PT) {
        const int row = q / PB, c = q % PB, P = P0 + c;
        Ni[row][c] = P < naux ? N[(int64_t)min(i0 + row, nocc - 1) * naux + P] : 0.0;
        Nj[row][c] = P < naux ? N[(int64_t)min(j0 + row, nocc - 1) * naux + P] : 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < PB; ++c) s += Ni[ti][c] * Nj[tj][c];
      __syncthreads();
    }
  }
  if (i >= nocc || j >= nocc) return;
  const int64_t p = (int64_t)i * nocc + j;
  const double dx = r[3 * i] - r[3 * j], dy = r[3 * i + 1] - r[3 * j + 1], dz = r[3 * i + 2] - r[3 * j + 2];
  double* f = feat + 4 * p;
  f[0] = sqrt(dx * dx + dy * dy + dz * dz) / 10.0;
  f[1] = log(nb[i]);
  f[2] = log(nb[j]);
  f[3] = (eo[i] + eo[j]) / 10.0;
  if (bound) bound[p] = 3.0 * s * s / (2.0 * *evmin - eo[i] - eo[j]);
}

// ---- network ------------------------------------------------------------------
// Four waves a workgroup, blocks of SB = 16 samples.  The 64 x 64 products run
// on v_mfma_f64_16x16x4 (lane l: A[l%16][l/16], B[l/16][l%16]; register r of
// lane l: D[4r + l/16][l%16]); wave w owns the hidden units [16 w, 16 w + 16).
// Latency-bound: a block is a few microseconds of dependent steps, so the
// blocks are spread over the CUs, one workgroup each.  (A first version, one
// wave for 32 samples with a thread per hidden unit and 64-way bank conflicts
// on W2's rows, took 122 us for 4096 samples' gradient, 15 us now, and its
// reduction 35, 4 us now.)
typedef double dbl4 __attribute__((ext_vector_type(4)));
constexpr int SB = 16, MAXW = 256;   // samples per block, workgroups of a gradient launch
constexpr int LD = H + 1;            // LDS row stride (no bank conflicts down a column)

struct MlpLds {
  double X[SB][NIN], W1[H][NIN], A1[SB][LD], T[SB][LD], y[SB];
};

// Hidden layers of one block for lane (g = l/16, c = l%16) of wave w: X is in
// LDS; writes A1 = silu(Z1) to LDS.  Element r of z1 and z2 is sample 4r + g,
// unit u = 16 w + c; w2[ks] = W2[u][4 ks + g].  Ends after a barrier that makes A1 visible.
__device__ __forceinline__ void mlp_hidden(MlpLds& L, int u, int g, int c, double b1, double b2, const double (&w2)[16],
                                           double (&z1)[4], dbl4& z2) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int s = 4 * r + g;
    double z = b1;
#pragma unroll
    for (int k = 0; k < NIN; ++k) z += L.W1[u][k] * L.X[s][k];
    z1[r] = z;
    L.A1[s][u] = silu(z);
  }
  __syncthreads();
  z2 = dbl4{b2, b2, b2, b2};
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) z2 = __builtin_amdgcn_mfma_f64_16x16x4f64(L.A1[c][4 * ks + g], w2[ks], z2, 0, 0, 0);
}
// out[s] = b3 + sum_u W3[u] T[s][u] for the block's samples (T = silu(Z2)): 16
// lanes a sample, fixed order; valid in the threads with threadIdx.x % 16 == 0.
__device__ __forceinline__ double mlp_out(const MlpLds& L, const double* P) {
  const int s = threadIdx.x >> 4, q = threadIdx.x & 15;
  double o = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) o += P[OW3 + q + 16 * k] * L.T[s][q + 16 * k];
#pragma unroll
  for (int d = 8; d > 0; d >>= 1) o += __shfl_down(o, d, 16);
  return o + P[OB3];
}
// Samples s0.. of x, or of its rows idx[s] (idx not null).
__device__ __forceinline__ void mlp_load(MlpLds& L, int64_t n, int64_t s0, const double* x, const int64_t* idx) {
  for (int q = threadIdx.x; q < SB * NIN; q += 256) {
    const int64_t s = s0 + q / NIN;
    L.X[q / NIN][q % NIN] = s < n ? x[(idx ? idx[s] : s) * NIN + q % NIN] : 0.0;
  }
}

__global__ __launch_bounds__(256) void mlp_forward_kernel(int64_t n, const double* x, const double* P, double* y) {
  __shared__ MlpLds L;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, g = lane >> 4, c = lane & 15, u = 16 * w + c;
  double w2[16];
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) w2[ks] = P[OW2 + u * H + 4 * ks + g];
  L.W1[t / NIN][t % NIN] = P[OW1 + t];
  const double b1 = P[OB1 + u], b2 = P[OB2 + u];
  const int64_t nb = (n + SB - 1) / SB;
  for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
    mlp_load(L, n, b * SB, x, nullptr);
    __syncthreads();
    double z1[4];
    dbl4 z2;
    mlp_hidden(L, u, g, c, b1, b2, w2, z1, z2);
#pragma unroll
    for (int r = 0; r < 4; ++r) L.T[4 * r + g][u] = silu(z2[r]);
    __syncthreads();
    const double o = mlp_out(L, P);
    const int64_t s = b * SB + (t >> 4);
    if ((t & 15) == 0 && s < n) y[s] = o;
  }
}

// Gradient of sum_s (y - t)^2 / n (and the loss part) over the workgroup's
// blocks blockIdx.x, blockIdx.x + gridDim.x, ... -> part[blockIdx][NP + 1]
__global__ __launch_bounds__(256) void mlp_backward_kernel(int64_t n, const double* x, const double* tgt,
                                                           const int64_t* idx, const double* P, double* part) {
  __shared__ MlpLds L;
  __shared__ double gs[4][H];   // b1, b2, W3 gradients, loss and b3 (per sample slot)
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, g = lane >> 4, c = lane & 15, u = 16 * w + c;
  double w2[16], w2t[16];       // W2[u][4 ks + g], W2[4 ks + g][u]
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) {
    w2[ks] = P[OW2 + u * H + 4 * ks + g];
    w2t[ks] = P[OW2 + (4 * ks + g) * H + u];
  }
  L.W1[t / NIN][t % NIN] = P[OW1 + t];
  const double b1 = P[OB1 + u], b2 = P[OB2 + u], w3 = P[OW3 + u];
  dbl4 gw2[4];                  // gradient of W2[16 w + 4r + g][16 nb + c]
#pragma unroll
  for (int q = 0; q < 4; ++q) gw2[q] = dbl4{0.0, 0.0, 0.0, 0.0};
  double gw1 = 0.0, gb1 = 0.0, gb2 = 0.0, gw3 = 0.0, gb3 = 0.0, loss = 0.0;
  const int64_t nblk = (n + SB - 1) / SB;
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    mlp_load(L, n, b * SB, x, idx);
    __syncthreads();
    double z1[4], a2[4];
    dbl4 z2;
    mlp_hidden(L, u, g, c, b1, b2, w2, z1, z2);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a2[r] = silu(z2[r]);
      L.T[4 * r + g][u] = a2[r];
    }
    __syncthreads();
    const double o = mlp_out(L, P);
    if ((t & 15) == 0) {
      const int64_t s = b * SB + (t >> 4);
      const double res = s < n ? o - tgt[idx ? idx[s] : s] : 0.0, dy = 2.0 * res / (double)n;
      L.y[t >> 4] = dy;
      gb3 += dy;
      loss += res * res / (double)n;
    }
    __syncthreads();
    // dZ2[s][u] = dy[s] W3[u] silu'(Z2[s][u]) into T
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double dy = L.y[4 * r + g], d = dy * w3 * dsilu(z2[r]);
      gw3 += dy * a2[r];
      gb2 += d;
      L.T[4 * r + g][u] = d;
    }
    __syncthreads();
    // W2 gradient: sum_s dZ2[s][m] A1[s][n]; dA1[s][u] = sum_m dZ2[s][m] W2[m][u]
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const double a = L.T[4 * ks + g][u];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        gw2[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, L.A1[4 * ks + g][16 * q + c], gw2[q], 0, 0, 0);
    }
    dbl4 da = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) da = __builtin_amdgcn_mfma_f64_16x16x4f64(L.T[c][4 * ks + g], w2t[ks], da, 0, 0, 0);
    __syncthreads();
    // dZ1 into A1, then the W1 gradient (thread: unit t / 4, input t % 4)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double d = da[r] * dsilu(z1[r]);
      gb1 += d;
      L.A1[4 * r + g][u] = d;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < SB; ++s) gw1 += L.A1[s][t / NIN] * L.X[s][t % NIN];
    __syncthreads();
  }
  double* out = part + (int64_t)blockIdx.x * (NP + 1);
  out[OW1 + t] = gw1;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) out[OW2 + (16 * w + 4 * r + g) * H + 16 * q + c] = gw2[q][r];
  // the four lane groups' parts of unit u, in order
  auto fold = [&](double v, int at) {
    gs[g][u] = v;
    __syncthreads();
    if (g == 0) out[at + u] = ((gs[0][u] + gs[1][u]) + gs[2][u]) + gs[3][u];
    __syncthreads();
  };
  fold(gb1, OB1);
  fold(gb2, OB2);
  fold(gw3, OW3);
  if ((t & 15) == 0) { gs[0][t >> 4] = gb3; gs[1][t >> 4] = loss; }
  __syncthreads();
  if (t < 2) {
    double v = 0.0;
    for (int s = 0; s < SB; ++s) v += gs[t][s];
    out[t == 0 ? OB3 : NP] = v;
  }
}
// One Adam step of parameter q with gradient gq.
struct AdamArgs {
  double *p, *m, *v;
  double c1, c2, lr, b1, b2, eps;
};
__device__ __forceinline__ void adam_step(const AdamArgs& a, int q, double gq) {
  const double mq = a.b1 * a.m[q] + (1.0 - a.b1) * gq, vq = a.b2 * a.v[q] + (1.0 - a.b2) * gq * gq;
  a.m[q] = mq;
  a.v[q] = vq;
  a.p[q] -= a.lr * (mq / a.c1) / (sqrt(vq / a.c2) + a.eps);
}
// The gradient of parameter q, the sum over workgroups of part[w][q] in a fixed
// order (16 lanes a parameter, each every 16th workgroup, then the lanes in
// order), goes to grad[q], or (ADAM) into an Adam step; loss = part[.][NP].
template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_reduce_kernel(const double* part, int nw, double* grad, double* loss,
                                                         AdamArgs a) {
  __shared__ double sh[16][17];
  const int e = threadIdx.x & 15, l = threadIdx.x >> 4, q = blockIdx.x * 16 + e;
  double s = 0.0;
  if (q <= NP) {
#pragma unroll 8
    for (int w = l; w < nw; w += 16) s += part[(int64_t)w * (NP + 1) + q];
  }
  sh[l][e] = s;
  __syncthreads();
  if (l != 0 || q > NP) return;
  for (int k = 1; k < 16; ++k) s += sh[k][e];
  if (q == NP) *loss = s;
  else if (ADAM) adam_step(a, q, s);
  else grad[q] = s;
}
__global__ __launch_bounds__(256) void adam_kernel(const double* g, AdamArgs a) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q < NP) adam_step(a, q, g[q]);
}
__global__ __launch_bounds__(256) void log_energy_kernel(int64_t n, const double* e, double* out) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s < n) out[s] = log10(fmax(-e[s], 1e-300));
}
// Predicted energy of the pairs i < j (both orders) whose prediction is below
// thr, in a fixed order over one workgroup's threads; skip (may be null)
// receives the mask.  Latency-bound (16.9 us with 256 threads at nocc = 100, 11
// with 1024).
constexpr int MT = 1024;
__device__ __forceinline__ double mask_energy(int nocc, const double* pred, double thr, uint8_t* skip, double* sh) {
  double acc = 0.0;
  for (int64_t p = threadIdx.x; p < (int64_t)nocc * nocc; p += MT) {
    const int i = (int)(p / nocc), j = (int)(p - (int64_t)i * nocc);
    const int a = min(i, j), b = max(i, j);
    const double pr = pred[(int64_t)a * nocc + b];
    const bool sk = (a != b) && pr < thr;
    if (skip) skip[p] = sk ? 1 : 0;
    if (sk) acc += pow(10.0, pr);
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = MT / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  const double e = sh[0];
  __syncthreads();
  return e;
}
__global__ __launch_bounds__(MT) void screen_mask_kernel(int nocc, const double* pred, double thr, uint8_t* skip,
                                                         double* skipped) {
  __shared__ double sh[MT];
  const double e = mask_energy(nocc, pred, thr, skip, sh);
  if (threadIdx.x == 0) *skipped = e;
}
// The bisection of [-30, 0] for the largest threshold whose mask_energy is at
// most budget (the same in every thread).  As 60 mask launches, each read back,
// it took 2.6 ms at nocc = 100; 0.5 ms here.
__global__ __launch_bounds__(MT) void budget_threshold_kernel(int nocc, const double* pred, double budget, int iters,
                                                              double* thr) {
  __shared__ double sh[MT];
  double lo = -30.0, hi = 0.0;
  for (int it = 0; it < iters; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (mask_energy(nocc, pred, mid, nullptr, sh) <= budget) lo = mid; else hi = mid;
  }
  if (threadIdx.x == 0) *thr = lo;
}

size_t align_up(size_t x) { return (x + 255) / 256 * 256; }
int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

extern "C" {

size_t rimp2_features_workspace_size(int32_t nocc, int32_t naux) {
  return align_up(8 * (size_t)nocc * naux) + align_up(8 * (size_t)nocc) + 256;
}

int rimp2_pair_features(int32_t nocc, int32_t nvir, int32_t naux, const double* B, const double* eps_occ,
                        const double* eps_vir, const double* centroids, double* features, double* bound,
                        void* workspace, size_t workspace_bytes, void* stream) {
  if (nocc < 1 || nvir < 1 || naux < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  if (!B || !eps_occ || !eps_vir || !centroids || !features || !workspace)
    return fail(RIMP2_EINVAL, "null pointer argument");
  if (workspace_bytes < rimp2_features_workspace_size(nocc, naux)) return fail(RIMP2_ENOMEM, "workspace too small");
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  double* N = (double*)ws;
  double* nb = (double*)(ws + align_up(8 * (size_t)nocc * naux));
  double* evmin = (double*)(ws + align_up(8 * (size_t)nocc * naux) + align_up(8 * (size_t)nocc));
  hipLaunchKernelGGL(colnorm_kernel, dim3((unsigned)(nocc * cdiv(naux, 64))), dim3(256), 0, st, B, nvir, naux, N);
  hipLaunchKernelGGL(rownorm_kernel, dim3(nocc), dim3(256), 0, st, N, naux, nb, eps_vir, nvir, evmin);
  const unsigned pt = (unsigned)cdiv(nocc, PT);
  hipLaunchKernelGGL(pair_kernel, dim3(pt, pt), dim3(PT * PT), 0, st, nocc, naux, N, nb, eps_occ, centroids, evmin,
                     features, bound);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

int rimp2_mlp_forward(int64_t n, const double* x, const double* params, double* y, void* stream) {
  if (n < 0 || (n > 0 && (!x || !params || !y))) return fail(RIMP2_EINVAL, "bad forward arguments");
  if (n == 0) return RIMP2_OK;
  if (cdiv(n, 64) * 64 > kMaxItems) return fail(RIMP2_EINVAL, "n = %lld is too large for one launch", (long long)n);
  const int64_t nwg = std::min<int64_t>(cdiv(n, SB), 4 * MAXW);
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((unsigned)nwg), dim3(256), 0, (hipStream_t)stream, n, x, params, y);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

size_t rimp2_mlp_workspace_size(int64_t n) {
  return align_up(8 * (size_t)std::min<int64_t>(cdiv(n, SB), MAXW) * (NP + 1));
}

int rimp2_mlp_loss_grad(int64_t n, const double* x, const double* target, const double* params, double* loss,
                        double* grad, void* workspace, size_t workspace_bytes, void* stream) {
  if (n < 1 || !x || !target || !params || !loss || !grad || !workspace) return fail(RIMP2_EINVAL, "bad arguments");
  if (workspace_bytes < rimp2_mlp_workspace_size(n)) return fail(RIMP2_ENOMEM, "workspace too small");
  hipStream_t st = (hipStream_t)stream;
  if (cdiv(n, 32) * 64 > kMaxItems) return fail(RIMP2_EINVAL, "n = %lld is too large for one launch", (long long)n);
  const int nw = (int)std::min<int64_t>(cdiv(n, SB), MAXW);
  hipLaunchKernelGGL(mlp_backward_kernel, dim3((unsigned)nw), dim3(256), 0, st, n, x, target, (const int64_t*)nullptr,
                     params, (double*)workspace);
  hipLaunchKernelGGL(mlp_reduce_kernel<false>, dim3((unsigned)cdiv(NP + 1, 16)), dim3(256), 0, st,
                     (const double*)workspace, nw, grad, loss, AdamArgs{});
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

int rimp2_mlp_adam(const double* grad, double* params, double* m, double* v, int64_t step, double lr, double beta1,
                   double beta2, double eps, void* stream) {
  if (!grad || !params || !m || !v || step < 1) return fail(RIMP2_EINVAL, "bad Adam arguments");
  const AdamArgs a{params, m, v, 1.0 - pow(beta1, (double)step), 1.0 - pow(beta2, (double)step), lr, beta1, beta2, eps};
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)cdiv(NP, 256)), dim3(256), 0, (hipStream_t)stream, grad, a);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

int rimp2_mlp_fit(int64_t n, int32_t steps, const double* x, const double* target, const int64_t* idx, double* params,
                  double* m, double* v, int64_t first_step, double lr, double beta1, double beta2, double eps,
                  double* loss, void* workspace, size_t workspace_bytes, void* stream) {
  if (n < 1 || steps < 0 || !x || !target || !idx || !params || !m || !v || first_step < 1 || !loss || !workspace)
    return fail(RIMP2_EINVAL, "bad fit arguments");
  if (workspace_bytes < rimp2_mlp_workspace_size(n)) return fail(RIMP2_ENOMEM, "workspace too small");
  if (cdiv(n, 32) * 64 > kMaxItems) return fail(RIMP2_EINVAL, "n = %lld is too large for one launch", (long long)n);
  hipStream_t st = (hipStream_t)stream;
  const int nw = (int)std::min<int64_t>(cdiv(n, SB), MAXW);
  for (int32_t k = 0; k < steps; ++k) {
    const double t = (double)(first_step + k);
    const AdamArgs a{params, m, v, 1.0 - pow(beta1, t), 1.0 - pow(beta2, t), lr, beta1, beta2, eps};
    hipLaunchKernelGGL(mlp_backward_kernel, dim3((unsigned)nw), dim3(256), 0, st, n, x, target, idx + k * n,
                       (const double*)params, (double*)workspace);
    hipLaunchKernelGGL(mlp_reduce_kernel<true>, dim3((unsigned)cdiv(NP + 1, 16)), dim3(256), 0, st,
                       (const double*)workspace, nw, (double*)nullptr, loss, a);
    HIP_TRY(hipGetLastError());
  }
  return RIMP2_OK;
}

int rimp2_log_energy(int64_t n, const double* e, double* out, void* stream) {
  if (n < 0 || (n > 0 && (!e || !out))) return fail(RIMP2_EINVAL, "bad arguments");
  if (n == 0) return RIMP2_OK;
  if (cdiv(n, 256) * 256 > kMaxItems) return fail(RIMP2_EINVAL, "n = %lld is too large for one launch", (long long)n);
  hipLaunchKernelGGL(log_energy_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, (hipStream_t)stream, n, e, out);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

int rimp2_screen_mask(int32_t nocc, const double* pred, double threshold_log10, uint8_t* skip, double* skipped_energy,
                      void* stream) {
  if (nocc < 1 || !pred || !skip || !skipped_energy) return fail(RIMP2_EINVAL, "bad arguments");
  hipLaunchKernelGGL(screen_mask_kernel, dim3(1), dim3(MT), 0, (hipStream_t)stream, nocc, pred, threshold_log10,
                     skip, skipped_energy);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

int rimp2_budget_threshold(int32_t nocc, const double* pred, double budget_Eh, int32_t iters, double* threshold_log10,
                           void* stream) {
  if (nocc < 1 || iters < 0 || !pred || !threshold_log10) return fail(RIMP2_EINVAL, "bad arguments");
  hipLaunchKernelGGL(budget_threshold_kernel, dim3(1), dim3(MT), 0, (hipStream_t)stream, nocc, pred, budget_Eh, iters,
                     threshold_log10);
  HIP_TRY(hipGetLastError());
  return RIMP2_OK;
}

}  // extern "C"
