// Host side of the C ABI declared in include/rimp2.h: argument checks,
// workspace planning and the launch sequence of the RI-MP2 fragment kernel.
//
// Path for one fragment (all on the caller's stream, no host synchronisation):
//   gap check -> for each slab group of g occupied orbitals k0..k0+g-1:
//     (ia|jb) slab GEMM  V[(k,a),(j,b)] = sum_P B[k,a,P] B[j,b,P]       (Eq. MP2_ints)
//     amplitude pass     X = V/D, T = 2X - X^T, e_kj = sum T V           (Appendix, X)
//     Gamma GEMM         Gamma[k,a,P] = sum_(j,b) T[k,a,j,b] B[j,b,P]    (Appendix, Gamma)
//     P_ab GEMM          P_ab += sum_(k,j,c) T[k,a,j,c] X[k,b,j,c]       (Appendix, D_ab)
//     P_ij GEMM          P_ij -= sum_(k,a,b) T[k,a,i,b] X[k,a,j,b]       (Appendix, D_ij)
//   -> compensated E = sum e_ij.
// Slab layout [kk][a][j][b]: the (ia|jb) and Gamma GEMMs see plain row-major
// matrices; P_ab and P_ij read the same slabs with a two-level reduction index.
// P_ab and P_ij are symmetric, so their GEMMs compute upper-triangular tiles
// and write each also transposed.  For P_ij every slab's contribution is
// symmetric.  For P_ab only the sum over both orders of each pair is
// (T_kj X_kj^T + T_jk X_jk^T = 2(X X^T + X^T X) - (X X + (X X)^T) with
// X = X_kj), so the mirrored partials of a slab group are not its own lower
// triangle; but the mirror of a sum is the sum of the mirrors, and the total
// over all groups is symmetric, so the accumulated lower triangle is exact.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "../../include/rimp2.h"
#include "../../include/rimp2_gradient.h"
#include "common.hpp"
#include "gemm_f64.hpp"
#include "kernels.hpp"
#include "split_int8.hpp"
#include "batch.hpp"

using namespace rimp2;

// Scratch space of rimp2_fragment_noalloc: one array per GPU, part of the
// library's code object, so each device that runs the library holds its own
// copy until the process ends.  Host code never uses the name `scratch` as an
// address: rimp2_fragment_noalloc takes the device address from
// hipGetSymbolAddress once per device (with that device current) and passes
// it to the kernels as the workspace.
constexpr size_t kScratchBytes = (size_t)RIMP2_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {


// ---- kernel timing -------------------------------------------------------
enum Role { R_GAP, R_INTS, R_AMP, R_GAMMA, R_PAB, R_PIJ, R_REDUCE, R_ESUM, R_STATUS, R_SPLIT, R_INTS8, R_GAMMA8,
            R_GAMMA_T, R_GAMMA_AO, R_LTERM, R_RESPONSE, R_GAMMA_T8, R_GAMMA_METRIC, R_TAIL, R_NROLES };
const char* const kRoleName[R_NROLES] = {"gap_check",  "ints_gemm",     "amplitude",  "gamma_gemm",
                                         "pab_gemm",   "pij_gemm",      "splitk_reduce", "energy_sum",
                                         "status_copy", "digit_split", "ints_oz8",   "gamma_oz8",
                                         "gamma_t_gemm", "gamma_ao_gemm", "l_terms_gemm", "response",
                                         "gamma_t_oz8", "gamma_metric", "small_gemms"};
struct TraceRec {
  int role;
  hipEvent_t e0, e1;
  double af, ef, ab;
};
struct Tracer {
  std::mutex mu;
  bool on = false;
  std::vector<TraceRec> recs;
  std::vector<hipEvent_t> pool;
};
Tracer& tracer() {
  static Tracer t;
  return t;
}

// Set while this thread runs rimp2_fragment_noalloc: no events are created
// or recorded (that entry point allocates nothing).
thread_local bool t_noalloc = false;

// Launches `launch` on stream st; while timing is on, brackets it with events.
template <class F>
int traced(int role, double af, double ef, double ab, hipStream_t st, F&& launch) {
  Tracer& T = tracer();
  hipEvent_t ev[2] = {nullptr, nullptr};
  bool on;
  {
    std::lock_guard<std::mutex> lk(T.mu);
    on = T.on && !t_noalloc;
    for (int i = 0; on && i < 2; ++i) {
      if (!T.pool.empty()) {
        ev[i] = T.pool.back();
        T.pool.pop_back();
      } else {
        HIP_TRY(hipEventCreate(&ev[i]));
      }
    }
  }
  if (on) HIP_TRY(hipEventRecord(ev[0], st));
  launch();
  HIP_TRY(hipGetLastError());
  if (on) {
    HIP_TRY(hipEventRecord(ev[1], st));
    std::lock_guard<std::mutex> lk(T.mu);
    T.recs.push_back(TraceRec{role, ev[0], ev[1], af, ef, ab});
  }
  return RIMP2_OK;
}

constexpr size_t kAlign = 256;
constexpr int kBK = 16;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// A dispatch's grid size is a 32-bit count of work-items (workgroups x 256 here).
constexpr int64_t kMaxWorkgroups = 0xffffffffLL / 256;
int check_grid(int64_t wgs, const char* what) {
  if (wgs <= 0 || wgs > kMaxWorkgroups)
    return fail(RIMP2_EINVAL, "%s grid of %lld workgroups is out of range (1..%lld)", what, (long long)wgs,
                (long long)kMaxWorkgroups);
  return RIMP2_OK;
}
int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- tile shape and split-K factor of a GEMM ------------------------------
// Measured on the NT kernel (us): with w workgroups resident on a CU, one
// chunk of kBK reduction indices takes a + b w, up to `resident` workgroups
// (tile 128: 2.35, 4.05; tile 96: 1.45, 2.45, 3.45; tile 64: 0.80, 1.25, 1.70,
// 2.15; tile 32: 0.39, 0.54, 0.71, .., 1.44 with 8); filling the pipeline and
// writing the tile take about kTileFill more.  Large tiles reach the higher
// rate (66 TFLOP/s at 512 tiles of 128, 62 at 1024 of 64), small ones fill the
// chip sooner (256 tiles of 64 run at 42, 64 tiles of 128 at 14).
struct TileCost {
  int bm;
  double a, b;
  int resident;
};
constexpr TileCost kTileCost[4] = {{128, 0.65, 1.70, 2}, {96, 0.47, 0.99, 3}, {64, 0.35, 0.45, 4}, {32, 0.24, 0.15, 8}};
constexpr double kTileFill = 5.0, kCUs = 256.0;
// Split-K costs one launch that reads the partials at about 3.5 TB/s (their
// writes run under the other workgroups' MFMAs).
constexpr double kReduceUs = 5.0, kReduceBytesPerUs = 3.5e6;
constexpr int64_t kMaxSplits = 1024;

double gemm_us(const TileCost& t, int64_t tiles, int64_t K, int64_t splits) {
  const double chunks = (double)cdiv(cdiv(K, splits), kBK);
  const int64_t w = cdiv(tiles * splits, (int64_t)kCUs), rounds = w / t.resident, rest = w % t.resident;
  return rounds * (kTileFill + chunks * (t.a + t.b * t.resident)) +
         (rest ? kTileFill + chunks * (t.a + t.b * rest) : 0.0);
}

// A smaller tile has to be estimated 3% faster than the larger one: it stages
// more operand bytes per multiply-add, which the table (operands in the
// caches) does not hold ((ia|jb) of 16/1800/6000: 79 ms with tiles of 128, 84
// with 64, estimated alike).
constexpr double kSmallerTile = 0.97;

// What the table does not hold of long reductions.  Tiles that live long drift
// apart, the operand panels they share fall out of the caches, and one sum of
// many terms rounds more than the sum of several: splits of at most kSplitLen,
// as far as kLongSplits go (P_ab of 6 orbitals' slabs of 200/1800, 2.2M long:
// 122 ms in 4 splits, 116 in 64; Gamma rows of 200/1800/6000, up to 360000 long,
// in 2 to 4 or 2 to 11: 673 ms in both, a sampled row 5.4e-15 or 1.6e-15 off).
// And operands that no cache holds reach the tiles at 8 TB/s of staged bytes at
// most (P_ij of the same slabs: 36 ms with tiles of 32, which the table prefers,
// 30 with 64).
constexpr int64_t kSplitLen = 32768, kLongSplits = 64;
constexpr double kCacheBytes = 256e6, kStageBytesPerUs = 8e6;

struct GemmChoice {
  int bm;           // square tile
  int64_t splits;   // split-K factor
};

const TileCost& tile_cost(int bm) {
  const TileCost* t = kTileCost;
  while (t->bm != bm) ++t;
  return *t;
}
int64_t square_tiles(int64_t M, int64_t N, int bm, bool tri) {
  const int64_t tm = cdiv(M, bm), tn = cdiv(N, bm);
  return tri ? tm * (tm + 1) / 2 : tm * tn;
}
// Estimate of an M x N x K product (`batch` of them in one launch) with choice
// c, its reduction included.
double product_us(int64_t M, int64_t N, int64_t K, bool tri, const GemmChoice& c, int64_t batch = 1) {
  const int64_t tiles = square_tiles(M, N, c.bm, tri) * batch;
  const bool streamed = 8.0 * (M + N) * K > kCacheBytes;
  const double staged = streamed ? 16.0 * tiles * c.bm * K / kStageBytesPerUs : 0.0;
  const double reduce = c.splits > 1 ? kReduceUs + 8.0 * (c.splits + 1) * M * N / kReduceBytesPerUs : 0.0;
  return std::max(gemm_us(tile_cost(c.bm), tiles, K, c.splits), staged) + reduce;
}

// The tile (one of `bms`, 0 ends the list) and split-K factor (at most smax)
// with the smallest estimate for an M x N x K product (tri: upper-triangular
// tiles).  Split factors tried: 1 to 4 (they fill a ragged last round of many
// tiles) and those that give every CU 1 to 8 workgroups.  With one tile shape
// and 64 splits of 2048 at most, P_ij of nocc = 61 ran on 64 workgroups (8.0 ms,
// 1.6 ms now) and Gamma of 20/100/400 on 64 (288 us, 90 us now).
// batch: that many such products in one launch.
GemmChoice choose_gemm(int64_t M, int64_t N, int64_t K, bool tri, const int* bms, int64_t smax = kMaxSplits,
                       int64_t batch = 1) {
  GemmChoice best{0, 1};
  double best_us = 0.0;
  smax = std::max<int64_t>(1, std::min<int64_t>(smax, K / (4 * kBK)));
  const int64_t smin = std::min<int64_t>({smax, kLongSplits, cdiv(K, kSplitLen)});
  for (; *bms; ++bms) {
    const int64_t tiles = square_tiles(M, N, *bms, tri) * batch;
    for (int64_t w = 1, last = 0; w <= 12; ++w) {
      const int64_t s = std::max<int64_t>(smin, std::min<int64_t>(smax, w <= 4 ? w : (w - 4) * (int64_t)kCUs / tiles));
      if (s == last) continue;
      last = s;
      const double us = product_us(M, N, K, tri, GemmChoice{*bms, s}, batch);
      if (best.bm == 0 || us < best_us * (*bms < best.bm ? kSmallerTile : 1.0)) {
        best_us = us;
        best = GemmChoice{*bms, s};
      }
    }
  }
  return best;
}
// Tile shapes instantiated for each product.
constexpr int kIntsTiles[] = {128, 64, 0}, kGammaTiles[] = {128, 64, 0}, kPabTiles[] = {128, 96, 64, 0},
              kPijTiles[] = {128, 96, 64, 32, 0}, kLtermTiles[] = {128, 64, 0}, kAoTiles[] = {128, 64, 0};

// Split-K factor of a grouped P_ab or P_ij product of K reduction indices: a
// wave's fragments fill the chip together, so the splits only keep its items
// short (klen).  With 64 splits whatever the length, the P_ij items of nocc =
// 60, nvir = 300 were 84000 long, and the launch waited for them.
constexpr int64_t kGroupedPab = 4096, kGroupedPij = 2048;
int64_t grouped_splits(int64_t K, int64_t klen) {
  return std::max<int64_t>(1, std::min<int64_t>(kMaxSplits, cdiv(K, klen)));
}
// Estimate of a grouped product's `tiles` of side bm, on a chip that the wave's
// other products keep full: P_ij of nocc = 30 costs a third with tiles of 32
// what it costs with 64, P_ab of nvir = 300 two thirds with 64 of 128.
double grouped_cost(int bm, int64_t tiles) {
  const TileCost& c = tile_cost(bm);
  return tiles * (c.a + c.b * c.resident) / c.resident;
}

struct Plan {
  int64_t nocc, nvir, naux;
  bool gamma, density;
  bool sym;                  // Gamma without P (FP64): (ia|jb) over pairs j >= k only
  bool g_fixed;              // slab_group given by the caller
  double budget;             // slab budget in bytes (slab_group == 0)
  bool split;                // RIMP2_SPLIT_INT8
  bool autotune;             // in-situ tile choice of the FP64 GEMMs
  bool general;              // FP64 GEMMs take the general loader only
  double part_bytes;         // cap of the split-K partial sums of each product
  int sv, sg;                // digits per operand of (ia|jb) and of Gamma
  int64_t kpv, kpg;          // padded reduction lengths of the split products
  size_t off_dbv, off_ev, off_dbg, off_eg, off_cmax, off_dt, off_et;
  // symmetric path with split products: digits of the transposed T blocks and
  // of the group's B rows (the transposed-block product), per group
  size_t off_dtt, off_ett, off_cmt, off_dbk, off_ebk;
  int64_t g;                 // occupied orbitals per slab group
  GemmChoice c_ab, c_ij, c_gam;   // tile and split-K factor of P_ab, P_ij and (ordered path) Gamma
  size_t off_status, off_V, off_T, off_e, off_pab, off_pij, off_gam, off_epart, total;
};

// Workgroups per pair block of an amplitude launch over `pairs` pair blocks
// of nvir x nvir: enough for about 8 waves of the resident workgroups, at
// most kAmpSplitMax and at most one per tile pair.
constexpr int64_t kAmpSplitMax = 64;
// Tile side of an amplitude launch (HBM-bound).  Rows of 64 doubles leave half
// as many partly written cache lines as rows of 32: E+Gamma of 97/485/1746
// 18.4 -> 8.8 ms (of that about 7 for X, which only P_ab and P_ij read and is
// no longer written without them), with P of 61/305/1098 2.83 -> 2.24 ms, of
// 37/211/733 384 -> 336 us.  A pass that writes nothing is faster with the
// small tile's 8 workgroups a CU (100/600: 4.6 ms against 6.6), and so are few
// virtual orbitals, which a tile of 64 would pad.
int64_t amp_tile(int64_t nvir, bool energy_only) { return !energy_only && nvir >= 192 ? 64 : 32; }
int64_t amp_splits(int64_t pairs, int64_t nvir, bool energy_only) {
  const int64_t t = amp_tile(nvir, energy_only), nt = cdiv(nvir, t), npt = nt * (nt + 1) / 2;
  const int64_t w = (6144 + pairs - 1) / pairs;
  return std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(w, kAmpSplitMax), npt));
}

// Occupied orbitals in the slab group that starts at k0.  The ordered path
// uses one size g for every group.  The symmetric path's slabs hold the
// columns j >= k0 only, so without a caller-given size each group takes the
// most orbitals whose two slabs fit the budget, and later groups grow.
int64_t group_at(const Plan& P, int64_t k0) {
  if (!P.sym || P.g_fixed) return std::min<int64_t>(P.g, P.nocc - k0);
  const double per_k = 2.0 * 8.0 * (double)(P.nocc - k0) * P.nvir * P.nvir;
  // at most as many rows as one reduction launch covers (its grid counts
  // work-items in 32 bits)
  const int64_t red = std::max<int64_t>(1, kMaxWorkgroups * 256 / (P.nvir * P.naux));
  return std::max<int64_t>(1, std::min<int64_t>({(int64_t)(P.budget / per_k), P.nocc - k0, red}));
}

// Largest split-K factor of an M x N product: its partial sums stay within the
// plan's cap, and one launch covers its reduction.
int64_t split_cap(const Plan& P, int64_t M, int64_t N) {
  if (cdiv(M * N, 256) > kMaxWorkgroups) return 1;
  return std::max<int64_t>(1, (int64_t)std::min((double)kMaxSplits, P.part_bytes / (8.0 * M * N)));
}

// Tile and split-K factor of the symmetric path's Gamma GEMM over the row
// blocks of a group of gc orbitals starting at k0 (reduction over the pairs
// j >= k0).
GemmChoice sym_gamma_choice(const Plan& P, int64_t k0, int64_t gc) {
  const int64_t M = gc * P.nvir;
  return choose_gemm(M, P.naux, (P.nocc - k0) * P.nvir, false, kGammaTiles, split_cap(P, M, P.naux));
}

// Each product's split-K partial sums take at most this share of the slab budget,
// or kPartFloor where that is more (kSplitLen's splits of a whole Gamma would take
// 14 GB beside the slabs of 279/5366/7205, and P_ab's as much; the splits that
// fill the chip stay below the floor).
constexpr double kPartShare = 1.0 / 8.0, kPartFloor = 2.0 * (1ull << 30);

// grouped: the fragment runs in a batch wave (whole slab, no split amplitude
// partials).  part_bytes: a tighter cap of each product's partial sums.
constexpr double kAnyPartBytes = 1e30;
int make_plan(int64_t nocc, int64_t nvir, int64_t naux, bool gamma, bool density, const rimp2_opts* o, Plan* p,
              bool grouped = false, double part_bytes = kAnyPartBytes) {
  if (nocc < 1 || nvir < 1 || naux < 1 || nocc > (1 << 20) || nvir > (1 << 24) || naux > (1 << 24))
    return fail(RIMP2_EINVAL, "sizes must be >= 1 (nocc=%lld nvir=%lld naux=%lld)", (long long)nocc,
                (long long)nvir, (long long)naux);
  if ((double)nocc * nvir * naux >= 4.6e18)
    return fail(RIMP2_EINVAL, "nocc*nvir*naux too large");
  if (o && o->precision != RIMP2_FP64 && o->precision != RIMP2_SPLIT_INT8)
    return fail(RIMP2_ENOTSUP, "precision %d is not supported", o->precision);
  p->nocc = nocc; p->nvir = nvir; p->naux = naux; p->gamma = gamma; p->density = density;
  p->split = o && o->precision == RIMP2_SPLIT_INT8;
  p->autotune = o && o->autotune != 0;
  if (o && (o->gemm_loader < 0 || o->gemm_loader > 1))
    return fail(RIMP2_EINVAL, "gemm_loader must be 0 or 1 (got %d)", o->gemm_loader);
  p->general = o && o->gemm_loader == 1;
  p->sv = (o && o->split_slices) ? o->split_slices : 7;
  p->sg = (o && o->split_slices_gamma) ? o->split_slices_gamma : 5;
  if (p->split && (p->sv < 3 || p->sv > 7 || p->sg < 3 || p->sg > 7))
    return fail(RIMP2_EINVAL, "split digit counts must be 3..7 (got %d and %d)", p->sv, p->sg);
  p->kpv = cdiv(naux, 64) * 64;
  p->kpg = cdiv(nocc * nvir, 64) * 64;
  const bool need_T = gamma || density;
  const double slab_per_k = (need_T ? 2.0 : 1.0) * 8.0 * (double)nocc * nvir * nvir;
  p->sym = gamma && !density && !grouped;
  p->g_fixed = o && o->slab_group > 0;
  p->budget = (o && o->slab_budget_bytes) ? (double)o->slab_budget_bytes : 64.0 * (1ull << 30);
  int64_t g;
  if (p->g_fixed) {
    g = std::min<int64_t>(o->slab_group, nocc);
  } else {
    g = (int64_t)(p->budget / slab_per_k);
    g = std::max<int64_t>(1, std::min<int64_t>(g, nocc));
  }
  p->g = g;
  p->part_bytes = std::min(part_bytes, std::max(kPartFloor, kPartShare * p->budget));
  p->c_ab = p->c_ij = p->c_gam = GemmChoice{0, 0};
  if (density && grouped) {
    p->c_ab.splits = grouped_splits(nocc * nocc * nvir, kGroupedPab);   // (the wave's lists choose the tiles)
    p->c_ij.splits = grouped_splits(nocc * nvir * nvir, kGroupedPij);
  } else if (density) {
    p->c_ab = choose_gemm(nvir, nvir, g * nocc * nvir, true, kPabTiles, split_cap(*p, nvir, nvir));
    p->c_ij = choose_gemm(nocc, nocc, g * nvir * nvir, true, kPijTiles, split_cap(*p, nocc, nocc));
  }
  if (gamma)
    p->c_gam = choose_gemm(g * nvir, naux, nocc * nvir, false, kGammaTiles,
                           grouped ? 1 : split_cap(*p, g * nvir, naux));
  // slab elements (g x ncols pair blocks) and Gamma split partials of the
  // largest group
  double slab_elems = (double)g * nocc * nvir * nvir, gam_part = (double)p->c_gam.splits * g * nvir * naux;
  if (p->sym) {
    slab_elems = gam_part = 0.0;
    for (int64_t k0 = 0; k0 < nocc;) {
      const int64_t gc = group_at(*p, k0), s = sym_gamma_choice(*p, k0, gc).splits;
      slab_elems = std::max(slab_elems, (double)gc * (nocc - k0) * nvir * nvir);
      if (s > 1) gam_part = std::max(gam_part, (double)s * gc * nvir * naux);
      k0 += gc;
    }
  }
  size_t off = 0;
  p->off_status = off; off = align_up(off + 64);
  p->off_V = off; off = align_up(off + (size_t)(8.0 * slab_elems));
  p->off_T = off; if (need_T) off = align_up(off + (size_t)(8.0 * slab_elems));
  p->off_e = off; off = align_up(off + 8 * (size_t)nocc * nocc);
  p->off_pab = off; if (density) off = align_up(off + 8 * (size_t)p->c_ab.splits * nvir * nvir);
  p->off_pij = off; if (density) off = align_up(off + 8 * (size_t)p->c_ij.splits * nocc * nocc);
  p->off_gam = off;
  // (grouped fragments run their Gamma GEMM without split-K: no partials)
  if (gamma && !p->split && !grouped && (p->sym || p->c_gam.splits > 1)) off = align_up(off + (size_t)(8.0 * gam_part));
  p->off_epart = off;
  if (!grouped) {  // largest partial array of the amplitude launches (see run_fragment)
    const bool eonly = !(gamma || density);
    int64_t most = 0;
    for (int64_t k0 = 0; k0 < nocc;) {
      const int64_t gc = group_at(*p, k0);
      const int64_t pairs = gc * ((eonly || p->sym) ? nocc - k0 : nocc);
      const int64_t W = amp_splits(pairs, nvir, eonly);
      if (W > 1) most = std::max(most, pairs * W);
      k0 += gc;
    }
    off = align_up(off + 16 * (size_t)most);
  }
  p->off_dbv = p->off_ev = p->off_dbg = p->off_eg = p->off_cmax = p->off_dt = p->off_et = off;
  p->off_dtt = p->off_ett = p->off_cmt = p->off_dbk = p->off_ebk = off;
  if (p->split) {
    const int64_t L = nocc * nvir;
    p->off_dbv = off; off = align_up(off + (size_t)p->sv * L * p->kpv);
    p->off_ev = off; off = align_up(off + 4 * (size_t)L);
    if (gamma && !p->sym) {
      p->off_dbg = off; off = align_up(off + (size_t)p->sg * naux * p->kpg);
      p->off_eg = off; off = align_up(off + 4 * (size_t)naux);
      p->off_cmax = off; off = align_up(off + 8 * (size_t)naux);
      p->off_dt = off; off = align_up(off + (size_t)p->sg * g * nvir * p->kpg);
      p->off_et = off; off = align_up(off + 4 * (size_t)g * nvir);
    } else if (gamma) {
      // per group at k0 (gc orbitals, Lc = (nocc - k0) nvir columns): T row
      // digits [S][gc nvir][pad(Lc)], B column digits of rows >= k0 nvir
      // [S][naux][pad(Lc)], T column digits of the later columns
      // [S][(nocc - k0 - gc) nvir][pad(gc nvir)], B column digits of the
      // group's rows [S][naux][pad(gc nvir)]; sized for the largest group
      double dt = 0, dbg = 0, dtt = 0, dbk = 0, rows = 0, cols = 0;
      int64_t grid = 0;   // largest digit-split grid (split_cols: 32 x 32 tiles)
      for (int64_t k0 = 0; k0 < nocc;) {
        const int64_t gc = group_at(*p, k0), kc = cdiv((nocc - k0) * nvir, 64) * 64, kg = cdiv(gc * nvir, 64) * 64;
        grid = std::max({grid, cdiv(kc, 32) * cdiv(naux, 32), cdiv(kg, 32) * cdiv((nocc - k0 - gc) * nvir, 32)});
        dt = std::max(dt, (double)gc * nvir * kc);
        dbg = std::max(dbg, (double)naux * kc);
        dtt = std::max(dtt, (double)(nocc - k0 - gc) * nvir * kg);
        dbk = std::max(dbk, (double)naux * kg);
        rows = std::max(rows, (double)gc * nvir);
        cols = std::max(cols, (double)(nocc - k0 - gc) * nvir);
        k0 += gc;
      }
      p->off_dbg = off; off = align_up(off + (size_t)(p->sg * dbg));
      p->off_eg = off; off = align_up(off + 4 * (size_t)naux);
      p->off_cmax = off; off = align_up(off + 8 * (size_t)naux);
      p->off_dt = off; off = align_up(off + (size_t)(p->sg * dt));
      p->off_et = off; off = align_up(off + (size_t)(4.0 * rows));
      p->off_dtt = off; off = align_up(off + (size_t)(p->sg * dtt));
      p->off_ett = off; off = align_up(off + (size_t)(4.0 * cols));
      p->off_cmt = off; off = align_up(off + (size_t)(8.0 * cols));
      p->off_dbk = off; off = align_up(off + (size_t)(p->sg * dbk));
      p->off_ebk = off; off = align_up(off + 4 * (size_t)naux);
      if (int rc = check_grid(grid, "digit split")) return rc;
    }
  }
  p->total = off;
  int rc;
  if (gamma && p->c_gam.splits > 1 && !p->sym && (rc = check_grid(cdiv(g * nvir * naux, 256), "reduction"))) return rc;
  if (p->sym && p->g_fixed && (rc = check_grid(cdiv(g * nvir * naux, 256), "reduction"))) return rc;
  if (p->split && ((rc = check_grid(nocc * nvir, "digit split")) || (rc = check_grid(cdiv(p->kpg, 32), "digit split"))))
    return rc;
  return RIMP2_OK;
}

// 16-byte loads need 16-byte aligned bases and even strides (so every pair of
// reduction indices, and every pair of N-contiguous columns, is aligned).
bool kop_vec(const KOperand& o, int64_t K) {
  const bool plain = o.kdiv >= K;
  return (uintptr_t)o.base % 16 == 0 && o.rs % 2 == 0 && (plain || (o.kdiv % 2 == 0 && o.ks1 % 2 == 0));
}

// 16-byte loads for a whole GEMM (the split length is a multiple of kBK, so
// even).  amc: A is M-contiguous (pairs of rows, like an N-contiguous B).
bool gemm_vec(const GemmParams& gp, bool nc, bool amc = false) {
  const bool a = amc ? ((uintptr_t)gp.Am.base % 16 == 0 && gp.Am.ld % 2 == 0) : kop_vec(gp.A, gp.K);
  if (gp.batch > 1 && (gp.batch_a % 2 || gp.batch_b % 2)) return false;
  return a && (nc ? ((uintptr_t)gp.Bn.base % 16 == 0 && gp.Bn.ld % 2 == 0) : kop_vec(gp.Bk, gp.K));
}

// The kernels' FAST level of a GEMM (0: the general loader).  It needs runs of
// the K operands at least one chunk long (a chunk crosses at most one run
// boundary), and of an M-contiguous A (N-contiguous B) an even number of rows
// (columns) or a whole tile of side bm to read pairs from.  2 when a K operand's
// runs are even and can end inside a chunk, 3 when they are odd; alignment, odd
// strides and odd lengths do not matter.  (Odd sizes took the general loader with 8-byte loads: Gamma of
// nocc = 97, nvir = 485, naux = 1746 ran at 57 TFLOP/s, and at 64 here.)
int fast_level(const GemmParams& gp, int bm, bool nc, bool amc = false) {
  auto runs = [&](const KOperand& o) { return o.kdiv >= gp.K || o.kdiv >= kBK; };
  auto pairs = [&](int64_t n) { return n % 2 == 0 || n >= bm; };
  auto level = [&](const KOperand& o) { return o.kdiv >= gp.K || o.kdiv % kBK == 0 ? 1 : o.kdiv % 2 == 0 ? 2 : 3; };
  if (!(gp.kchunk % kBK == 0 && (amc ? pairs(gp.M) : runs(gp.A)) && (nc ? pairs(gp.N) : runs(gp.Bk)))) return 0;
  return std::max(amc ? 1 : level(gp.A), nc ? 1 : level(gp.Bk));
}

// Output tiles (of one split) a GEMM launches workgroups for: the upper
// triangle, the tiles a pair_upper launch keeps (decode_pair_tile), or all.
int64_t gemm_tiles(const GemmParams& gp, int64_t bm, int64_t bn, bool tri) {
  if (tri) return (int64_t)gp.tiles_m * (gp.tiles_m + 1) / 2;
  int64_t n = (int64_t)gp.tiles_m * gp.tiles_n;
  if (gp.pair_upper)
    for (int64_t m = 0; m < gp.tiles_m; m += gp.group_m) {
      int64_t from;
      n -= std::min<int64_t>(gp.group_m, gp.tiles_m - m) *
           pair_cols_skipped(gp.skip_k0 + m * bm / gp.skip_nvir, gp.skip_j0, gp.pair_lo, gp.skip_nvir, bn, gp.tiles_n,
                             &from);
    }
  return n;
}

template <int BM, int BN, bool NC, int ROLE, bool TRI>
int launch_gemm(GemmParams gp, hipStream_t st, int role, double af, double ab, bool general) {
  gp.tiles_m = (int32_t)cdiv(gp.M, BM);
  gp.tiles_n = (int32_t)cdiv(gp.N, BN);
  gp.group_m = 8;
  if (gp.kchunk <= 0) gp.kchunk = gp.K;
  gp.kchunk = cdiv(gp.kchunk, kBK) * kBK;
  gp.splits = (int32_t)cdiv(gp.K, gp.kchunk);
  if (TRI && (gp.M != gp.N || BM != BN)) return fail(RIMP2_EINVAL, "triangular GEMM needs a square tile grid");
  if (gp.pair_upper && gp.splits != 1) return fail(RIMP2_EINVAL, "pair_upper GEMM without split-K only");
  if (gp.batch > 1 && (gp.splits != 1 || !role_batched(ROLE)))
    return fail(RIMP2_EINVAL, "batched GEMM without split-K only");
  const int64_t tiles = gemm_tiles(gp, BM, BN, TRI), nwg = tiles * std::max(gp.splits, gp.batch);
  gp.pair_map = gp.pair_upper && tiles < (int64_t)gp.tiles_m * gp.tiles_n;
  if (int rc = check_grid(nwg, "GEMM")) return rc;
  constexpr bool AMC = role_a_mcontig(ROLE);
  if (AMC && gp.splits != 1) return fail(RIMP2_EINVAL, "M-contiguous GEMM without split-K only");
  if (gp.accumulate && (TRI || gp.splits != 1)) return fail(RIMP2_EINVAL, "accumulating GEMM without split-K only");
  const bool vec = gemm_vec(gp, NC, AMC);
  double ef = (TRI ? 0.5 * (1.0 + 1.0 / gp.tiles_m) : 1.0) * 2.0 * (double)gp.M * gp.N * gp.K;
  if (gp.pair_upper) {  // tiles not skipped: those with a pair j >= k or j < pair_lo (see tile_screened)
    int64_t kept = 0;
    for (int64_t tm = 0; tm < gp.tiles_m; ++tm) {
      const int64_t k_lo = gp.skip_k0 + tm * BM / gp.skip_nvir;
      const int64_t below = std::max<int64_t>(0, cdiv((k_lo - gp.skip_j0) * gp.skip_nvir - BN + 1, BN));
      const int64_t from = std::max<int64_t>(0, cdiv((gp.pair_lo - gp.skip_j0) * gp.skip_nvir, BN));
      kept += gp.tiles_n - std::max<int64_t>(0, std::min<int64_t>(below, gp.tiles_n) - from);
    }
    ef *= (double)kept / ((double)gp.tiles_m * gp.tiles_n);
  }
  const int fast = general ? 0 : fast_level(gp, BM, NC, AMC);
  const int64_t grid = nwg + (ROLE == ROLE_INTS && gp.gap_status ? 1 : 0);
  // the roles whose K operands have runs
  constexpr bool RUNS = ROLE == ROLE_PAB || ROLE == ROLE_PIJ || ROLE == ROLE_LTERM;
  if (!RUNS && fast > 1) return fail(RIMP2_EINVAL, "GEMM role %d with a two-level reduction", ROLE);
  return traced(role, af, ef, ab, st, [&] {
    if (fast == 1)
      hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, kBK, NC, ROLE, true, TRI, 1>), dim3((unsigned)grid), dim3(256), 0,
                         st, gp);
    else if (RUNS && fast == 2)
      hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, kBK, NC, ROLE, true, TRI, RUNS ? 2 : 0>), dim3((unsigned)grid),
                         dim3(256), 0, st, gp);
    else if (RUNS && fast == 3)
      hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, kBK, NC, ROLE, true, TRI, RUNS ? 3 : 0>), dim3((unsigned)grid),
                         dim3(256), 0, st, gp);
    else if (vec)
      hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, kBK, NC, ROLE, true, TRI>), dim3((unsigned)grid), dim3(256), 0, st, gp);
    else
      hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, kBK, NC, ROLE, false, TRI>), dim3((unsigned)grid), dim3(256), 0, st, gp);
  });
}


// Sizes and pair fields of the (ia|jb) product of the slab group of gc orbitals
// at k0: rows (kk, a) from k0, columns (j, b) over all orbitals, or (energy only
// and the symmetric Gamma path, where pairs j < k come from their mirror) over
// j >= k0.  Pairs with both orbitals in the group: blocks (k, j < k) are not
// computed and the amplitude pass forms them from their transposes.
GemmParams ints_product(const Plan& P, int64_t k0, int64_t gc) {
  GemmParams gp{};
  const int64_t j0 = (P.sym || !(P.gamma || P.density)) ? k0 : 0;
  gp.M = gc * P.nvir; gp.N = (P.nocc - j0) * P.nvir; gp.K = P.naux; gp.kchunk = P.naux;
  gp.skip_nvir = (int32_t)P.nvir; gp.skip_k0 = (int32_t)k0; gp.skip_j0 = (int32_t)j0; gp.skip_nocc = (int32_t)P.nocc;
  gp.pair_upper = 1;
  gp.pair_lo = (int32_t)k0;
  return gp;
}
// Estimate of an (ia|jb) product over the tiles it keeps (no split-K: the
// amplitude pass needs whole sums), and the tile with the smallest.
double ints_us(GemmParams gp, int bm) {
  // (raster groups of one row: exactly the tiles that are not skipped)
  gp.tiles_m = (int32_t)cdiv(gp.M, bm); gp.tiles_n = (int32_t)cdiv(gp.N, bm); gp.group_m = 1;
  return gemm_us(tile_cost(bm), gemm_tiles(gp, bm, bm, false), gp.K, 1);
}
int ints_tile(const GemmParams& gp) {
  int best = 0;
  double best_us = 0.0;
  for (const int* t = kIntsTiles; *t; ++t) {
    const double us = ints_us(gp, *t);
    if (best == 0 || us < best_us * kSmallerTile) {
      best = *t;
      best_us = us;
    }
  }
  return best;
}

// Estimate of a plan's products and of the launches of its slab groups, which
// compares plans of one fragment (the amplitude passes, alike in all of them,
// are left out; split products count as FP64 ones).
constexpr double kGroupUs = 20.0;   // five or six launches a group
double plan_us(const Plan& P) {
  double us = 0.0;
  for (int64_t k0 = 0, gc = 0; k0 < P.nocc; k0 += gc) {
    gc = group_at(P, k0);
    const GemmParams gp = ints_product(P, k0, gc);
    us += kGroupUs + ints_us(gp, ints_tile(gp));
    if (P.gamma) {
      GemmChoice c = P.sym ? sym_gamma_choice(P, k0, gc) : P.c_gam;
      if (P.split) c.splits = 1;
      us += product_us(gp.M, P.naux, gp.N, false, c);
    }
    if (const int64_t later = (P.nocc - k0 - gc) * P.nvir; P.sym && later > 0)   // the transposed blocks' product
      us += product_us(later, P.naux, gp.M, false, choose_gemm(later, P.naux, gp.M, false, kGammaTiles, 1));
    if (P.density)
      us += product_us(P.nvir, P.nvir, gc * P.nocc * P.nvir, true, P.c_ab) +
            product_us(P.nocc, P.nocc, gc * P.nvir * P.nvir, true, P.c_ij);
  }
  return us;
}

// ---- in-situ tile autotuner (Sec. "GEMM runtime auto-tuning") -------------
// Candidates are output tile shapes; the split length (and with it every
// element's summation order) comes from the plan and is the same for all.
struct TileShape {
  int bm, bn;
};
constexpr int kTuneVars = 4, kTuneTrials = 2;

// Candidate tile shapes of a role's GEMM: bm0 (the plan's choice) first.
int tile_candidates(int role, int bm0, TileShape* c) {
  const int* t = role == R_PAB ? kPabTiles : role == R_PIJ ? kPijTiles : kGammaTiles;
  int n = 0;
  c[n++] = {bm0, bm0};
  for (; *t; ++t)
    if (*t != bm0) c[n++] = {*t, *t};
  return n;
}

// The GEMM of `role` with square tiles of side bm (one of its candidates).
int launch_role(int role, int bm, const GemmParams& gp, hipStream_t st, double af, double ab, bool general) {
  switch (role) {
    case R_INTS:
      return bm == 64 ? launch_gemm<64, 64, false, ROLE_INTS, false>(gp, st, role, af, ab, general)
                      : launch_gemm<128, 128, false, ROLE_INTS, false>(gp, st, role, af, ab, general);
    case R_GAMMA:
      return bm == 64 ? launch_gemm<64, 64, true, ROLE_GAMMA, false>(gp, st, role, af, ab, general)
                      : launch_gemm<128, 128, true, ROLE_GAMMA, false>(gp, st, role, af, ab, general);
    case R_GAMMA_T:
      return bm == 64 ? launch_gemm<64, 64, true, ROLE_GAMMA_T, false>(gp, st, role, af, ab, general)
                      : launch_gemm<128, 128, true, ROLE_GAMMA_T, false>(gp, st, role, af, ab, general);
    case R_PAB:
      return bm == 64   ? launch_gemm<64, 64, false, ROLE_PAB, true>(gp, st, role, af, ab, general)
             : bm == 96 ? launch_gemm<96, 96, false, ROLE_PAB, true>(gp, st, role, af, ab, general)
                        : launch_gemm<128, 128, false, ROLE_PAB, true>(gp, st, role, af, ab, general);
    case R_PIJ:
      return bm == 32    ? launch_gemm<32, 32, false, ROLE_PIJ, true>(gp, st, role, af, ab, general)
             : bm == 96  ? launch_gemm<96, 96, false, ROLE_PIJ, true>(gp, st, role, af, ab, general)
             : bm == 128 ? launch_gemm<128, 128, false, ROLE_PIJ, true>(gp, st, role, af, ab, general)
                         : launch_gemm<64, 64, false, ROLE_PIJ, true>(gp, st, role, af, ab, general);
    default:
      return fail(RIMP2_EINVAL, "no GEMM for role %d", role);
  }
}

// bm0: the plan's own tile, candidate 0.  Two plans of one fragment (other slab
// groups) can give a shape different tiles, and an entry's trials and decision
// name candidates by their place.  vec: 16-byte loads (+ 2: the general loader
// only); 2 with `general` telling the loaders apart for a grouped launch.
struct TuneKey {
  int dev, role, vec, general, bm0;
  int64_t M, N, K, kchunk;
  bool operator<(const TuneKey& o) const {
    return std::tie(dev, role, vec, general, bm0, M, N, K, kchunk) <
           std::tie(o.dev, o.role, o.vec, o.general, o.bm0, o.M, o.N, o.K, o.kchunk);
  }
};
struct TunePending {
  int var;
  hipEvent_t e0, e1;
};
struct TuneEntry {
  int nvar = 0, best = -1;
  TileShape cand[kTuneVars] = {};
  int launched[kTuneVars] = {}, timed[kTuneVars] = {};
  double min_ms[kTuneVars] = {};
  int64_t uses = 0;
  std::vector<TunePending> pend;
};
struct Tuner {
  std::mutex mu;
  std::map<TuneKey, TuneEntry> tab;
  std::vector<hipEvent_t> pool;
};
Tuner& tuner() {
  static Tuner t;
  return t;
}

// Folds the completed trials of e into its timings without blocking, and
// decides once every candidate has kTuneTrials of them: the fastest (by its
// fastest trial), unless it beats the default by less than 2%.  Caller holds
// the tuner lock.
void tune_poll(Tuner& U, TuneEntry& e) {
  for (size_t i = 0; i < e.pend.size();) {
    const TunePending q = e.pend[i];
    const hipError_t r = hipEventQuery(q.e1);
    if (r == hipErrorNotReady) {
      (void)hipGetLastError();
      ++i;
      continue;
    }
    float ms = 0.f;
    if (r == hipSuccess && hipEventElapsedTime(&ms, q.e0, q.e1) == hipSuccess) {
      e.min_ms[q.var] = e.timed[q.var] ? std::min(e.min_ms[q.var], (double)ms) : (double)ms;
      e.timed[q.var] += 1;
    } else {
      (void)hipGetLastError();
      e.launched[q.var] -= 1;  // trial lost: it is run again
    }
    U.pool.push_back(q.e0);
    U.pool.push_back(q.e1);
    e.pend[i] = e.pend.back();
    e.pend.pop_back();
  }
  if (e.best >= 0) return;
  int best = 0;
  for (int v = 0; v < e.nvar; ++v) {
    if (e.timed[v] < kTuneTrials) return;
    if (e.min_ms[v] < e.min_ms[best] && e.min_ms[v] < 0.98 * e.min_ms[0]) best = v;
  }
  e.best = best;
}

// Runs launch(v) for the candidate v of `key` that the tuner picks (see
// tune_poll): the decided one, else a candidate still owed a trial (bracketed
// by events on st, unless st is capturing), else candidate 0.
template <class F>
int tuned(const TuneKey& key, int nvar, const TileShape* cand, hipStream_t st, F&& launch) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
    (void)hipGetLastError();
    cs = hipStreamCaptureStatusActive;
  }
  const bool capturing = cs != hipStreamCaptureStatusNone;
  Tuner& U = tuner();
  int v = 0;
  bool trial = false;
  hipEvent_t ev[2] = {nullptr, nullptr};
  {
    std::lock_guard<std::mutex> lk(U.mu);
    TuneEntry& e = U.tab[key];
    if (e.nvar == 0) {
      e.nvar = nvar;
      for (int i = 0; i < nvar; ++i) e.cand[i] = cand[i];
    }
    e.uses += 1;
    if (!capturing) tune_poll(U, e);
    if (e.best >= 0) {
      v = e.best;
    } else if (!capturing) {
      for (int i = 0; i < nvar && !trial; ++i)
        if (e.launched[i] < kTuneTrials) { v = i; trial = true; }
    }
    for (int i = 0; trial && i < 2; ++i) {
      if (!U.pool.empty()) {
        ev[i] = U.pool.back();
        U.pool.pop_back();
      } else if (hipEventCreate(&ev[i]) != hipSuccess) {
        (void)hipGetLastError();
        if (i == 1) U.pool.push_back(ev[0]);
        trial = false;
        v = 0;
      }
    }
    if (trial) e.launched[v] += 1;
  }
  const bool rec0 = trial && hipEventRecord(ev[0], st) == hipSuccess;
  const int rc = launch(v);
  if (trial) {
    const bool ok = rec0 && rc == RIMP2_OK && hipEventRecord(ev[1], st) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    std::lock_guard<std::mutex> lk(U.mu);
    TuneEntry& e = U.tab[key];
    if (ok) {
      e.pend.push_back(TunePending{v, ev[0], ev[1]});
    } else {
      e.launched[v] -= 1;
      U.pool.push_back(ev[0]);
      U.pool.push_back(ev[1]);
    }
  }
  return rc;
}

// Launches the GEMM of `role` with tiles of side bm0, or with autotuning the
// shape's tuned candidate.
int launch_tuned(int role, int bm0, const GemmParams& gp, bool autotune, bool general, hipStream_t st, double af,
                 double ab) {
  if (!autotune) return launch_role(role, bm0, gp, st, af, ab, general);
  TileShape c[kTuneVars];
  const int nvar = tile_candidates(role, bm0, c);
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  // the key's loader field: 16-byte loads, and whether the fast loaders are allowed
  const int loader = (gemm_vec(gp, role == R_GAMMA || role == R_GAMMA_T, role == R_GAMMA_T) ? 1 : 0) + (general ? 2 : 0);
  const TuneKey key{dev, role, loader, 0, bm0, gp.M, gp.N, gp.K, gp.kchunk};
  return tuned(key, nvar, c, st, [&](int v) { return launch_role(role, c[v].bm, gp, st, af, ab, general); });
}


template <int S>
void launch_split_rows(const double* X, int64_t rows, int64_t K, int64_t ld, int8_t* D, int64_t kp, int32_t* e,
                       const int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(split_rows_kernel<S>, dim3((unsigned)rows), dim3(256), 0, st, X, rows, K, ld, D, kp, e, status);
}
template <int S>
void launch_split_cols(const double* X, int64_t K, int64_t N, int64_t ld, const unsigned long long* cmax, int8_t* D,
                       int64_t kp, int32_t* e, const int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(split_cols_kernel<S>, dim3((unsigned)cdiv(kp, 32), (unsigned)cdiv(N, 32)), dim3(256), 0, st, X, K,
                     N, ld, cmax, D, kp, e, status);
}
// Output tiles a split-product launch holds workgroups for (as gemm_tiles).
int64_t oz8_tiles(const OzParams& op, int bm, int bn) {
  GemmParams gp{};
  gp.tiles_m = op.tiles_m; gp.tiles_n = op.tiles_n; gp.group_m = op.group_m;
  gp.pair_upper = op.pair_nvir > 0; gp.skip_nvir = op.pair_nvir; gp.skip_k0 = op.pair_k0; gp.skip_j0 = op.pair_j0;
  gp.pair_lo = op.pair_lo;
  return gemm_tiles(gp, bm, bn, false);
}
// Outputs' worth of 64 x 64 tiles at which the 128 x 128 tile of at most 5
// digits (OzWide) computes one, measured 2.5 against 2.1 POP/s.
constexpr double kOzWideRate = 1.2;
// Tile side of a split product with S digits: 128 where its rate outweighs its
// padding and it gives every CU a workgroup or more (8000 x 720, 378 tiles of
// 128: 0.260 ms against 0.267).
int oz8_side(int S, double tiles64, double tiles128) {
  return S <= 5 && tiles128 >= 256 && 4.0 * tiles128 < kOzWideRate * tiles64 ? 128 : 64;
}
template <int S>
void launch_oz8(OzParams op, int side, bool windowed, hipStream_t st) {
  const int64_t nwg = oz8_tiles(op, side, side);
  if (S <= 5 && side == 128)
    hipLaunchKernelGGL((gemm_oz8_kernel<S <= 5 ? S : 5, 2, OzWide>), dim3((unsigned)nwg), dim3(512), 0, st, op);
  // one LDS stage (two workgroups per CU) unless a windowed product with at
  // most 5 digits, where the double-buffered stage (still two per CU) was faster
  else if (windowed && S <= 5)
    hipLaunchKernelGGL((gemm_oz8_kernel<S <= 5 ? S : 5, 2, OzSmall>), dim3((unsigned)nwg), dim3(256), 0, st, op);
  else
    hipLaunchKernelGGL((gemm_oz8_kernel<S, 1, OzSmall>), dim3((unsigned)nwg), dim3(256), 0, st, op);
}
#define RIMP2_SWITCH_S(S, CALL)                                   \
  switch (S) {                                                    \
    case 3: { constexpr int SS = 3; CALL; } break;                \
    case 4: { constexpr int SS = 4; CALL; } break;                \
    case 5: { constexpr int SS = 5; CALL; } break;                \
    case 6: { constexpr int SS = 6; CALL; } break;                \
    default: { constexpr int SS = 7; CALL; } break;               \
  }

__global__ void zero_u64_kernel(unsigned long long* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

// A reduction longer than kOzWindowMax runs in windows of kOzWindow, one
// launch each in stream order, every later window adding into C, with a
// narrower raster (4 row tiles per group).  The tiles of one launch then
// stream digit panels short enough for the caches they share: over the whole
// 360000-long reduction of the Gamma product the launch fetched more than its
// staging bytes from beyond the L2, and the windows made the product about
// 1.7x faster (windows of 5632: 1.6x).
constexpr int64_t kOzWindow = 2816, kOzWindowMax = 8192;
static_assert(kOzWindowMax <= kOzMaxK, "INT32 levels");

// C[m, n] (m < M, n < N) from split digits; A rows start at a_row0.
// acc0: the first window adds into C too (C already holds a partial sum).
// pairs: null, or the pair fields of an (ia|jb) launch (OzParams).
struct OzPairs {
  int64_t nvir, k0, j0, lo;
};
int run_oz8(int S, const int8_t* A, int64_t a_slice, int64_t a_row0, const int32_t* ea, const int8_t* B,
            int64_t b_slice, const int32_t* eb, int64_t M, int64_t N, int64_t kp, double* C, int64_t ldc,
            const int32_t* status, int role, double af, double ab, hipStream_t st, int acc0 = 0,
            const OzPairs* pairs = nullptr) {
  OzParams op{};
  op.M = M; op.N = N; op.kp = kp;
  op.A = A; op.a_slice = a_slice; op.a_row0 = a_row0;
  op.B = B; op.b_slice = b_slice; op.ea = ea; op.eb = eb;
  op.C = C; op.ldc = ldc;
  const bool windowed = kp > kOzWindowMax;
  const int side = oz8_side(S, (double)cdiv(M, 64) * cdiv(N, 64), (double)cdiv(M, 128) * cdiv(N, 128));
  op.tiles_m = (int32_t)cdiv(M, side); op.tiles_n = (int32_t)cdiv(N, side); op.group_m = windowed && side == 64 ? 4 : 8;
  op.status = status;
  if (pairs) {
    op.pair_nvir = (int32_t)pairs->nvir; op.pair_k0 = (int32_t)pairs->k0; op.pair_j0 = (int32_t)pairs->j0;
    op.pair_lo = (int32_t)pairs->lo;
  }
  const int64_t nwg = oz8_tiles(op, side, side);
  op.pair_map = nwg < (int64_t)op.tiles_m * op.tiles_n;
  if (int rc = check_grid(nwg * (side / 64), "split GEMM")) return rc;
  const double ef = 2.0 * (double)M * N * kp * ((double)nwg / ((double)op.tiles_m * op.tiles_n));
  const int64_t kc = windowed ? kOzWindow : kp;
  for (int64_t k0 = 0;; k0 += kc) {
    op.k0 = k0;
    op.kc = std::min(kc, kp - k0);
    op.accumulate = (k0 > 0 || acc0) ? 1 : 0;
    const double fr = kp > 0 ? (double)op.kc / (double)kp : 1.0;
    if (int rc = traced(role, af * fr, ef * fr, ab * fr, st,
                        [&] { RIMP2_SWITCH_S(S, launch_oz8<SS>(op, side, windowed, st)); }))
      return rc;
    if (k0 + kc >= kp) return RIMP2_OK;
  }
}

KOperand kop(const double* base, int64_t rs, int64_t kdiv, int64_t ks1) { return KOperand{base, rs, kdiv, ks1}; }

// tiles, splits and group size of a GEMM, as launch_gemm sets them, but raster
// groups of one row for (ia|jb): a group of 8 also keeps tiles that only some of
// its rows need, and their workgroups, which end at once, fall unevenly on the
// CUs of a grouped launch (24 of 40/200/720: 19.6 ms with groups of 8, 18.3 with
// one; persistent workgroups that passed such tiles over: 18.5)
int64_t finalize_gemm(GemmParams& gp, int BM, int BN, bool tri) {
  gp.tiles_m = (int32_t)cdiv(gp.M, BM);
  gp.tiles_n = (int32_t)cdiv(gp.N, BN);
  gp.group_m = gp.pair_upper ? 1 : 8;
  if (gp.kchunk <= 0) gp.kchunk = gp.K;
  gp.kchunk = cdiv(gp.kchunk, kBK) * kBK;
  gp.splits = (int32_t)cdiv(gp.K, gp.kchunk);
  const int64_t tiles = gemm_tiles(gp, BM, BN, tri);
  gp.pair_map = gp.pair_upper && tiles < (int64_t)gp.tiles_m * gp.tiles_n;
  return tiles * gp.splits;
}

int launch_finish(const FinishParams& f, hipStream_t st) {
  if (f.n > 1 && f.first[f.n] >= kMaxWorkgroups) {   // more than one launch covers: the first reduction by itself
    FinishParams a = f, b = f;
    a.n = 1;
    a.E = nullptr;
    b.n = f.n - 1;
    for (int i = 0; i < b.n; ++i) {
      b.r[i] = f.r[i + 1];
      b.first[i + 1] = f.first[i + 2] - f.first[1];
    }
    if (int rc = launch_finish(a, st)) return rc;
    return launch_finish(b, st);
  }
  const int64_t grid = f.first[f.n] + (f.E ? 1 : 0);
  double bytes = f.E ? 8.0 * f.count : 0.0;
  for (int i = 0; i < f.n; ++i) bytes += 8.0 * (f.r[i].splits + 1 + f.r[i].accumulate) * f.r[i].M * f.r[i].N;
  return traced(f.n ? R_REDUCE : R_ESUM, 0, 0, bytes, st,
                [&] { hipLaunchKernelGGL(finish_kernel, dim3((unsigned)grid), dim3(256), 0, st, f); });
}

// Loader level (2 or 3) of gemm_f64_tail for a fragment's Gamma, P_ab and P_ij
// products, 0: separate launches.  One launch where the plan gives all of them
// small tiles (no product fills the chip by itself with large ones); the
// general loader and the autotuner's trials run apart.
int tail_level(const Plan& P, GemmParams gg, GemmParams ga, GemmParams gi) {
  if (P.autotune || P.general || P.c_gam.bm != 64 || P.c_ab.bm != 64 || P.c_ij.bm != 32) return 0;
  for (GemmParams* p : {&gg, &ga, &gi}) p->kchunk = cdiv(p->kchunk, kBK) * kBK;
  const int fg = fast_level(gg, 64, true), fa = fast_level(ga, 64, false), fi = fast_level(gi, 32, false);
  return fg && fa && fi ? std::max({2, fa, fi}) : 0;
}

int launch_tail(int level, const GemmParams& gg, const GemmParams& ga, const GemmParams& gi, double af, double ab,
                hipStream_t st) {
  TailParams t{gg, ga, gi, 0, 0};
  t.n_gam = (int32_t)finalize_gemm(t.gam, 64, 64, false);
  t.n_ab = (int32_t)finalize_gemm(t.ab, 64, 64, true);
  const int64_t grid = t.n_gam + t.n_ab + finalize_gemm(t.ij, 32, 32, true);
  if (int rc = check_grid(grid, "small GEMMs")) return rc;
  return traced(R_TAIL, af, af, ab, st, [&] {
    if (level == 3)
      hipLaunchKernelGGL(gemm_f64_tail<3>, dim3((unsigned)grid), dim3(256), 0, st, t);
    else
      hipLaunchKernelGGL(gemm_f64_tail<2>, dim3((unsigned)grid), dim3(256), 0, st, t);
  });
}

// Estimate of a first (ia|jb) product up to which the gap check is one more of
// its workgroups instead of a launch before it.  The launch costs 4 to 5 us (of
// 31 at 5/25/90, of 184 at 20/100/400, with products of 9 and 68); a fragment
// that the check rejects pays for the product, so a long one waits for the check.
constexpr double kFoldGapUs = 100.0;

// Enqueue the whole path for one fragment.  Pointers already validated.
int run_fragment(const Plan& P, const double* B, const double* eo, const double* ev, double* E, double* Gam,
                 double* Pij, double* Pab, double* e_user, char* ws, const uint8_t* skip, hipStream_t st) {
  const int64_t nocc = P.nocc, nvir = P.nvir, naux = P.naux, L = nocc * nvir;
  const double o = (double)nocc, v = (double)nvir, x = (double)naux;
  int32_t* status = (int32_t*)(ws + P.off_status);
  double* V = (double*)(ws + P.off_V);
  double* T = (double*)(ws + P.off_T);
  double* ep = e_user ? e_user : (double*)(ws + P.off_e);
  int rc;
  bool fold_gap = false;   // the gap check runs inside the first (ia|jb) launch
  if (!P.split) {
    const GemmParams first = ints_product(P, 0, group_at(P, 0));
    fold_gap = ints_us(first, ints_tile(first)) <= kFoldGapUs;
  }
  if (!fold_gap && (rc = traced(R_GAP, 0, 0, 8.0 * (o + v), st, [&] {
         hipLaunchKernelGGL(gap_check_kernel, dim3(1), dim3(256), 0, st, eo, (int)nocc, ev, (int)nvir, status);
       })))
    return rc;
  const bool energy_only = !(P.gamma || P.density);
  int8_t* dbv = (int8_t*)(ws + P.off_dbv);
  int32_t* exv = (int32_t*)(ws + P.off_ev);
  int8_t* dbg = (int8_t*)(ws + P.off_dbg);
  int32_t* exg = (int32_t*)(ws + P.off_eg);
  int8_t* dt = (int8_t*)(ws + P.off_dt);
  int32_t* ext = (int32_t*)(ws + P.off_et);
  if (P.split) {
    // digits of every B row (both operands of the (ia|jb) products)
    if ((rc = traced(R_SPLIT, 0, 0, 8.0 * L * naux + (double)P.sv * L * P.kpv, st, [&] {
           RIMP2_SWITCH_S(P.sv, launch_split_rows<SS>(B, L, naux, naux, dbv, P.kpv, exv, status, st));
         })))
      return rc;
    if (P.gamma && !P.sym) {
      // column-scaled, transposed digits of B as the [(j,b)][P] operand of Gamma
      // (the symmetric path splits the rows each group needs, per group)
      unsigned long long* cmax = (unsigned long long*)(ws + P.off_cmax);
      if ((rc = traced(R_SPLIT, 0, 0, 8.0 * naux, st, [&] {
             hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)cdiv(naux, 256)), dim3(256), 0, st, cmax, naux);
           })))
        return rc;
      if ((rc = traced(R_SPLIT, 0, 0, 8.0 * L * naux, st, [&] {
             hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)cdiv(naux, 256), (unsigned)cdiv(L, 1024)), dim3(256), 0,
                                st, B, L, naux, naux, cmax, status);
           })))
        return rc;
      if ((rc = traced(R_SPLIT, 0, 0, 8.0 * L * naux + (double)P.sg * naux * P.kpg, st, [&] {
             RIMP2_SWITCH_S(P.sg, launch_split_cols<SS>(B, L, naux, naux, cmax, dbg, P.kpg, exg, status, st));
           })))
        return rc;
    }
  }
  FinishParams fin{};
  fin.e = ep; fin.count = nocc * nocc; fin.E = E; fin.status = status;
  // queues a split-K reduction of the group for its finish launch
  auto reduce = [&](double* out, const double* W, int64_t M, int64_t N, int64_t splits, double alpha, int acc) {
    fin.r[fin.n] = ReduceDesc{out, W, status, N, N, M * N, M, N, alpha, (int32_t)splits, acc};
    fin.first[fin.n + 1] = fin.first[fin.n] + (int32_t)reduce_blocks(M * N, splits);
    ++fin.n;
  };
  for (int64_t k0 = 0, gc = 0; k0 < nocc; k0 += gc) {
    gc = group_at(P, k0);
    GemmParams gp = ints_product(P, k0, gc);
    const int64_t j0 = gp.skip_j0, ncols = nocc - j0, Lc = ncols * nvir;
    const double g = (double)gc, slab = 8.0 * g * (double)ncols * v * v;
    {
      gp.A = kop(B + k0 * nvir * naux, naux, INT64_MAX, 0);
      gp.Bk = kop(B + j0 * nvir * naux, naux, INT64_MAX, 0);
      gp.C = V; gp.ldc = Lc; gp.split_stride = 0; gp.status = status;
      gp.skip = skip;
      if (k0 == 0 && fold_gap) {
        gp.status = nullptr;
        gp.gap_status = status; gp.gap_eo = eo; gp.gap_ev = ev;
        gp.gap_nocc = (int32_t)nocc; gp.gap_nvir = (int32_t)nvir;
      }
      // algorithmic FLOPs: unordered pairs whose first orbital is in the group
      // (energy only: exactly the pairs (k, j >= k) computed; otherwise the
      // unordered-pair share of the ordered pairs computed)
      const double npairs = (energy_only || P.sym) ? g * o - (g * (double)k0 + g * (g - 1.0) / 2.0)
                                                   : g * o * (o + 1.0) / (2.0 * o);
      const double af = 2.0 * v * v * x * npairs;
      if (P.split) {
        // digit sums are exact and symmetric in the two operands, so the blocks
        // the amplitude pass takes from their transposes are bit for bit those
        // a product would give; leaving them out halves the product of a
        // one-slab fragment (MFMA and staging bound; 40/900/3000, 7 digits:
        // 100 -> 52 ms)
        const OzPairs pairs{nvir, k0, j0, k0};
        if ((rc = run_oz8(P.sv, dbv, L * P.kpv, k0 * nvir, exv, dbv + j0 * nvir * P.kpv, L * P.kpv, exv + j0 * nvir,
                          gc * nvir, Lc, P.kpv, V, Lc, status, R_INTS8, af,
                          (double)P.sv * (g * v + o * v) * P.kpv + slab, st, 0, &pairs)))
          return rc;
      } else if ((rc = launch_tuned(R_INTS, ints_tile(gp), gp, P.autotune, P.general, st, af,
                                    8.0 * (g + o) * v * x + slab))) {
        return rc;
      }
    }
    {
      const int64_t W = amp_splits(gc * ncols, nvir, energy_only);
      double* epart = (double*)(ws + P.off_epart);
      const int sym = energy_only ? 1 : (P.sym ? 3 : 2);
      if ((rc = check_grid(gc * ncols * W, "amplitude"))) return rc;
      if ((rc = traced(R_AMP, 0, 0, energy_only ? slab : (P.density ? 3.0 : 2.0) * slab, st, [&] {
             const int wx = P.density ? 1 : 0, eo_only = energy_only ? 1 : 0;
             if (amp_tile(nvir, energy_only) == 64)
               hipLaunchKernelGGL((amplitude_kernel<64, 512>), dim3((unsigned)(gc * ncols * W)), dim3(512), 0, st, V, T,
                                  eo, ev, (int)nocc, (int)nvir, (int)k0, (int)j0, (int)ncols, sym, (int)gc, eo_only, wx,
                                  skip, ep, (int)W, epart, status);
             else
               hipLaunchKernelGGL((amplitude_kernel<32, 256>), dim3((unsigned)(gc * ncols * W)), dim3(256), 0, st, V, T,
                                  eo, ev, (int)nocc, (int)nvir, (int)k0, (int)j0, (int)ncols, sym, (int)gc, eo_only, wx,
                                  skip, ep, (int)W, epart, status);
             if (W > 1)
               hipLaunchKernelGGL(pair_energy_reduce_kernel, dim3((unsigned)cdiv(gc * ncols, 256)), dim3(256), 0, st,
                                  (const double*)epart, (int)W, (int)nocc, (int)k0, (int)j0, (int)gc, (int)ncols, sym,
                                  ep, status);
           })))
        return rc;
    }
    if (P.gamma && P.sym) {
      // Gamma rows of the group: Gamma[k] (+)= sum over pairs (k, j >= k0) of T_kj B_j
      const GemmChoice cg = sym_gamma_choice(P, k0, gc);
      const int acc = k0 > 0 ? 1 : 0;   // earlier groups' transposed blocks are already in these rows
      GemmParams gp{};
      gp.M = gc * nvir; gp.N = naux; gp.K = Lc;
      gp.kchunk = cdiv(Lc, cg.splits);
      gp.A = kop(T, Lc, INT64_MAX, 0);
      gp.Bn = NOperand{B + j0 * nvir * naux, naux};
      gp.status = status;
      double* out = Gam + k0 * nvir * naux;
      const double c = (double)ncols;
      const double af = 2.0 * g * v * x * c * v, ab = slab + 8.0 * c * v * x + 8.0 * (1 + acc) * g * v * x;
      const int64_t splits = cdiv(Lc, cdiv(cdiv(Lc, cg.splits), kBK) * kBK);
      if (P.split) {
        // row product: T rows of the group (reduction over (j >= k0, b)) times
        // the column digits of B's rows j >= k0
        const int64_t kc = cdiv(Lc, 64) * 64;
        unsigned long long* cmax = (unsigned long long*)(ws + P.off_cmax);
        const double* Bj = B + j0 * nvir * naux;
        if ((rc = traced(R_SPLIT, 0, 0, slab + 16.0 * c * v * x + (double)P.sg * (g * v + x) * kc, st, [&] {
               RIMP2_SWITCH_S(P.sg, launch_split_rows<SS>(T, gc * nvir, Lc, Lc, dt, kc, ext, status, st));
               hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)cdiv(naux, 256)), dim3(256), 0, st, cmax, naux);
               hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)cdiv(naux, 256), (unsigned)cdiv(Lc, 1024)), dim3(256),
                                  0, st, Bj, Lc, naux, naux, cmax, status);
               RIMP2_SWITCH_S(P.sg, launch_split_cols<SS>(Bj, Lc, naux, naux, cmax, dbg, kc, exg, status, st));
             })))
          return rc;
        if ((rc = run_oz8(P.sg, dt, gc * nvir * kc, 0, ext, dbg, naux * kc, exg, gc * nvir, naux, kc, out, naux,
                          status, R_GAMMA8, af, (double)P.sg * (g * v + x) * kc + 8.0 * (1 + acc) * g * v * x, st,
                          acc)))
          return rc;
      } else if (splits > 1) {
        double* W = (double*)(ws + P.off_gam);
        gp.C = W; gp.ldc = naux; gp.split_stride = gc * nvir * naux;
        if ((rc = launch_tuned(R_GAMMA, cg.bm, gp, P.autotune, P.general, st, af, ab))) return rc;
        const int64_t n = gc * nvir * naux;
        if ((rc = traced(R_REDUCE, 0, 0, 8.0 * (splits + 1 + acc) * n, st, [&] {
               hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)reduce_blocks(n, splits)), dim3(256), 0, st, out,
                                  naux, W, naux, gc * nvir * naux, (int)splits, gc * nvir, naux, 1.0, acc, status);
             })))
          return rc;
      } else {
        gp.C = out; gp.ldc = naux; gp.split_stride = 0; gp.accumulate = acc;
        if ((rc = launch_tuned(R_GAMMA, cg.bm, gp, P.autotune, P.general, st, af, ab))) return rc;
      }
      // Gamma rows of the later orbitals j >= k0 + gc, from the transposed
      // blocks: Gamma[j, b, P] += sum over (kk, a) of T_kj[a, b] B[k0 + kk, a, P]
      // (T_jk = T_kj^T), with the T slab read as an M-contiguous operand
      if (ncols > gc) {
        const int64_t rows = (ncols - gc) * nvir;
        GemmParams gt{};
        gt.M = rows; gt.N = naux; gt.K = gc * nvir; gt.kchunk = gt.K;
        gt.Am = NOperand{T + gc * nvir, Lc};
        gt.Bn = NOperand{B + k0 * nvir * naux, naux};
        gt.C = Gam + (k0 + gc) * nvir * naux; gt.ldc = naux; gt.split_stride = 0; gt.accumulate = acc;
        gt.status = status;
        const double r = (double)(ncols - gc);
        const double aft = 2.0 * r * v * x * g * v, abt = 8.0 * g * v * r * v + 8.0 * g * v * x + 8.0 * (1 + acc) * r * v * x;
        if (P.split) {
          // transposed-block product: the T columns (j >= k0 + gc, b) over the
          // group's rows (kk, a) as column digits [S][rows][pad(gc nvir)], and
          // the group's B rows as column digits [S][naux][pad(gc nvir)]
          const int64_t kg = cdiv(gc * nvir, 64) * 64;
          int8_t* dtt = (int8_t*)(ws + P.off_dtt);
          int32_t* ett = (int32_t*)(ws + P.off_ett);
          unsigned long long* cmt = (unsigned long long*)(ws + P.off_cmt);
          int8_t* dbk = (int8_t*)(ws + P.off_dbk);
          int32_t* ebk = (int32_t*)(ws + P.off_ebk);
          unsigned long long* cmax = (unsigned long long*)(ws + P.off_cmax);
          const double* Tt = T + gc * nvir;
          const double* Bk = B + k0 * nvir * naux;
          if ((rc = traced(R_SPLIT, 0, 0, 16.0 * g * v * r * v + 16.0 * g * v * x + (double)P.sg * (r * v + x) * kg, st,
                           [&] {
                             hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)cdiv(rows, 256)), dim3(256), 0, st,
                                                cmt, rows);
                             hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)cdiv(rows, 256),
                                                                    (unsigned)cdiv(gc * nvir, 1024)),
                                                dim3(256), 0, st, Tt, gc * nvir, rows, Lc, cmt, status);
                             RIMP2_SWITCH_S(P.sg, launch_split_cols<SS>(Tt, gc * nvir, rows, Lc, cmt, dtt, kg, ett,
                                                                        status, st));
                             hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)cdiv(naux, 256)), dim3(256), 0, st,
                                                cmax, naux);
                             hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)cdiv(naux, 256),
                                                                    (unsigned)cdiv(gc * nvir, 1024)),
                                                dim3(256), 0, st, Bk, gc * nvir, naux, naux, cmax, status);
                             RIMP2_SWITCH_S(P.sg, launch_split_cols<SS>(Bk, gc * nvir, naux, naux, cmax, dbk, kg, ebk,
                                                                        status, st));
                           })))
            return rc;
          if ((rc = run_oz8(P.sg, dtt, rows * kg, 0, ett, dbk, naux * kg, ebk, rows, naux, kg,
                            Gam + (k0 + gc) * nvir * naux, naux, status, R_GAMMA_T8, aft,
                            (double)P.sg * (r * v + x) * kg + 8.0 * (1 + acc) * r * v * x, st, acc)))
            return rc;
        } else if ((rc = launch_tuned(R_GAMMA_T, choose_gemm(gt.M, gt.N, gt.K, false, kGammaTiles, 1).bm, gt,
                                      P.autotune, P.general, st, aft, abt))) {
          return rc;
        }
      }
    }
    GemmParams gg{};   // ordered path: Gamma[k, a, P] = sum over (j, b) of T[k, a, j, b] B[j, b, P]
    const bool gam64 = P.gamma && !P.sym && !P.split;
    double afg = 0.0, abg = 0.0;
    if (P.gamma && !P.sym) {
      double* out = Gam + k0 * nvir * naux;
      afg = 2.0 * g * v * x * o * v;
      abg = slab + 8.0 * o * v * x + 8.0 * g * v * x;
      if (P.split) {
        if ((rc = traced(R_SPLIT, 0, 0, slab + (double)P.sg * g * v * P.kpg, st, [&] {
               RIMP2_SWITCH_S(P.sg, launch_split_rows<SS>(T, gc * nvir, L, L, dt, P.kpg, ext, status, st));
             })))
          return rc;
        if ((rc = run_oz8(P.sg, dt, gc * nvir * P.kpg, 0, ext, dbg, naux * P.kpg, exg, gc * nvir, naux, P.kpg, out,
                          naux, status, R_GAMMA8, afg, (double)P.sg * (g * v + x) * P.kpg + 8.0 * g * v * x, st)))
          return rc;
      } else {
        gg.M = gc * nvir; gg.N = naux; gg.K = L; gg.kchunk = cdiv(L, P.c_gam.splits);
        gg.A = kop(T, L, INT64_MAX, 0);
        gg.Bn = NOperand{B, naux};
        gg.C = out; gg.ldc = naux; gg.status = status;
        if (P.c_gam.splits > 1) {
          gg.C = (double*)(ws + P.off_gam);
          gg.split_stride = gg.M * naux;
          reduce(out, gg.C, gg.M, naux, cdiv(L, cdiv(gg.kchunk, kBK) * kBK), 1.0, 0);
        }
      }
    }
    GemmParams ga{}, gi{};
    if (P.density) {
      const int accumulate = k0 > 0 ? 1 : 0;
      // P_ab[a,b] += sum over (kk, j, c) of T[kk,a,j,c] X[kk,b,j,c]
      ga.M = nvir; ga.N = nvir; ga.K = gc * L; ga.kchunk = cdiv(ga.K, P.c_ab.splits);
      ga.A = kop(T, L, L, nvir * L);
      ga.Bk = kop(V, L, L, nvir * L);
      ga.C = (double*)(ws + P.off_pab); ga.ldc = nvir; ga.split_stride = nvir * nvir; ga.status = status;
      reduce(Pab, ga.C, nvir, nvir, cdiv(ga.K, cdiv(ga.kchunk, kBK) * kBK), 1.0, accumulate);
      // P_ij[i,j] -= sum over (kk, a, b) of T[kk,a,i,b] X[kk,a,j,b]; each slab's
      // contribution is symmetric: upper-triangular tiles, mirrored
      gi.M = nocc; gi.N = nocc; gi.K = gc * nvir * nvir; gi.kchunk = cdiv(gi.K, P.c_ij.splits);
      gi.A = kop(T, nvir, nvir, L);
      gi.Bk = kop(V, nvir, nvir, L);
      gi.C = (double*)(ws + P.off_pij); gi.ldc = nocc; gi.split_stride = nocc * nocc; gi.status = status;
      reduce(Pij, gi.C, nocc, nocc, cdiv(gi.K, cdiv(gi.kchunk, kBK) * kBK), -1.0, accumulate);
    }
    const double afa = 2.0 * v * v * g * o * v, aba = 2.0 * slab + 8.0 * v * v, afi = 2.0 * o * o * g * v * v,
                 abi = 2.0 * slab + 8.0 * o * o;
    int tail = 0;
    if (gam64 && P.density) tail = tail_level(P, gg, ga, gi);
    if (tail) {
      if ((rc = launch_tail(tail, gg, ga, gi, afg + afa + afi, abg + aba + abi, st))) return rc;
    } else {
      if (gam64 && (rc = launch_tuned(R_GAMMA, P.c_gam.bm, gg, P.autotune, P.general, st, afg, abg))) return rc;
      if (P.density && ((rc = launch_tuned(R_PAB, P.c_ab.bm, ga, P.autotune, P.general, st, afa, aba)) ||
                        (rc = launch_tuned(R_PIJ, P.c_ij.bm, gi, P.autotune, P.general, st, afi, abi))))
        return rc;
    }
    // the group's reductions, and with the last group's the energy
    const bool last = k0 + gc >= nocc;
    if (fin.n > 0 && !last) {
      FinishParams f = fin;
      f.E = nullptr;
      if ((rc = launch_finish(f, st))) return rc;
      fin.n = 0;
    }
  }
  return launch_finish(fin, st);
}

int want_of(const double* Gam, const double* Pij, const double* Pab, int* want) {
  if ((Pij == nullptr) != (Pab == nullptr))
    return fail(RIMP2_EINVAL, "P_ij and P_ab must both be given or both be NULL");
  *want = (Gam ? RIMP2_WANT_GAMMA : 0) | (Pij ? RIMP2_WANT_DENSITY : 0);
  return RIMP2_OK;
}


// ---- scratch space of the entry point that allocates nothing ----------------
// The array `scratch` is declared at file scope at the top of this file.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
int scratch_address(char** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(RIMP2_EDEVICE, "device %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      return fail(RIMP2_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = (char*)g_scratch_ptr[dev];
  return RIMP2_OK;
}

// Bytes of the largest array of split-K partial sums that fewer splits would shrink.
double largest_part(const Plan& P) {
  auto part = [](const GemmChoice& c, double elems) { return c.splits > 1 ? 8.0 * c.splits * elems : 0.0; };
  double most = std::max(part(P.c_ab, (double)P.nvir * P.nvir), part(P.c_ij, (double)P.nocc * P.nocc));
  if (P.gamma && !P.split && !P.sym) most = std::max(most, part(P.c_gam, (double)P.g * P.nvir * P.naux));
  if (P.gamma && !P.split && P.sym)
    for (int64_t k0 = 0, gc = 0; k0 < P.nocc; k0 += gc) {
      gc = group_at(P, k0);
      most = std::max(most, part(sym_gamma_choice(P, k0, gc), (double)gc * P.nvir * P.naux));
    }
  return most;
}

// The plan of rimp2_fragment_noalloc: the caller's options with, unless the
// caller fixed the slab group, the largest slab budget whose workspace fits
// the scratch array.  Slabs and split-K partial sums share the array, so plans
// with ever smaller partial sums are tried until one holds the whole fragment in
// a slab or has no splits left, and the smallest estimate is taken.  (The plan's
// own factors or else one split of each product, nothing between: P_ij of
// 51/427/1404 summed 182000 terms a workgroup.)
int noalloc_plan(int64_t nocc, int64_t nvir, int64_t naux, int want, const rimp2_opts* opts, Plan* P) {
  rimp2_opts o{};
  if (opts) o = *opts;
  if (o.autotune) return fail(RIMP2_ENOTSUP, "autotuning records events: not available without allocation");
  const bool gamma = want & RIMP2_WANT_GAMMA, density = want & RIMP2_WANT_DENSITY;
  int rc;
  double best_us = -1.0;
  Plan Q;
  for (double part_bytes = kAnyPartBytes;; part_bytes = largest_part(Q) / 2.0) {
    if (o.slab_group == 0) o.slab_budget_bytes = kScratchBytes;
    if ((rc = make_plan(nocc, nvir, naux, gamma, density, &o, &Q, false, part_bytes))) return rc;
    for (int it = 0; o.slab_group == 0 && it < 64 && Q.total > kScratchBytes; ++it) {
      const size_t over = Q.total - kScratchBytes;
      if (o.slab_budget_bytes <= over + 1) break;
      o.slab_budget_bytes -= over + 1;   // the slabs shrink by at least the overshoot (or g reaches 1)
      if ((rc = make_plan(nocc, nvir, naux, gamma, density, &o, &Q, false, part_bytes))) return rc;
    }
    if (Q.total <= kScratchBytes) {
      const bool whole = group_at(Q, 0) == nocc;
      const double us = whole && best_us < 0.0 ? 0.0 : plan_us(Q);
      if (best_us < 0.0 || us < best_us) {
        best_us = us;
        *P = Q;
      }
      if (whole) break;
    }
    if (largest_part(Q) == 0.0) break;
  }
  if (best_us < 0.0)
    return fail(RIMP2_ENOMEM, "fragment nocc=%lld nvir=%lld naux=%lld needs %zu bytes of scratch, more than the "
                "%zu of rimp2_fragment_noalloc", (long long)nocc, (long long)nvir, (long long)naux, Q.total,
                kScratchBytes);
  return RIMP2_OK;
}


// One digit split of one fragment in a batch wave (split precision): rows of
// X [N][K] (row stride ld) into D [S][N][kp] with exps e[N] (split_row), or
// columns of X [K][N] into D [S][N][kp] with column maxima cmax[N]
// (colmax_block, split_cols_tile).  gx: the op's blocks along its first grid
// dimension (columns: cdiv(N, 256) for the maxima, cdiv(kp, 32) for the
// digits, which use one op entry each).
struct DigitOp {
  const double* X;
  int64_t K, N, ld, kp, gx;
  int8_t* D;
  int32_t* e;
  unsigned long long* cmax;
  const int32_t* status;
};

// ---- batches -----------------------------------------------------------------
// Grouped GEMMs of a wave: every role has two candidate tile choices, each a
// table of all its problems, sorted into lists of one tile side and loader (0, 1,
// 2: the fast loader's levels 1, 2, 3; 3: the general loader with 16-byte loads,
// 4: the general loader, 8-byte loads), largest problem first.
constexpr int kGLoaders = 5, kGKeys = 4 * kGLoaders;
struct GemmList {
  int bm, loader, first, n;   // entries [first, first + n) of the table
  int64_t items;              // work items (tiles x splits)
  size_t pre;                 // offset of its prefix array within the table's prefixes
};
struct GemmEntry {
  int bm, loader;
  GemmParams p;
  int64_t items;
};
struct Wave {
  std::vector<int32_t> frags;   // original fragment indices, largest first
  size_t tab_bytes = 0;         // bytes of device tables at the start of the wave region
  size_t host_off = 0;          // offset of this wave's tables in the pinned blob
  size_t bytes = 0;             // tables + fragment partitions
  // offsets within the tables
  size_t o_fs, o_idx, o_amp, o_amp_pre[2], o_red, o_red_pre;   // o_amp_pre: tiles of 32, of 64 (amp_tile)
  size_t o_g[4][2], o_pre[4][2];   // tables and prefixes by role and candidate
  std::vector<GemmList> lists[4][2];
  int n_g[4] = {0, 0, 0, 0};       // problems of each role
  int tile_g[4][2] = {};           // tile side of the largest problem (autotuner report)
  uint64_t sig = 0;             // hash of the wave's fragment sizes (autotuner key)
  int nred = 0;                 // split-K reductions
  int64_t amp_blocks[2], red_blocks = 0;
  // split products (precision RIMP2_SPLIT_INT8): grouped (ia|jb) and Gamma
  // product lists, run in reduction windows (win_* launches each)
  size_t o_oz[2] = {0, 0}, o_oz_pre[2] = {0, 0};
  int n_oz[2] = {0, 0};
  int64_t items_oz[2] = {0, 0};
  int win_oz[2] = {0, 0};
  int side_oz[2] = {64, 64};      // tile side of each product
  // grouped digit splits: lists 0 (B rows), 1 (B columns: zero, maxima), 2 (B
  // column digits), 3 (T rows); each with its op table and four prefix arrays
  // (one per mode; only the one its launch uses is read)
  static constexpr int kDigitLists = 4;
  size_t o_dop[kDigitLists] = {0, 0, 0, 0}, o_dpre[kDigitLists][4] = {};
  int n_dop[kDigitLists] = {0, 0, 0, 0};
  int64_t blocks_dop[kDigitLists][4] = {};
};
}  // namespace

struct rimp2_batch_s {
  bool autotune = false;
  bool general = false;            // FP64 GEMMs take the general loader only
  bool split = false;              // grouped split-precision products
  std::vector<rimp2_frag_desc> d;
  std::vector<int32_t> solo;       // fragments run alone
  std::vector<Plan> plan;          // per fragment (solo: own plan; grouped: full-slab plan)
  std::vector<Wave> waves;
  std::vector<char> blob;          // tables of every wave, as laid out at the start of the workspace
  char* host = nullptr;            // pinned copy of blob (handle path)
  size_t tables_total = 0, ws_bytes = 0;
};

namespace {

uint64_t rel(size_t off) { return kRelTag | (uint64_t)off; }
template <class T>
T* relp(size_t off) { return (T*)(uintptr_t)rel(off); }
bool aligned16(const void* p) { return ((uintptr_t)p & ~kRelTag) % 16 == 0; }
bool kop_vec_rel(const KOperand& o, int64_t K) {
  const bool plain = o.kdiv >= K;
  return aligned16(o.base) && o.rs % 2 == 0 && (plain || (o.kdiv % 2 == 0 && o.ks1 % 2 == 0));
}

// Grouped GEMM roles of a wave and their tiles (those launch_group_list has).
const int kBatchRole[4] = {R_INTS, R_GAMMA, R_PAB, R_PIJ};
constexpr int kBatchPijTiles[] = {96, 64, 32, 0};
const int* const kBatchTiles[4] = {kIntsTiles, kGammaTiles, kPabTiles, kBatchPijTiles};
// loader of a grouped GEMM (see GemmList); vec: 16-byte loads are aligned;
// general: the general loader only
int loader_of(const GemmParams& g, int bm, bool nc, bool vec, bool general) {
  const int f = general ? 0 : fast_level(g, bm, nc);
  return f ? f - 1 : vec ? 3 : 4;
}

size_t place(size_t& off, size_t bytes) {
  const size_t o = off;
  off = align_up(off + bytes);
  return o;
}

int batch_plan(int32_t nfrag, const rimp2_frag_desc* d, const rimp2_opts* opts, rimp2_batch_s* B) {
  if (nfrag < 0 || (nfrag > 0 && !d)) return fail(RIMP2_EINVAL, "bad batch arguments");
  if (opts && opts->precision != RIMP2_FP64 && opts->precision != RIMP2_SPLIT_INT8)
    return fail(RIMP2_ENOTSUP, "precision %d is not supported", opts->precision);
  if (opts && opts->pair_skip) return fail(RIMP2_ENOTSUP, "pair_skip is not supported for batches");
  const bool split = opts && opts->precision == RIMP2_SPLIT_INT8;
  B->split = split;
  B->d.assign(d, d + nfrag);
  B->autotune = opts && opts->autotune;
  if (opts && (opts->gemm_loader < 0 || opts->gemm_loader > 1))
    return fail(RIMP2_EINVAL, "gemm_loader must be 0 or 1 (got %d)", opts->gemm_loader);
  const bool general = opts && opts->gemm_loader == 1;
  B->general = general;
  B->plan.resize(nfrag);
  const size_t budget = (opts && opts->slab_budget_bytes) ? opts->slab_budget_bytes : (size_t)64 << 30;
  std::vector<int32_t> order(nfrag), grouped;
  std::vector<char> solo(nfrag, 0);
  for (int32_t f = 0; f < nfrag; ++f) {
    if (!d[f].B || !d[f].eps_occ || !d[f].eps_vir || !d[f].E)
      return fail(RIMP2_EINVAL, "fragment %d: B, eps_occ, eps_vir and E must not be NULL", f);
    int want, rc;
    if ((rc = want_of(d[f].Gamma, d[f].P_ij, d[f].P_ab, &want))) return fail(rc, "fragment %d: %s", f, g_err);
    rimp2_opts o{};
    o.slab_group = d[f].nocc;     // whole slab
    if (split) {
      o.precision = RIMP2_SPLIT_INT8;
      o.split_slices = opts->split_slices;
      o.split_slices_gamma = opts->split_slices_gamma;
    }
    Plan P;
    if ((rc = make_plan(d[f].nocc, d[f].nvir, d[f].naux, want & 1, want & 2, &o, &P, true)))
      return fail(rc, "fragment %d: %s", f, g_err);
    if (P.total > budget) {
      solo[f] = 1;
      if ((rc = make_plan(d[f].nocc, d[f].nvir, d[f].naux, want & 1, want & 2, opts, &P)))
        return fail(rc, "fragment %d: %s", f, g_err);
    }
    B->plan[f] = P;
    order[f] = f;
  }
  auto cost = [&](int32_t f) { return (double)d[f].nocc * d[f].nocc * d[f].nvir * d[f].nvir * d[f].naux; };
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return cost(a) > cost(b); });
  size_t ws = kAlign, max_solo = 0;
  for (int32_t f : order) {
    if (solo[f]) { B->solo.push_back(f); max_solo = std::max(max_solo, B->plan[f].total); }
    else grouped.push_back(f);
  }
  // pack waves greedily (largest first) by the sum of full-slab plans
  for (size_t i = 0; i < grouped.size();) {
    Wave W;
    size_t sum = 0;
    while (i < grouped.size() && (W.frags.empty() || sum + B->plan[grouped[i]].total <= budget)) {
      sum += B->plan[grouped[i]].total;
      W.frags.push_back(grouped[i++]);
    }
    B->waves.push_back(W);
  }
  // table layout of every wave (sizes depend only on the wave's fragment count)
  size_t tab = 0;
  for (Wave& W : B->waves) {
    const int n = (int)W.frags.size();
    size_t t = 0;
    W.o_fs = place(t, sizeof(FragSmall) * n);
    W.o_idx = place(t, sizeof(int32_t) * n);
    W.o_amp = place(t, sizeof(AmpDesc) * n);
    for (size_t& o : W.o_amp_pre) o = place(t, sizeof(int64_t) * (n + 1));
    W.o_red = place(t, sizeof(ReduceDesc) * 2 * n);
    W.o_red_pre = place(t, sizeof(int64_t) * (2 * n + 1));
    for (int r = 0; r < 4; ++r)
      for (int c = 0; c < 2; ++c) {
        W.o_g[r][c] = place(t, sizeof(GemmParams) * n);
        W.o_pre[r][c] = place(t, sizeof(int64_t) * (n + kGKeys));
      }
    if (split) {
      for (int r = 0; r < 2; ++r) {
        W.o_oz[r] = place(t, sizeof(OzParams) * n);
        W.o_oz_pre[r] = place(t, sizeof(int64_t) * (n + 1));
      }
      // windows of every fragment in the wave (at most this many launches per product)
      for (int32_t f : W.frags) {
        const Plan& P = B->plan[f];
        W.win_oz[0] = std::max<int>(W.win_oz[0], (int)cdiv(P.kpv, kOzWindow));
        if (P.gamma) W.win_oz[1] = std::max<int>(W.win_oz[1], (int)cdiv(P.kpg, kOzWindow));
      }
      // one tile shape for the wave's Gamma products, by their tiles together
      // ((ia|jb) runs at 64: its defaults are 7 digits)
      double t64 = 0.0, t128 = 0.0;
      for (int32_t f : W.frags)
        if (const Plan& P = B->plan[f]; P.gamma) {
          t64 += (double)cdiv(P.nocc * P.nvir, 64) * cdiv(P.naux, 64);
          t128 += (double)cdiv(P.nocc * P.nvir, 128) * cdiv(P.naux, 128);
        }
      W.side_oz[1] = oz8_side(B->plan[W.frags[0]].sg, t64, t128);
      for (int r = 0; r < Wave::kDigitLists; ++r) {
        W.o_dop[r] = place(t, sizeof(DigitOp) * n);
        for (int m = 0; m < 4; ++m) W.o_dpre[r][m] = place(t, sizeof(int64_t) * (n + 1));
      }
    }
    W.tab_bytes = t;
    W.host_off = tab;
    tab = align_up(tab + t);
  }
  B->tables_total = tab;
  B->blob.assign(tab, 0);
  for (Wave& W : B->waves) {
    const int n = (int)W.frags.size();
    std::vector<FragSmall> fs(n);
    std::vector<int32_t> idx(n);
    std::vector<AmpDesc> amp(n);
    std::vector<int64_t> amp_pre[2] = {std::vector<int64_t>(n + 1, 0), std::vector<int64_t>(n + 1, 0)};
    std::vector<ReduceDesc> red;
    std::vector<int64_t> red_pre(1, 0);
    std::vector<GemmEntry> ge[4][2];
    std::vector<OzParams> oz[2];
    std::vector<int64_t> oz_pre[2] = {{0}, {0}};
    std::vector<DigitOp> dop[Wave::kDigitLists];
    std::vector<int64_t> dpre[Wave::kDigitLists][4];
    for (auto& l : dpre)
      for (auto& v : l) v.assign(1, 0);
    // op f of list r: workgroups per mode
    auto add_dop = [&](int r, const DigitOp& o, int64_t rows_wgs, int64_t zero_wgs, int64_t max_wgs, int64_t dig_wgs) {
      dop[r].push_back(o);
      const int64_t w[4] = {rows_wgs, zero_wgs, max_wgs, dig_wgs};
      for (int m = 0; m < 4; ++m) dpre[r][m].push_back(dpre[r][m].back() + w[m]);
    };
    // a GEMM goes to both candidates' tables of its role: with the tile of the
    // smallest grouped_cost, and with the next best
    auto add = [&](int rho, const GemmParams& g0, bool vec) {
      int best[2] = {0, 0};
      double cost[2] = {0.0, 0.0};
      for (const int* t = kBatchTiles[rho]; *t; ++t) {
        GemmParams g = g0;
        const double c = grouped_cost(*t, finalize_gemm(g, *t, *t, rho >= 2) / g.splits);
        if (best[0] == 0 || c < kSmallerTile * cost[0]) {
          best[1] = best[0]; cost[1] = cost[0];
          best[0] = *t; cost[0] = c;
        } else if (best[1] == 0 || c < cost[1]) {
          best[1] = *t; cost[1] = c;
        }
      }
      for (int c = 0; c < 2; ++c) {
        GemmEntry e{best[c], 0, g0, 0};
        e.items = finalize_gemm(e.p, e.bm, e.bm, rho >= 2);
        e.loader = loader_of(e.p, e.bm, rho == 1, vec, general);
        if (ge[rho][c].empty()) W.tile_g[rho][c] = e.bm;
        ge[rho][c].push_back(e);
      }
    };
    uint64_t sig = 1469598103934665603ull;  // FNV-1a over the fragment sizes and outputs
    size_t poff = tab;   // fragment partitions follow all tables (shared by the waves)
    for (int i = 0; i < n; ++i) {
      const int32_t f = W.frags[i];
      const rimp2_frag_desc& q = d[f];
      const Plan& P = B->plan[f];
      const size_t base = poff;
      poff = align_up(poff + P.total);
      const int64_t nocc = q.nocc, nvir = q.nvir, naux = q.naux, L = nocc * nvir;
      for (int64_t w : {nocc, nvir, naux, (int64_t)P.gamma, (int64_t)P.density}) sig = (sig ^ (uint64_t)w) * 1099511628211ull;
      int32_t* status = relp<int32_t>(base + P.off_status);
      double* V = relp<double>(base + P.off_V);
      double* T = relp<double>(base + P.off_T);
      double* ep = q.e_pair ? q.e_pair : relp<double>(base + P.off_e);
      fs[i] = FragSmall{q.eps_occ, q.eps_vir, ep, q.E, status, q.nocc, q.nvir};
      idx[i] = f;
      amp[i] = AmpDesc{V, T, q.eps_occ, q.eps_vir, ep, status, q.nocc, q.nvir, (P.gamma || P.density) ? 0 : 1,
                       P.density ? 1 : 0};
      const int big = amp_tile(nvir, !(P.gamma || P.density)) == 64 ? 1 : 0;
      for (int b = 0; b < 2; ++b) amp_pre[b][i + 1] = amp_pre[b][i] + (b == big ? nocc * nocc : 0);
      if (split) {  // (ia|jb) and Gamma as INT8 digit products of the whole slab
        OzParams z{};
        z.M = L; z.N = L; z.kp = P.kpv; z.k0 = 0; z.kc = P.kpv;
        z.A = relp<int8_t>(base + P.off_dbv); z.a_slice = L * P.kpv; z.a_row0 = 0;
        z.B = z.A; z.b_slice = z.a_slice;
        z.ea = relp<int32_t>(base + P.off_ev); z.eb = z.ea;
        z.C = V; z.ldc = L;
        const int64_t sz = W.side_oz[0];
        z.tiles_m = (int32_t)cdiv(L, sz); z.tiles_n = z.tiles_m; z.group_m = 8;
        // blocks j < k: the amplitude pass mirrors them (pair_k0 = pair_j0 = pair_lo = 0)
        z.pair_nvir = (int32_t)nvir;
        z.status = status;
        const int64_t tiles = oz8_tiles(z, sz, sz);
        z.pair_map = tiles < (int64_t)z.tiles_m * z.tiles_n;
        oz[0].push_back(z);
        oz_pre[0].push_back(oz_pre[0].back() + tiles);
        // digits of every B row (both operands of the (ia|jb) products)
        add_dop(0, DigitOp{q.B, naux, L, naux, P.kpv, 0, relp<int8_t>(base + P.off_dbv),
                           relp<int32_t>(base + P.off_ev), nullptr, status}, L, 0, 0, 0);
        if (P.gamma) {
          OzParams y{};
          y.M = L; y.N = naux; y.kp = P.kpg; y.k0 = 0; y.kc = P.kpg;
          y.A = relp<int8_t>(base + P.off_dt); y.a_slice = L * P.kpg; y.a_row0 = 0;
          y.B = relp<int8_t>(base + P.off_dbg); y.b_slice = naux * P.kpg;
          y.ea = relp<int32_t>(base + P.off_et); y.eb = relp<int32_t>(base + P.off_eg);
          y.C = q.Gamma; y.ldc = naux;
          const int64_t sy = W.side_oz[1];
          y.tiles_m = (int32_t)cdiv(L, sy); y.tiles_n = (int32_t)cdiv(naux, sy); y.group_m = 8;
          y.status = status;
          oz[1].push_back(y);
          oz_pre[1].push_back(oz_pre[1].back() + oz8_tiles(y, sy, sy));
          // column digits of B (maxima first) and row digits of the T slab
          unsigned long long* cm = relp<unsigned long long>(base + P.off_cmax);
          const int64_t gxm = cdiv(naux, 256), gxd = cdiv(P.kpg, 32);
          add_dop(1, DigitOp{q.B, L, naux, naux, P.kpg, gxm, nullptr, nullptr, cm, status}, 0, gxm,
                  gxm * cdiv(L, 1024), 0);
          add_dop(2, DigitOp{q.B, L, naux, naux, P.kpg, gxd, relp<int8_t>(base + P.off_dbg),
                             relp<int32_t>(base + P.off_eg), cm, status}, 0, 0, 0, gxd * cdiv(naux, 32));
          add_dop(3, DigitOp{relp<double>(base + P.off_T), L, L, L, P.kpg, 0, relp<int8_t>(base + P.off_dt),
                             relp<int32_t>(base + P.off_et), nullptr, status}, L, 0, 0, 0);
        }
      }
      if (!split) {  // (ia|jb)
        GemmParams gp{};
        gp.M = nocc * nvir; gp.N = L; gp.K = naux; gp.kchunk = naux;
        gp.A = KOperand{q.B, naux, INT64_MAX, 0};
        gp.Bk = KOperand{q.B, naux, INT64_MAX, 0};
        gp.C = V; gp.ldc = L; gp.status = status;
        gp.skip_nvir = (int32_t)nvir; gp.skip_nocc = (int32_t)nocc; gp.pair_upper = 1;
        add(0, gp, kop_vec_rel(gp.A, gp.K) && kop_vec_rel(gp.Bk, gp.K));
      }
      if (P.gamma && !split) {
        GemmParams gp{};
        gp.M = nocc * nvir; gp.N = naux; gp.K = L; gp.kchunk = L;
        gp.A = KOperand{T, L, INT64_MAX, 0};
        gp.Bn = NOperand{q.B, naux};
        gp.C = q.Gamma; gp.ldc = naux; gp.status = status;
        add(1, gp, kop_vec_rel(gp.A, gp.K) && aligned16(q.B) && naux % 2 == 0);
      }
      if (P.density) {
        double* Wab = relp<double>(base + P.off_pab);
        double* Wij = relp<double>(base + P.off_pij);
        GemmParams ga{};
        ga.M = nvir; ga.N = nvir; ga.K = nocc * L; ga.kchunk = cdiv(ga.K, P.c_ab.splits);
        ga.A = KOperand{T, L, L, nvir * L};
        ga.Bk = KOperand{V, L, L, nvir * L};
        ga.C = Wab; ga.ldc = nvir; ga.split_stride = nvir * nvir; ga.status = status;
        add(2, ga, kop_vec_rel(ga.A, ga.K) && kop_vec_rel(ga.Bk, ga.K));
        (void)finalize_gemm(ga, 64, 64, true);   // splits for the reduction
        GemmParams gi{};
        gi.M = nocc; gi.N = nocc; gi.K = nocc * nvir * nvir; gi.kchunk = cdiv(gi.K, P.c_ij.splits);
        gi.A = KOperand{T, nvir, nvir, L};
        gi.Bk = KOperand{V, nvir, nvir, L};
        gi.C = Wij; gi.ldc = nocc; gi.split_stride = nocc * nocc; gi.status = status;
        add(3, gi, kop_vec_rel(gi.A, gi.K) && kop_vec_rel(gi.Bk, gi.K));
        (void)finalize_gemm(gi, 64, 64, true);
        ReduceDesc ra{q.P_ab, Wab, status, nvir, nvir, nvir * nvir, nvir, nvir, 1.0, ga.splits, 0};
        ReduceDesc ri{q.P_ij, Wij, status, nocc, nocc, nocc * nocc, nocc, nocc, -1.0, gi.splits, 0};
        red.push_back(ra); red_pre.push_back(red_pre.back() + reduce_blocks(nvir * nvir, ga.splits));
        red.push_back(ri); red_pre.push_back(red_pre.back() + reduce_blocks(nocc * nocc, gi.splits));
      }
    }
    W.bytes = poff;
    ws = std::max(ws, poff);
    for (int b = 0; b < 2; ++b) W.amp_blocks[b] = amp_pre[b][n];
    W.nred = (int)red.size();
    W.red_blocks = red_pre.back();
    W.sig = sig;
    char* blob = B->blob.data() + W.host_off;
    auto put = [&](size_t off, const void* src, size_t bytes) { if (bytes) memcpy(blob + off, src, bytes); };
    put(W.o_fs, fs.data(), sizeof(FragSmall) * n);
    put(W.o_idx, idx.data(), sizeof(int32_t) * n);
    put(W.o_amp, amp.data(), sizeof(AmpDesc) * n);
    for (int b = 0; b < 2; ++b) put(W.o_amp_pre[b], amp_pre[b].data(), sizeof(int64_t) * (n + 1));
    put(W.o_red, red.data(), sizeof(ReduceDesc) * red.size());
    put(W.o_red_pre, red_pre.data(), sizeof(int64_t) * red_pre.size());
    for (int r = 0; r < 4; ++r)
      for (int c = 0; c < 2; ++c) {
        std::vector<GemmEntry>& e = ge[r][c];
        std::stable_sort(e.begin(), e.end(), [](const GemmEntry& x, const GemmEntry& y) {
          return x.bm != y.bm ? x.bm > y.bm : x.loader < y.loader;
        });
        W.n_g[r] = (int)e.size();
        size_t pre = W.o_pre[r][c];
        for (size_t i = 0; i < e.size();) {
          GemmList l{e[i].bm, e[i].loader, (int)i, 0, 0, pre};
          std::vector<int64_t> prefix(1, 0);
          for (; i < e.size() && e[i].bm == l.bm && e[i].loader == l.loader; ++i, ++l.n) {
            put(W.o_g[r][c] + sizeof(GemmParams) * i, &e[i].p, sizeof(GemmParams));
            prefix.push_back(l.items += e[i].items);
          }
          put(pre, prefix.data(), sizeof(int64_t) * prefix.size());
          pre += sizeof(int64_t) * prefix.size();
          W.lists[r][c].push_back(l);
        }
      }
    if (split) {
      for (int r = 0; r < 2; ++r) {
        W.n_oz[r] = (int)oz[r].size();
        W.items_oz[r] = oz_pre[r].back();
        put(W.o_oz[r], oz[r].data(), sizeof(OzParams) * oz[r].size());
        put(W.o_oz_pre[r], oz_pre[r].data(), sizeof(int64_t) * oz_pre[r].size());
      }
      for (int r = 0; r < Wave::kDigitLists; ++r) {
        W.n_dop[r] = (int)dop[r].size();
        put(W.o_dop[r], dop[r].data(), sizeof(DigitOp) * dop[r].size());
        for (int m = 0; m < 4; ++m) {
          W.blocks_dop[r][m] = dpre[r][m].back();
          put(W.o_dpre[r][m], dpre[r][m].data(), sizeof(int64_t) * dpre[r][m].size());
        }
      }
    }
  }
  // solo fragments use the workspace after all tables
  B->ws_bytes = std::max(ws, align_up(tab + max_solo));
  return RIMP2_OK;
}

// Items of a grouped launch that go to one XCD in turn, at most `most`: 64 (an 8
// x 8 block of tiles) for the products that wait for their operands (split, P_ab
// and P_ij); 8 for FP64 (ia|jb) and Gamma, which are MFMA-bound and whose tiles
// are long (up to milliseconds), so that the XCDs finish together (24 monomers'
// Gamma: 35.4 ms with 64, 34.2 with 8).
constexpr int kLongBlock = 8, kOperandBlock = 64;
int grouped_block(int64_t items, int most) { return (int)std::max<int64_t>(1, std::min<int64_t>(most, items / 64)); }
int64_t grouped_grid(int64_t items, int most) {
  const int64_t per = 8 * grouped_block(items, most);
  return cdiv(items, per) * per;
}

template <int BM, int BN, bool NC, int ROLE, bool VEC, bool TRI, int FAST>
int launch_grouped(const Grouped<GemmParams>& G, int64_t items, int role, hipStream_t st) {
  const int64_t grid = grouped_grid(items, role == R_INTS || role == R_GAMMA ? kLongBlock : kOperandBlock);
  if (int rc = check_grid(grid, "grouped GEMM")) return rc;
  return traced(role, 0, 0, 0, st, [&] {
    hipLaunchKernelGGL((gemm_f64_grouped<BM, BN, kBK, NC, ROLE, VEC, TRI, FAST>), dim3((unsigned)grid), dim3(256), 0,
                       st, G);
  });
}

// One grouped launch of batch role rho over a list of one tile side and loader
// (see GemmList).
int launch_group_list(int rho, int bm, int loader, const Grouped<GemmParams>& G, int64_t items, hipStream_t st) {
  const int role = kBatchRole[rho];
#define RIMP2_G(BM, NC, ROLE, TRI, F2, F3)                                                            \
  switch (loader) {                                                                                   \
    case 0: return launch_grouped<BM, BM, NC, ROLE, true, TRI, 1>(G, items, role, st);                \
    case 1: return launch_grouped<BM, BM, NC, ROLE, true, TRI, F2>(G, items, role, st);               \
    case 2: return launch_grouped<BM, BM, NC, ROLE, true, TRI, F3>(G, items, role, st);               \
    case 3: return launch_grouped<BM, BM, NC, ROLE, true, TRI, 0>(G, items, role, st);                \
    default: return launch_grouped<BM, BM, NC, ROLE, false, TRI, 0>(G, items, role, st);              \
  }
  // (ia|jb) and Gamma have no runs: their lists hold loader 0 or a general one
  switch (rho * 1000 + bm) {
    case 128: RIMP2_G(128, false, ROLE_INTS, false, 1, 1);
    case 64: RIMP2_G(64, false, ROLE_INTS, false, 1, 1);
    case 1128: RIMP2_G(128, true, ROLE_GAMMA, false, 1, 1);
    case 1064: RIMP2_G(64, true, ROLE_GAMMA, false, 1, 1);
    case 2128: RIMP2_G(128, false, ROLE_PAB, true, 2, 3);
    case 2096: RIMP2_G(96, false, ROLE_PAB, true, 2, 3);
    case 2064: RIMP2_G(64, false, ROLE_PAB, true, 2, 3);
    case 3096: RIMP2_G(96, false, ROLE_PIJ, true, 2, 3);
    case 3064: RIMP2_G(64, false, ROLE_PIJ, true, 2, 3);
    case 3032: RIMP2_G(32, false, ROLE_PIJ, true, 2, 3);
    default: return fail(RIMP2_EINVAL, "no grouped GEMM for role %d with tiles of %d", role, bm);
  }
#undef RIMP2_G
}

__device__ __forceinline__ int digit_op_at(const int64_t* prefix, int n, int64_t t) {
  int lo = 0, hi = n - 1;   // last f with prefix[f] <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Grouped digit splits: one launch over every op of a list (prefix counts
// each op's workgroups).  mode 0: rows; 1: zero cmax; 2: column maxima;
// 3: column digits.
template <int S, int MODE>
__global__ __launch_bounds__(256) void digit_split_grouped(const DigitOp* ops, const int64_t* prefix, int n) {
  const int f = digit_op_at(prefix, n, blockIdx.x);
  const DigitOp o = ops[f];
  if (o.status != nullptr && *o.status != 0) return;
  const int64_t u = (int64_t)blockIdx.x - prefix[f];
  if constexpr (MODE == 0) {
    split_row<S>(o.X, o.N, o.K, o.ld, o.D, o.kp, o.e, u);
  } else if constexpr (MODE == 1) {
    const int64_t i = u * 256 + threadIdx.x;
    if (i < o.N) o.cmax[i] = 0ull;
  } else if constexpr (MODE == 2) {
    colmax_block(o.X, o.K, o.N, o.ld, o.cmax, u % o.gx, u / o.gx);
  } else {
    split_cols_tile<S>(o.X, o.K, o.N, o.ld, o.cmax, o.D, o.kp, o.e, u % o.gx, u / o.gx);
  }
}

__global__ void relocate_digit_kernel(char* base, DigitOp* ops, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    DigitOp& o = ops[i];
    reloc_t(o.X, base); reloc_t(o.D, base); reloc_t(o.e, base); reloc_t(o.cmax, base); reloc_t(o.status, base);
  }
}

__global__ void relocate_oz_kernel(char* base, OzParams* z, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    OzParams& p = z[i];
    reloc_t(p.A, base); reloc_t(p.B, base); reloc_t(p.ea, base); reloc_t(p.eb, base);
    reloc_t(p.C, base); reloc_t(p.status, base);
  }
}

// One grouped split-product launch over reduction window `window` of every
// problem in G (the shapes and buffering of launch_oz8 for a windowed product).
template <int S>
int launch_oz8_grouped(const Grouped<OzParams>& G, int64_t items, int side, int64_t window, int role, hipStream_t st) {
  if (G.nprob == 0 || items == 0) return RIMP2_OK;
  const int64_t grid = grouped_grid(items, kOperandBlock);
  if (int rc = check_grid(grid * (side / 64), "grouped split product")) return rc;
  return traced(role, 0, 0, 0, st, [&] {
    if (S <= 5 && side == 128)
      hipLaunchKernelGGL((gemm_oz8_grouped<S <= 5 ? S : 5, 2, OzWide>), dim3((unsigned)grid), dim3(512), 0, st, G,
                         window, kOzWindow);
    else
      hipLaunchKernelGGL((gemm_oz8_grouped<S, S <= 5 ? 2 : 1, OzSmall>), dim3((unsigned)grid), dim3(256), 0, st, G,
                         window, kOzWindow);
  });
}

// upload: 0 = tables already in the workspace, 1 = copy them from B->host (pinned) on the stream
int batch_run(rimp2_batch_s* B, int32_t* status_dev, void* workspace, size_t bytes, hipStream_t st, int upload) {
  if (!workspace) return fail(RIMP2_EINVAL, "workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  if (bytes < B->ws_bytes) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", bytes, B->ws_bytes);
  char* ws = (char*)workspace;
  int rc;
  if (upload && B->tables_total) {
    if (!B->host) return fail(RIMP2_EINVAL, "batch tables are not resident");
    HIP_TRY(hipMemcpyAsync(ws, B->host, B->tables_total, hipMemcpyHostToDevice, st));
  }
  // solo fragments run with their own workspace layout after the tables
  char* solo_ws = ws + B->tables_total;
  for (int32_t f : B->solo) {
    const rimp2_frag_desc& q = B->d[f];
    if ((rc = run_fragment(B->plan[f], q.B, q.eps_occ, q.eps_vir, q.E, q.Gamma, q.P_ij, q.P_ab, q.e_pair, solo_ws,
                           nullptr, st)))
      return fail(rc, "fragment %d: %s", f, g_err);
    if (status_dev && (rc = traced(R_STATUS, 0, 0, 8.0, st, [&] {
                         hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(64), 0, st,
                                            (const int32_t*)(solo_ws + B->plan[f].off_status), status_dev, (int)f);
                       })))
      return rc;
  }
  for (const Wave& W : B->waves) {
    const int n = (int)W.frags.size();
    auto at = [&](size_t o) { return ws + W.host_off + o; };
    if ((rc = traced(R_STATUS, 0, 0, 0, st, [&] {
           // relocate every table
           for (int r = 0; r < 4; ++r)
             for (int c = 0; c < (B->autotune ? 2 : 1); ++c)
               if (W.n_g[r])
                 hipLaunchKernelGGL(relocate_tables_kernel, dim3((unsigned)cdiv(W.n_g[r], 256)), dim3(256), 0, st, ws,
                                    (GemmParams*)at(W.o_g[r][c]), W.n_g[r], (AmpDesc*)nullptr, 0, (ReduceDesc*)nullptr,
                                    0, (FragSmall*)nullptr, 0);
           const int m = std::max(n, W.nred);
           hipLaunchKernelGGL(relocate_tables_kernel, dim3((unsigned)cdiv(m, 256)), dim3(256), 0, st, ws,
                              (GemmParams*)nullptr, 0, (AmpDesc*)at(W.o_amp), n, (ReduceDesc*)at(W.o_red), W.nred,
                              (FragSmall*)at(W.o_fs), n);
           hipLaunchKernelGGL(gap_check_grouped, dim3((unsigned)n), dim3(256), 0, st, (const FragSmall*)at(W.o_fs));
           if (B->split) {
             for (int r = 0; r < 2; ++r)
               if (W.n_oz[r])
                 hipLaunchKernelGGL(relocate_oz_kernel, dim3((unsigned)cdiv(W.n_oz[r], 256)), dim3(256), 0, st, ws,
                                    (OzParams*)at(W.o_oz[r]), W.n_oz[r]);
             for (int r = 0; r < Wave::kDigitLists; ++r)
               if (W.n_dop[r])
                 hipLaunchKernelGGL(relocate_digit_kernel, dim3((unsigned)cdiv(W.n_dop[r], 256)), dim3(256), 0, st,
                                    ws, (DigitOp*)at(W.o_dop[r]), W.n_dop[r]);
           }
         })))
      return rc;
    // each GEMM role: the lists of one candidate (with autotuning the tuned one
    // for this wave's fragment sizes)
    auto run_role = [&](int rho) -> int {
      if (W.n_g[rho] == 0) return RIMP2_OK;
      auto launch = [&](int c) -> int {
        for (const GemmList& l : W.lists[rho][c]) {
          const Grouped<GemmParams> G{(const GemmParams*)at(W.o_g[rho][c]) + l.first, (const int64_t*)at(l.pre), l.n,
                                      grouped_block(l.items, rho < 2 ? kLongBlock : kOperandBlock)};
          if (int r = launch_group_list(rho, l.bm, l.loader, G, l.items, st)) return r;
        }
        return RIMP2_OK;
      };
      if (!B->autotune) return launch(0);
      int dev = 0;
      HIP_TRY(hipGetDevice(&dev));
      int64_t items[2] = {0, 0};
      for (int c = 0; c < 2; ++c)
        for (const GemmList& l : W.lists[rho][c]) items[c] += l.items;
      const TuneKey key{dev, kBatchRole[rho], 2,        B->general ? 1 : 0,    W.tile_g[rho][0],
                        n,   items[0],        items[1], (int64_t)(W.sig >> 1)};
      const TileShape cand[2] = {{W.tile_g[rho][0], W.tile_g[rho][0]}, {W.tile_g[rho][1], W.tile_g[rho][1]}};
      return tuned(key, 2, cand, st, launch);
    };
    // split products: the per-fragment digit splits, then one grouped launch
    // per reduction window (r = 0: (ia|jb), r = 1: Gamma)
    auto run_split = [&](int r) -> int {
      int rc2;
      // the digit splits of every fragment of the wave: one launch per list and mode
      auto dlaunch = [&](int list, int mode, int S) -> int {
        const int64_t blocks = W.blocks_dop[list][mode];
        if (W.n_dop[list] == 0 || blocks == 0) return RIMP2_OK;
        if (int rc3 = check_grid(blocks, "digit split")) return rc3;
        const DigitOp* ops = (const DigitOp*)at(W.o_dop[list]);
        const int64_t* pre = (const int64_t*)at(W.o_dpre[list][mode]);
        return traced(R_SPLIT, 0, 0, 0, st, [&] {
          switch (mode) {
            case 0: RIMP2_SWITCH_S(S, hipLaunchKernelGGL((digit_split_grouped<SS, 0>), dim3((unsigned)blocks),
                                                        dim3(256), 0, st, ops, pre, W.n_dop[list])); break;
            case 1: hipLaunchKernelGGL((digit_split_grouped<1, 1>), dim3((unsigned)blocks), dim3(256), 0, st, ops,
                                       pre, W.n_dop[list]); break;
            case 2: hipLaunchKernelGGL((digit_split_grouped<1, 2>), dim3((unsigned)blocks), dim3(256), 0, st, ops,
                                       pre, W.n_dop[list]); break;
            default: RIMP2_SWITCH_S(S, hipLaunchKernelGGL((digit_split_grouped<SS, 3>), dim3((unsigned)blocks),
                                                         dim3(256), 0, st, ops, pre, W.n_dop[list])); break;
          }
        });
      };
      const int sv = B->plan[W.frags[0]].sv, sg = B->plan[W.frags[0]].sg;
      if (r == 0) {
        if ((rc2 = dlaunch(0, 0, sv))) return rc2;
      } else if ((rc2 = dlaunch(1, 1, sg)) || (rc2 = dlaunch(1, 2, sg)) || (rc2 = dlaunch(2, 3, sg)) ||
                 (rc2 = dlaunch(3, 0, sg))) {
        return rc2;
      }
      if (W.n_oz[r] == 0) return RIMP2_OK;
      const int S = r == 0 ? B->plan[W.frags[0]].sv : B->plan[W.frags[0]].sg;
      for (int w = 0; w < W.win_oz[r]; ++w) {
        const Grouped<OzParams> G{(const OzParams*)at(W.o_oz[r]), (const int64_t*)at(W.o_oz_pre[r]), W.n_oz[r],
                                  grouped_block(W.items_oz[r], kOperandBlock)};
        const int role = r == 0 ? R_INTS8 : R_GAMMA8;
        RIMP2_SWITCH_S(S, rc2 = launch_oz8_grouped<SS>(G, W.items_oz[r], W.side_oz[r], w, role, st));
        if (rc2) return rc2;
      }
      return RIMP2_OK;
    };
    if ((rc = B->split ? run_split(0) : run_role(0))) return rc;
    if ((rc = traced(R_AMP, 0, 0, 0, st, [&] {
           if (W.amp_blocks[0])
             hipLaunchKernelGGL((amplitude_grouped<32, 256>), dim3((unsigned)W.amp_blocks[0]), dim3(256), 0, st,
                                (const AmpDesc*)at(W.o_amp), (const int64_t*)at(W.o_amp_pre[0]), n);
           if (W.amp_blocks[1])
             hipLaunchKernelGGL((amplitude_grouped<64, 512>), dim3((unsigned)W.amp_blocks[1]), dim3(512), 0, st,
                                (const AmpDesc*)at(W.o_amp), (const int64_t*)at(W.o_amp_pre[1]), n);
         })))
      return rc;
    if ((rc = B->split ? run_split(1) : run_role(1)) || (rc = run_role(2)) || (rc = run_role(3))) return rc;
    if (W.nred && (rc = traced(R_REDUCE, 0, 0, 0, st, [&] {
                        hipLaunchKernelGGL(reduce_grouped, dim3((unsigned)W.red_blocks), dim3(256), 0, st,
                                           (const ReduceDesc*)at(W.o_red), (const int64_t*)at(W.o_red_pre), W.nred);
                      })))
      return rc;
    if ((rc = traced(R_ESUM, 0, 0, 0, st, [&] {
           hipLaunchKernelGGL(energy_sum_grouped, dim3((unsigned)n), dim3(256), 0, st, (const FragSmall*)at(W.o_fs));
           if (status_dev)
             hipLaunchKernelGGL(status_copy_grouped, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st,
                                (const FragSmall*)at(W.o_fs), (const int32_t*)at(W.o_idx), n, status_dev);
         })))
      return rc;
  }
  return RIMP2_OK;
}

}  // namespace

extern "C" {

int rimp2_version(void) { return 10000; }

const char* rimp2_last_error(void) { return g_err; }

const char* rimp2_status_string(int s) {
  switch (s) {
    case RIMP2_OK: return "RIMP2_OK";
    case RIMP2_EINVAL: return "RIMP2_EINVAL";
    case RIMP2_ENOMEM: return "RIMP2_ENOMEM";
    case RIMP2_EWORKSPACE: return "RIMP2_EWORKSPACE";
    case RIMP2_EDEVICE: return "RIMP2_EDEVICE";
    case RIMP2_EGAP: return "RIMP2_EGAP";
    case RIMP2_ENOTSUP: return "RIMP2_ENOTSUP";
    case RIMP2_ENOCONV: return "RIMP2_ENOCONV";
    default: return "unknown rimp2 status";
  }
}

int rimp2_workspace_size(int32_t nocc, int32_t nvir, int32_t naux, int32_t want, const rimp2_opts* opts,
                         size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  if (want & ~(RIMP2_WANT_GAMMA | RIMP2_WANT_DENSITY)) return fail(RIMP2_EINVAL, "bad want mask %d", want);
  Plan P;
  int rc = make_plan(nocc, nvir, naux, want & RIMP2_WANT_GAMMA, want & RIMP2_WANT_DENSITY, opts, &P);
  if (rc) return rc;
  *bytes = P.total;
  return RIMP2_OK;
}

int rimp2_fragment(int32_t nocc, int32_t nvir, int32_t naux, const double* B, const double* eps_occ,
                   const double* eps_vir, double* E, double* Gamma, double* P_ij, double* P_ab, double* e_pair,
                   void* workspace, size_t workspace_bytes, const rimp2_opts* opts, void* stream) {
  if (!B || !eps_occ || !eps_vir || !E || !workspace)
    return fail(RIMP2_EINVAL, "B, eps_occ, eps_vir, E and workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  int want, rc;
  if ((rc = want_of(Gamma, P_ij, P_ab, &want))) return rc;
  Plan P;
  if ((rc = make_plan(nocc, nvir, naux, want & RIMP2_WANT_GAMMA, want & RIMP2_WANT_DENSITY, opts, &P))) return rc;
  if (workspace_bytes < P.total)
    return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
  return run_fragment(P, B, eps_occ, eps_vir, E, Gamma, P_ij, P_ab, e_pair, (char*)workspace,
                      opts ? opts->pair_skip : nullptr, (hipStream_t)stream);
}

int rimp2_fragment_noalloc(int32_t nocc, int32_t nvir, int32_t naux, const double* B, const double* eps_occ,
                           const double* eps_vir, double* E, double* Gamma, double* P_ij, double* P_ab,
                           double* e_pair, int32_t* status_dev, const rimp2_opts* opts, void* stream) {
  if (!B || !eps_occ || !eps_vir || !E) return fail(RIMP2_EINVAL, "B, eps_occ, eps_vir and E must not be NULL");
  int want, rc;
  if ((rc = want_of(Gamma, P_ij, P_ab, &want))) return rc;
  Plan P;
  if ((rc = noalloc_plan(nocc, nvir, naux, want, opts, &P))) return rc;
  char* ws = nullptr;
  if ((rc = scratch_address(&ws))) return rc;
  hipStream_t st = (hipStream_t)stream;
  t_noalloc = true;
  rc = run_fragment(P, B, eps_occ, eps_vir, E, Gamma, P_ij, P_ab, e_pair, ws, opts ? opts->pair_skip : nullptr, st);
  if (rc == RIMP2_OK && status_dev) {
    rc = traced(R_STATUS, 0, 0, 8.0, st, [&] {
      hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(64), 0, st, (const int32_t*)(ws + P.off_status),
                         status_dev, 0);
    });
  }
  t_noalloc = false;
  return rc;
}

int rimp2_read_status(const void* workspace, void* stream, int32_t* status) {
  if (!workspace || !status) return fail(RIMP2_EINVAL, "workspace and status must not be NULL");
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  HIP_TRY(hipMemcpy(status, workspace, sizeof(int32_t), hipMemcpyDeviceToHost));
  return RIMP2_OK;
}

int rimp2_batch_create(int32_t nfrag, const rimp2_frag_desc* descs, const rimp2_opts* opts, rimp2_batch* batch,
                       size_t* workspace_bytes) {
  if (!batch || !workspace_bytes) return fail(RIMP2_EINVAL, "batch and workspace_bytes must not be NULL");
  rimp2_batch_s* B = new rimp2_batch_s();
  int rc = batch_plan(nfrag, descs, opts, B);
  if (!rc && B->tables_total) {
    if (hipHostMalloc((void**)&B->host, B->tables_total, hipHostMallocDefault) != hipSuccess) {
      B->host = nullptr;
      rc = fail(RIMP2_EDEVICE, "hipHostMalloc of %zu bytes failed", B->tables_total);
    } else {
      memcpy(B->host, B->blob.data(), B->tables_total);
    }
  }
  if (rc) {
    if (B->host) (void)hipHostFree(B->host);
    delete B;
    return rc;
  }
  *batch = B;
  *workspace_bytes = B->ws_bytes;
  return RIMP2_OK;
}

int rimp2_batch_run(rimp2_batch batch, int32_t* status_dev, void* workspace, size_t workspace_bytes, void* stream) {
  if (!batch) return fail(RIMP2_EINVAL, "batch is NULL");
  return batch_run(batch, status_dev, workspace, workspace_bytes, (hipStream_t)stream, 1);
}

int rimp2_batch_destroy(rimp2_batch batch) {
  if (!batch) return RIMP2_OK;
  if (batch->host) HIP_TRY(hipHostFree(batch->host));
  delete batch;
  return RIMP2_OK;
}

int rimp2_batch_workspace_size(int32_t nfrag, const rimp2_frag_desc* descs, const rimp2_opts* opts, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  rimp2_batch_s B;
  const int rc = batch_plan(nfrag, descs, opts, &B);
  if (rc) return rc;
  *bytes = B.ws_bytes;
  return RIMP2_OK;
}

int rimp2_fragment_batch(int32_t nfrag, const rimp2_frag_desc* descs, int32_t* status_dev, void* workspace,
                         size_t workspace_bytes, const rimp2_opts* opts, void* stream) {
  if (!workspace) return fail(RIMP2_EINVAL, "workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  rimp2_batch_s B;
  int rc = batch_plan(nfrag, descs, opts, &B);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  if (workspace_bytes < B.ws_bytes)
    return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, B.ws_bytes);
  // earlier work on the stream may still use the workspace: wait, then upload the tables synchronously
  HIP_TRY(hipStreamSynchronize(st));
  if (B.tables_total) HIP_TRY(hipMemcpy(workspace, B.blob.data(), B.tables_total, hipMemcpyHostToDevice));
  return batch_run(&B, status_dev, workspace, workspace_bytes, st, 0);
}

int rimp2_timing_enable(int enable) {
  Tracer& T = tracer();
  std::lock_guard<std::mutex> lk(T.mu);
  for (auto& r : T.recs) {
    T.pool.push_back(r.e0);
    T.pool.push_back(r.e1);
  }
  T.recs.clear();
  T.on = enable != 0;
  return RIMP2_OK;
}

int rimp2_timing_collect(rimp2_kernel_stat* stats, int32_t capacity, int32_t* count) {
  if (!count || (capacity > 0 && !stats)) return fail(RIMP2_EINVAL, "bad timing_collect arguments");
  Tracer& T = tracer();
  std::lock_guard<std::mutex> lk(T.mu);
  rimp2_kernel_stat acc[R_NROLES];
  memset(acc, 0, sizeof acc);
  for (int r = 0; r < R_NROLES; ++r) snprintf(acc[r].name, sizeof acc[r].name, "%s", kRoleName[r]);
  for (auto& r : T.recs) {
    HIP_TRY(hipEventSynchronize(r.e1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, r.e0, r.e1));
    rimp2_kernel_stat& a = acc[r.role];
    a.launches += 1;
    a.total_ms += ms;
    a.alg_flops += r.af;
    a.exec_flops += r.ef;
    a.alg_bytes += r.ab;
    T.pool.push_back(r.e0);
    T.pool.push_back(r.e1);
  }
  T.recs.clear();
  int32_t n = 0;
  for (int r = 0; r < R_NROLES; ++r)
    if (acc[r].launches > 0) {
      if (n < capacity) stats[n] = acc[r];
      ++n;
    }
  *count = std::min(n, capacity);
  return RIMP2_OK;
}

int rimp2_autotune_report(rimp2_tune_stat* stats, int32_t capacity, int32_t* count) {
  if (!count || (capacity > 0 && !stats)) return fail(RIMP2_EINVAL, "bad autotune_report arguments");
  Tuner& U = tuner();
  std::lock_guard<std::mutex> lk(U.mu);
  int32_t n = 0;
  for (auto& kv : U.tab) {
    TuneEntry& e = kv.second;
    tune_poll(U, e);
    if (n >= capacity) break;
    rimp2_tune_stat& t = stats[n++];
    memset(&t, 0, sizeof t);
    snprintf(t.role, sizeof t.role, "%s", kRoleName[kv.first.role]);
    t.device = kv.first.dev;
    t.nvar = e.nvar;
    t.best = e.best;
    t.vec = kv.first.vec;
    t.M = kv.first.M; t.N = kv.first.N; t.K = kv.first.K; t.kchunk = kv.first.kchunk;
    for (int v = 0; v < e.nvar && v < 4; ++v) {
      t.tile_m[v] = e.cand[v].bm;
      t.tile_n[v] = e.cand[v].bn;
      t.timed[v] = e.timed[v];
      t.min_ms[v] = e.min_ms[v];
    }
    t.uses = e.uses;
  }
  *count = n;
  return RIMP2_OK;
}

int rimp2_autotune_reset(void) {
  Tuner& U = tuner();
  std::lock_guard<std::mutex> lk(U.mu);
  for (auto& kv : U.tab)
    for (auto& q : kv.second.pend) {
      U.pool.push_back(q.e0);
      U.pool.push_back(q.e1);
    }
  U.tab.clear();
  return RIMP2_OK;
}

// ---- adjacent gradient steps (include/rimp2_gradient.h) --------------------

namespace {
// GEMMs of the gradient steps, with the tile of the smallest estimate (no
// split-K unless the caller planned it): A M-contiguous; A and B K-contiguous
// (bm given); A K-contiguous and B N-contiguous.
int launch_ao(const GemmParams& gp, hipStream_t st, int role, double af, double ab) {
  const int bm = choose_gemm(gp.M, gp.N, gp.K, false, kAoTiles, 1, std::max(1, gp.batch)).bm;
  return bm == 64 ? launch_gemm<64, 64, true, ROLE_AO, false>(gp, st, role, af, ab, false)
                  : launch_gemm<128, 128, true, ROLE_AO, false>(gp, st, role, af, ab, false);
}
int launch_lterm(int bm, const GemmParams& gp, hipStream_t st, int role, double af, double ab) {
  return bm == 64 ? launch_gemm<64, 64, false, ROLE_LTERM, false>(gp, st, role, af, ab, false)
                  : launch_gemm<128, 128, false, ROLE_LTERM, false>(gp, st, role, af, ab, false);
}
int launch_batch(const GemmParams& gp, hipStream_t st, int role, double af, double ab) {
  const int bm = choose_gemm(gp.M, gp.N, gp.K, false, kAoTiles, 1, std::max(1, gp.batch)).bm;
  return bm == 64 ? launch_gemm<64, 64, true, ROLE_BATCH, false>(gp, st, role, af, ab, false)
                  : launch_gemm<128, 128, true, ROLE_BATCH, false>(gp, st, role, af, ab, false);
}
}  // namespace

int rimp2_gamma_metric(int32_t nocc, int32_t nvir, int32_t naux, const double* Gamma, const double* Jm, double* out,
                       void* stream) {
  if (nocc < 1 || nvir < 1 || naux < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  if (!Gamma || !Jm || !out) return fail(RIMP2_EINVAL, "Gamma, Jm and out must not be NULL");
  const int64_t M = (int64_t)nocc * nvir, n = naux;
  const char *g0 = (const char*)Gamma, *g1 = (const char*)(Gamma + M * n), *o0 = (const char*)out,
             *o1 = (const char*)(out + M * n);
  if (o0 < g1 && g0 < o1) return fail(RIMP2_EINVAL, "out must not overlap Gamma");
  GemmParams gp{};
  gp.M = M; gp.N = n; gp.K = n; gp.kchunk = n;
  gp.A = kop(Gamma, n, INT64_MAX, 0);   // row (i,a), reduction Q
  gp.Bk = kop(Jm, n, INT64_MAX, 0);     // row P, reduction Q
  gp.C = out; gp.ldc = n;
  return launch_lterm(choose_gemm(M, n, n, false, kLtermTiles, 1).bm, gp, (hipStream_t)stream, R_GAMMA_METRIC,
                      2.0 * M * n * n, 8.0 * (2.0 * M * n + n * n));
}

int rimp2_gamma_ao_workspace_size(int32_t nocc, int32_t nao, int32_t pcount, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  if (nocc < 1 || nao < 1 || pcount < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  *bytes = align_up(64) + align_up((size_t)8 * nocc * nao * pcount);
  return RIMP2_OK;
}

int rimp2_gamma_ao(int32_t nocc, int32_t nvir, int32_t nao, int32_t naux, int32_t p0, int32_t pcount,
                   const double* Gamma, const double* C_occ, const double* C_vir, double* out, void* workspace,
                   size_t workspace_bytes, void* stream) {
  if (nocc < 1 || nvir < 1 || nao < 1 || naux < 1 || pcount < 1 || p0 < 0 || (int64_t)p0 + pcount > naux)
    return fail(RIMP2_EINVAL, "sizes must be >= 1 and 0 <= p0, p0 + pcount <= naux (nocc=%d nvir=%d nao=%d naux=%d "
                "p0=%d pcount=%d)", nocc, nvir, nao, naux, p0, pcount);
  if (!Gamma || !C_occ || !C_vir || !out || !workspace)
    return fail(RIMP2_EINVAL, "Gamma, C_occ, C_vir, out and workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  size_t need = 0;
  int rc;
  if ((rc = rimp2_gamma_ao_workspace_size(nocc, nao, pcount, &need))) return rc;
  if (workspace_bytes < need) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, need);
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  unsigned long long* status = (unsigned long long*)ws;
  double* H = (double*)(ws + align_up(64));
  const int64_t pc = pcount, na = nao;
  if ((rc = traced(R_STATUS, 0, 0, 8.0, st, [&] {
         hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(256), 0, st, status, 1);
       })))
    return rc;
  // H[i][n][P] = sum_a C_vir[a][n] Gamma[i][a][p0 + P]: one launch over the
  // occupied orbitals (one launch each held 4 workgroups at nao = pcount = 240:
  // 40 x 35 us, 30 us now)
  {
    GemmParams gp{};
    gp.M = na; gp.N = pc; gp.K = nvir; gp.kchunk = nvir;
    gp.Am = NOperand{C_vir, na};
    gp.Bn = NOperand{Gamma + p0, naux};
    gp.batch = nocc; gp.batch_a = 0; gp.batch_b = (int64_t)nvir * naux; gp.split_stride = na * pc;
    gp.C = H; gp.ldc = pc; gp.status = (const int32_t*)status;
    if ((rc = launch_ao(gp, st, R_GAMMA_AO, 2.0 * nocc * na * pc * nvir, 8.0 * nocc * (nvir * (na + pc) + na * pc))))
      return rc;
  }
  // out[m][(n, P)] = sum_i C_occ[i][m] H[i][(n, P)]
  GemmParams gp{};
  gp.M = na; gp.N = na * pc; gp.K = nocc; gp.kchunk = nocc;
  gp.Am = NOperand{C_occ, na};
  gp.Bn = NOperand{H, na * pc};
  gp.C = out; gp.ldc = na * pc; gp.status = (const int32_t*)status;
  return launch_ao(gp, st, R_GAMMA_AO, 2.0 * na * na * pc * nocc, 8.0 * (nocc * na + nocc * na * pc + na * na * pc));
}

namespace {
// Split-K plan of the two L-term GEMMs: M x N outputs over reduction K.
struct LPlan {
  GemmChoice c1, c2;
  size_t part_bytes;
};
LPlan l_plan(int64_t nocc, int64_t nvir, int64_t nmo, int64_t naux) {
  LPlan L;
  L.c1 = choose_gemm(nocc, nmo, nvir * naux, false, kLtermTiles);
  L.c2 = choose_gemm(nvir, nmo, nocc * naux, false, kLtermTiles);
  L.part_bytes = std::max((size_t)8 * L.c1.splits * nocc * nmo, (size_t)8 * L.c2.splits * nvir * nmo);
  return L;
}
}  // namespace

int rimp2_l_terms_workspace_size(int32_t nocc, int32_t nvir, int32_t nmo, int32_t naux, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  if (nocc < 1 || nvir < 1 || nmo < 1 || naux < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  *bytes = align_up(64) + align_up(l_plan(nocc, nvir, nmo, naux).part_bytes);
  return RIMP2_OK;
}

int rimp2_l_terms(int32_t nocc, int32_t nvir, int32_t nmo, int32_t naux, const double* Gamma, const double* I_qa,
                  const double* I_iq, double* L1, double* L2, void* workspace, size_t workspace_bytes, void* stream) {
  if (nocc < 1 || nvir < 1 || nmo < 1 || naux < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  if (!Gamma || !workspace) return fail(RIMP2_EINVAL, "Gamma and workspace must not be NULL");
  if ((L1 == nullptr) != (I_qa == nullptr) || (L2 == nullptr) != (I_iq == nullptr))
    return fail(RIMP2_EINVAL, "L1 needs I_qa and L2 needs I_iq (both or neither)");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  size_t need = 0;
  int rc;
  if ((rc = rimp2_l_terms_workspace_size(nocc, nvir, nmo, naux, &need))) return rc;
  if (workspace_bytes < need) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, need);
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  int32_t* status = (int32_t*)ws;
  double* W = (double*)(ws + align_up(64));
  const LPlan lp = l_plan(nocc, nvir, nmo, naux);
  const double o = nocc, v = nvir, q = nmo, x = naux;
  if ((rc = traced(R_STATUS, 0, 0, 8.0, st, [&] {
         hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(256), 0, st, (unsigned long long*)status, 1);
       })))
    return rc;
  auto run = [&](GemmParams gp, const GemmChoice& c, double* out, double af, double ab) -> int {
    gp.kchunk = cdiv(gp.K, c.splits);
    gp.C = W; gp.ldc = gp.N; gp.split_stride = gp.M * gp.N; gp.status = status;
    const int64_t splits = cdiv(gp.K, cdiv(gp.kchunk, kBK) * kBK);
    int r;
    if ((r = launch_lterm(c.bm, gp, st, R_LTERM, af, ab))) return r;
    const int64_t n = gp.M * gp.N;
    return traced(R_REDUCE, 0, 0, 8.0 * (splits + 1) * n, st, [&] {
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)reduce_blocks(n, splits)), dim3(256), 0, st, out, gp.N,
                         (const double*)W, gp.N, gp.M * gp.N, (int)splits, gp.M, gp.N, 1.0, 0, status);
    });
  };
  if (L1) {   // L'[i][q] = sum over (a, P) of Gamma[i][a][P] I_qa[q][a][P]
    GemmParams gp{};
    gp.M = nocc; gp.N = nmo; gp.K = (int64_t)nvir * naux;
    gp.A = kop(Gamma, gp.K, INT64_MAX, 0);
    gp.Bk = kop(I_qa, gp.K, INT64_MAX, 0);
    if ((rc = run(gp, lp.c1, L1, 2.0 * o * q * v * x, 8.0 * (o + q) * v * x + 8.0 * o * q))) return rc;
  }
  if (L2) {   // L''[a][q] = sum over (i, P) of Gamma[i][a][P] I_iq[i][q][P]
    GemmParams gp{};
    gp.M = nvir; gp.N = nmo; gp.K = (int64_t)nocc * naux;
    gp.A = kop(Gamma, naux, naux, (int64_t)nvir * naux);
    gp.Bk = kop(I_iq, naux, naux, (int64_t)nmo * naux);
    if ((rc = run(gp, lp.c2, L2, 2.0 * v * q * o * x, 8.0 * (v + q) * o * x + 8.0 * v * q))) return rc;
  }
  return RIMP2_OK;
}

}  // extern "C"

// ---- orbital response: antisymmetrised-integral term, Z-vector, W ---------------
namespace {

// The nonzero block of a density: D_rs = D[(r - r0) * ld + s - c0] for r0 <= r
// < r0 + nr, c0 <= s < c0 + nc, and 0 outside it.
struct DBlock {
  const double* D;
  int64_t ld, r0, nr, c0, nc;
};

// c_part[z][P] = sum over the pairs (r, s) of chunk z of the density's block
// of Bf[r][s][P] D[r][s] (fixed chunking: deterministic after the ordered
// reduction).
__global__ __launch_bounds__(256) void coulomb_vector_kernel(const double* Bf, DBlock d, int64_t nmo, int64_t naux,
                                                             int64_t chunk, double* part, const int32_t* status) {
  if (*status != 0) return;
  const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x, z = blockIdx.y;
  if (P >= naux) return;
  const int64_t rs0 = z * chunk, rs1 = min(d.nr * d.nc, rs0 + chunk);
  int64_t r = rs0 / d.nc, q = rs0 - r * d.nc;
  double s = 0.0;
#pragma unroll 8
  for (int64_t rs = rs0; rs < rs1; ++rs) {
    s += Bf[((d.r0 + r) * nmo + d.c0 + q) * naux + P] * d.D[r * d.ld + q];
    const bool next = ++q == d.nc;
    q = next ? 0 : q;
    r += next ? 1 : 0;
  }
  part[z * naux + P] = s;
}

// The antisymmetrised term G[p][q] = 2 sum_P Bf[r0 + p][c0 + q][P] c[P] - sum_s
// Kp[s][p][q] (the splits of the exchange product) for p < nrows, q < ncols.
// A workgroup takes kCombine neighbouring (p, q): its waves two each for the sum
// over P (lanes over P), all of them together for the sums over the splits
// (lanes over the pairs first, so that a split's row is read in whole sectors);
// every sum in a fixed order.  Bound by the read of Bf.  A launch
// of its own for the splits before one wave per (p, q) took 7 + 11 us at 200 x
// 40 pairs of 720; the splits read by that wave, one double a sector, 18; this 13.
// ROLE 0 writes G to F (row stride ldf).  For the Z-vector's rows a and columns
// i (gap = (eps_a - eps_i)/2):
//   ROLE 1  F = gap x[a][i] + G                                (operator)
//   ROLE 2  F = L2[a][i] - L1[i][nocc + a] - G (right-hand side), diag = gap +
//           sum_P Bf[a][i][P]^2 (the operator's diagonal), x = F / diag
struct ZElem {
  const double *eo, *ev, *L1, *L2;
  double *x, *diag;
};
constexpr int kCombine = 8;
template <int ROLE>
__global__ __launch_bounds__(256) void antisym_combine_kernel(const double* Bf, int64_t nmo, int64_t naux,
                                                              int64_t r0, int64_t nrows, int64_t c0, int64_t ncols,
                                                              const double* c, const double* Kp, int splits,
                                                              double* F, int64_t ldf, ZElem z,
                                                              const int32_t* status) {
  if (*status != 0) return;
  __shared__ double sk[4][kCombine], ss[kCombine], sd[kCombine];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t n = nrows * ncols, e0 = (int64_t)blockIdx.x * kCombine;
  // the last workgroup's missing pairs repeat the last pair
  const int64_t e1 = min(n - 1, e0 + 2 * wave), e2 = min(n - 1, e0 + 2 * wave + 1);
  const double* row1 = Bf + ((r0 + e1 / ncols) * nmo + c0 + e1 % ncols) * naux;
  const double* row2 = Bf + ((r0 + e2 / ncols) * nmo + c0 + e2 % ncols) * naux;
  const int64_t ek = min(n - 1, e0 + (t & (kCombine - 1)));
  double k = 0.0, s1 = 0.0, s2 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll 2
  for (int sp = t / kCombine; sp < splits; sp += 256 / kCombine) k += Kp[sp * n + ek];
#pragma unroll 4
  for (int64_t P = lane; P < naux; P += 64) {
    const double b1 = row1[P], b2 = row2[P], cp = c[P];
    s1 += b1 * cp;
    s2 += b2 * cp;
    if (ROLE == 2) { d1 += b1 * b1; d2 += b2 * b2; }
  }
  for (int off = 32; off > 0; off >>= 1) {
    if (off >= kCombine) k += __shfl_down(k, off, 64);
    s1 += __shfl_down(s1, off, 64);
    s2 += __shfl_down(s2, off, 64);
    if (ROLE == 2) { d1 += __shfl_down(d1, off, 64); d2 += __shfl_down(d2, off, 64); }
  }
  if (lane < kCombine) sk[wave][lane] = k;
  if (lane == 0) {
    ss[2 * wave] = s1; ss[2 * wave + 1] = s2;
    if (ROLE == 2) { sd[2 * wave] = d1; sd[2 * wave + 1] = d2; }
  }
  __syncthreads();
  const int64_t e = e0 + t;
  if (t >= kCombine || e >= n) return;
  const int64_t p = e / ncols, q = e - p * ncols;
  const double g = 2.0 * ss[t] - (((sk[0][t] + sk[1][t]) + sk[2][t]) + sk[3][t]);
  if (ROLE == 0) {
    F[p * ldf + q] = g;
    return;
  }
  const double gap = (z.ev[p] - z.eo[q]) / 2.0;
  if (ROLE == 1) {
    F[e] = gap * z.x[e] + g;
  } else {
    const double rhs = (z.L2[p * nmo + q] - z.L1[q * nmo + ncols + p]) - g, dg = gap + sd[t];
    F[e] = rhs;
    z.diag[e] = dg;
    z.x[e] = rhs / dg;
  }
}

struct AntisymPlan {
  int64_t nmo, naux, nrows, ncols, nr, nc, chunks, chunk;
  bool rows_first;
  GemmChoice c_k;
  size_t off_status, off_cpart, off_c, off_Y, off_Kp, total;
};

// nrows x ncols results from a density whose nonzero block is nr x nc.
AntisymPlan antisym_plan(int64_t nmo, int64_t naux, int64_t nrows, int64_t ncols, int64_t nr, int64_t nc) {
  AntisymPlan A{};
  A.nmo = nmo; A.naux = naux; A.nrows = nrows; A.ncols = ncols; A.nr = nr; A.nc = nc;
  const int64_t npairs = nr * nc;
  A.chunks = std::max<int64_t>(1, std::min<int64_t>(256, npairs / 32));
  A.chunk = cdiv(npairs, A.chunks);
  A.chunks = cdiv(npairs, A.chunk);
  // the exchange part's order: D against Bf's columns (Y) or rows (Z) first,
  // whichever takes fewer multiply-adds
  A.rows_first =
      (double)nrows * nr * nc + (double)nrows * ncols * nr < (double)nc * ncols * nr + (double)nrows * ncols * nc;
  A.c_k = choose_gemm(nrows, ncols, (A.rows_first ? nr : nc) * naux, false, kLtermTiles);
  size_t off = 0;
  A.off_status = off; off = align_up(off + 64);
  A.off_cpart = off; off = align_up(off + 8 * (size_t)A.chunks * naux);
  A.off_c = off; off = align_up(off + 8 * (size_t)naux);
  A.off_Y = off; off = align_up(off + 8 * (size_t)(A.rows_first ? nrows * nr : nc * ncols) * naux);
  A.off_Kp = off; off = align_up(off + 8 * (size_t)A.c_k.splits * nrows * ncols);
  A.total = off;
  return A;
}

// F[p - r0][q - c0] (row stride ldf) = sum_rs G_pq^rs D_rs for the rows
// [r0, r0 + nrows) and columns [c0, c0 + ncols), with G_pq^rs = 2 (pq|rs) -
// (ps|rq) and (pq|rs) = sum_P Bf[p][q][P] Bf[r][s][P]; r and s run over D's
// nonzero block only:
//   Coulomb  2 sum_P Bf[p][q][P] c_P,   c_P = sum_rs Bf[r][s][P] D_rs
//   exchange sum_(s,P) Bf[p][s][P] Y[s][q][P],   Y[s][q][P] = sum_r D_rs Bf[r][q][P]
//         or sum_(r,P) Z[p][r][P] Bf[r][q][P],   Z[p][r][P] = sum_s Bf[p][s][P] D_rs
// A Z-vector operator application (only the virtual-occupied block of D holds
// the vector) at 40/200/720 took 480 us over the whole of D and 80 us over
// its block.  The workspace's status word must be zero (the callers clear it).
template <int ROLE>
int antisym_run(const AntisymPlan& A, const double* Bf, const DBlock& d, int64_t r0, int64_t c0, double* F, int64_t ldf,
                const ZElem& z, char* ws, hipStream_t st) {
  const int64_t nmo = A.nmo, naux = A.naux, nrows = A.nrows, ncols = A.ncols;
  const int32_t* status = (const int32_t*)(ws + A.off_status);
  double* cpart = (double*)(ws + A.off_cpart);
  double* c = (double*)(ws + A.off_c);
  double* Y = (double*)(ws + A.off_Y);
  double* Kp = (double*)(ws + A.off_Kp);
  int rc;
  // c is the trace of Z over r = p, or of Y over s = q, where those run over the
  // same orbitals (the Z-vector's operator, every full density); else a pass
  // over Bf of its own.  At 40/200/720 the pass and its reduction took 24 us, the
  // trace 5.
  const bool trace = A.rows_first ? (r0 == d.r0 && nrows == d.nr) : (c0 == d.c0 && ncols == d.nc);
  auto sum_c = [&](const double* part, int64_t terms, int64_t stride) {
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)reduce_blocks(naux, terms)), dim3(256), 0, st, c, naux,
                       part, naux, stride, (int)terms, (int64_t)1, naux, 1.0, 0, status);
  };
  if (!trace && (rc = traced(R_RESPONSE, 0, 0, 8.0 * d.nr * d.nc * (naux + 1), st, [&] {
         hipLaunchKernelGGL(coulomb_vector_kernel, dim3((unsigned)cdiv(naux, 256), (unsigned)A.chunks), dim3(256), 0,
                            st, Bf, d, nmo, naux, A.chunk, cpart, status);
         sum_c(cpart, A.chunks, naux);
       })))
    return rc;
  GemmParams gk{};
  gk.M = nrows; gk.N = ncols;
  if (A.rows_first) {
    // Z[p][r][P] = sum_s D[r][s] Bf[r0 + p][s][P], one product per row p
    GemmParams gp{};
    gp.M = d.nr; gp.N = naux; gp.K = d.nc; gp.kchunk = d.nc;
    gp.A = kop(d.D, d.ld, INT64_MAX, 0);
    gp.Bn = NOperand{Bf + (r0 * nmo + d.c0) * naux, naux};
    gp.batch = (int32_t)nrows; gp.batch_a = 0; gp.batch_b = nmo * naux; gp.split_stride = d.nr * naux;
    gp.C = Y; gp.ldc = naux; gp.status = status;
    if ((rc = launch_batch(gp, st, R_RESPONSE, 2.0 * nrows * d.nr * d.nc * naux,
                           8.0 * (d.nr * d.nc + (double)nrows * (d.nr + d.nc) * naux))))
      return rc;
    // K[p][q] = sum over (r, P) of Z[p][r][P] Bf[r][c0 + q][P]
    gk.K = d.nr * naux;
    gk.A = kop(Y, d.nr * naux, INT64_MAX, 0);
    gk.Bk = kop(Bf + (d.r0 * nmo + c0) * naux, naux, naux, nmo * naux);
  } else {
    // Y[s][(q, P)] = sum_r D[r][s] Bf[r][c0 + q][P]
    GemmParams gp{};
    gp.M = d.nc; gp.N = ncols * naux; gp.K = d.nr; gp.kchunk = d.nr;
    gp.Am = NOperand{d.D, d.ld};
    gp.Bn = NOperand{Bf + (d.r0 * nmo + c0) * naux, nmo * naux};
    gp.C = Y; gp.ldc = ncols * naux; gp.status = status;
    if ((rc = launch_ao(gp, st, R_RESPONSE, 2.0 * d.nr * d.nc * ncols * naux,
                        8.0 * (d.nr * d.nc + (double)(d.nr + d.nc) * ncols * naux))))
      return rc;
    // K[p][q] = sum over (s, P) of Bf[r0 + p][s][P] Y[s][q][P]
    gk.K = d.nc * naux;
    gk.A = kop(Bf + (r0 * nmo + d.c0) * naux, nmo * naux, INT64_MAX, 0);
    gk.Bk = kop(Y, naux, naux, ncols * naux);
  }
  if (trace) {
    const int64_t terms = A.rows_first ? d.nr : d.nc, width = A.rows_first ? d.nr : ncols;
    if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * (terms + 1) * naux, st, [&] { sum_c(Y, terms, (width + 1) * naux); })))
      return rc;
  }
  gk.kchunk = cdiv(gk.K, A.c_k.splits);
  gk.C = Kp; gk.ldc = ncols; gk.split_stride = nrows * ncols; gk.status = status;
  const int64_t splits = cdiv(gk.K, cdiv(gk.kchunk, kBK) * kBK), n = nrows * ncols;
  if ((rc = launch_lterm(A.c_k.bm, gk, st, R_RESPONSE, 2.0 * n * gk.K, 8.0 * (nrows + ncols) * gk.K))) return rc;
  return traced(R_RESPONSE, 0, 0, 8.0 * n * (naux + splits + 1), st, [&] {
    hipLaunchKernelGGL(antisym_combine_kernel<ROLE>, dim3((unsigned)cdiv(n, kCombine)), dim3(256), 0, st, Bf, nmo, naux,
                       r0, nrows, c0, ncols, (const double*)c, (const double*)Kp, (int)splits, F, ldf, z, status);
  });
}

// D[nmo][nmo]: the blocks given (any may be null: zero); the occupied-virtual
// block is the transpose of D_vo when ov != 0, else zero; hf adds the
// identity on the occupied block.
__global__ __launch_bounds__(256) void assemble_density_kernel(int64_t nocc, int64_t nvir, const double* Doo,
                                                               const double* Dvv, const double* Dvo, int ov, int hf,
                                                               double* D) {
  const int64_t nmo = nocc + nvir, e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nmo * nmo) return;
  const int64_t p = e / nmo, q = e - p * nmo;
  double v = 0.0;
  if (p < nocc && q < nocc) v = Doo ? Doo[p * nocc + q] : 0.0;
  else if (p >= nocc && q >= nocc) v = Dvv ? Dvv[(p - nocc) * nvir + (q - nocc)] : 0.0;
  else if (p >= nocc) v = Dvo ? Dvo[(p - nocc) * nocc + q] : 0.0;
  else v = (Dvo && ov) ? Dvo[(q - nocc) * nocc + p] : 0.0;
  if (hf && p == q && p < nocc) v += 1.0;
  D[e] = v;
}

// CG's vector algebra, one workgroup (its sums in a fixed order), on vectors of
// nov elements; scal = (p.q, r.(r / diag), r.r, rhs.rhs, iterations).  Both set
// the status word once there is nothing left to iterate (r.r <= tol^2 rhs.rhs, or
// the break below), which empties every launch that follows.  Latency-bound: as one
// launch per dot product and update, with a read-back for each dot product, an
// iteration at nov = 8000 spent about 90 us on them; as one launch and one
// read-back about 30, 18 of them in the kernel with its sums over LDS in ten
// barriers each and every vector read once a pass, 11 like this.
constexpr int kCgThreads = 1024;
constexpr int kCgWaves = kCgThreads / 64;
// The sums of N values over the workgroup: a shuffle tree in each wave, then
// one over the waves' totals, which every wave does for itself.
template <int N>
__device__ __forceinline__ void cg_sum(double (&v)[N]) {
  __shared__ double sh[N][kCgWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    for (int off = 32; off > 0; off >>= 1) v[i] += __shfl_down(v[i], off, 64);
    if (lane == 0) sh[i][wave] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    v[i] = sh[i][lane & (kCgWaves - 1)];
    for (int off = kCgWaves / 2; off > 0; off >>= 1) v[i] += __shfl_xor(v[i], off, 64);
  }
}
// x = p (the first iterate), r = rhs - q, p = r / diag.  x is the caller's
// array, first written here, after every read of the caller's inputs: it may lie
// over them.
__global__ __launch_bounds__(kCgThreads) void cg_start_kernel(int64_t n, const double* rhs, const double* diag,
                                                              const double* q, double* x, double* r, double* p,
                                                              double* scal, double tol, int32_t* status) {
  double sum[3] = {0.0, 0.0, 0.0};   // r.(r / diag), r.r, rhs.rhs
  for (int64_t k = threadIdx.x; k < n; k += kCgThreads) {
    const double b = rhs[k], rk = b - q[k], d = diag[k];
    x[k] = p[k];
    r[k] = rk;
    p[k] = rk / d;
    sum[0] += rk * rk / d;
    sum[1] += rk * rk;
    sum[2] += b * b;
  }
  cg_sum(sum);
  if (threadIdx.x == 0) {
    scal[1] = sum[0]; scal[2] = sum[1]; scal[3] = sum[2]; scal[4] = 0.0;
    if (!(sum[1] > tol * tol * sum[2])) *status = 1;
  }
}
// One iteration after q = A p: alpha = rz / p.q, x += alpha p, r -= alpha q,
// p = r / diag + (rz_new / rz) p.  Only scal[0] is written when p.q is not > 0
// (the operator is not positive definite along p).  The first kCgHeld elements
// of each thread stay in registers from the loads to the stores, all loads
// being issued at once; the rest of a longer vector is read again in each of
// the three passes.
constexpr int kCgHeld = 8;
__global__ __launch_bounds__(kCgThreads) void cg_step_kernel(int64_t n, const double* diag, const double* q, double* x,
                                                             double* r, double* p, double* scal, double tol,
                                                             int32_t* status) {
  if (*status != 0) return;
  const int64_t t = threadIdx.x, rest = t + (int64_t)kCgHeld * kCgThreads;
  const double rz = scal[1];
  double hp[kCgHeld], hq[kCgHeld], hr[kCgHeld], hd[kCgHeld], hx[kCgHeld];
#pragma unroll
  for (int j = 0; j < kCgHeld; ++j) {
    const int64_t k = t + (int64_t)j * kCgThreads;
    const bool in = k < n;
    hp[j] = in ? p[k] : 0.0;
    hq[j] = in ? q[k] : 0.0;
    hr[j] = in ? r[k] : 0.0;
    hd[j] = in ? diag[k] : 1.0;
    hx[j] = in ? x[k] : 0.0;
  }
  double pq[1] = {0.0};
#pragma unroll
  for (int j = 0; j < kCgHeld; ++j) pq[0] += hp[j] * hq[j];
  for (int64_t k = rest; k < n; k += kCgThreads) pq[0] += p[k] * q[k];
  cg_sum(pq);
  if (t == 0) scal[0] = pq[0];
  if (!(pq[0] > 0.0)) {
    if (t == 0) *status = 1;
    return;
  }
  const double alpha = rz / pq[0];
  double sum[2] = {0.0, 0.0};   // r.(r / diag), r.r
#pragma unroll
  for (int j = 0; j < kCgHeld; ++j) {
    hr[j] -= alpha * hq[j];
    hd[j] = hr[j] / hd[j];
    sum[0] += hr[j] * hd[j];
    sum[1] += hr[j] * hr[j];
  }
  for (int64_t k = rest; k < n; k += kCgThreads) {
    const double rk = r[k] - alpha * q[k];
    x[k] += alpha * p[k];
    r[k] = rk;
    sum[0] += rk * (rk / diag[k]);
    sum[1] += rk * rk;
  }
  cg_sum(sum);
  const double beta = sum[0] / rz;
#pragma unroll
  for (int j = 0; j < kCgHeld; ++j) {
    const int64_t k = t + (int64_t)j * kCgThreads;
    if (k < n) {
      x[k] = hx[j] + alpha * hp[j];
      r[k] = hr[j];
      p[k] = hd[j] + beta * hp[j];
    }
  }
  for (int64_t k = rest; k < n; k += kCgThreads) p[k] = r[k] / diag[k] + beta * p[k];
  if (t == 0) {
    scal[1] = sum[0]; scal[2] = sum[1]; scal[4] += 1.0;
    if (!(sum[1] > tol * tol * scal[3])) *status = 1;
  }
}

// W[p][q] = (eps_p + eps_q)/2 D[p][q] + (p < nocc ? F[p][q] + L1[p][q] : L2[p - nocc][q]),
// D including the HF identity on the occupied block.
__global__ __launch_bounds__(256) void w_assemble_kernel(int64_t nocc, int64_t nvir, const double* eo,
                                                         const double* ev, const double* D, const double* F,
                                                         const double* L1, const double* L2, double* W) {
  const int64_t nmo = nocc + nvir, e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nmo * nmo) return;
  const int64_t p = e / nmo, q = e - p * nmo;
  const double ep = p < nocc ? eo[p] : ev[p - nocc], eq = q < nocc ? eo[q] : ev[q - nocc];
  double w = (ep + eq) / 2.0 * D[e];
  w += p < nocc ? F[e] + L1[e] : L2[(p - nocc) * nmo + q];
  W[e] = w;
}

struct ZPlan {
  AntisymPlan full, vo;   // right-hand side (both diagonal blocks of D), operator (the virtual-occupied block)
  size_t off_D, off_rhs, off_diag, off_r, off_p, off_q, off_dot, total;
};

ZPlan zvector_plan(int64_t nocc, int64_t nvir, int64_t naux) {
  ZPlan Z{};
  const int64_t nmo = nocc + nvir, nov = nocc * nvir;
  Z.full = antisym_plan(nmo, naux, nvir, nocc, nmo, nmo);
  Z.vo = antisym_plan(nmo, naux, nvir, nocc, nvir, nocc);
  size_t off = std::max(Z.full.total, Z.vo.total);
  Z.off_D = off; off = align_up(off + 8 * (size_t)nmo * nmo);
  for (size_t* o : {&Z.off_rhs, &Z.off_diag, &Z.off_r, &Z.off_p, &Z.off_q}) {
    *o = off;
    off = align_up(off + 8 * (size_t)nov);
  }
  Z.off_dot = off; off = align_up(off + 64);
  Z.total = off;
  return Z;
}

int response_sizes(int32_t nocc, int32_t nvir, int32_t naux) {
  if (nocc < 1 || nvir < 1 || naux < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  const double nmo = (double)nocc + nvir;
  if (nmo * nmo * naux >= 4.6e18 || nmo > (1 << 20)) return fail(RIMP2_EINVAL, "sizes too large");
  return RIMP2_OK;
}

int clear_status(char* ws, hipStream_t st) {
  return traced(R_STATUS, 0, 0, 8.0, st, [&] {
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(256), 0, st, (unsigned long long*)ws, 1);
  });
}

// Reads the CG scalars back (one synchronisation for kCgBatch iterations: a
// read-back and the empty queue after it cost 25 us at 40/200/720, the launches
// of an iteration after the last, which the status word empties, 15).
constexpr int kCgBatch = 4;
int read_scal(const double* d, double* h, hipStream_t st) {
  HIP_TRY(hipMemcpyAsync(h, d, 5 * sizeof(double), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  return RIMP2_OK;
}

}  // namespace

extern "C" {

int rimp2_antisym_workspace_size(int32_t nmo, int32_t naux, int32_t nrows, int32_t ncols, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  if (nmo < 1 || naux < 1 || nrows < 1 || ncols < 1) return fail(RIMP2_EINVAL, "sizes must be >= 1");
  *bytes = antisym_plan(nmo, naux, nrows, ncols, nmo, nmo).total;
  return RIMP2_OK;
}

int rimp2_antisym_term(int32_t nmo, int32_t naux, int32_t r0, int32_t nrows, int32_t c0, int32_t ncols,
                       const double* Bf, const double* D, double* F, int64_t ldf, void* workspace,
                       size_t workspace_bytes, void* stream) {
  if (nmo < 1 || naux < 1 || nrows < 1 || ncols < 1 || r0 < 0 || c0 < 0 || (int64_t)r0 + nrows > nmo ||
      (int64_t)c0 + ncols > nmo || ldf < ncols)
    return fail(RIMP2_EINVAL, "rows [r0, r0 + nrows) and columns [c0, c0 + ncols) must lie in [0, nmo), ldf >= ncols");
  if (!Bf || !D || !F || !workspace) return fail(RIMP2_EINVAL, "Bf, D, F and workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  const AntisymPlan A = antisym_plan(nmo, naux, nrows, ncols, nmo, nmo);
  if (workspace_bytes < A.total) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, A.total);
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = clear_status((char*)workspace, st))) return rc;
  return antisym_run<0>(A, Bf, DBlock{D, nmo, 0, nmo, 0, nmo}, r0, c0, F, ldf, ZElem{}, (char*)workspace, st);
}

int rimp2_zvector_workspace_size(int32_t nocc, int32_t nvir, int32_t naux, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  int rc;
  if ((rc = response_sizes(nocc, nvir, naux))) return rc;
  *bytes = zvector_plan(nocc, nvir, naux).total;
  return RIMP2_OK;
}

int rimp2_zvector(int32_t nocc, int32_t nvir, int32_t naux, const double* Bf, const double* eps_occ,
                  const double* eps_vir, const double* P_ij, const double* P_ab, const double* L1, const double* L2,
                  double* D_ai, double tol, int32_t max_iter, int32_t* iterations, double* rel_residual,
                  void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = response_sizes(nocc, nvir, naux))) return rc;
  if (!Bf || !eps_occ || !eps_vir || !P_ij || !P_ab || !L1 || !L2 || !D_ai || !workspace)
    return fail(RIMP2_EINVAL, "Bf, eps_occ, eps_vir, P_ij, P_ab, L1, L2, D_ai and workspace must not be NULL");
  if (!(tol > 0.0) || max_iter < 1) return fail(RIMP2_EINVAL, "tol must be > 0 and max_iter >= 1");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  const ZPlan Z = zvector_plan(nocc, nvir, naux);
  if (workspace_bytes < Z.total) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, Z.total);
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const int64_t no = nocc, nv = nvir, nmo = no + nv, nov = no * nv;
  double* D = (double*)(ws + Z.off_D);
  double* rhs = (double*)(ws + Z.off_rhs);
  double* diag = (double*)(ws + Z.off_diag);
  double* r = (double*)(ws + Z.off_r);
  double* pv = (double*)(ws + Z.off_p);
  double* q = (double*)(ws + Z.off_q);
  double* scal = (double*)(ws + Z.off_dot);
  double* x = D_ai;
  // out = (eps_a - eps_i)/2 v_ai + sum_bj G_ai^bj v_bj
  auto apply = [&](double* v, double* out) -> int {
    return antisym_run<1>(Z.vo, Bf, DBlock{v, no, no, nv, 0, no}, no, 0, out, no,
                          ZElem{eps_occ, eps_vir, nullptr, nullptr, v, nullptr}, ws, st);
  };
  if ((rc = clear_status(ws, st))) return rc;
  // right-hand side L''_ai - L'_ia - sum_pq G_ai^pq Dbar_pq, Dbar = D_ij (+)
  // D_ab; Jacobi preconditioner: the operator's diagonal; first iterate rhs /
  // diagonal, in pv
  if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * nmo * nmo, st, [&] {
         hipLaunchKernelGGL(assemble_density_kernel, dim3((unsigned)cdiv(nmo * nmo, 256)), dim3(256), 0, st, no, nv,
                            P_ij, P_ab, (const double*)nullptr, 0, 0, D);
       })))
    return rc;
  if ((rc = antisym_run<2>(Z.full, Bf, DBlock{D, nmo, 0, nmo, 0, nmo}, no, 0, rhs, no,
                           ZElem{eps_occ, eps_vir, L1, L2, pv, diag}, ws, st)))
    return rc;
  // preconditioned conjugate gradients
  int32_t* done = (int32_t*)(ws + Z.vo.off_status);
  double h[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if ((rc = apply(pv, q))) return rc;
  if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * 5 * nov, st, [&] {
         hipLaunchKernelGGL(cg_start_kernel, dim3(1), dim3(kCgThreads), 0, st, nov, (const double*)rhs,
                            (const double*)diag, (const double*)q, x, r, pv, scal, tol, done);
       })))
    return rc;
  double bb, rr, target;
  int it = 0;
  do {
    for (int b = std::min(kCgBatch, max_iter - it); b > 0; --b) {
      if ((rc = apply(pv, q))) return rc;
      if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * 8 * nov, st, [&] {
             hipLaunchKernelGGL(cg_step_kernel, dim3(1), dim3(kCgThreads), 0, st, nov, (const double*)diag,
                                (const double*)q, x, r, pv, scal, tol, done);
           })))
        return rc;
    }
    if ((rc = read_scal(scal, h, st))) return rc;
    rr = h[2]; bb = h[3]; target = tol * tol * bb; it = (int)h[4];
    // h[0] = p.q: the operator is not positive definite along p
  } while (rr > target && it < max_iter && h[0] > 0.0);
  if (iterations) *iterations = it;
  const double rel_res = bb > 0.0 ? sqrt(rr / bb) : sqrt(rr);
  if (rel_residual) *rel_residual = rel_res;
  if (!(rr <= target))
    return fail(RIMP2_ENOCONV, "Z-vector CG stopped after %d iterations at relative residual %.3e (tol %.3e)", it,
                rel_res, tol);
  return RIMP2_OK;
}

int rimp2_energy_weighted_density_workspace_size(int32_t nocc, int32_t nvir, int32_t naux, size_t* bytes) {
  if (!bytes) return fail(RIMP2_EINVAL, "bytes is NULL");
  int rc;
  if ((rc = response_sizes(nocc, nvir, naux))) return rc;
  const int64_t nmo = (int64_t)nocc + nvir;
  const AntisymPlan A = antisym_plan(nmo, naux, nocc, nmo, nmo, nmo);
  *bytes = A.total + align_up(8 * (size_t)nmo * nmo) * 2;
  return RIMP2_OK;
}

int rimp2_energy_weighted_density(int32_t nocc, int32_t nvir, int32_t naux, const double* Bf, const double* eps_occ,
                                  const double* eps_vir, const double* P_ij, const double* P_ab, const double* D_ai,
                                  const double* L1, const double* L2, double* W, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = response_sizes(nocc, nvir, naux))) return rc;
  if (!Bf || !eps_occ || !eps_vir || !P_ij || !P_ab || !D_ai || !L1 || !L2 || !W || !workspace)
    return fail(RIMP2_EINVAL, "Bf, eps_occ, eps_vir, P_ij, P_ab, D_ai, L1, L2, W and workspace must not be NULL");
  if ((uintptr_t)workspace % kAlign) return fail(RIMP2_EWORKSPACE, "workspace must be 256-byte aligned");
  size_t need = 0;
  if ((rc = rimp2_energy_weighted_density_workspace_size(nocc, nvir, naux, &need))) return rc;
  if (workspace_bytes < need) return fail(RIMP2_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, need);
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const int64_t no = nocc, nv = nvir, nmo = no + nv;
  const AntisymPlan A = antisym_plan(nmo, naux, nocc, nmo, nmo, nmo);
  double* Dm = (double*)(ws + A.total);
  double* F = (double*)(ws + A.total + align_up(8 * (size_t)nmo * nmo));
  const unsigned gd = (unsigned)cdiv(nmo * nmo, 256);
  if ((rc = clear_status(ws, st))) return rc;
  // D^MP2 (every block) for the antisymmetrised term of the occupied rows
  if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * nmo * nmo, st, [&] {
         hipLaunchKernelGGL(assemble_density_kernel, dim3(gd), dim3(256), 0, st, no, nv, P_ij, P_ab, D_ai, 1, 0, Dm);
       })))
    return rc;
  if ((rc = antisym_run<0>(A, Bf, DBlock{Dm, nmo, 0, nmo, 0, nmo}, 0, 0, F, nmo, ZElem{}, ws, st))) return rc;
  // D = D^HF + D^MP2 for the energy-weighted piece
  if ((rc = traced(R_RESPONSE, 0, 0, 8.0 * nmo * nmo, st, [&] {
         hipLaunchKernelGGL(assemble_density_kernel, dim3(gd), dim3(256), 0, st, no, nv, P_ij, P_ab, D_ai, 1, 1, Dm);
       })))
    return rc;
  return traced(R_RESPONSE, 0, 0, 8.0 * 4 * nmo * nmo, st, [&] {
    hipLaunchKernelGGL(w_assemble_kernel, dim3(gd), dim3(256), 0, st, no, nv, eps_occ, eps_vir, (const double*)Dm,
                       (const double*)F, L1, L2, W);
  });
}

}  // extern "C"
