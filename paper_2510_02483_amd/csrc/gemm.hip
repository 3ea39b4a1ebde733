// The matrix products: choice of tile and split of K, launch order, and the
// kernels that finish a split K.  The product kernel itself is in gemm_tile.h,
// instantiated per operand layout in gemm_nt.hip, gemm_nn.hip and gemm_tn.hip.
#include <algorithm>
#include <atomic>

#include "gemm_tile.h"

namespace ls {

namespace {

// F (already holding slice 0's result, with the accumulate read) += the
// partial sums of slices 1 .. ksplit-1, added in slice order.  N % 4 == 0.
__global__ __launch_bounds__(256) void kpart_reduce_kernel(GemmArgs p) {
  const int64_t per = (int64_t)p.M * p.N, n4 = per / 4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const int64_t e = 4 * i;
    const int m = (int)(e / p.N), n = (int)(e - (int64_t)m * p.N);
    const int sg = m >= p.f_start[2] ? 2 : (m >= p.f_start[1] ? 1 : 0);
    float* base = sg == 2 ? p.F[2] : (sg == 1 ? p.F[1] : p.F[0]);
    const int fs = sg == 2 ? p.f_start[2] : (sg == 1 ? p.f_start[1] : 0);
    float* dst = base + (int64_t)(m - fs) * p.ldf + n;
    f32x4 v = *(const f32x4*)dst;
    for (int j = 0; j < p.ksplit - 1; ++j) v += *(const f32x4*)(p.kpart + j * per + e);
    *(f32x4*)dst = v;
  }
}

// Finishes a bf16-output product whose K was split: the slices' fp32 partial
// sums ([slice][M][N]) are added in slice order and go through the product's
// epilogue.  A thread takes 8 columns of a row (and their partner columns: the
// other half of the head, the up feature).  Bound by memory: reads ksplit M N
// fp32 values, at most the last-level cache's size (make_plan) and most of them
// still in it (12.4 MB for 2 slices of 504 x 3072: 5 us).
LS_DEV void sum_slices8(const GemmArgs& p, int m, int n, float v[8]) {
  const float* src = p.kpart + (int64_t)m * p.N + n;
  const int64_t per = (int64_t)p.M * p.N;
  f32x4 lo = *(const f32x4*)src, hi = *(const f32x4*)(src + 4);
  for (int j = 1; j < p.ksplit; ++j) {
    lo += *(const f32x4*)(src + j * per);
    hi += *(const f32x4*)(src + j * per + 4);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = lo[e];
    v[4 + e] = hi[e];
  }
}
template <int EPI>
__global__ __launch_bounds__(256) void ksplit_finish_kernel(GemmArgs p) {
  constexpr bool PAIR = EPI == EPI_ROPE || EPI == EPI_ROPE64;
  // items per row: features (SwiGLU forward), column pairs (RoPE) or columns, 8 at a time
  const int per_row = (EPI == EPI_GLU_FWD ? p.glu_I : PAIR ? p.N / 2 : p.N) / 8;
  const int64_t items = (int64_t)p.M * per_row;
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < items; x += (int64_t)gridDim.x * 256) {
    const int m = (int)(x / per_row), c = (int)(x - (int64_t)m * per_row) * 8;
    float a[8], b[8];
    if constexpr (EPI == EPI_GLU_FWD) {
      const int n = (c >> 6) * 128 + (c & 63);  // gate column of feature c; up: 64 further
      sum_slices8(p, m, n, a);
      sum_slices8(p, m, n + 64, b);
      store_glu_fwd8(p, m, c, a, b);
    } else if constexpr (PAIR) {
      constexpr int HD = EPI == EPI_ROPE ? 128 : 64;
      const int n = c / (HD / 2) * HD + c % (HD / 2);
      sum_slices8(p, m, n, a);
      sum_slices8(p, m, n + HD / 2, b);
      store_rope8<HD>(p, m, n, a, b);
    } else {
      sum_slices8(p, m, c, a);
      if constexpr (EPI == EPI_GLU_BWD) store_glu_bwd8(p, m, c, a);
      else if constexpr (EPI == EPI_RESID) store_resid8(p, m, c, a);
      else *(u32x4*)(p.C + (int64_t)m * p.ldc + c) = pack8f(a);
    }
  }
}

int compute_units() {
  static const int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        v <= 0)
      v = 256;
    return v;
  }();
  return n;
}

constexpr int64_t LLC_BYTES = (int64_t)256 << 20;  // last-level cache

// Tile rows per group of the launch order (map_tile) for an M x N x K product
// in BM x BN tiles.  Two caches decide it.  The workgroups an XCD runs at once
// (one per CU, 32) cover g tile rows x 32/g tile columns and stream g A panels
// of BM rows and 32/g B panels of BN rows along K through its 4 MB L2: fewer
// panel rows, fewer L2 misses (4 for 256 x 192 tiles, 8 for 192 x 256).  And
// the panels the whole chip reads in its first round of workgroups should fit
// the 256 MB last-level cache, or every round fetches them from HBM again:
// for K = 16384 and 368 MB of operands only g = 2 keeps a round within it.
// So: among g = 8, 4, 2 whose first round fits, the fewest panel rows (the
// larger g on a tie); if none fits, the smallest first-round footprint.
int group_rows(int M, int N, int K, int bm, int bn) {
  const int tiles_m = (M + bm - 1) / bm, tiles_n = (N + bn - 1) / bn;
  const int ncu = compute_units(), round = std::min(tiles_m * tiles_n, ncu), per_xcd = std::max(ncu / 8, 1);
  constexpr int MAX_TILES = 4096;  // per dimension (no allocation in a call): larger grids keep 8
  if (tiles_m > MAX_TILES || tiles_n > MAX_TILES) return 8;
  int best = 8;
  bool best_fits = false;
  int64_t best_rows = 0, best_bytes = 0;
  char used_m[MAX_TILES], used_n[MAX_TILES];
  for (int g : {8, 4, 2}) {
    std::fill(used_m, used_m + tiles_m, 0);
    std::fill(used_n, used_n + tiles_n, 0);
    for (int wg = 0; wg < round; ++wg) {
      int tm, tn;
      map_tile(wg, tiles_m, tiles_n, g, tm, tn);
      used_m[tm] = used_n[tn] = 1;
    }
    const int64_t panels = (int64_t)std::count(used_m, used_m + tiles_m, 1) * bm +
                           (int64_t)std::count(used_n, used_n + tiles_n, 1) * bn;
    const int64_t bytes = panels * K * 2, rows = (int64_t)g * bm + (int64_t)(per_xcd / g) * bn;
    const bool fits = bytes <= LLC_BYTES;
    const bool better = g == 8 || (fits && !best_fits) || (fits == best_fits && (fits ? rows < best_rows : bytes < best_bytes));
    if (better) {
      best = g;
      best_fits = fits;
      best_rows = rows;
      best_bytes = bytes;
    }
  }
  return best;
}

std::atomic<int> g_tile_override{0};  // 0: automatic, else 1000 * BM + BN

// ---- choice of the tile and of the split of K ------------------------------------
//
// Each candidate's time is estimated from the number of rounds of workgroups it
// takes and the time of one workgroup, k tiles x time per k tile + fixed part
// (first loads, epilogue, hand-over), with constants measured on the card in us:
//   256 x 256        1.3 per k tile with the chip full (1.05 with a quarter of it), fixed 9
//   narrower sides   proportional to the area, 10% more per 192-wide side (more LDS traffic per flop),
//                    3% for 192 columns with a k-contiguous A (whose B has a third LDS stage)
//   256 x 128        one workgroup per CU, three stages: 0.85 per k tile full, 0.45 with few
//                    workgroups, fixed 6; 8% more with a k-strided operand
//   128 x 128        one workgroup per CU, four LDS stages: 0.49 per k tile full, 0.34 at a third
//                    of the chip, fixed 4.5; two per CU with two stages (more tiles than CUs):
//                    0.97 per k tile of the pair, fixed 6; 12% more with a k-strided operand
//   finishing a split  4.5 and its partial sums written and read back at 2.5 TB/s
// What is about the same for every candidate is left out: the estimate ranks
// them and is no prediction.  Large launches take longer, most of all those whose
// epilogue moves much (SwiGLU backward reads 2 M N saved values and writes as
// many): 8192 x 3072 x 16384 NN 532 estimated, 628 measured; 8192 x 8192 x 3072
// with the SwiGLU backward 286 and 430.
//
// Measured with these choices against 256 x 256 or 256 x 192 alone: 2048 x 2048
// x 22016 327 -> 169 us (256 workgroups where there were 88), 504 x 3072 x 8192
// 106 -> 37 us (two slices), 2048 x 2560 x 2048 36 -> 28 us, 256 x 512 x 256
// 10 -> 6 us; 8192 x 16384 x 3072 stays 256 x 256 (620 us against 760 with 128 x 128).
//
// Grids of more than one round are split as well where that leaves less of the
// last round empty.  Partial sums are held to the size of the last-level cache.
// They are the caller's workspace, and beyond the cache they go to memory and
// back, which leaves little of the gain: 8192 x 6656 x 35840 in three slices (624
// MiB, doubling the MLP's workspace) 3317 us against 3410 unsplit, 4096 rows of it
// (312 MiB) 1560 against 1648.  Within it: 9536 x 2560 x 24816 in two slices (186
// MiB) 1159 against 1396, 4864 x 3400 x 28544 in four (252 MiB) 932 against 1017,
// 12288 x 2048 x 17888 in two (192 MiB) 845 against 957; 432 x 40128 x 8192 with
// the SwiGLU backward in two (132 MiB) 356 against 422 and 128 x 67200 x 6656 with
// the forward (66 MiB) 317 against 325; 5190 x 3328 x 27264 906 in three (198
// MiB), 880 in four (264 MiB), 931 unsplit.

// Slices of K for an fp32 weight-gradient product whose 256 x 256 tiles fill
// at most half the compute units: as many as fill them, at most 8, each at
// least 8 k tiles deep.
int ksplit_of(int M, int N, int K) {
  const int64_t tiles = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  const int ncu = compute_units();
  if (N % 4 != 0 || tiles == 0 || 2 * tiles > ncu) return 1;
  const int64_t s = std::min<int64_t>(std::min<int64_t>(ncu / tiles, ((int64_t)K + KT - 1) / KT / 8), 8);
  return s < 2 ? 1 : (int)s;
}

// Floats of kpart that `ks` slices need (slice 0 of a weight gradient goes to its buffer).
int64_t kpart_need(const GemmArgs& a, int ks) {
  return ks <= 1 ? 0 : (int64_t)(a.epi == EPI_F32 ? ks - 1 : ks) * a.M * a.N;
}

// forced: 0, or the tile shape of ls_gemm_tile_override (1000 BM + BN).
GemmPlan make_plan(const GemmArgs& a, int64_t kpart_floats, int forced) {
  const bool nt = a.a_kcontig && a.b_kcontig, f32 = a.epi == EPI_F32;
  // 192-wide tiles of a k-contiguous B put a wave's blocks in two 64-row segments: one buffer only
  const bool n192 = nt ? (a.epi == EPI_BF16 || a.epi == EPI_RESID) && a.b_start[1] >= a.N : a.epi != EPI_GLU_BWD;
  const bool m192 = f32;
  const int ncu = compute_units();
  const int64_t ktiles = ((int64_t)a.K + KT - 1) / KT;
  GemmPlan best;
  if (forced) {
    const int bm = forced / 1000, bn = forced % 1000;
    if ((bm == 256 || m192) && (bn == 256 || n192)) {
      best.bm = bm;
      best.bn = bn;
    }
    if (f32) best.ks = ksplit_of(a.M, a.N, a.K);
    while (best.ks > 1 && kpart_need(a, best.ks) > kpart_floats) --best.ks;
    if (best.ks > 1) best.bm = best.bn = 256;
    return best;
  }
  double best_us = 0.0;
  auto consider = [&](int bm, int bn, int ks) {
    if (kpart_need(a, ks) > std::min(kpart_floats, LLC_BYTES / 4)) return;
    const int64_t wgs = (int64_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * ks;
    const double kt = (double)((ktiles + ks - 1) / ks);
    GemmPlan p;
    p.bm = bm;
    p.bn = bn;
    p.ks = ks;
    double us;
    if (bn == 128 && bm == 256) {
      const double fill = std::min(1.0, (double)wgs / ncu);
      us = (double)((wgs + ncu - 1) / ncu) * (kt * (0.45 + 0.40 * fill) * (nt ? 1.0 : 1.08) + 6.0);
    } else if (bm == 128) {
      p.deep = wgs <= ncu;
      const int64_t slots = p.deep ? ncu : 2 * ncu;
      const double fill = std::min(1.0, (double)wgs / slots);
      const double per = (p.deep ? 0.26 + 0.23 * fill : 0.30 + 0.67 * fill) * (nt ? 1.0 : 1.12);
      us = (double)((wgs + slots - 1) / slots) * (kt * per + (p.deep ? 4.5 : 6.0));
    } else {
      const double fill = std::min(1.0, (double)wgs / ncu);
      const double per = (0.95 + 0.35 * fill) * (bm * bn / 65536.0) * (bm == 192 ? 1.1 : 1.0) *
                         (bn == 192 ? (a.a_kcontig ? 1.03 : 1.1) : 1.0);
      us = (double)((wgs + ncu - 1) / ncu) * (kt * per + 9.0);
    }
    if (ks > 1) us += 4.5 + (double)ks * a.M * a.N * 4.0 / 2.5e6;
    if (best_us == 0.0 || us < best_us) {
      best = p;
      best_us = us;
    }
  };
  for (int bm : {256, 192})
    for (int bn : {256, 192})
      if ((bm == 256 || m192) && (bn == 256 || n192)) consider(bm, bn, 1);
  if (f32) {
    const int ks = ksplit_of(a.M, a.N, a.K);
    if (ks > 1) consider(256, 256, ks);
  }
  // slices at least 8 k tiles deep
  for (int ks = 1; ks <= 8 && (ks == 1 || ktiles >= 8 * ks); ++ks) {
    consider(128, 128, ks);
    consider(256, 128, ks);
    if (ks > 1 && !f32 && a.epi != EPI_GLU_FWD) consider(256, 256, ks);
  }
  return best;
}

}  // namespace

int gemm_tile_override(int bm, int bn) {
  if (bm == 0 && bn == 0) {
    g_tile_override.store(0);
    return 0;
  }
  if ((bm != 256 && bm != 192) || (bn != 256 && bn != 192)) return -1;
  g_tile_override.store(bm * 1000 + bn);
  return 0;
}

// Workspace sizes come from this, so it does not look at the tile override: a
// workspace serves every setting, and one switched by another thread during a
// call cannot make a launch need more than the call has checked.
int64_t gemm_kpart_floats(const GemmArgs& a) {
  int64_t need = kpart_need(a, make_plan(a, INT64_MAX, 0).ks);
  // the split a forced tile shape would use
  if (a.epi == EPI_F32) need = std::max(need, kpart_need(a, ksplit_of(a.M, a.N, a.K)));
  return need;
}

GemmPlan gemm_plan(const GemmArgs& a, int64_t kpart_floats) {
  return make_plan(a, kpart_floats, g_tile_override.load(std::memory_order_relaxed));
}

hipError_t gemm(const GemmArgs& args, hipStream_t s) {
  GemmArgs a = args;
  // A k-contiguous B split over buffers (or gate/up interleaved) is loaded a
  // wave's 64 rows at a time from one buffer: segments start at multiples of 64.
  if (a.b_kcontig && ((a.b_start[1] % 64 && a.b_start[1] < a.N) || (a.b_start[2] % 64 && a.b_start[2] < a.N)))
    return hipErrorInvalidValue;
  if (!a.a_kcontig && a.b_kcontig) return hipErrorInvalidValue;
  const GemmPlan p = gemm_plan(a, a.kpart ? a.kpart_floats : 0);
  a.ksplit = p.ks;
  a.group_m = group_rows(a.M, a.N, a.K, p.bm, p.bn);
  const GemmTile t = p.bm == 128 ? (p.deep ? TILE_128_DEEP : TILE_128)
                     : p.bn == 128 ? TILE_256x128
                                 : p.bm == 256 ? (p.bn == 256 ? TILE_256 : TILE_256x192)
                                               : (p.bn == 256 ? TILE_192x256 : TILE_192);
  const int epi = a.epi;
  if (p.ks > 1 && t == TILE_256 && epi != EPI_F32) a.epi = EPI_PART;
  hipError_t e = a.a_kcontig ? (a.b_kcontig ? gemm_nt(a, t, s) : gemm_nn(a, t, s)) : gemm_tn(a, t, s);
  a.epi = epi;
  if (e != hipSuccess || p.ks == 1) return e;
  const int64_t items = a.epi == EPI_F32 ? (int64_t)a.M * a.N / 4 : (int64_t)a.M * a.N / 8;
  const dim3 grid((unsigned)std::min<int64_t>((items + 255) / 256, 256 * 8)), block(256);
  switch (a.epi) {
    case EPI_F32: hipLaunchKernelGGL(kpart_reduce_kernel, grid, block, 0, s, a); break;
    case EPI_BF16: hipLaunchKernelGGL((ksplit_finish_kernel<EPI_BF16>), grid, block, 0, s, a); break;
    case EPI_RESID: hipLaunchKernelGGL((ksplit_finish_kernel<EPI_RESID>), grid, block, 0, s, a); break;
    case EPI_ROPE:
      if (a.head_dim == 64) hipLaunchKernelGGL((ksplit_finish_kernel<EPI_ROPE64>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((ksplit_finish_kernel<EPI_ROPE>), grid, block, 0, s, a);
      break;
    case EPI_GLU_FWD: hipLaunchKernelGGL((ksplit_finish_kernel<EPI_GLU_FWD>), grid, block, 0, s, a); break;
    case EPI_GLU_BWD: hipLaunchKernelGGL((ksplit_finish_kernel<EPI_GLU_BWD>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ls
