// Host-side planning of the kernels' work: the march's workspace layout,
// sample capacity and light-march order; the conv layers' tile heights and
// split-K factors; the channel adapters' supported widths.  Host code only
// (no kernels), shared by the entry points and the kernels' launchers.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace lnm {

// ---------------------------------------------------------------- march
int march_capacity(const MarchDev& m) {
  double d2 = 0.0;
  const int n[3] = {m.nx, m.ny, m.nz};
  for (int a = 0; a < 3; ++a) d2 += (1.0 + 1.0 / n[a]) * (1.0 + 1.0 / n[a]);
  return (int)std::ceil(std::sqrt(d2) / (double)m.h) + 2;
}

static size_t a256(size_t x) { return (x + 255) / 256 * 256; }
int bricks_along(int n) { return (n >> 2) + 1; }
size_t bricks_bytes(int nx, int ny, int nz) {
  return sizeof(float) * kBrickSlot * (size_t)bricks_along(nx) * bricks_along(ny) * bricks_along(nz);
}

// Bricked grids above this size (the eight XCDs' L2s together) take the z
// order: at 256^3 / 1024^2 the march took 4.30 ms in bands, 2.73 in z order on
// bricks and takes 1.7 on plane pairs.  Smaller grids whose planes do not fit
// in LDS stay in bands, which took 0.68 to 1.5 of the z order's time with pairs
// (7 to 30 MB of bricks, planes of 160 x 160 to 200 x 200, 64 to 700 pixels a
// side; 2 to 4 times on planes of 700 columns); so do the left/right lights,
// whose marches leave their z cell: 0.61 to 1.2 below the border (112^3 at 367 x
// 662 2.1), 0.62 to 1.4 above it.
constexpr size_t kZOrderBytes = (size_t)32 << 20;
static int tiles_per_band(int W, int H) { return (((W + kTile - 1) / kTile) * ((H + kTile - 1) / kTile) + 7) / 8; }

// Scratch: [K][P] planes t, A, T_{n-1}, T_top, T_bottom; per-pixel counts; the
// counter block; 8 band work lists of (pixel, k) with room for every sample
// of the band's pixels (not in cell order); in the z orders the [K][P]
// z-bucket plane and the z-ordered list (room for every sample); the plane
// pairs, or the bricked grid unless the caller supplies it.
size_t march_scratch_bytes(const MarchDev& m, int K, int W, int H) {
  const size_t P = (size_t)W * H, plane = a256(sizeof(float) * (size_t)K * P);
  const size_t cap = (size_t)tiles_per_band(W, H) * kTile * kTile * K;
  return 5 * plane + a256(sizeof(int) * P) + a256(kCounterBytes) +
         (m.zorder != kOrderCells ? a256(8 * cap * sizeof(int2)) : 0) +
         (m.zorder ? a256((size_t)K * P) + a256(sizeof(int2) * (size_t)K * P) : 0) +
         (m.pairs ? a256(pairs_bytes(m.nx, m.ny, m.nz)) : m.brick ? 0 : a256(bricks_bytes(m.nx, m.ny, m.nz)));
}

// Cell order: the two planes of a cell in LDS, beside the kernel's own
// arrays, within the 160 KB a gfx950 workgroup may allocate; at most 255
// cells (z buckets).
size_t cell_planes_bytes(int nx, int ny) { return 2 * sizeof(float) * (size_t)(nx + 3) * (ny + 3); }
static bool cells_fit(int nx, int ny, int nz) { return cell_planes_bytes(nx, ny) <= kCellLdsBytes && nz < kZBuckets; }

int march_order(int work_order, int light_set, int nx, int ny, int nz) {
  if (work_order == LNM_ORDER_BANDS) return kOrderBands;
  if (work_order == LNM_ORDER_Z) return kOrderLayers;
  if (work_order == LNM_ORDER_CELLS) return cells_fit(nx, ny, nz) ? kOrderCells : -1;
  if (bricks_bytes(nx, ny, nz) > kZOrderBytes) return kOrderLayers;
  return light_set == LNM_LIGHTS_TOP_BOTTOM && cells_fit(nx, ny, nz) ? kOrderCells : kOrderBands;
}

// Plane pairs (z order): a sample is two 16-byte loads (rows j and j + 1 of
// its cell's pair of planes) instead of a brick's four 8-byte ones, and the
// gathers cost by the instruction (17 to 38 cycles for 64 lanes, 8 bytes and
// 16 alike), which bounds the z order's light marches: 1950 -> 1275 us at 256^3
// / 1024^2.  Building them takes what building the bricks takes.  In cell
// order, whose light marches read LDS, they gained nothing over the bricks.
//
// Where the caller gives bricks, the light marches' samples have to repay the
// copy.  Their number goes with the primary samples inside the grid (pixels x
// mean chord / h), the share of them that meet density (pair_hits of 256
// points, looked at on the device) and the steps of a light march beyond the
// dozen that cost alike either way: the copy is made from kPairCost voxels'
// worth on.  140 marches over 136^3 to 256^3 grids, cubic and not, 64 to 512
// pixels a side, both projections, steps of 2, 4 and 8 voxels, full and nearly
// empty grids, buffers cold: below 1.2 products per voxel pairs took 0.83 to
// 1.38 of the bricks' time, above it 0.63 to 0.99 (256^3 at 512^2 0.86).  (The
// bricks for the primary march and the copy once its records are counted: 0.82
// to 1.04 there, as both copies of the grid are then read.)
size_t pairs_bytes(int nx, int ny, int nz) { return 2 * sizeof(float) * (size_t)(nx + 2) * (ny + 2) * (nz + 1); }
// Mean length of a view's rays inside the support box, from 8 x 8 of them.
static double mean_chord(const MarchDev& m, const CamDev& c) {
  const double n[3] = {(double)m.nx, (double)m.ny, (double)m.nz};
  double sum = 0.0;
  for (int p = 0; p < 64; ++p) {
    const double sx = ((p % 8 + 0.5) / 4 - 1) * c.aspect, sy = 1 - (p / 8 + 0.5) / 4;
    double o[3], d[3], len = 0.0;
    for (int a = 0; a < 3; ++a) {
      const double side = sx * c.r[a] + sy * c.u[a];
      o[a] = c.eye[a] + (c.proj == LNM_ORTHOGRAPHIC ? c.half_extent * side : 0.0);
      d[a] = c.f[a] + (c.proj == LNM_ORTHOGRAPHIC ? 0.0 : c.tan_half * side);
      len += d[a] * d[a];
    }
    double t0 = 0.0, t1 = INFINITY;
    for (int a = 0; a < 3; ++a) {
      const double lo = -0.5 / n[a] - o[a], hi = 1 + 0.5 / n[a] - o[a];
      if (d[a] == 0.0) {
        if (lo > 0 || hi < 0) t1 = -1.0;
        continue;
      }
      t0 = std::max(t0, std::min(lo / d[a], hi / d[a]));
      t1 = std::min(t1, std::max(lo / d[a], hi / d[a]));
    }
    if (t1 > t0) sum += (t1 - t0) * std::sqrt(len);
  }
  return sum / 64;
}

constexpr double kPairCost = 1.2;

int march_pairs(MarchDev* m, const CamDev& c) {
  m->pair_hits = m->pair_shift = 0;
  if (m->zorder != kOrderLayers || pairs_bytes(m->nx, m->ny, m->nz) > 0xFFFFFFFFull) return kPairsNone;
  while (m->pair_shift < kBrickShift && (m->nz - 1) >> m->pair_shift >= kZBuckets) ++m->pair_shift;
  if (!m->brick) return kPairsAlways;
  const double steps = 1.0 / m->h, voxels = (double)m->nx * m->ny * m->nz;
  const double samples = (double)c.W * c.H * mean_chord(*m, c) * steps * std::max(steps - 12.0, steps / 8.0);
  const double hits = std::ceil(256.0 * kPairCost * voxels / samples);
  if (!(hits <= 256.0)) return kPairsNone;
  m->pair_hits = (int)hits;
  return kPairsAsked;
}

// Light marches of few steps across the grid do not pay for staging planes in
// LDS and sorting the records.  220 marches of 5 to 20 steps over 16^3 to 128^3
// and oblong grids, views of 32 to 1024 pixels a side: up to 16 steps the bands
// took 0.73 to 1.10 of the cells' time (one march 1.19; the mean 0.91), from
// 16 to 20 0.84 to 1.09 where the view takes under 50000 primary samples in the
// grid and 0.89 to 1.28 above.  (24 x 48 x 192, 19 steps, 348 x 1080: 256 us in
// band order, 210 in cells.)
int march_order_short(int work_order, int order, const MarchDev& m, const CamDev& c) {
  if (work_order != LNM_ORDER_AUTO || order != kOrderCells || 20.0f * m.h < 1.0f) return order;
  return 16.0f * m.h >= 1.0f || (double)c.W * c.H * mean_chord(m, c) < 50000.0 * m.h ? kOrderBands : order;
}

MarchBuf march_buffers(void* ws, const MarchDev& m, int K, int W, int H) {
  char* p = static_cast<char*>(ws);
  const size_t P = (size_t)W * H, plane = a256(sizeof(float) * (size_t)K * P);
  MarchBuf b;
  b.t = reinterpret_cast<float*>(p);
  b.a = reinterpret_cast<float*>(p + plane);
  b.tp = reinterpret_cast<float*>(p + 2 * plane);
  b.tl = reinterpret_cast<float*>(p + 3 * plane);  // two planes
  p += 5 * plane;
  b.cnt = reinterpret_cast<int*>(p);
  p += a256(sizeof(int) * P);
  b.ctr = reinterpret_cast<int*>(p);
  p += a256(kCounterBytes);
  b.cap = (size_t)tiles_per_band(W, H) * kTile * kTile * K;
  b.rec = nullptr;  // cell order reads the records through the per-pixel counts
  if (m.zorder != kOrderCells) {
    b.rec = reinterpret_cast<int2*>(p);
    p += a256(8 * b.cap * sizeof(int2));
  }
  b.zb = nullptr;
  b.srt = nullptr;
  if (m.zorder) {
    b.zb = reinterpret_cast<uint8_t*>(p);
    p += a256((size_t)K * P);
    b.srt = reinterpret_cast<int2*>(p);
    p += a256(sizeof(int2) * (size_t)K * P);
  }
  b.brick = m.pairs || m.brick ? nullptr : reinterpret_cast<float*>(p);
  b.pair = m.pairs ? reinterpret_cast<float*>(p) : nullptr;
  b.nbx = bricks_along(m.nx);
  b.nby = bricks_along(m.ny);
  b.nbz = bricks_along(m.nz);
  b.K = K;
  b.P = (int)P;
  return b;
}

// ---------------------------------------------------------------- conv layers
int conv_splits(long wgs, int nchunks, int target) {
  // grow the split until the layer has `target` workgroups; keep at least
  // two chunks per split
  int s = 1;
  while (wgs * s < target && 2 * (s * 2) <= nchunks && s < 16) s *= 2;
  return s;
}

// Tile height and split-K factor of conv layer i at level size h x w (tiles
// of th x 16 pixels x 32 output channels); the 3-channel input layer is
// never split.  The split grows until the layer has 256 workgroups (fp32) or
// 512 (bf16, fp8), the targets measured fastest per precision with the
// split-K reductions counted (the fp32 networks of nine small inputs with 512
// instead: 0.98 to 1.06 of the time, with 128 0.99 to 1.02).  The height given
// here is that of the fp32 instruction's kernel, which training and calibration
// run, and, for layers too small for more, of the bf16 and fp8 kernel; the split
// fp32 kernel takes its own.  4-row tiles where they need a smaller split than
// 8-row tiles (the deep levels: twice the workgroups without partial sums to
// write, read and reduce) or where 8-row tiles leave one workgroup per CU
// (nothing else on the CU hides a workgroup's chunk-boundary stalls); fp8
// layers, whose LDS footprint lets five 4-row workgroups share a CU, throughout.
//
// The split and the tile height follow the workgroup count of one image, so
// an image's sums (whose order the split sets) are the same alone and in any
// batch.  Where a batch fills the chip without the split (two 8-row
// workgroups per CU), bf16 and fp8 layers run their splits one after the
// other in each workgroup: the same sums without the partial tensors (16 x
// 256^2, 4-level base-32 bf16: 84 us of reductions and the partial stores).
LayerTiling conv_layer_tiling(const lnm_net_s* net, int i, int B, int h, int w) {
  const LayerDesc& d = net->layers[i];
  if (d.ci == 3) return {8, 1, 1};
  const int target = d.prec == LNM_FP32 ? 256 : 512, nch = d.ci_pad / d.ck;
  auto wgs = [&](int th) { return (long)((w + 15) / 16) * ((h + th - 1) / th) * (d.co_pad / kBN); };
  const int s8 = conv_splits(wgs(8), nch, target);
  LayerTiling t{8, s8, 1};
  const bool fp8 = d.prec == LNM_FP8_E4M3;
  if (s8 > 1 || wgs(8) <= 256 || fp8) {
    // the longest fp32 layers (16+ chunks) split on to two workgroups per CU
    // (a 256^2 frame 308 us against 318, other small inputs up to 6%)
    const int s4 = conv_splits(wgs(4), nch, d.prec == LNM_FP32 && nch >= 16 ? 512 : target);
    if (s4 < s8 || wgs(8) <= 256 || fp8) t = {4, s4, 1};
  }
  if (t.splits > 1 && d.prec != LNM_FP32 && B * wgs(8) >= 512 && rows_fit(h, 8)) t = {8, 1, t.splits};
  return t;
}

// Weight gradient of a layer: 32 x 32 channels per workgroup (16 where the
// layer has no more), its pixel tiles cut into as many groups as give the
// layer at most 512 workgroups, the two per CU that fit at once (with 768 the
// second round leaves half the CUs idle: 1010 against 910 us for the layers
// of 8 x 256^2, 4 levels, base 32).  More groups cost partial sums written
// and read back (37 KB per workgroup and way), fewer leave CUs idle.
WgradTiling wgrad_tiling(int co, int ci, int B, int h, int w) {
  WgradTiling t;
  t.wm = co > 16 ? 2 : 1;
  t.wn = ci > 16 ? 2 : 1;
  const int bm = 16 * t.wm, bc = 16 * t.wn;
  t.co_pad = (co + bm - 1) / bm * bm;
  t.ci_pad = (ci + bc - 1) / bc * bc;
  const int tiles = B * ((w + 15) / 16) * ((h + 7) / 8), pairs = (t.co_pad / bm) * (t.ci_pad / bc);
  const int want = std::max(1, std::min(tiles, 512 / pairs));
  t.tiles_per_group = (tiles + want - 1) / want;
  t.groups = (tiles + t.tiles_per_group - 1) / t.tiles_per_group;
  return t;
}

// ---------------------------------------------------------------- channel adapters
bool adapter_width_supported(int c) { return c == 16 || c == 32 || c == 48 || c == 64; }

int adapter_tail_blocks_per_image(int H, int W) { return (H * W + 255) / 256; }

// One wavefront per run of pixels and convolution: at least 256 pixels, at
// most 256 runs (the partial sums stay small beside the pixels' own values).
int adapter_wgrad_run(size_t P) { return (int)std::max<size_t>(256, ((P + 255) / 256 + 15) / 16 * 16); }

// conv5, conv4, conv3, conv1 of three groups: 3 (1 + 2 + 1 + 2) c^2 per run
size_t adapter_wgrad_partial_bytes(size_t P, int c) {
  const size_t run = adapter_wgrad_run(P);
  return sizeof(float) * ((P + run - 1) / run) * 18 * (size_t)c * c;
}

int adapter_tiles(int H, int W) {
  return ((H + kAdaptTileY - 1) / kAdaptTileY) * ((W + kAdaptTileX - 1) / kAdaptTileX);
}

}  // namespace lnm
