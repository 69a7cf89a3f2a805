// forward.cpp -- forward rendering entry points: vr_render (whole volume or
// bricks + composite), vr_render_bricks and vr_composite (the two halves of
// sort-last compositing, paper Sec. 2.4 and 2.5).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "forward.h"
#include "plan.h"
#include "runtime.h"
#include "vr_internal.h"

namespace vr {

namespace {

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// Ring march limits: window floats per slot, and wavefronts per compute unit
// the kernel's registers allow (78 VGPRs: 6 per SIMD).
constexpr int32_t kRingCap = 8192;
constexpr int32_t kRingMaxWaves = 24;
constexpr int32_t kRingWantWaves = 12;  // below this the march starts to wait on its loads
constexpr int32_t kRingMinWaves = 2;
// register-staged cells march: its registers leave room for 4 wavefronts per SIMD
constexpr int32_t kRingRegWaves = 16;
constexpr int32_t kLdsPerCu = 160 * 1024;
// perspective views with rays closer than this many voxels (on the plane
// through the box centre): cells hold 20 rays on average there (their sizes
// follow the brick's densest point) and gathers are as fast (two views of
// 1024 x 1024 x 768 at 1.6 voxels: 8.0 ms against 8.8)
constexpr double kPerspCellPitch = 1.8;
// further apart: samples per second of the cells, and the chains of cells a
// compute unit's wavefronts take one after another (near bricks' wide windows
// leave room for few).  The 24 GiB cube at 3.2 voxels: 11.7 ms per view, 14.7 by
// gathers; 1000^3 at 1.9 and 3.5 voxels: 5.1 and 3.0 ms, 4.0 and 2.0 by gathers
constexpr double kPerspCellRate = 106e9, kPerspChains = 5.0;
// whole-ray termination: every ray through all its bricks in one launch for a
// view on its own (512^3 in 64 bricks at 768^2 1.53 -> 1.24 ms, 700^3 2.28 ->
// 1.88), for rays less than a voxel apart (two views of 300^3 at 768^2 1.15 ->
// 1.03) and for views whose gathers are estimated below this (0.3 ms per 200^2
// view of 64 bricks against 1.6 in 10 launches).  Otherwise launches per front
// of bricks, each working on a compact part of the volume, the views' side by
// side (two views of 1024 x 1024 x 512 6.2 ms against 6.9)
constexpr double kThruBelow = 0.4e-3;
// what a view by cells costs beside its march: their size is searched on the host
// and the launch takes more kernels (checkpointing forward, three views of 35 x 40
// rays through 16 x 6 x 57 voxels 181 us by cells, 81 by gathers; masked 21 x 29
// view of 24 x 23 x 14 voxels 105 and 28)
constexpr double kCellsFixed = 60e-6;

bool near_rays(const Camera& cam) {
  return cam.S / (double)cam.W < 1.1 && (int64_t)cam.W * cam.H >= ((int64_t)1 << 16);
}

// Estimated time of a view's gathers with D lanes per ray: the wavefronts' set-up
// (pixels x D / 64 of them, a bricked view's pixels those of its rectangles, 0.87 ns
// each over the device, more with the table each workgroup copies), the longest ray's
// chain of loads (0.5 us for D samples) and the samples at 182 G/s, falling with the
// distance of the rays, faster the fewer lanes lie along a ray.  Calibrated on 765
// views of one volume (6 to 700 voxels a side, 30 k to 1.7 M pixels, 64 to 4096
// entries, each measured with 1, 4 and 16 lanes): chosen so, a view takes 1.06 times
// its best number's time on average (1.17 with 16 always) and at worst 1.16 times its
// time with 16 lanes.  10 x 301 x 393 in perspective, three 486 x 450 views at step
// 2.7: 143 us with 16 lanes, 61 with 4; two 287 x 821 views of 143 x 117 x 812: 149
// and 315; two 622 x 824 views of 973 x 100 x 78 in eight bricks 114 and 166; two
// 1130 x 1179 views of 8 x 9 x 7: 157 with 4, 76 with 1.
double lanes_time(const Camera& cam, const BoxSums& boxes, double step, int32_t M, int32_t D) {
  const double waves = (double)boxes.pixels * D / 64.0, apart = std::max(1.0, cam.S / (double)cam.W / 1.2);
  const double chord = cam.persp ? 1.5 * boxes.chord : boxes.chord;  // (other rays' ways are longer)
  return waves * 0.87e-9 * (1.0 + M / 1500.0) + chord / step / D * 0.5e-6 +
         boxes.samples * (D == 16 ? std::sqrt(apart) : apart) / 182e9;
}

}  // namespace

int32_t gather_lanes(const Camera& cam, const BoxSums& boxes, double step, int32_t M) {
  const int64_t pixels = boxes.pixels;
  auto time = [&](int32_t D) { return lanes_time(cam, boxes, step, M, D); };
  // (few rays fill the device with 16 lanes only, below 2^18 not with one)
  if (!near_rays(cam) && (pixels < ((int64_t)1 << 15) || time(4) >= 0.95 * time(16))) return 16;
  return pixels >= ((int64_t)1 << 18) && time(1) < 0.7 * time(4) ? 1 : 4;
}

void add_box(BoxSums& s, const Camera& cam, const Box& b, int64_t pixels, double step) {
  const double pitch = cam.S / (double)cam.W;
  const double* d = cam.e3;
  const double e[3] = {(double)(b.hi[0] - b.lo[0]), (double)(b.hi[1] - b.lo[1]), (double)(b.hi[2] - b.lo[2])};
  const double vol = e[0] * e[1] * e[2];
  const double area = std::fabs(d[0]) * e[1] * e[2] + std::fabs(d[1]) * e[0] * e[2] + std::fabs(d[2]) * e[0] * e[1];
  const double rays = std::min(area / (pitch * pitch), (double)cam.W * cam.H);
  s.samples += rays * vol / std::max(area, 1.0) / step;
  s.bytes += 4.0 * vol;
  s.pixels += pixels;
  double way = 1e30;
  for (int i = 0; i < 3; i++) way = std::min(way, e[i] / std::max(std::fabs(d[i]), 1e-9));
  s.chord = std::max(s.chord, way);
  for (int i = 0; i < 3; i++) s.most[i] = std::max(s.most[i], b.hi[i] - b.lo[i]);
}

// Estimated times of a view (seconds) by the cell march with the shape fs
// (infinite when null) and by gathers, for boxes marched side by side (and
// `views` views on streams of their own).
//   gathers: 230 G samples/s with rays less than 1.1 voxels apart (4 lanes
//     per ray), else 182 falling with the distance (cache lookups of four row pairs
//     per sample, then lines used by fewer and fewer rays): 140 to 165 measured
//     at 1.7 voxels, 110 to 150 at 2.4, 75 to 150 at 2.9, 65 to 95 at 4.6;
//   cells: the larger of 300 G samples/s (vector instructions and LDS), 2.3
//     times the boxes' bytes at 7.2 TB/s (window traffic), and the chain of one
//     wavefront (1.0 us a layer with rays a voxel apart, 1.3 at three, more with
//     the wide windows beyond), which no number of wavefronts shortens; slower where windows leave room
//     for fewer than 12 wavefronts on a compute unit (an 800^3 view at 4.6
//     voxels: 2 wavefronts 2.3 ms, 10 0.8, gathers 0.5 to 0.8).  Rays less than
//     0.75 voxels apart, where the narrowest cells hold more than 64 of them,
//     are left to the gathers (300^3 at 800^2, 0.65 voxels: 1.1 ms by cells,
//     0.49 by gathers).
MarchTimes march_times(const Camera& cam, const BoxSums& boxes, const FootShape* fs, int views) {
  MarchTimes t;
  t.pitch = cam.S / (double)cam.W;
  const double samples = boxes.samples, bytes = boxes.bytes;
  const int64_t layers = fs ? boxes.most[fs->axis] : 0;
  t.samples = samples;
  t.gather = 20e-6 + samples * std::pow(std::max(1.0, t.pitch / 1.2), 0.75) / (near_rays(cam) ? 230e9 : 182e9);
  if (!fs || t.pitch < 0.75) return t;
  t.chain = (double)layers * (0.9e-6 + 0.13e-6 * t.pitch) * (1.0 + std::max(0.0, t.pitch - 4.0) / 4.0);
  t.cells = std::max(std::max(samples / 300e9, 2.3 * bytes / 7.2e12), t.chain / (double)std::max(1, views));
  if (fs->waves > 0) t.cells *= std::max(1.0, 12.0 / (double)fs->waves);
  t.cells += kCellsFixed;
  return t;
}

bool pick_foot(const Camera& cam, const int64_t n[3], int32_t M, bool plain, bool reg_on, int32_t nslots,
               double rays, int32_t pad, int32_t kmax, FootShape& fs, int32_t max_px, int32_t axis) {
  // register-staged cells: a lane's offset inside a window's rows (at most
  // kRingRegLoads instructions of up to 16 rows) must stay below 4 GiB
  const int64_t row_stride = std::max(n[0], n[0] * n[1]);
  const bool reg = plain && reg_on && nslots != 3 && ((int64_t)kRingRegLoads * 16 * row_stride + 256) * 4 < ((int64_t)1 << 32);
  const bool two = rays > 64.0;  // two pixels per lane: half the wavefronts, twice the window loads
  const int32_t rw = two ? kRingRegWaves / 2 : kRingRegWaves;
  return choose_foot(cam, kRingCap, M, kRingMaxWaves, reg ? rw : kRingWantWaves, rays, plain ? nslots : 3, fs, pad,
                     kmax, reg ? rw : 0, two ? 2 * kRingRegLoads : kRingRegLoads, max_px, axis);
}

bool brick_rows_readable(const vr_volume* vol, int32_t brick, int32_t pitch) {
  const int64_t tail = vol->owned || (vol->bricked && vol->materialized) ? 64 : 0;
  int64_t lo[3] = {0, 0, 0}, hi[3], n[3];
  for (int i = 0; i < 3; i++) {
    n[i] = vol->n[i];
    hi[i] = n[i] - 1;
    if (!vol->bricked) continue;
    lo[i] = vol->bdesc[brick].slo[i];
    hi[i] = vol->bdesc[brick].shi[i];
    if (!vol->materialized) {
      if (i == 0) lo[0] = std::min(lo[0], std::max<int64_t>(0, hi[0] + 1 - pitch));  // DevBrick::wlo
      continue;
    }
    hi[i] -= lo[i];  // storage of its own
    lo[i] = 0;
    n[i] = hi[i] + 1;
  }
  return rows_readable(lo, hi, n, pitch, tail);
}

void foot_args(const vr_ctx* ctx, const FootShape& fs, MarchArgs& a, int& wpb) {
  a.foot = 1;
  a.slab_axis = fs.axis;
  a.ring_slot = fs.slot;
  a.ring_nslots = fs.nslots;
  a.ring_reg = fs.reg;
  wpb = fs.reg && ctx->cells_wpb > 0 ? ctx->cells_wpb : fs.wpb;
  // The wavefronts of a workgroup hold its LDS until the last is done, and
  // cells side by side along g (a few rows wide) cross a brick in about the
  // same number of layers, along f (28 or 60 voxels) they do not: numbered
  // along g, marches bound by their own work are 5 to 20 % faster (two
  // views of eight 512^3 bricks 2.19 -> 1.90 ms, six bricks 1.47 -> 1.38).
  // Along f neighbours share a line of every window row, which counts where
  // traffic binds: cells of many rows, most of them no neighbour's (rays 3
  // voxels apart: 2 to 9 % faster along f).
  a.cols = fs.reg && fs.blk_f == 0 && fs.Tg < 16.0 && fs.ng >= 1.4 * fs.Tg;
  if (fs.reg && ctx->cells_waves > 0) {
    // at most cells_waves wavefronts per compute unit: reserve LDS so that
    // one workgroup more would not fit (more wavefronts ran slower: their
    // windows crowd each other out of the caches)
    const int32_t nwg = std::max(1, ctx->cells_waves / wpb);
    a.lds_floor = kLdsPerCu / (nwg + 1) + 1024;
  }
  a.foot_nf = fs.nf;
  a.foot_ng = fs.ng;
  a.foot_Tf = fs.Tf;
  a.foot_Tg = fs.Tg;
  a.fa_u = fs.fa_u;
  a.fa_v = fs.fa_v;
  a.fb_u = fs.fb_u;
  a.fb_v = fs.fb_v;
}

int32_t foot_brick(const Camera& cam, const FootShape& fs, const Box& box, DevBrickView& b) {
  int32_t ncf, ncg;
  foot_cells(cam, fs, box, b.cf0, b.cg0, ncf, ncg, b.fa0, b.fb0);
  b.tiles_x = ncf;
  if (fs.blk_f > 0) {
    b.blocks_x = (ncf + fs.blk_f - 1) / fs.blk_f;
    return b.blocks_x * ((ncg + fs.blk_g - 1) / fs.blk_g);
  }
  b.blocks_x = ncg;  // cells along g
  return ncf * ncg;
}

// Plan one view of a bricked volume: rectangles, culling (empty rectangle or
// transparent brick), launch order (brick index order, which keeps
// neighbouring bricks together), arena offsets and the front-to-back layers.
void plan_bricked_view(const vr_volume* vol, const Camera& cam, const vr_params* p, int32_t tile_w,
                       const float* tf, int32_t M, double vmin, double vmax, ViewPlan& vp) {
  const Partition& P = vol->part;
  const int32_t nb = (int32_t)P.boxes.size();
  const int32_t tile_h = 64 / tile_w;
  std::vector<Rect> rects((size_t)nb);
  std::vector<int32_t> slot((size_t)nb, -1);
  vp.bv.clear();
  vp.layers_order.clear();
  int32_t tiles = 0;
  int64_t pix = 0;
  for (int32_t b = 0; b < nb; b++) {
    rects[b] = brick_rect(cam, P.boxes[b]);
    if (rects[b].w == 0 || rects[b].h == 0) continue;
    if (p->ess && p->mode == VR_MODE_DVR &&
        brick_transparent(vol->bricks[b].vmin, vol->bricks[b].vmax, tf, M, vmin, vmax))
      continue;
    DevBrickView v;
    std::memset(&v, 0, sizeof v);
    v.brick = b;
    v.x0 = rects[b].x0;
    v.y0 = rects[b].y0;
    v.w = rects[b].w;
    v.h = rects[b].h;
    v.tiles_x = (v.w + tile_w - 1) / tile_w;
    v.tile_begin = tiles;
    v.img_off = pix;
    tiles += v.tiles_x * ((v.h + tile_h - 1) / tile_h);
    pix += (int64_t)v.w * v.h;
    slot[b] = (int32_t)vp.bv.size();
    vp.bv.push_back(v);
  }
  std::vector<int32_t> order;
  depth_order(P, cam, order);
  for (int32_t b : order)
    if (slot[b] >= 0) vp.layers_order.push_back(slot[b]);
  vp.ntiles = tiles;
  vp.pixels = pix;
  vp.wave_begin.clear();
  vp.wave_tiles.clear();
}

void plan_waves(const vr_volume* vol, const Camera& cam, int32_t tile_w, ViewPlan& vp) {
  const int32_t tile_h = 64 / tile_w;
  std::vector<int32_t> wave;
  const int32_t nw = brick_waves(vol->part, cam, wave);
  std::vector<DevBrickView> by_wave;
  by_wave.reserve(vp.bv.size());
  for (int32_t w = 0; w < nw; w++) {
    const int32_t first = (int32_t)by_wave.size();
    int32_t t = 0;
    for (const DevBrickView& b : vp.bv)
      if (wave[b.brick] == w) {
        DevBrickView c = b;
        c.tile_begin = t;
        t += c.tiles_x * ((c.h + tile_h - 1) / tile_h);
        by_wave.push_back(c);
      }
    if (t == 0) continue;
    vp.wave_begin.push_back(first);
    vp.wave_tiles.push_back(t);
  }
  vp.wave_begin.push_back((int32_t)by_wave.size());
  vp.bv.swap(by_wave);
  vp.layers_order.clear();  // no brick images to composite
}

int render_forward(vr_ctx* ctx, vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p,
                   float* out, hipStream_t s) {
  const bool bricked = vol->bricked;
  const int32_t W = views[0].W, H = views[0].H;
  double vmin, vmax;
  VR_TRY(resolve_window(ctx, vol, s, vmin, vmax));
  MarchArgs base;
  std::memset(&base, 0, sizeof base);
  int32_t tuned_tile, budget, mode;
  tuned_shape(ctx, vol, W, H, p, tuned_tile, budget, mode);
  vr_params pt = *p;
  pt.tile = tuned_tile;
  fill_march_common(base, vol, &pt, vmin, vmax, ctx->d_tf, ctx->tf_m);
  if (ctx->mask_n > 0) {
    if (vol->n[vol->spectral_axis] != ctx->mask_n)
      return fail(VR_EINVAL, "mask length %d differs from the volume's axis-3 size %lld", ctx->mask_n,
                  (long long)vol->n[vol->spectral_axis]);
    base.mask = ctx->d_mask;
    base.mask_n = ctx->mask_n;
  }
  VR_TRY(prepare_macrocells(ctx, vol, p, vmin, vmax, base, s));
  const int32_t tw = base.tile_w, th = base.tile_h;
  // opacity tested over the whole ray: bricks marched in front-to-back waves
  // straight into the frame, each ray carrying its state from brick to brick
  const bool global = bricked && out && !base.mip && p->ert_scope == VR_ERT_GLOBAL;
  // the march is chosen per view (the default shapes, no other march forced);
  // forced: windows in LDS wherever they fit, whatever the estimates say
  const bool pick = (mode == 0 || mode == 3) && tw == 8, forced = mode == 3;
  if (pick && base.mc > 0) {
    // few clear macrocells: what the walk from macrocell to macrocell and the
    // 16-sample blocks around the others cost outweighs the samples saved (a
    // block-gathered sample costs about twice a sample of the cell march)
    const int64_t cells = vol->mcn[0] * vol->mcn[1] * vol->mcn[2];
    const bool indexed = std::max({vol->n[0], vol->n[1], vol->n[2]}) <= kSkipIndex;
    if (forced || !indexed || 2 * vol->mc_nclear < cells) base.mc = 0;
  }

  std::vector<ViewPlan> plans((size_t)nviews);
  std::vector<Camera> cams((size_t)nviews);
  int64_t arena_pix = 0;
  for (int32_t v = 0; v < nviews; v++) {
    make_camera(views[v], vol->n, cams[v]);
    ViewPlan& vp = plans[v];
    if (bricked) {
      plan_bricked_view(vol, cams[v], p, tw, ctx->h_tf.data(), ctx->tf_m, vmin, vmax, vp);
      if (!global) arena_pix = std::max(arena_pix, vp.pixels);
    } else {
      DevBrickView b;
      std::memset(&b, 0, sizeof b);
      b.brick = 0;
      b.w = W;
      b.h = H;
      b.tiles_x = (W + tw - 1) / tw;
      b.tile_begin = 0;
      b.img_off = (int64_t)v * W * H;
      vp.bv.assign(1, b);
      vp.ntiles = b.tiles_x * ((H + th - 1) / th);
      vp.pixels = (int64_t)W * H;
    }
  }
  // tiles of e x e pixels, numbered by blocks of 2 x 2
  auto gather_tiles = [](ViewPlan& vp, int32_t first, int32_t last, int32_t e) {
    int32_t t = 0;
    for (int32_t i = first; i < last; i++) {
      DevBrickView& b = vp.bv[i];
      b.tiles_x = (b.w + 2 * e - 1) / (2 * e);
      b.tile_begin = t;
      t += 4 * b.tiles_x * ((b.h + 2 * e - 1) / (2 * e));
    }
    return t;
  };
  // a view marched by gathers: 64 / depth pixels a wavefront (8 x 8 with macrocell skipping)
  auto gather_view = [&](ViewPlan& vp, int32_t depth) {
    if (vp.thru) depth = std::max(depth, 4);
    vp.deep = depth;
    if (depth == 1) return;  // 8 x 8 pixels, as planned
    const int32_t e = vp.skip ? 8 : depth == 16 ? 2 : 4;
    if (global && !vp.thru)
      for (size_t w = 0; w + 1 < vp.wave_begin.size(); w++)
        vp.wave_tiles[w] = gather_tiles(vp, vp.wave_begin[w], vp.wave_begin[w + 1], e);
    else if (vp.thru) vp.ntiles = 4 * ((W + 2 * e - 1) / (2 * e)) * ((H + 2 * e - 1) / (2 * e));
    else vp.ntiles = gather_tiles(vp, 0, (int32_t)vp.bv.size(), e);
  };
  // every ray through all its bricks in one launch: bricks front to back
  auto thru_order = [&](int32_t v) {
    ViewPlan& vp = plans[v];
    std::vector<DevBrickView> o;
    o.reserve(vp.bv.size());
    for (int32_t i : vp.layers_order) o.push_back(vp.bv[i]);
    vp.bv.swap(o);
    vp.layers_order.clear();
    vp.thru = true;
  };
  Box whole;
  for (int i = 0; i < 3; i++) {
    whole.lo[i] = 0;
    whole.hi[i] = vol->n[i] - 1;
    whole.closed[i] = 1;
  }
  std::vector<BoxSums> sums((size_t)nviews);
  for (int32_t v = 0; v < nviews && pick; v++)
    for (const DevBrickView& b : plans[v].bv)
      add_box(sums[v], cams[v], bricked ? vol->part.boxes[b.brick] : whole, (int64_t)b.w * b.h, p->step);
  for (int32_t v = 0; v < nviews; v++) {
    ViewPlan& vp = plans[v];
    const bool choose = pick && !vp.bv.empty();
    if (choose && base.mc > 0) {
      if (global) thru_order(v);
      vp.skip = true;
      gather_view(vp, 16);
    } else if (global) {
      const MarchTimes t = march_times(cams[v], sums[v], nullptr);
      if (choose && !forced && (nviews == 1 || t.pitch < 1.0 || t.gather < kThruBelow)) {
        thru_order(v);
        BoxSums rays = sums[v], all;
        add_box(all, cams[v], whole, (int64_t)W * H, p->step);
        rays.chord = all.chord;  // a ray's chain runs through all its bricks
        rays.pixels = all.pixels;
        gather_view(vp, gather_lanes(cams[v], rays, p->step, base.M));
        continue;
      }
      plan_waves(vol, cams[v], tw, vp);
      if (choose && !forced && (base.mask || cams[v].persp || vp.wave_begin.size() > 8))
        gather_view(vp, t.pitch < 2.0 ? 4 : 16);
    }
  }
  // perspective views: footprint cells sized per brick (the plain march of
  // emission-absorption or MIP, register-staged), each brick along the slab
  // axis along which the eye lies outside its slab; the bricks neither axis
  // suits, and views with rays less than kPerspCellPitch voxels apart, by
  // gathers
  auto persp_faster = [&](const Camera& cam, const BoxSums& boxes) {
    FootShape any;
    any.axis = std::fabs(cam.e3[1]) >= std::fabs(cam.e3[2]) ? 1 : 2;
    const MarchTimes t = march_times(cam, boxes, &any);
    return t.samples / kPerspCellRate + kPerspChains * t.chain <= t.gather;
  };
  for (int32_t v = 0; v < nviews; v++) {
    ViewPlan& vp = plans[v];
    if (!pick || !cams[v].persp || vp.bv.empty() || vp.deep || global) continue;
    const bool cells = bricked && ctx->persp_cells && (!base.mask || base.mask_n <= kCellsMaskMax) &&
                       ctx->ring_reg > 0 && ctx->ring_nslots != 3 &&
                       (forced || (cams[v].S / W >= kPerspCellPitch && persp_faster(cams[v], sums[v])));
    const int first_axis = std::fabs(cams[v].e3[1]) >= std::fabs(cams[v].e3[2]) ? 1 : 2;
    std::vector<int32_t> axis(vp.bv.size(), 0);
    bool any = false;
    for (size_t i = 0; cells && i < vp.bv.size(); i++) {
      DevBrickView& b = vp.bv[i];
      Rect rc;
      rc.x0 = b.x0;
      rc.y0 = b.y0;
      rc.w = b.w;
      rc.h = b.h;
      for (int tryax : {first_axis, 3 - first_axis}) {
        PerspCells pc;
        if (!persp_cells(cams[v], tryax, vol->part.boxes[b.brick], rc, ctx->foot_rays, ctx->persp_kmax, kRingCap,
                         kRingRegLoads, pc, ctx->foot_maxpx) ||
            !brick_rows_readable(vol, b.brick, pc.pitch) || !samples_countable(cams[v], vol->part.boxes[b.brick], p->step))
          continue;
        axis[i] = tryax;
        any = true;
        b.tiles_x = pc.ncf;
        b.cf0 = pc.cf0;
        b.cg0 = pc.cg0;
        b.blocks_x = pc.ncg;  // cells along g (the cell count is tiles_x x blocks_x)
        b.pTf = pc.Tf;
        b.pTg = pc.Tg;
        b.ppitch = pc.pitch;
        b.png = pc.ng;
        break;
      }
    }
    if (!any) {
      gather_view(vp, gather_lanes(cams[v], sums[v], p->step, base.M));
      continue;
    }
    std::vector<DevBrickView> grouped;
    std::vector<int32_t> where(vp.bv.size(), -1);
    for (const int32_t ax : {1, 2, 0}) {
      const int32_t first = (int32_t)grouped.size();
      int32_t t = 0;
      for (size_t i = 0; i < vp.bv.size(); i++) {
        if (axis[i] != ax) continue;
        DevBrickView b = vp.bv[i];
        b.tile_begin = t;
        if (ax != 0) t += b.tiles_x * b.blocks_x;
        where[i] = (int32_t)grouped.size();
        grouped.push_back(b);
      }
      if ((int32_t)grouped.size() == first) continue;
      vp.class_begin.push_back(first);
      vp.class_axis.push_back(ax);
      vp.class_tiles.push_back(t);
    }
    vp.class_begin.push_back((int32_t)grouped.size());
    for (int32_t& l : vp.layers_order) l = where[l];
    vp.bv.swap(grouped);
    if (vp.class_axis.back() == 0)
      vp.class_tiles.back() =
          gather_tiles(vp, vp.class_begin[vp.class_begin.size() - 2], (int32_t)vp.bv.size(), 2);
  }
  // parallel rays on the ring march: footprint cells instead of 8 x 8 pixel
  // tiles (the cell counts replace the tile counts of the plan)
  const bool plain_ring = base.mc == 0 && !base.mask;
  const int32_t table_rows = cells_table_rows(base);
  for (int32_t v = 0; v < nviews; v++) {
    ViewPlan& vp = plans[v];
    if (!pick || cams[v].persp || vp.deep) continue;
    FootShape fs;
    // gathers for certain: their estimate is below the cells' best (the slab
    // axis with fewer layers), without sizing the cells on the host (80 us)
    if (!forced && !global && ctx->foot && !vp.bv.empty()) {
      bool sure = true;
      for (int axis : {1, 2}) {
        FootShape any;
        any.axis = axis;
        const MarchTimes t = march_times(cams[v], sums[v], &any);
        sure = sure && t.gather < t.cells;
      }
      if (sure) {
        gather_view(vp, gather_lanes(cams[v], sums[v], p->step, base.M));
        continue;
      }
    }
    auto shape = [&](bool plain) {
      return ctx->foot && pick_foot(cams[v], vol->n, plain ? table_rows : base.M, plain, ctx->ring_reg > 0,
                                    ctx->ring_nslots, ctx->foot_rays, ctx->foot_pad, ctx->foot_kmax, fs, ctx->foot_maxpx);
    };
    bool cells = shape(base.mc == 0 && (!base.mask || base.mask_n <= kCellsMaskMax));
    // a channel mask: register-staged cells or three slots
    if (base.mask && (!cells || !fs.reg)) cells = shape(false);
    // staged windows read whole rows, past a narrow volume's end too
    if (cells && fs.reg)
      for (const DevBrickView& b : vp.bv) cells = cells && brick_rows_readable(vol, b.brick, (fs.nf + 3) & ~3);
    Box widest = whole;
    for (int i = 0; i < 3; i++) widest.hi[i] = sums[v].most[i];
    cells = cells && samples_countable(cams[v], widest, p->step);
    if (!forced && !global && ctx->foot && !vp.bv.empty()) {
      const MarchTimes t = march_times(cams[v], sums[v], cells ? &fs : nullptr);
      if (ctx->debug_plan)
        std::fprintf(stderr, "[vr] view %d: estimated cells %.0f us, gathers %.0f us\n", v, t.cells * 1e6, t.gather * 1e6);
      if (t.gather < t.cells) {
        gather_view(vp, gather_lanes(cams[v], sums[v], p->step, base.M));
        continue;
      }
    }
    if (!cells) continue;
    // blocks of cells (the plain march, emission-absorption or MIP): one
    // workgroup per block, one window per layer; the window's rows must fit
    // inside every brick along axis 1
    if (plain_ring && ctx->foot_block != 0) {
      int64_t ext[3] = {INT64_MAX, 0, 0};
      for (const DevBrickView& b : vp.bv) {
        const Box& bx = bricked ? vol->part.boxes[b.brick] : whole;
        ext[0] = std::min<int64_t>(ext[0], bx.hi[0] - bx.lo[0]);
        for (int i = 1; i < 3; i++) ext[i] = std::max<int64_t>(ext[i], bx.hi[i] - bx.lo[i]);
      }
      const Box& b0 = bricked ? vol->part.boxes[vp.bv.empty() ? 0 : vp.bv[0].brick] : whole;
      int64_t typ[3];
      for (int i = 0; i < 3; i++) typ[i] = b0.hi[i] - b0.lo[i];
      typ[0] = std::min(typ[0], ext[0]);
      choose_foot_block(cams[v], fs, typ, base.M, kRingRegWaves, kRingRegWaves, kRingRegLoads,
                        ctx->foot_block > 0 ? ctx->foot_block_f : 0, ctx->foot_block > 0 ? ctx->foot_block_g : 0);
    }
    if (ctx->debug_plan)
      std::fprintf(stderr, "[vr] view %d: cells axis %d Tf %.1f Tg %.2f nf %d ng %d slot %d nslots %d reg %d wpb %d waves %d rf %.3f rg %.3f blocks %dx%d nf %d ng %d waves %d\n",
                   v, fs.axis, fs.Tf, fs.Tg, fs.nf, fs.ng, fs.slot, fs.nslots, fs.reg, fs.wpb, fs.waves, fs.rf, fs.rg,
                   fs.blk_f, fs.blk_g, fs.blk_nf, fs.blk_ng, fs.blk_waves);
    vp.foot = true;
    vp.fs = fs;
    int32_t tiles = 0;
    size_t w = 0;  // wave of the brick (whole-ray termination)
    for (size_t i = 0; i < vp.bv.size(); i++) {
      DevBrickView& b = vp.bv[i];
      if (global) {
        while (w + 1 < vp.wave_begin.size() && (int32_t)i >= vp.wave_begin[w + 1]) w++;
        if ((int32_t)i == vp.wave_begin[w]) tiles = 0;
      }
      b.tile_begin = tiles;
      tiles += foot_brick(cams[v], fs, bricked ? vol->part.boxes[b.brick] : whole, b);
      if (global) vp.wave_tiles[w] = tiles;
    }
    if (!global) vp.ntiles = tiles;
  }
  if (bricked && arena_pix > 0) VR_TRY(ensure_device(&ctx->d_arena, &ctx->arena_bytes, (size_t)arena_pix * 16));
  // overflow lists of the footprint-cell marches: one per stream a view may use
  int64_t foot_tiles = 0;  // cells of a launch (a block holds blk_f x blk_g)
  for (const ViewPlan& vp : plans) {
    if (vp.foot) {
      const int64_t per = vp.fs.blk_f > 0 ? (int64_t)vp.fs.blk_f * vp.fs.blk_g : 1;
      foot_tiles = std::max<int64_t>(foot_tiles, vp.ntiles * per);
      for (int32_t t : vp.wave_tiles) foot_tiles = std::max<int64_t>(foot_tiles, t * per);
    }
    for (size_t c = 0; c < vp.class_tiles.size(); c++)
      if (vp.class_axis[c] != 0) foot_tiles = std::max<int64_t>(foot_tiles, vp.class_tiles[c]);
  }
  const size_t ovf_stride = align16(256 + 4 * (size_t)foot_tiles);
  if (foot_tiles > 0) VR_TRY(ensure_device(&ctx->d_ovf, &ctx->ovf_bytes, ovf_stride * vr_ctx::kAux));
  float4* arena = reinterpret_cast<float4*>(ctx->d_arena);

  // pack: [whole-volume brick] then per view [DevBrickView...][CompLayer...]
  std::vector<size_t> off_bv((size_t)nviews), off_cl((size_t)nviews);
  size_t bytes = align16(sizeof(DevBrick));
  for (int32_t v = 0; v < nviews; v++) {
    off_bv[v] = bytes;
    bytes = align16(bytes + sizeof(DevBrickView) * plans[v].bv.size());
    off_cl[v] = bytes;
    bytes = align16(bytes + sizeof(CompLayer) * plans[v].layers_order.size());
  }
  std::vector<unsigned char> host(bytes, 0);
  std::memcpy(host.data(), &vol->whole, sizeof(DevBrick));
  for (int32_t v = 0; v < nviews; v++) {
    const ViewPlan& vp = plans[v];
    std::memcpy(host.data() + off_bv[v], vp.bv.data(), sizeof(DevBrickView) * vp.bv.size());
    CompLayer* cl = reinterpret_cast<CompLayer*>(host.data() + off_cl[v]);
    for (size_t i = 0; i < vp.layers_order.size(); i++) {
      const DevBrickView& b = vp.bv[vp.layers_order[i]];
      cl[i].x0 = b.x0;
      cl[i].y0 = b.y0;
      cl[i].w = b.w;
      cl[i].h = b.h;
      cl[i].rgba = arena + b.img_off;
    }
  }
  void* dtab = nullptr;
  VR_TRY(stage_begin(ctx, VR_STAGE_SETUP, s));
  VR_TRY(upload_tables(ctx, s, host.data(), bytes, &dtab));
  VR_TRY(stage_end(ctx, s));
  unsigned char* dt = reinterpret_cast<unsigned char*>(dtab);

  // views with the opacity test over whole rays write disjoint frames and use
  // no shared arena: their wave sequences run side by side on the side streams
  // (small front and back waves of one view leave most of the chip idle)
  const bool side = global && nviews > 1;
  if (global) VR_TRY(stage_begin(ctx, VR_STAGE_MARCH, s));
  if (side) VR_TRY(aux_fork(ctx, s));
  for (int32_t v = 0; v < nviews; v++) {
    const ViewPlan& vp = plans[v];
    MarchArgs a = base;
    a.cam = cams[v];
    a.nbv = (int32_t)vp.bv.size();
    a.ntiles = vp.ntiles;
    a.bv = reinterpret_cast<const DevBrickView*>(dt + off_bv[v]);
    if (bricked) {
      a.bricks = vol->d_bricks;
      a.img = arena;
    } else {
      a.bricks = reinterpret_cast<const DevBrick*>(dt);
      a.img = reinterpret_cast<float4*>(out);
    }
    bool lds = false, ring = false;
    int ring_wpb = 4;
    a.lds_budget = budget;
    a.depth = vp.deep;
    a.skip = vp.skip ? 1 : 0;
    a.thru = vp.thru ? 1 : 0;
    if (vp.deep && ctx->debug_plan)
      std::fprintf(stderr, "[vr] view %d: gathers lanes %d skip %d thru %d\n", v, vp.deep, a.skip, a.thru);
    // fewer bricks than XCDs: the cells of one brick spread over all of them
    // in runs (a whole volume 604 -> 553 us for two views, six bricks 1.70 ->
    // 1.59 ms); from 8 bricks on each XCD keeps bricks of its own (2.39 ms for
    // eight bricks against 2.66)
    a.xcd_chunk = a.nbv < 8 ? 16 : 0;
    if (vp.foot) {
      const FootShape& fs = vp.fs;
      ring = true;
      foot_args(ctx, fs, a, ring_wpb);
      if (fs.blk_f > 0) {
        // one window per block: its rows and slot replace the cell's
        a.blk_f = fs.blk_f;
        a.blk_g = fs.blk_g;
        a.foot_nf = fs.blk_nf;
        a.foot_ng = fs.blk_ng;
        a.ring_slot = fs.blk_slot;
        a.ring_nslots = 2;
      }
      unsigned char* ovf = reinterpret_cast<unsigned char*>(ctx->d_ovf) + (global ? (size_t)(v % vr_ctx::kAux) * ovf_stride : 0);
      a.ovf_count = reinterpret_cast<unsigned int*>(ovf);
      a.ovf_tiles = reinterpret_cast<int32_t*>(ovf + 256);
      // pixels of the brick images (or of the frame) whose rays have no
      // sample are not written by the cells: clear them first
      if (!global) {
        VR_HIP(launch_zero(bricked ? arena : reinterpret_cast<float4*>(out) + (int64_t)v * W * H,
                           bricked ? vp.pixels : (int64_t)W * H, s));
      }
    } else if ((mode == 0 || mode == 3) && a.tile_w == 8) {
      if (!cams[v].persp && !vp.deep) {
        int32_t waves3 = 0;
        ring = choose_ring(cams[v], kRingCap, a.M, kRingMaxWaves, kRingWantWaves, kRingMinWaves, a.slab_axis,
                           a.ring_slot, ring_wpb, 3, &waves3);
        a.ring_nslots = 3;
        // two LDS slots per wavefront (the next layer's loads no longer overlap
        // the wavefront's own sampling, but more wavefronts fit): taken
        // whenever they fit more wavefronts on a compute unit than three (on
        // 24 GiB cubes the march follows the wavefront count, not the
        // lookahead: 12 -> 16 wavefronts took one view from 12.1 to 9.3 ms, a
        // fourth slot at fewer wavefronts cost 35 %), or when forced; plain
        // march and maximum intensity projection only
        if (ring && !a.mask && ctx->ring_nslots != 3) {
          int32_t ax2 = 0, slot2 = 0, wpb2 = 4, waves2 = 0;
          if (choose_ring(cams[v], kRingCap, a.M, kRingMaxWaves, kRingWantWaves, kRingMinWaves, ax2, slot2, wpb2, 2,
                          &waves2) &&
              (ctx->ring_nslots == 2 || waves2 > waves3)) {
            a.slab_axis = ax2;
            a.ring_slot = slot2;
            ring_wpb = wpb2;
            a.ring_nslots = 2;
          }
        }
      }
    }
    if (ring && !vp.foot && ctx->debug_plan)
      std::fprintf(stderr, "[vr] view %d: tiles axis %d slot %d nslots %d wpb %d\n", v, a.slab_axis, a.ring_slot,
                   a.ring_nslots, ring_wpb);
    if (ring) {
      a.tile_order = ctx->tile_order;
      a.tile_bw = ctx->tile_bw;
      a.tile_bh = ctx->tile_bh;
    }
    // (the slab march has no MIP and no mask)
    if (!ring && mode != 1 && !a.mip && !a.mask && !vp.deep && vp.class_begin.empty()) {
      lds = choose_slab(cams[v], a.tile_w, a.tile_h, budget, a.slab_axis, a.slab_T);
      // rays nearly parallel to axis 1 need a wider slab box: retry with twice the budget
      if (!lds && budget < 8192 && choose_slab(cams[v], a.tile_w, a.tile_h, 8192, a.slab_axis, a.slab_T)) {
        lds = true;
        a.lds_budget = 8192;
      }
    }
    if (global) {
      // waves in order, each continuing the rays the previous left in the frame
      float4* frame = reinterpret_cast<float4*>(out) + (int64_t)v * W * H;
      hipStream_t vs = side ? ctx->aux[v % vr_ctx::kAux] : s;
      lds = false;  // the slab march does not carry state
      a.img = frame;
      if (vp.thru) {
        VR_HIP(launch_march(a, vs));
        continue;
      }
      a.carry = 1;
      VR_HIP(launch_carry(frame, (int64_t)W * H, false, vs));
      const DevBrickView* wbv = a.bv;
      for (size_t w = 0; w + 1 < vp.wave_begin.size(); w++) {
        a.bv = wbv + vp.wave_begin[w];
        a.nbv = vp.wave_begin[w + 1] - vp.wave_begin[w];
        a.ntiles = vp.wave_tiles[w];
        VR_HIP(ring ? launch_march_ring(a, ring_wpb, vs) : launch_march(a, vs));
      }
      VR_HIP(launch_carry(frame, (int64_t)W * H, true, vs));
      continue;
    }
    VR_TRY(stage_begin(ctx, VR_STAGE_MARCH, s));
    if (!vp.class_begin.empty()) {
      // perspective footprint cells: the brick images' pixels without samples
      // are not written, so the arena is cleared first; one launch per slab
      // axis, the largest window as the slot, then the bricks by gathers
      VR_HIP(launch_zero(arena, vp.pixels, s));
      const DevBrickView* cbv = a.bv;
      for (size_t c = 0; c + 1 < vp.class_begin.size(); c++) {
        MarchArgs ac = a;
        const int32_t first = vp.class_begin[c], count = vp.class_begin[c + 1] - first;
        ac.bv = cbv + first;
        ac.nbv = count;
        ac.ntiles = vp.class_tiles[c];
        if (vp.class_axis[c] == 0) {
          ac.depth = 16;
          if (ctx->debug_plan) std::fprintf(stderr, "[vr] view %d gathers class %zu: bricks %d lanes 16\n", v, c, count);
          VR_HIP(launch_march(ac, s));
          continue;
        }
        int32_t slot = 0, mpitch = 0, mng = 0;
        for (int32_t k = first; k < first + count; k++) {
          slot = std::max(slot, vp.bv[k].ppitch * vp.bv[k].png);
          mpitch = std::max(mpitch, vp.bv[k].ppitch);
          mng = std::max(mng, vp.bv[k].png);
        }
        ac.foot = 1;
        ac.blk_f = ac.blk_g = 0;
        ac.slab_axis = vp.class_axis[c];
        ac.ring_slot = slot;
        ac.ring_nslots = 2;
        ac.ring_reg = 1;
        ac.foot_nf = mpitch;
        ac.foot_ng = mng;
        int32_t waves = 0;
        int cwpb = ring_waves_per_block(slot, cells_table_rows(ac), kRingRegWaves, &waves, 2);
        if (ctx->cells_wpb > 0) cwpb = ctx->cells_wpb;
        if (ctx->cells_waves > 0) {
          const int32_t nwg = std::max(1, ctx->cells_waves / cwpb);
          ac.lds_floor = kLdsPerCu / (nwg + 1) + 1024;
        }
        unsigned char* ovf = reinterpret_cast<unsigned char*>(ctx->d_ovf);
        ac.ovf_count = reinterpret_cast<unsigned int*>(ovf);
        ac.ovf_tiles = reinterpret_cast<int32_t*>(ovf + 256);
        if (ctx->debug_plan)
          std::fprintf(stderr, "[vr] view %d cells class %zu: bricks %d cells %d axis %d slot %d pitch<=%d ng<=%d wpb %d waves %d\n",
                       v, c, count, ac.ntiles, ac.slab_axis, slot, mpitch, mng, cwpb, waves);
        VR_HIP(launch_march_ring(ac, cwpb, s));
      }
    } else {
      VR_HIP(ring ? launch_march_ring(a, ring_wpb, s) : (lds ? launch_march_lds(a, s) : launch_march(a, s)));
    }
    VR_TRY(stage_end(ctx, s));
    if (bricked && out) {
      CompArgs c;
      std::memset(&c, 0, sizeof c);
      c.layers = reinterpret_cast<const CompLayer*>(dt + off_cl[v]);
      c.n = (int32_t)vp.layers_order.size();
      c.W = W;
      c.H = H;
      c.mip = base.mip;
      c.out = reinterpret_cast<float4*>(out) + (int64_t)v * W * H;
      VR_TRY(stage_begin(ctx, VR_STAGE_COMPOSITE, s));
      VR_HIP(launch_composite(c, s));
      VR_TRY(stage_end(ctx, s));
    }
  }
  if (side) VR_TRY(aux_join(ctx, s));
  if (global) VR_TRY(stage_end(ctx, s));
  return VR_OK;
}

int validate_render(vr_ctx* ctx, const vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p) {
  if (!ctx || !vol || !views) return fail(VR_EINVAL, "ctx, vol and views must be non-NULL");
  if (vol->ctx != ctx) return fail(VR_EINVAL, "volume belongs to another context");
  if (nviews < 1) return fail(VR_EINVAL, "nviews must be >= 1");
  VR_TRY(check_params(p));
  for (int32_t v = 0; v < nviews; v++) {
    VR_TRY(check_view(&views[v], vol->n));
    if (views[v].W != views[0].W || views[v].H != views[0].H)
      return fail(VR_EINVAL, "all views of one call must share W and H");
  }
  if (!ctx->tf_set) return fail(VR_ESTATE, "no transfer function set (vr_tf_set)");
  if (!vol->bricked && vol->n[0] * vol->n[1] * vol->n[2] >= ((int64_t)1 << 31))
    return fail(VR_EUNSUPPORTED, "unbricked rendering needs fewer than 2^31 voxels; brick the volume");
  return VR_OK;
}

}  // namespace vr

using namespace vr;

extern "C" {

int vr_render(vr_ctx* ctx, const vr_volume* cvol, const vr_view* views, int32_t nviews, const vr_params* p,
              float* out, uintptr_t stream, vr_state** save) {
  clear_error();
  VR_TRY(validate_render(ctx, cvol, views, nviews, p));
  if (!out) return fail(VR_EINVAL, "out is NULL");
  vr_volume* vol = const_cast<vr_volume*>(cvol);
  DeviceGuard g(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  if (save) return render_with_state(ctx, vol, views, nviews, p, out, s, save);
  VR_TRY(ctx_begin(ctx, s));
  if (!vol->twin || !vol->bricked) {
    VR_TRY(render_forward(ctx, vol, views, nviews, p, out, s));
    return ctx_end(ctx, s);
  }
  // views looking mostly along axis 1 (the contiguous one) are rendered from
  // the permuted copy, whose contiguous axis is axis 2: the same rays in
  // permuted coordinates (view axes permuted like the volume's)
  auto along1 = [](const vr_view& v) {
    return std::fabs(v.R[6]) > std::max(std::fabs(v.R[7]), std::fabs(v.R[8]));
  };
  const int64_t frame = (int64_t)views[0].W * views[0].H * 4;
  for (int32_t v0 = 0; v0 < nviews;) {
    const bool tw = along1(views[v0]);
    int32_t v1 = v0 + 1;
    while (v1 < nviews && along1(views[v1]) == tw) v1++;
    if (tw) {
      std::vector<vr_view> pv(views + v0, views + v1);
      for (vr_view& q : pv)
        for (int r = 0; r < 3; r++) {
          const double x = q.R[3 * r], y = q.R[3 * r + 1], z = q.R[3 * r + 2];
          q.R[3 * r] = y;
          q.R[3 * r + 1] = z;
          q.R[3 * r + 2] = x;
        }
      VR_TRY(render_forward(ctx, vol->twin, pv.data(), v1 - v0, p, out + v0 * frame, s));
    } else {
      VR_TRY(render_forward(ctx, vol, views + v0, v1 - v0, p, out + v0 * frame, s));
    }
    v0 = v1;
  }
  return ctx_end(ctx, s);
}

int vr_render_bricks(vr_ctx* ctx, const vr_volume* cvol, const vr_view* view, const vr_params* p,
                     vr_brick_image* imgs, int32_t* nimg, int32_t* order, uintptr_t stream) {
  clear_error();
  VR_TRY(validate_render(ctx, cvol, view, 1, p));
  if (!imgs || !nimg || !order) return fail(VR_EINVAL, "imgs, nimg and order must be non-NULL");
  if (!cvol->bricked) return fail(VR_ESTATE, "volume is not bricked (vr_volume_brick)");
  if (p->ert_scope == VR_ERT_GLOBAL)
    return fail(VR_EUNSUPPORTED, "per-brick images exist only with VR_ERT_LOCAL (global termination carries rays "
                                 "across bricks)");
  vr_volume* vol = const_cast<vr_volume*>(cvol);
  DeviceGuard g(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  VR_TRY(ctx_begin(ctx, s));
  // plan first to check capacity
  double vmin, vmax;
  VR_TRY(resolve_window(ctx, vol, s, vmin, vmax));
  Camera cam;
  make_camera(*view, vol->n, cam);
  ViewPlan vp;
  int32_t tw, budget, mode;
  tuned_shape(ctx, vol, view->W, view->H, p, tw, budget, mode);
  plan_bricked_view(vol, cam, p, tw, ctx->h_tf.data(), ctx->tf_m, vmin, vmax, vp);
  if ((int32_t)vp.bv.size() > *nimg)
    return fail(VR_EINVAL, "capacity %d below the %d rendered bricks", *nimg, (int)vp.bv.size());
  VR_TRY(render_forward(ctx, vol, view, 1, p, nullptr, s));
  float4* arena = reinterpret_cast<float4*>(ctx->d_arena);
  for (size_t i = 0; i < vp.bv.size(); i++) {
    const DevBrickView& b = vp.bv[i];
    imgs[i].brick = b.brick;
    imgs[i].x0 = b.x0;
    imgs[i].y0 = b.y0;
    imgs[i].w = b.w;
    imgs[i].h = b.h;
    imgs[i].reserved = 0;
    imgs[i].rgba = reinterpret_cast<float*>(arena + b.img_off);
  }
  for (size_t i = 0; i < vp.layers_order.size(); i++) order[i] = vp.layers_order[i];
  *nimg = (int32_t)vp.bv.size();
  return ctx_end(ctx, s);
}

int vr_composite(vr_ctx* ctx, const vr_brick_image* imgs, int32_t n, const int32_t* order, int32_t W, int32_t H,
                 float* out, uintptr_t stream) {
  clear_error();
  if (!ctx || !out || (n > 0 && !imgs)) return fail(VR_EINVAL, "ctx, out (and imgs when n > 0) must be non-NULL");
  if (n < 0) return fail(VR_EINVAL, "n must be >= 0");
  if (W < 1 || H < 1 || W > 16384 || H > 16384) return fail(VR_EINVAL, "image size outside [1, 16384]");
  std::vector<CompLayer> layers((size_t)n);
  std::vector<char> seen((size_t)n, 0);
  for (int32_t i = 0; i < n; i++) {
    const int32_t j = order ? order[i] : i;
    if (j < 0 || j >= n) return fail(VR_EINVAL, "order[%d] = %d out of range", i, j);
    if (seen[j]) return fail(VR_EINVAL, "order lists image %d twice", j);
    seen[j] = 1;
    const vr_brick_image& im = imgs[j];
    if (im.w < 0 || im.h < 0 || im.x0 < 0 || im.y0 < 0 || (int64_t)im.x0 + im.w > W || (int64_t)im.y0 + im.h > H)
      return fail(VR_EINVAL, "image %d rectangle (%d,%d,%d,%d) outside %dx%d", j, im.x0, im.y0, im.w, im.h, W, H);
    if (im.w > 0 && im.h > 0 && !im.rgba) return fail(VR_EINVAL, "image %d has no pixels pointer", j);
    layers[i] = CompLayer{im.x0, im.y0, im.w, im.h, reinterpret_cast<const float4*>(im.rgba)};
  }
  DeviceGuard g(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  VR_TRY(ctx_begin(ctx, s));
  void* d = nullptr;
  CompLayer dummy{0, 0, 0, 0, nullptr};
  VR_TRY(upload_tables(ctx, s, n > 0 ? (const void*)layers.data() : (const void*)&dummy,
                       sizeof(CompLayer) * (size_t)std::max(n, 1), &d));
  CompArgs c;
  std::memset(&c, 0, sizeof c);
  c.layers = reinterpret_cast<const CompLayer*>(d);
  c.n = n;
  c.W = W;
  c.H = H;
  c.out = reinterpret_cast<float4*>(out);
  VR_TRY(stage_begin(ctx, VR_STAGE_COMPOSITE, s));
  VR_HIP(launch_composite(c, s));
  VR_TRY(stage_end(ctx, s));
  return ctx_end(ctx, s);
}

}  // extern "C"
