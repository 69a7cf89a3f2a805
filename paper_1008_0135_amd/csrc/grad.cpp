// grad.cpp -- the differentiable forward (vr_render with save) and
// vr_render_backward: state ownership, validation and launch sequence.
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

struct vr_state {
  vr_ctx* ctx = nullptr;
  const vr_volume* vol = nullptr;
  uint64_t vol_version = 0, tf_version = 0;
  std::vector<vr_view> views;
  vr_params p;
  double vmin = 0.0, vmax = 0.0;
  int32_t W = 0, H = 0, nviews = 0, K = 32, nseg = 0;
  // per view: checkpoint layout.  Ring views keep, per group of L cell layers
  // along the slab axis, T at a ray's start of the group, and at its end; the
  // others keep T before every K-th sample.
  struct View {
    bool ring = false;
    bool exact = false;  // T of the adjoint's own samples (saved by gathers), not of the image's
    int32_t axis = 0, slot = 0, L = 0, smax = 0, ngrp = 0;
    int64_t off = 0;  // offset of this view's checkpoints in d_ckpt
    int32_t parts = 1, part_groups = 0;  // workgroups per tile and the groups each takes
    int64_t sums = 0;                    // offset of this view's sums in d_sums
    int32_t band[9] = {};  // ring adjoint: tiles per XCD (all zero: equal counts)
  };
  std::vector<View> vs;
  float* d_ckpt = nullptr;     // checkpoints, all views
  double4* d_sums = nullptr;   // behind the checkpoints: views in parts
  int32_t* d_nused = nullptr;  // [view][pixel], then the adjoint's bound flag
  size_t ckpt_bytes = 0, nused_bytes = 0;  // allocated sizes
  int32_t* d_flag = nullptr;   // set by the adjoint when a group held more samples than its bound
};

namespace vr {

namespace {

constexpr int32_t kPartBlocks = 4096, kMaxParts = 16;
// tables with (nearly) opaque entries: no parts.  Behind a sample of opacity 1
// the forward's sums hold nothing, but its own gradient needs what lies there.
constexpr float kPartAlpha = 0.99f;

float table_max_alpha(const vr_ctx* ctx) {
  float m = 0.f;
  for (int32_t i = 0; i < ctx->tf_m; i++) m = std::max(m, ctx->h_tf[4 * (size_t)i + 3]);
  return m;
}

// Largest change of the opacity per unit of the normalised value.
float table_slope(const vr_ctx* ctx) {
  float m = 0.f;
  for (int32_t i = 0; i + 1 < ctx->tf_m; i++)
    m = std::max(m, std::fabs(ctx->h_tf[4 * (size_t)i + 7] - ctx->h_tf[4 * (size_t)i + 3]));
  return m * (float)(ctx->tf_m - 1);
}

// Device tables of one view of a whole-volume render: [DevBrick][DevBrickView].
struct WholeTables {
  size_t bytes = 0, off_bv = 0;
};

void pack_whole(const vr_volume* vol, int32_t W, int32_t H, int32_t tw, int32_t th, int32_t nviews,
                std::vector<unsigned char>& host, std::vector<size_t>& off_bv) {
  size_t bytes = (sizeof(DevBrick) + 15) & ~(size_t)15;
  off_bv.resize((size_t)nviews);
  for (int32_t v = 0; v < nviews; v++) {
    off_bv[v] = bytes;
    bytes += (sizeof(DevBrickView) + 15) & ~(size_t)15;
  }
  host.assign(bytes, 0);
  std::memcpy(host.data(), &vol->whole, sizeof(DevBrick));
  for (int32_t v = 0; v < nviews; v++) {
    DevBrickView b;
    std::memset(&b, 0, sizeof b);
    b.w = W;
    b.h = H;
    b.tiles_x = (W + tw - 1) / tw;
    b.img_off = (int64_t)v * W * H;
    std::memcpy(host.data() + off_bv[v], &b, sizeof b);
  }
}

int ntiles_of(int32_t W, int32_t H, int32_t tw, int32_t th) { return ((W + tw - 1) / tw) * ((H + th - 1) / th); }

// Estimated work of each 8 x 8 tile of a whole-volume view, for splitting a
// ring march's tile groups into XCD bands: a fixed set-up plus the samples of
// the tile's longest ray, taken as the longest of its four corner rays through
// the volume (a wavefront walks its tile's rays in lockstep).
std::vector<double> tile_costs(const Camera& cam, const double hi[3], double step, int32_t W, int32_t H) {
  const int tx_n = (W + 7) / 8, ty_n = (H + 7) / 8;
  std::vector<int64_t> cn((size_t)(tx_n + 1) * (ty_n + 1), 0);  // samples of the corner rays
  for (int cy = 0; cy <= ty_n; cy++)
    for (int cx = 0; cx <= tx_n; cx++) {
      double o[3], tin;
      int64_t n = 0;
      pixel_origin(cam, std::min(cx * 8, W - 1), std::min(cy * 8, H - 1), o);
      if (ray_lattice(o, cam.e3, hi, step, tin, n)) cn[(size_t)cy * (tx_n + 1) + cx] = n;
    }
  std::vector<double> c((size_t)tx_n * ty_n);
  for (int t = 0; t < tx_n * ty_n; t++) {
    const size_t i = (size_t)(t / tx_n) * (tx_n + 1) + (size_t)(t % tx_n);
    c[(size_t)t] = 32.0 + (double)std::max(std::max(cn[i], cn[i + 1]), std::max(cn[i + tx_n + 1], cn[i + tx_n + 2]));
  }
  return c;
}

// Tile groups (wpb consecutive tiles) in 8 contiguous bands of about equal
// work, one per XCD.  Equal counts of groups leave the XCDs holding the
// image's border idle while those holding its middle, where rays are
// longest, still work.
void xcd_bands(const std::vector<double>& cost, int wpb, int32_t band[9]) {
  const int nt = (int)cost.size(), ng = (nt + wpb - 1) / wpb;
  std::vector<double> pre((size_t)ng + 1, 0.0);
  for (int g = 0; g < ng; g++) {
    double c = 0.0;
    for (int t = g * wpb; t < std::min(nt, (g + 1) * wpb); t++) c += cost[(size_t)t];
    pre[g + 1] = pre[g] + c;
  }
  band[0] = 0;
  for (int x = 1; x < 8; x++) {
    const double target = pre[ng] * (double)x / 8.0;
    const int b = (int)(std::lower_bound(pre.begin(), pre.end(), target) - pre.begin());
    band[x] = std::max(band[x - 1], std::min(b, ng));
  }
  band[8] = ng;
}

// Ring layout for the differentiable pair of one view: slab axis, window slot
// and cell layers per checkpoint group (about K samples, the adjoint's windows of
// one tile within 160 KB of LDS).  False when the view needs the sample-segment
// kernels (perspective; rays along axis 1).
bool plan_ring_view(const Camera& cam, const vr_params* p, int32_t M, const int64_t n[3], int layer_cap,
                    vr_state::View& rv) {
  if (p->tile != 0 && p->tile != 8) return false;
  if (cam.persp) return false;  // the ring adjoint assumes parallel rays
  int32_t axis = 0, slot = 0, wpb = 4;
  if (!choose_ring(cam, 4096, M, 24, 12, 2, axis, slot, wpb)) {
    // rays so far apart that no tile's windows fit: the same adjoint without
    // windows (corners from memory, voxel gradients by global atomics, which
    // hardly meet there), 4 lanes per ray and in parts, against one lane walking
    // segments: four views of 51 x 83 rays through 55 x 82 x 438 voxels 1.37 ->
    // 0.66 ms, of 64^2 through 256^3 5.6 -> 1.6
    axis = std::fabs(cam.e3[1]) >= std::fabs(cam.e3[2]) ? 1 : 2;
    if (std::fabs(cam.e3[axis]) < 0.05) return false;
    slot = 4;
    layer_cap = std::max(layer_cap, 8);
  }
  const double db = std::fabs(cam.e3[axis]);
  // layers per group: about K samples, at most `layer_cap` (LDS per wavefront
  // grows with the group and occupancy falls)
  const int Lmax = std::max(1, std::min(layer_cap, (int)std::lround((double)p->ckpt_K * p->step * db)));
  for (int L = Lmax; L >= 1; L = L > 1 ? L / 2 : 0) {
    const int smax = (int)std::floor((double)L / (p->step * db)) + 3;
    if (bwd_ring_lds_bytes(M, L, slot, smax, true) > 160 * 1024) continue;
    rv.ring = true;
    rv.axis = axis;
    rv.slot = slot;
    rv.L = L;
    rv.smax = smax;
    rv.ngrp = (int32_t)((n[axis] - 1 + L - 1) / L) + 1;
    return true;
  }
  return false;
}

}  // namespace

int render_with_state(vr_ctx* ctx, vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p,
                      float* out, hipStream_t s, vr_state** save) {
  if (vol->bricked) return fail(VR_EUNSUPPORTED, "saving forward state needs an unbricked volume");
  if (p->mode != VR_MODE_DVR) return fail(VR_EUNSUPPORTED, "the adjoint implements VR_MODE_DVR only");
  if (ctx->mask_n > 0) return fail(VR_EUNSUPPORTED, "the adjoint takes no channel mask (vr_mask_set(ctx, NULL, 0))");
  if (p->ckpt_K > 64) return fail(VR_EINVAL, "ckpt_K must be <= 64");
  const int32_t W = views[0].W, H = views[0].H;
  VR_TRY(ctx_begin(ctx, s));
  double vmin, vmax;
  VR_TRY(resolve_window(ctx, vol, s, vmin, vmax));
  vr_state* st = new (std::nothrow) vr_state();
  if (!st) return fail(VR_ENOMEM, "out of host memory");
  st->ctx = ctx;
  st->vol = vol;
  st->vol_version = vol->version;
  st->tf_version = ctx->tf_version;
  st->views.assign(views, views + nviews);
  st->p = *p;
  st->vmin = vmin;
  st->vmax = vmax;
  st->W = W;
  st->H = H;
  st->nviews = nviews;
  st->K = p->ckpt_K;
  double diag = 0.0;
  for (int i = 0; i < 3; i++) diag += (double)(vol->n[i] - 1) * (double)(vol->n[i] - 1);
  const int64_t nmax = (int64_t)std::ceil(std::sqrt(diag) / p->step) + 2;
  st->nseg = (int32_t)((nmax + st->K - 1) / st->K);
  const int64_t npix = (int64_t)W * H;
  // per-view layout and checkpoint offsets
  std::vector<Camera> cams((size_t)nviews);
  st->vs.assign((size_t)nviews, vr_state::View());
  int64_t ck_total = 0, sums_total = 0;
  const float max_alpha = table_max_alpha(ctx);
  Box whole;
  for (int i = 0; i < 3; i++) {
    whole.lo[i] = 0;
    whole.hi[i] = vol->n[i] - 1;
    whole.closed[i] = 1;
  }
  std::vector<FootShape> shapes((size_t)nviews);  // (axis 0: no cells)
  std::vector<int32_t> cells((size_t)nviews, 0);
  for (int32_t v = 0; v < nviews; v++) {
    make_camera(views[v], vol->n, cams[v]);
    vr_state::View& rv = st->vs[v];
    rv.off = ck_total;
    if (ctx->march_mode == 1 || !plan_ring_view(cams[v], p, ctx->tf_m, vol->n, ctx->bwd_layer_cap, rv)) {
      ck_total += (int64_t)st->nseg * npix;
      continue;
    }
    ck_total += (int64_t)rv.ngrp * npix;
    // the forward's march: footprint cells along the slab axis of the groups
    // where they are estimated faster, else gathers (three of the side streams
    // run at a time)
    FootShape fs;
    fs.axis = rv.axis;
    BoxSums box;
    add_box(box, cams[v], whole, npix, p->step);
    const MarchTimes t = march_times(cams[v], box, &fs, ctx->bwd_side ? std::min(nviews, 3) : 1);
    if (ctx->foot && (ctx->march_mode == 3 || t.cells <= t.gather) &&
        pick_foot(cams[v], vol->n, ctx->tf_m, true, ctx->ring_reg > 0, ctx->ring_nslots, ctx->foot_rays,
                  ctx->foot_pad, ctx->foot_kmax, fs, ctx->foot_maxpx, rv.axis) &&
        fs.reg && brick_rows_readable(vol, 0, (fs.nf + 3) & ~3) && samples_countable(cams[v], whole, p->step)) {
      shapes[v] = fs;
      if (ctx->debug_plan) std::fprintf(stderr, "[vr] view %d: saved by cells of %.1f x %.1f\n", v, fs.Tf, fs.Tg);
      continue;
    }
    rv.exact = true;
    // Few tiles leave most compute units without a workgroup of the adjoint, and
    // its time is one tile's chain of groups: parts of the groups side by side
    // until there are kPartBlocks workgroups (two views of 100 x 92 rays through
    // 61 x 83 x 72 voxels: 202 -> 95 us per view, the step 720 -> 585; one view of
    // 256^2 rays through 128^3: 690 -> 600; 16384 gains nothing more)
    const int32_t tiles = ntiles_of(W, H, 8, 8) * nviews, groups = rv.ngrp - 1;
    const int32_t want =
        max_alpha > kPartAlpha ? 1 : std::max(1, std::min({kPartBlocks / std::max(1, tiles), kMaxParts, groups / 2}));
    rv.part_groups = (groups + want - 1) / want;
    rv.parts = (groups + rv.part_groups - 1) / rv.part_groups;
    if (ctx->debug_plan) std::fprintf(stderr, "[vr] view %d: saved by gathers, %d parts\n", v, rv.parts);
    if (rv.parts > 1) {
      rv.sums = sums_total;
      sums_total += (int64_t)rv.parts * npix;
    }
  }
  const size_t sums_at = (sizeof(float) * (size_t)std::max<int64_t>(ck_total, 1) + 31) & ~(size_t)31;
  const size_t ck_bytes = sums_at + sizeof(double4) * (size_t)sums_total;
  const size_t nu_bytes = sizeof(int32_t) * ((size_t)nviews * npix + 64);
  // the buffers of the last destroyed state when they are large enough
  vr_ctx::StateBufs& sp = ctx->spare;
  if (sp.ckpt && sp.ckpt_bytes >= ck_bytes && sp.nused_bytes >= nu_bytes) {
    st->d_ckpt = sp.ckpt;
    st->d_nused = sp.nused;
    st->ckpt_bytes = sp.ckpt_bytes;
    st->nused_bytes = sp.nused_bytes;
    sp = vr_ctx::StateBufs();
  } else {
    st->ckpt_bytes = ck_bytes;
    st->nused_bytes = nu_bytes;
    if (dev_malloc(&st->d_ckpt, ck_bytes) != hipSuccess || dev_malloc(&st->d_nused, nu_bytes) != hipSuccess) {
      (void)hipGetLastError();
      vr_state_destroy(st);
      return fail(VR_ENOMEM, "hipMalloc for %zu bytes of checkpoints failed", ck_bytes);
    }
  }
  st->d_sums = reinterpret_cast<double4*>(reinterpret_cast<unsigned char*>(st->d_ckpt) + sums_at);
  st->d_flag = st->d_nused + (size_t)nviews * npix;
  {
    const hipError_t e = launch_fill(reinterpret_cast<float*>(st->d_flag), 1, 0.f, s);
    if (e != hipSuccess) {
      vr_state_destroy(st);
      return fail(VR_EHIP, "flag clear: %s", hipGetErrorString(e));
    }
  }
  MarchArgs base;
  std::memset(&base, 0, sizeof base);
  fill_march_common(base, vol, p, vmin, vmax, ctx->d_tf, ctx->tf_m);
  std::vector<unsigned char> host;
  std::vector<size_t> off_bv;
  pack_whole(vol, W, H, base.tile_w, base.tile_h, nviews, host, off_bv);
  int32_t most = 0;
  for (int32_t v = 0; v < nviews; v++) {
    if (shapes[v].axis == 0) continue;
    DevBrickView b;
    std::memcpy(&b, host.data() + off_bv[v], sizeof b);
    cells[v] = foot_brick(cams[v], shapes[v], whole, b);
    std::memcpy(host.data() + off_bv[v], &b, sizeof b);
    most = std::max(most, cells[v]);
  }
  const size_t ovf_stride = (256 + 4 * (size_t)most + 15) & ~(size_t)15;
  if (most > 0) {
    const int oc = ensure_device(&ctx->d_ovf, &ctx->ovf_bytes, ovf_stride * vr_ctx::kAux);
    if (oc != VR_OK) {
      vr_state_destroy(st);
      return oc;
    }
  }
  void* dtab = nullptr;
  int rc = upload_tables(ctx, s, host.data(), host.size(), &dtab);
  // views write disjoint frames and checkpoints: side by side on the side
  // streams, as the adjoint runs them
  const bool side = ctx->bwd_side && nviews > 1;
  if (rc == VR_OK && side) rc = stage_begin(ctx, VR_STAGE_MARCH, s);
  if (rc == VR_OK && side) rc = aux_fork(ctx, s);
  for (int32_t v = 0; v < nviews && rc == VR_OK; v++) {
    const hipStream_t vs = side ? ctx->aux[v % vr_ctx::kAux] : s;
    const vr_state::View& rv = st->vs[v];
    MarchArgs a = base;
    a.cam = cams[v];
    a.nbv = 1;
    a.ntiles = ntiles_of(W, H, a.tile_w, a.tile_h);
    a.bricks = reinterpret_cast<const DevBrick*>(dtab);
    a.bv = reinterpret_cast<const DevBrickView*>(reinterpret_cast<unsigned char*>(dtab) + off_bv[v]);
    a.img = reinterpret_cast<float4*>(out);
    SaveArgs sa;
    std::memset(&sa, 0, sizeof sa);
    sa.ckpt = st->d_ckpt + rv.off;
    sa.nused = st->d_nused + (int64_t)v * npix;
    sa.K = rv.ring ? rv.L : st->K;
    sa.npix = (int32_t)npix;
    sa.parts = rv.parts;
    sa.part_groups = rv.part_groups;
    sa.sums = st->d_sums + rv.sums;
    sa.vmin = vmin;
    sa.inv_range = vmax > vmin ? 1.0 / (vmax - vmin) : 0.0;
    if (rv.ring && ctx->bwd_bands)  // XCD bands of the adjoint
      xcd_bands(tile_costs(cams[v], base.hi, p->step, W, H), 1, st->vs[v].band);
    if (!side) rc = stage_begin(ctx, VR_STAGE_MARCH, s);
    if (rc == VR_OK) {
      hipError_t e;
      a.slab_axis = rv.axis;
      if (rv.ring && shapes[v].axis != 0) {
        int wpb = 4;
        foot_args(ctx, shapes[v], a, wpb);
        a.xcd_chunk = 16;
        a.ntiles = cells[v];
        unsigned char* ovf = reinterpret_cast<unsigned char*>(ctx->d_ovf) + (size_t)(v % vr_ctx::kAux) * ovf_stride;
        a.ovf_count = reinterpret_cast<unsigned int*>(ovf);
        a.ovf_tiles = reinterpret_cast<int32_t*>(ovf + 256);
        // pixels without samples are not written by the cells
        e = launch_zero(a.img + (int64_t)v * npix, npix, vs);
        if (e == hipSuccess) e = launch_fill(reinterpret_cast<float*>(sa.nused), npix, 0.f, vs);
        if (e == hipSuccess) e = launch_march_ring(a, wpb, vs, &sa);
      } else if (rv.ring) {
        a.ntiles = 4 * ((W + 3) / 4) * ((H + 3) / 4);  // blocks of 2 x 2 tiles of 2 x 2 pixels
        e = launch_march_save(a, sa, vs);
      } else {
        e = launch_fwd_save(a, sa, vs);
      }
      if (e != hipSuccess) rc = fail(VR_EHIP, "forward launch: %s", hipGetErrorString(e));
    }
    if (rc == VR_OK && !side) rc = stage_end(ctx, s);
  }
  if (rc == VR_OK && side) rc = aux_join(ctx, s);
  if (rc == VR_OK && side) rc = stage_end(ctx, s);
  if (rc == VR_OK) rc = ctx_end(ctx, s);
  if (rc != VR_OK) {
    vr_state_destroy(st);
    return rc;
  }
  *save = st;
  return VR_OK;
}

}  // namespace vr

using namespace vr;

extern "C" {

int vr_state_destroy(vr_state* st) {
  if (!st) return VR_OK;
  DeviceGuard g(st->ctx->device);
  vr_ctx::StateBufs& sp = st->ctx->spare;
  if (!sp.ckpt && st->d_ckpt && st->d_nused) {
    // kept for the context's next forward with state (calls on a context are
    // ordered, so no work of this state can still be reading them then)
    sp.ckpt = st->d_ckpt;
    sp.nused = st->d_nused;
    sp.ckpt_bytes = st->ckpt_bytes;
    sp.nused_bytes = st->nused_bytes;
  } else {
    (void)hipDeviceSynchronize();
    if (st->d_ckpt) (void)hipFree(st->d_ckpt);
    if (st->d_nused) (void)hipFree(st->d_nused);
  }
  delete st;
  return VR_OK;
}

int vr_state_info(const vr_state* st, int32_t view, int32_t* ring, int32_t* layers_per_group, double* samples_per_group) {
  clear_error();
  if (!st || view < 0 || view >= st->nviews) return fail(VR_EINVAL, "state NULL or view out of range");
  const vr_state::View& rv = st->vs[view];
  if (ring) *ring = rv.ring ? 1 : 0;
  if (layers_per_group) *layers_per_group = rv.ring ? rv.L : 0;
  if (samples_per_group) {
    if (rv.ring) {
      const double* e3 = st->views[view].R + 6;
      *samples_per_group = (double)rv.L / (st->p.step * std::fabs(e3[rv.axis]));
    } else {
      *samples_per_group = (double)st->K;
    }
  }
  return VR_OK;
}

int vr_render_backward(vr_ctx* ctx, const vr_volume* vol, const vr_state* st, const float* grad_out, float* grad_tf,
                       float* grad_vol, int accumulate, uintptr_t stream) {
  clear_error();
  if (!ctx || !vol || !st || !grad_out || !grad_tf)
    return fail(VR_EINVAL, "ctx, vol, st, grad_out and grad_tf must be non-NULL");
  if (st->ctx != ctx || st->vol != vol) return fail(VR_ESTATE, "state belongs to another context or volume");
  if (st->vol_version != vol->version) return fail(VR_ESTATE, "volume was re-bricked since the forward");
  if (st->tf_version != ctx->tf_version) return fail(VR_ESTATE, "transfer function changed since the forward");
  DeviceGuard g(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  VR_TRY(ctx_begin(ctx, s));
  const int32_t M = ctx->tf_m, W = st->W, H = st->H;
  const int64_t npix = (int64_t)W * H;
  if (!accumulate) {
    VR_HIP(launch_fill(grad_tf, (int64_t)M * 4, 0.f, s));
    if (grad_vol) VR_HIP(launch_fill(grad_vol, vol->n[0] * vol->n[1] * vol->n[2], 0.f, s));
  }
  MarchArgs base;
  std::memset(&base, 0, sizeof base);
  vr_params p = st->p;
  p.tile = 8;
  fill_march_common(base, vol, &p, st->vmin, st->vmax, ctx->d_tf, M);
  std::vector<unsigned char> host;
  std::vector<size_t> off_bv;
  pack_whole(vol, W, H, base.tile_w, base.tile_h, st->nviews, host, off_bv);
  void* dtab = nullptr;
  VR_TRY(upload_tables(ctx, s, host.data(), host.size(), &dtab));
  MarchArgs a0 = base;
  a0.ntiles = ntiles_of(W, H, base.tile_w, base.tile_h);
  // every view's workgroups write their table partials into a region of their
  // own, so the views can run side by side (a view's tiles differ in ray
  // length; alone, its launch leaves compute units idle at its tail) and one
  // fixed-order reduction sums them all
  std::vector<int64_t> pbase((size_t)st->nviews + 1, 0);
  for (int32_t v = 0; v < st->nviews; v++) {
    const vr_state::View& rv = st->vs[v];
    BwdArgs bb;
    std::memset(&bb, 0, sizeof bb);
    std::memcpy(bb.band, rv.band, sizeof bb.band);
    bb.parts = rv.parts;
    bb.run = bwd_ring_run(a0.ntiles, M);
    pbase[v + 1] = pbase[v] + (rv.ring ? bwd_ring_blocks(a0, bb) : bwd_blocks(a0));
  }
  // T between checkpoints by division only where what it divides by is what the
  // checkpoints were made of, or nearly
  const bool opaque = table_max_alpha(ctx) > kMaxDivAlpha, steep = table_slope(ctx) > kMaxDivSlope;
  bool replayed = false;
  const bool side = ctx->bwd_side && st->nviews > 1;
  int64_t nslots = 1;
  for (int32_t v = 0; v < st->nviews; v++) nslots = std::max(nslots, pbase[v + 1] - pbase[v]);
  if (side) nslots = std::max<int64_t>(pbase.back(), 1);
  VR_TRY(ensure_device(&ctx->d_scratch, &ctx->scratch_bytes,
                       sizeof(double) * 4 * (size_t)M * ((size_t)nslots + (size_t)tf_reduce_slices())));
  double* part = reinterpret_cast<double*>(ctx->d_scratch);
  double* slices = part + 4 * (size_t)M * (size_t)nslots;
  VR_TRY(stage_begin(ctx, VR_STAGE_BACKWARD, s));
  if (side) VR_TRY(aux_fork(ctx, s));
  for (int32_t v = 0; v < st->nviews; v++) {
    const vr_state::View& rv = st->vs[v];
    const hipStream_t vs = side ? ctx->aux[v % vr_ctx::kAux] : s;
    MarchArgs a = base;
    make_camera(st->views[v], vol->n, a.cam);
    a.nbv = 1;
    a.ntiles = a0.ntiles;
    a.bricks = reinterpret_cast<const DevBrick*>(dtab);
    a.bv = reinterpret_cast<const DevBrickView*>(reinterpret_cast<unsigned char*>(dtab) + off_bv[v]);
    BwdArgs ba;
    std::memset(&ba, 0, sizeof ba);
    ba.ckpt = st->d_ckpt + rv.off;
    ba.nused = st->d_nused + (int64_t)v * npix;
    ba.gout = reinterpret_cast<const float4*>(grad_out) + (int64_t)v * npix;
    ba.gvol = grad_vol;
    ba.tf_part = part + (side ? 4 * (size_t)M * (size_t)pbase[v] : 0);
    ba.vmin = st->vmin;
    ba.inv_range = st->vmax > st->vmin ? 1.0 / (st->vmax - st->vmin) : 0.0;
    ba.K = rv.ring ? rv.L : st->K;
    ba.npix = (int32_t)npix;
    ba.smax = rv.smax;
    ba.replay = opaque || (steep && !rv.exact) ? 1 : 0;
    replayed = replayed || ba.replay != 0;
    std::memcpy(ba.band, rv.band, sizeof ba.band);
    ba.flag = st->d_flag;
    ba.parts = rv.parts;
    ba.run = bwd_ring_run(a.ntiles, M);
    ba.part_groups = rv.part_groups;
    ba.sums = st->d_sums + rv.sums;
    if (rv.ring) {
      a.slab_axis = rv.axis;
      a.ring_slot = rv.slot;
      VR_HIP(launch_bwd_ring(a, ba, vs));
    } else {
      VR_HIP(launch_bwd(a, ba, vs));
    }
    if (!side) VR_HIP(launch_tf_reduce(part, (int)(pbase[v + 1] - pbase[v]), M * 4, grad_tf, slices, s));
  }
  if (side) {
    VR_TRY(aux_join(ctx, s));
    VR_HIP(launch_tf_reduce(part, (int)pbase.back(), M * 4, grad_tf, slices, s));
  }
  VR_TRY(stage_end(ctx, s));
  VR_TRY(ctx_end(ctx, s));
  // the replay's bound on the samples of one ray in one checkpoint group holds
  // by construction; a group that exceeded it is reported, not clamped (only
  // the replay can).  Either way the call ends with its stream idle.
  if (!replayed) {
    VR_HIP(hipStreamSynchronize(s));
    return VR_OK;
  }
  int32_t flag = 0;
  VR_HIP(hipMemcpyAsync(&flag, st->d_flag, sizeof flag, hipMemcpyDeviceToHost, s));
  VR_HIP(hipStreamSynchronize(s));
  if (flag) return fail(VR_EHIP, "adjoint: a ray held more samples in one checkpoint group than the planned bound");
  return VR_OK;
}

}  // extern "C"
