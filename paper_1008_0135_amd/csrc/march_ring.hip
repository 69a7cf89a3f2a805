// march_ring.hip -- forward march with per-layer voxel windows kept in an LDS
// ring and filled by direct global->LDS loads (gfx950).
//
// Same samples, same per-sample arithmetic and the same order as the gather
// march (paper Sec. 2.4: each ray is sampled between its entry and exit points
// and accumulated front to back with early termination); only the way the
// eight trilinear corners reach the lanes differs.
//
// A wavefront owns an 8 x 8 tile of pixel rays inside one brick and walks the
// brick one cell layer at a time along a slab axis b (y or z, chosen per view
// on the host so that rows along x -- the contiguous storage axis -- stay
// long).  Cell layer c is sampled from voxel layers c and c + 1.  For every
// voxel layer V the wavefront loads a window of rows along x: the box that
// holds the cells of every sample of its 64 rays lying between the planes
// b = V - 1 and b = V + 1, bounded from the four corner rays of the tile (the
// rays are parallel, so the corners bound the bundle on any plane).  Windows
// go into a ring of three LDS slots: while cell layer c is sampled from the
// slots of V = c and c + 1, the window of the layer after next is already in
// flight (global_load_lds_dwordx4: 16 bytes per lane straight into LDS, no
// registers, no store instructions).  Every voxel layer is read once per
// tile, with no halo layer read twice.
//
// The layer index, the window origins and the slot addresses are uniform over
// the wavefront (scalar registers); lanes step through their own samples of
// the current layer (two to three on typical views).  Four wavefronts share a
// workgroup only to share the transfer-function table in LDS; after loading it
// each wavefront runs on its own, with no workgroup barrier.
//
// Carried state (a.carry, opacity tested over the whole ray): the image is the
// output frame holding each ray's (C, T) from the bricks in front of this
// one; a ray starts from it (and not at all once 1 - T >= tau) and leaves its
// new state there.
#include <cstring>

#include "ring_common.h"
#include "sample.h"
#include "vr_internal.h"

namespace vr {

namespace {

using namespace ring;

constexpr int kSlotsMax = 3;

// MIP: maximum intensity projection (no table).
template <bool MIP, bool TWO, bool MASK>
__global__ __launch_bounds__(256) void k_march_ring(MarchArgs a) {
  static_assert(!(MASK && TWO), "the channel mask: three-slot forward marches");
  constexpr int kSlots = TWO ? 2 : 3;
  extern __shared__ float4 smem[];
  float4* s_tf = smem;
  for (int i = threadIdx.x; i < a.M; i += blockDim.x) s_tf[i] = a.tf[i];
  __syncthreads();

  const int wpb = (int)(blockDim.x >> 6);
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int slot = a.ring_slot;  // floats per ring slot
  float* s_ring = reinterpret_cast<float*>(smem + a.M) + (size_t)wave * kSlots * slot;

  // XCD-aware order: workgroup b runs on XCD b % 8; give each XCD a
  // contiguous range of tiles so that neighbouring tiles share its L2
  const int ngroups = (a.ntiles + wpb - 1) / wpb;
  const int per = (ngroups + 7) >> 3;
  int grp = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  const int tile = grp * wpb + wave;
  if (tile >= a.ntiles) return;

  int lo = 0, hi = a.nbv - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.bv[mid].tile_begin <= tile) lo = mid;
    else hi = mid - 1;
  }
  const DevBrickView bvw = a.bv[lo];
  const DevBrick br = a.bricks[bvw.brick];
  const int t = tile - bvw.tile_begin;
  // Footprint cells (parallel rays): the wavefront's rays are the pixels whose
  // rays cross the brick-local plane b = 0 inside cell (ci, cj) of the
  // Tf x Tg grid in (f, g).  Each image row holds one run of them (the cell
  // coordinate is monotone along a row); lane r measures the run of row
  // vrow0 + r, and a wave scan numbers the cell's pixels row by row.  The
  // wavefront marches the cell's first 64 pixels.
  const bool foot = a.foot != 0;
  int ci = 0, cj = 0;
  FootRuns fr;
  int tx = 0, ty = 0;
  if (foot) {
    foot_cell(a, bvw, t, ci, cj);
    fr = foot_runs(a, bvw, ci, cj, lane);
    // cells of more than 64 pixels: the pixels past the 64th are marched by
    // k_march_ring_ovf after this launch
    if (fr.n > 64 && lane == 0) a.ovf_tiles[atomicAdd(a.ovf_count, 1u)] = tile * 8;
  } else {
    // tile numbering inside the brick's rectangle.  Tiles started together run
    // at about the same layer; the L2 keeps a line only a few microseconds, so
    // lines two windows share (the partial 128-byte ends of rows, the halo
    // rows) are fetched once only when the two tiles are close in this order.
    // Blocks of tiles put neighbours on both image axes close, whichever way
    // the view turns the image against the storage axes.
    if (a.tile_order == 1) {
      const int th = (bvw.h + 7) >> 3;
      tx = t / th;
      ty = t - tx * th;
    } else if (a.tile_order == 2) {
      // blocks of bw x bh tiles in row order (tiles in a block in row order),
      // then the tiles right of the last whole block column, then those below
      // the last whole block row
      const int tw = bvw.tiles_x, th = (bvw.h + 7) >> 3, bw = a.tile_bw, bh = a.tile_bh;
      const int fw = tw / bw, fh = th / bh, nfull = fw * fh * bw * bh;
      if (t < nfull) {
        const int q = t / (bw * bh), r = t - q * (bw * bh), qy = q / fw;
        const int ry = r / bw;
        tx = (q - qy * fw) * bw + (r - ry * bw);
        ty = qy * bh + ry;
      } else {
        int r = t - nfull;
        const int rw = tw - fw * bw;
        if (r < rw * th) {
          ty = r / rw;
          tx = fw * bw + (r - ty * rw);
        } else {
          r -= rw * th;
          const int lw = fw * bw;
          const int ry = r / lw;
          tx = r - ry * lw;
          ty = fh * bh + ry;
        }
      }
    } else {
      ty = t / bvw.tiles_x;
      tx = t - ty * bvw.tiles_x;
    }
  }
  // the march of the wavefront's 64 rays (a single pass: early exits leave it)
  do {
  int lx, ly, u, v;
  bool valid;
  if (foot) {
    int ur, vr;
    foot_pixel(fr, lane, ur, vr);
    valid = lane < fr.n;
    u = valid ? ur : 0;
    v = valid ? vr : 0;
    lx = u - bvw.x0;
    ly = v - bvw.y0;
  } else {
    lx = tx * 8 + (lane & 7);
    ly = ty * 8 + (lane >> 3);
    valid = lx < bvw.w && ly < bvw.h;
    u = bvw.x0 + min(lx, bvw.w - 1);
    v = bvw.y0 + min(ly, bvw.h - 1);
  }
  // a footprint cell's pixel lies in the brick's rectangle whenever its ray
  // has samples here; the image arena (or output) was cleared before the
  // march, so only pixels with samples are written
  const bool inrect = lx >= 0 && lx < bvw.w && ly >= 0 && ly < bvw.h;

  // ---- per-lane ray setup (double precision, shared with every march)
  double o[3];
  const double* d = a.cam.e3;
  pixel_origin(a.cam, u, v, o);
  int cnt = 0;
  float px = 0.f, py = 0.f, pz = 0.f;
  float4* const dst =
      a.carry ? a.img + (int64_t)v * a.cam.W + u : a.img + bvw.img_off + (int64_t)ly * bvw.w + lx;
  const bool wr_ok = a.carry || !foot || inrect;  // dst is this pixel's place
  float4 carried = make_float4(0.f, 0.f, 0.f, 1.f);
  if (a.carry && valid) carried = *dst;
  const bool live = !a.carry || 1.f - carried.w < a.tau;
  double tin;
  int64_t n;
  if (valid && live && ray_lattice(o, d, a.hi, a.step, tin, n)) {
    int64_t k0, k1;
    brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0, k1);
    if (k1 > k0) {
      const double t0 = tin + ((double)k0 + 0.5) * a.step;
      px = (float)(o[0] + t0 * d[0] - (double)br.lo[0]);
      py = (float)(o[1] + t0 * d[1] - (double)br.lo[1]);
      pz = (float)(o[2] + t0 * d[2] - (double)br.lo[2]);
      cnt = (int)(k1 - k0);
    }
  }
  const float sx = (float)(a.step * d[0]), sy = (float)(a.step * d[1]), sz = (float)(a.step * d[2]);

  // ---- frame: b = slab axis (axis 2 or 3), g = the other of axes 2/3, f = axis 1
  const bool by = a.slab_axis == 1;
  const float pb = by ? py : pz, sb = by ? sy : sz;
  const int cloB = by ? br.clo[1] : br.clo[2], chiB = by ? br.chi[1] : br.chi[2];
  const int cloG = by ? br.clo[2] : br.clo[1], chiG = by ? br.chi[2] : br.chi[1];
  const int cloF = br.clo[0], chiF = br.chi[0];
  const double db = by ? d[1] : d[2], dg = by ? d[2] : d[1];
  const bool up = db > 0.0;

  // cell layers (along b) of the lane's first and last samples
  int c_first = up ? 0x7fffffff : -0x7fffffff, c_last = up ? -0x7fffffff : 0x7fffffff;
  if (cnt > 0) {
    c_first = (int)floorf(__builtin_amdgcn_fmed3f(pb, (float)cloB, (float)chiB));
    c_last = (int)floorf(__builtin_amdgcn_fmed3f(fmaf((float)(cnt - 1), sb, pb), (float)cloB, (float)chiB));
  }
  int Lbeg, Lend;  // first and last cell layer in marching order
  if (up) {
    Lbeg = uni(wave_imin(c_first));
    Lend = uni(wave_imax(c_last));
  } else {
    Lbeg = uni(wave_imax(c_first));
    Lend = uni(wave_imin(c_last));
  }
  if (up ? Lbeg > Lend : Lbeg < Lend) {
    if (valid && !a.carry && !foot) *dst = make_float4(0.f, 0.f, 0.f, 0.f);
    continue;
  }
  const int nlay = up ? Lend - Lbeg + 1 : Lbeg - Lend + 1;  // cell layers

  // ---- window geometry from the tile's corner rays (lanes 0..3)
  // A corner ray meets the plane b = P at f = Af + P rf, g = Ag + P rg.
  const double rfd = d[0] / db, rgd = dg / db;
  const float rf = (float)rfd, rg = (float)rgd;
  float Af = 0.f, Ag = 0.f;
  if (!foot) {
    const int cx = bvw.x0 + tx * 8, cy = bvw.y0 + ty * 8;
    const int ex = min(cx + 7, bvw.x0 + bvw.w - 1), ey = min(cy + 7, bvw.y0 + bvw.h - 1);
    const int cc = lane & 3;
    double oc[3];
    pixel_origin(a.cam, (cc & 1) ? ex : cx, (cc & 2) ? ey : cy, oc);
    const double ob = (by ? oc[1] : oc[2]) - (double)(by ? br.lo[1] : br.lo[2]);
    Af = (float)(oc[0] - (double)br.lo[0] - ob * rfd);
    Ag = (float)((by ? oc[2] : oc[1]) - (double)(by ? br.lo[2] : br.lo[1]) - ob * rgd);
  }
  float Af_lo = unif(wmin4(Af)), Af_hi = unif(wmax4(Af));
  float Ag_lo = unif(wmin4(Ag)), Ag_hi = unif(wmax4(Ag));
  if (foot) {  // the cell's rectangle on the plane b = 0
    Af_lo = (float)((double)ci * a.foot_Tf);
    Af_hi = (float)((double)(ci + 1) * a.foot_Tf);
    Ag_lo = (float)((double)cj * a.foot_Tg);
    Ag_hi = (float)((double)(cj + 1) * a.foot_Tg);
  }
  const float arf = fabsf(rf), arg = fabsf(rg);
  // window extents: f_hi - f_lo + 1 <= floor(span + 0.1) + 3 for the 0.05 margins
  int NF, NG;
  if (foot) {
    NF = a.foot_nf;
    NG = a.foot_ng;
  } else {
    NF = uni((int)floorf(Af_hi - Af_lo + 2.f * arf + 0.2f) + 3);
    NG = uni((int)floorf(Ag_hi - Ag_lo + 2.f * arg + 0.2f) + 3);
  }
  const int pitch = (NF + 3) & ~3;
  NG = min(NG, chiG + 2 - cloG);
  const int ysl = br.sy, zsl = br.sz;
  const int sB = by ? ysl : zsl, sG = by ? zsl : ysl;
  gfloat* gbase = (gfloat*)br.base;

  float Cr = carried.x, Cg = carried.y, Cb = carried.z, T = carried.w, mx = 0.f;
  int j = 0;
  bool done = cnt == 0;

  if (pitch > chiF + 2 - cloF || pitch * NG > slot || pitch > 256 ||
      ((int64_t)(64 / (pitch >> 2)) * sG + pitch) * 4 >= ((int64_t)1 << 32)) {
    // the window does not fit: read the corners from global memory
    while (!done) {
      const Cell c = cell_of(sample_pos(j, px, py, pz, sx, sy, sz), br);
      gfloat* p = gbase + (c.iz * zsl + c.iy * ysl + c.ix);
      const float val = trilerp(p[0], p[1], p[ysl], p[ysl + 1], p[zsl], p[zsl + 1], p[zsl + ysl], p[zsl + ysl + 1], c);
      ++j;
      if (MIP) {
        float s = norm_value(val, a.vmin, a.inv_range);
        if constexpr (MASK) s *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], c);
        mx = fmaxf(mx, s);
        if (j >= cnt || mx >= 1.f) done = true;
      } else {
        Classified k = classify(val, a.vmin, a.inv_range, a.M, s_tf);
        if constexpr (MASK) k.a *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], c);
        accumulate(k, Cr, Cg, Cb, T);
        if (j >= cnt || 1.f - T >= a.tau) done = true;
      }
    }
    // carried state: only rays with samples here write (another brick of the
    // wave whose rectangle holds the pixel may update it)
    if (valid && cnt > 0 && wr_ok)
      *dst = MIP ? make_float4(mx, mx, mx, mx) : make_float4(Cr, Cg, Cb, a.carry ? T : 1.f - T);
    else if (valid && !a.carry && !foot)
      *dst = make_float4(0.f, 0.f, 0.f, 0.f);
    continue;
  }

  // window of voxel layer V (brick-local): rows [g0, g0 + NG), columns [f0, f0 + pitch)
  auto window = [&](int V) {
    Window w;
    const float Pf = (float)V * rf, Pg = (float)V * rg;
    const int flo = max((int)floorf(Af_lo + Pf - arf - 0.05f), cloF);
    const int glo = max((int)floorf(Ag_lo + Pg - arg - 0.05f), cloG);
    w.f0 = uni(max(cloF, min(flo, chiF + 2 - pitch)));
    w.g0 = uni(max(cloG, min(glo, chiG + 2 - NG)));
    return w;
  };
  // chunk (16 bytes) i of a window: row i / (pitch / 4), column 4 (i % (pitch / 4))
  // A load instruction carries R whole rows (R = 64 / (pitch / 4) lanes per
  // row group; the remaining lanes idle), so a lane's offset from the group's
  // first row is fixed for the tile and only the uniform group base moves.
  const int nf4 = pitch >> 2;
  const int R = uni(64 / nf4);
  const int rl = lane / nf4, c4l = lane - rl * nf4;
  const bool lane_on = rl < R;
  const int nload = uni((NG + R - 1) / R);  // load instructions per layer
  const unsigned voff = (unsigned)(rl * sG + 4 * c4l) * 4u;
  const int64_t gstep = (int64_t)R * sG;
  const unsigned lstep = (unsigned)(R * pitch) * 4u;
  auto issue = [&](int V, const Window& w, float* sdst) {
    gfloat* gb = gbase + ((int64_t)V * sB + (int64_t)w.g0 * sG + w.f0);
    const unsigned l0 = uni(lds_addr(sdst));
    for (int k = 0; k < nload; ++k)
      if (lane_on && k * R + rl < NG) lds_dma16(unip(gb + k * gstep), voff, (unsigned)uni((int)(l0 + (unsigned)k * lstep)));
  };

  // voxel layers in marching order: V_k = Lbeg + k (up) or Lbeg + 1 - k (down);
  // cell layer c_k = Lbeg +- k reads V_k and V_{k+1}
  const int vstep = up ? 1 : -1;
  const int V0 = up ? Lbeg : Lbeg + 1;
  const float fclo = (float)cloB, fchi = (float)chiB;
  Window w0 = window(V0), w1 = window(V0 + vstep);
  issue(V0, w0, s_ring);
  issue(V0 + vstep, w1, s_ring + slot);
  int s0 = 0;  // slot of V_k
  for (int k = 0; k < nlay; ++k) {
    wait_loads();  // V_k and V_{k+1} are in LDS
    // start V_{k+2} into the slot V_{k-1} used (cell layer c_{k-1} is finished);
    // with two slots, into the slot of V_k once c_k is finished
    const int s1 = s0 == kSlots - 1 ? 0 : s0 + 1;
    const int s2 = s1 == kSlots - 1 ? 0 : s1 + 1;
    Window w2;
    if (k + 1 < nlay) {
      const int V2 = V0 + (k + 2) * vstep;
      w2 = window(V2);
      if (!TWO) issue(V2, w2, s_ring + s2 * slot);
    }
    // lower and upper voxel layer of cell layer c_k
    const int c = up ? Lbeg + k : Lbeg - k;
    const Window& wl = up ? w0 : w1;
    const Window& wu = up ? w1 : w0;
    const int sl = up ? s0 : s1, su = up ? s1 : s0;
    const float* baseL = s_ring + (sl * slot - wl.g0 * pitch - wl.f0);
    const int dU = (su * slot - wu.g0 * pitch - wu.f0) - (sl * slot - wl.g0 * pitch - wl.f0);
    while (!done) {
      const SamplePos q = sample_pos(j, px, py, pz, sx, sy, sz);
      const int ib = (int)floorf(__builtin_amdgcn_fmed3f(by ? q.y : q.z, fclo, fchi));
      if (ib != c) break;
      const Cell cl = cell_of(q, br);
      const int ig = by ? cl.iz : cl.iy;
      const float* p = baseL + (__mul24(ig, pitch) + cl.ix);
      const float* pu = p + dU;
      // corners v[dz][dy][dx]: within a window rows run along g, layers along b
      const float l00 = p[0], l01 = p[1], l10 = p[pitch], l11 = p[pitch + 1];
      const float u00 = pu[0], u01 = pu[1], u10 = pu[pitch], u11 = pu[pitch + 1];
      const float val = by ? trilerp(l00, l01, u00, u01, l10, l11, u10, u11, cl)
                           : trilerp(l00, l01, l10, l11, u00, u01, u10, u11, cl);
      ++j;
      if (MIP) {
        float s = norm_value(val, a.vmin, a.inv_range);
        if constexpr (MASK) s *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], cl);
        mx = fmaxf(mx, s);
        if (j >= cnt || mx >= 1.f) done = true;
      } else {
        Classified k = classify(val, a.vmin, a.inv_range, a.M, s_tf);
        if constexpr (MASK) k.a *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], cl);
        accumulate(k, Cr, Cg, Cb, T);
        if (j >= cnt || 1.f - T >= a.tau) done = true;
      }
    }
    if (__all(done)) break;
    if (TWO && k + 1 < nlay) issue(V0 + (k + 2) * vstep, w2, s_ring + s0 * slot);
    s0 = s1;
    w0 = w1;
    w1 = w2;
  }
  wait_loads();  // no load may still target LDS when the wavefront ends (or the next batch starts)
  if (valid && wr_ok && (cnt > 0 || (!a.carry && !foot)))
    *dst = MIP ? make_float4(mx, mx, mx, mx) : make_float4(Cr, Cg, Cb, a.carry ? T : 1.f - T);
  } while (false);

}

// Pixels past the 64th of footprint cells (listed by the march): one ray per
// lane, its corners read from global memory; the same samples, arithmetic and
// order as every march.  Wavefronts take listed cells in turn until the list
// is done.
template <bool MIP, bool MASK, bool SAVE = false>
__global__ __launch_bounds__(256) void k_march_ring_ovf(MarchArgs a, SaveArgs sa) {
  extern __shared__ float4 smem[];
  float4* s_tf = smem;
  for (int i = threadIdx.x; i < a.M; i += blockDim.x) s_tf[i] = a.tf[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int nw = (int)(gridDim.x * (blockDim.x >> 6));
  const int n_listed = (int)*a.ovf_count;
  for (int e = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); e < n_listed; e += nw) {
    const int tile = a.ovf_tiles[e] >> 3, w = a.ovf_tiles[e] & 7;
    const DevBrickView bvw = a.bv[find_bv(a, tile)];
    const DevBrick br = a.bricks[bvw.brick];
    int ci, cj;
    if (a.blk_f > 0) block_cell(a, bvw, tile - bvw.tile_begin, w, ci, cj);
    else foot_cell(a, bvw, tile - bvw.tile_begin, ci, cj);
    const FootRuns fr = a.cam.persp ? foot_runs_persp(a, bvw, br, ci, cj, lane) : foot_runs(a, bvw, ci, cj, lane);
    gfloat* gb = (gfloat*)br.base;
    const int ys = br.sy, zs = br.sz;
    for (int k0 = 64; k0 < fr.n; k0 += 64) {
      int uu, vv;
      foot_pixel(fr, k0 + lane, uu, vv);
      if (k0 + lane >= fr.n) continue;
      const int lx = uu - bvw.x0, ly = vv - bvw.y0;
      const bool inr = lx >= 0 && lx < bvw.w && ly >= 0 && ly < bvw.h;
      float4* const dst =
          a.carry ? a.img + (int64_t)vv * a.cam.W + uu : a.img + bvw.img_off + (int64_t)ly * bvw.w + lx;
      float4 c0 = make_float4(0.f, 0.f, 0.f, 1.f);
      if (a.carry) c0 = *dst;
      if (a.carry && !(1.f - c0.w < a.tau)) continue;
      double o[3], d[3];
      pixel_ray(a.cam, uu, vv, o, d);  // parallel rays: the view direction
      double tin;
      int64_t n, k0b, k1b;
      if (!ray_lattice(o, d, a.hi, a.step, tin, n)) continue;
      brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0b, k1b);
      if (k1b <= k0b) continue;
      const double t0 = tin + ((double)k0b + 0.5) * a.step;
      const float px = (float)(o[0] + t0 * d[0] - (double)br.lo[0]);
      const float py = (float)(o[1] + t0 * d[1] - (double)br.lo[1]);
      const float pz = (float)(o[2] + t0 * d[2] - (double)br.lo[2]);
      const float sx = (float)(a.step * d[0]), sy = (float)(a.step * d[1]), sz = (float)(a.step * d[2]);
      const int cnt = (int)(k1b - k0b);
      float Cr = c0.x, Cg = c0.y, Cb = c0.z, T = c0.w, mx = 0.f;
      [[maybe_unused]] int grp = -1;
      [[maybe_unused]] double Td = 1.0;  // T as the checkpoints have it: a double product
      int j = 0;
      while (j < cnt) {
        const Cell c = cell_of(sample_pos(j, px, py, pz, sx, sy, sz), br);
        if constexpr (SAVE) {
          const int b = a.slab_axis, ib = b == 1 ? c.iy : c.iz;
          const int gi = (a.cam.e3[b] > 0.0 ? ib - br.clo[b] : br.chi[b] - ib) / sa.K;
          // (the groups without a sample in front of it too, as k_march_save)
          for (int g = grp < 0 ? gi : grp + 1; g <= gi; ++g) sa.ckpt[(int64_t)g * sa.npix + vv * a.cam.W + uu] = (float)Td;
          grp = gi;
        }
        gfloat* p = gb + (c.iz * zs + c.iy * ys + c.ix);
        const float val = trilerp(p[0], p[1], p[ys], p[ys + 1], p[zs], p[zs + 1], p[zs + ys], p[zs + ys + 1], c);
        ++j;
        if (MIP) {
          float sv = norm_value(val, a.vmin, a.inv_range);
          if constexpr (MASK) sv *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], c);
          mx = fmaxf(mx, sv);
          if (mx >= 1.f) break;
        } else {
          Classified k = classify(val, a.vmin, a.inv_range, a.M, s_tf);
          if constexpr (MASK) k.a *= channel_weight(a.mask, a.mask_axis, br.lo[a.mask_axis], c);
          accumulate(k, Cr, Cg, Cb, T);
          if constexpr (SAVE) Td = fma(-Td, (double)k.a, Td);
          if (1.f - T >= a.tau) break;
        }
      }
      if constexpr (SAVE) {
        sa.ckpt[(int64_t)(grp + 1) * sa.npix + vv * a.cam.W + uu] = (float)Td;
        sa.nused[vv * a.cam.W + uu] = j;
      }
      if (a.carry || inr)
        *dst = MIP ? make_float4(mx, mx, mx, mx) : make_float4(Cr, Cg, Cb, a.carry ? T : 1.f - T);
    }
  }
}

__global__ void k_ovf_reset(unsigned int* count) { *count = 0u; }

}  // namespace

size_t ring_lds_bytes(const MarchArgs& a, int wpb) {
  const int ns = a.ring_nslots == 2 ? 2 : kSlotsMax;
  return sizeof(float4) * (size_t)a.M + sizeof(float) * (size_t)wpb * ns * (size_t)a.ring_slot;
}

static hipError_t launch_march_ring_main(const MarchArgs& a, int wpb, hipStream_t s);

hipError_t launch_march_ring(const MarchArgs& a, int wpb, hipStream_t s, const SaveArgs* sa) {
  if (a.ntiles <= 0) return hipSuccess;
  if (sa && (!a.foot || !a.ring_reg || a.blk_f > 0)) return hipErrorInvalidValue;  // (saved by the cells march)
  if (!a.foot) return launch_march_ring_main(a, wpb, s);
  // footprint cells: clear the overflow list, march, then the listed cells' pixels past the 64th
  // (perspective views: the register-staged cell march only)
  if ((a.cam.persp && (!a.ring_reg || a.blk_f > 0)) || !a.ovf_count || !a.ovf_tiles) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_ovf_reset, dim3(1), dim3(1), 0, s, a.ovf_count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = a.blk_f > 0 ? launch_march_block(a, s)
                   : (a.ring_reg ? launch_march_cells(a, wpb, s, sa) : launch_march_ring_main(a, wpb, s));
  if (e != hipSuccess) return e;
  const dim3 g(256), b(256);
  const size_t lds = sizeof(float4) * (size_t)a.M;
  SaveArgs save;
  std::memset(&save, 0, sizeof save);
  if (sa) save = *sa;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, lds, s, a, save); };
  if (sa) go(k_march_ring_ovf<false, false, true>);
  else if (a.mip && a.mask) go(k_march_ring_ovf<true, true>);
  else if (a.mip) go(k_march_ring_ovf<true, false>);
  else if (a.mask) go(k_march_ring_ovf<false, true>);
  else go(k_march_ring_ovf<false, false>);
  return hipGetLastError();
}

static hipError_t launch_march_ring_main(const MarchArgs& a, int wpb, hipStream_t s) {
  if (a.tile_w != 8 || a.ring_slot <= 0 || (a.ring_slot & 3) != 0 || (wpb != 1 && wpb != 2 && wpb != 4))
    return hipErrorInvalidValue;
  const int groups = (a.ntiles + wpb - 1) / wpb;
  const int grid = ((groups + 7) / 8) * 8;
  const dim3 g(grid), b(64 * wpb);
  const size_t lds = ring_lds_bytes(a, wpb);
  if (a.mc > 0 || a.cam.persp) return hipErrorInvalidValue;  // (gather marches, perspective cells)
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, lds, s, a); };
  if (a.mask) {
    // the channel mask lives in instantiations of its own (three slots)
    if (a.ring_nslots == 2) return hipErrorInvalidValue;
    if (a.mip) go(k_march_ring<true, false, true>);
    else go(k_march_ring<false, false, true>);
  } else if (a.ring_nslots == 2) {
    if (a.mip) go(k_march_ring<true, true, false>);
    else go(k_march_ring<false, true, false>);
  } else {
    if (a.mip) go(k_march_ring<true, false, false>);
    else go(k_march_ring<false, false, false>);
  }
  return hipGetLastError();
}

}  // namespace vr
