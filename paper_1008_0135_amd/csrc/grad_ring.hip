// grad_ring.hip -- the adjoint march on the ring-window layout (gfx950).
//
// The differentiable forward (k_march_cells, k_march_ring_ovf, k_march_save)
// stores, for every group of L consecutive cell layers along the slab axis b
// (counted in marching order from the box's first) that a ray has samples in,
// its transmittance at the group's start, and after the last one at its end.
// This kernel walks the groups of an 8 x 8 ray tile from the last to the first.  A workgroup
// of four wavefronts takes one tile: four neighbouring lanes share a ray and
// hold four consecutive samples of it, so a ray's chain is a quarter as long
// and the tile's windows serve four wavefronts.  For a group it
//   1. copies the L + 1 voxel windows the group's samples read into LDS
//      (rows along axis 1, as in the forward) beside L + 1 gradient windows;
//   2. takes the group's samples four per ray from the last to the first with
//      the recursion
//        dL/dc_k = g_rgb T_{k-1} a_k,
//        dL/da_k = T_{k-1} (h_k - S_k),  h_k = g_rgb . c_k + g_A,
//        S_{k-1} = a_k h_k + (1 - a_k) S_k
//      (S: the output gradient times what the ray gathers behind a sample, per
//      unit of transmittance), carrying S from block to block; table gradients
//      go to double LDS accumulators (one set per workgroup, reduced by
//      k_tf_reduce), voxel gradients to the gradient windows with LDS double
//      atomics;
//   3. adds the finished gradient windows to the gradient volume with one float
//      atomic per non-zero window voxel, row after row (coalesced), instead of
//      eight scattered atomics per sample.
// In small views several workgroups share a tile, each a part of its groups:
// what a ray gathers behind a part is known from the forward (BwdArgs::sums, in
// double precision), so S can start there.
// T before a block comes from the group's end by division by its samples'
// 1 - a (every sample is evaluated once), or, for tables whose opacity exceeds
// kMaxDivAlpha (or, after a forward by cells, changes faster than kMaxDivSlope),
// from a replay of the group from its start (REPLAY).
// Samples are evaluated at double-precision positions (start + j step, one
// rounding per axis; cell_d), with the trilinear value, the table lookup, the
// recursion and the gradient algebra in double precision; which group a
// sample belongs to follows the forward's single-precision position, so the
// stored transmittances fit.  A tile whose window would not fit reads its
// corners from global memory and adds its voxel gradients with global atomics
// directly (same groups, same arithmetic).
//
// Bound by the LDS atomics (16 double adds per sample, 28 to 33 cycles per
// wavefront instruction on one compute unit) and the double-precision vector
// work.
#include <algorithm>

#include "ring_common.h"
#include "sample.h"
#include "vr_internal.h"

namespace vr {

namespace {

using namespace ring;

struct Eval {
  double a, r, g, b;  // table opacity and colour
  double w;           // table weight
  double sraw;        // unclamped normalised value
  double wx, wy, wz;  // trilinear fractions
  int i;              // table interval
  float4 t0, t1;      // its entries
};

// A sample in double precision: position start + j step (one rounding per
// axis), base cell clamped to the stored range, fractions.  The adjoint
// differentiates the definition at these positions, not the forward's
// single-precision ones.
struct CellD {
  int ix, iy, iz;
  double wx, wy, wz;
};

__device__ __forceinline__ CellD cell_d(int j, const double (&p0)[3], const double (&sv)[3], const DevBrick& br) {
  CellD c;
  const double kk = (double)j;
  const double qx = fma(kk, sv[0], p0[0]), qy = fma(kk, sv[1], p0[1]), qz = fma(kk, sv[2], p0[2]);
  c.ix = min(max((int)floor(qx), br.clo[0]), br.chi[0]);
  c.iy = min(max((int)floor(qy), br.clo[1]), br.chi[1]);
  c.iz = min(max((int)floor(qz), br.clo[2]), br.chi[2]);
  c.wx = qx - (double)c.ix;
  c.wy = qy - (double)c.iy;
  c.wz = qz - (double)c.iz;
  return c;
}

// Trilinear value (lerp along 1, then 2, then 3) and table lookup in double
// precision from the eight corners v[dz][dy][dx].
__device__ __forceinline__ Eval eval_d(const float (&v)[8], const CellD& c, double vmin, double inv_range, int M,
                                       const float4* s_tf) {
  Eval e;
  e.wx = c.wx;
  e.wy = c.wy;
  e.wz = c.wz;
  const double c00 = fma(e.wx, (double)v[1] - (double)v[0], (double)v[0]);
  const double c01 = fma(e.wx, (double)v[3] - (double)v[2], (double)v[2]);
  const double c10 = fma(e.wx, (double)v[5] - (double)v[4], (double)v[4]);
  const double c11 = fma(e.wx, (double)v[7] - (double)v[6], (double)v[6]);
  const double c0 = fma(e.wy, c01 - c00, c00), c1 = fma(e.wy, c11 - c10, c10);
  const double val = fma(e.wz, c1 - c0, c0);
  e.sraw = (val - vmin) * inv_range;
  const double s = fmin(fmax(e.sraw, 0.0), 1.0);
  const double u = s * (double)(M - 1);
  e.i = min((int)u, M - 2);
  e.w = u - (double)e.i;
  e.t0 = s_tf[e.i];
  e.t1 = s_tf[e.i + 1];
  e.r = fma(e.w, (double)e.t1.x - (double)e.t0.x, (double)e.t0.x);
  e.g = fma(e.w, (double)e.t1.y - (double)e.t0.y, (double)e.t0.y);
  e.b = fma(e.w, (double)e.t1.z - (double)e.t0.z, (double)e.t0.z);
  e.a = fma(e.w, (double)e.t1.w - (double)e.t0.w, (double)e.t0.w);
  return e;
}

// LDS of one tile in floats: L + 1 voxel windows (float), L + 1 gradient
// windows (double), window offsets, layer ranges, and, for the replay, T before
// every block of four samples of the group.
__host__ __device__ constexpr size_t tile_floats(int L, int slot, int smax, bool replay) {
  return (size_t)3 * (L + 1) * slot + 64 + (replay ? (size_t)((smax + 3) / 4) * 128 : 0);
}

// value of v in lane I of the four lanes that share a ray
template <int I>
__device__ __forceinline__ double quad_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x55 * I, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x55 * I, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double quad_pick(int dl, double v0, double v1, double v2, double v3) {
  const double lo = dl & 1 ? v1 : v0, hi = dl & 1 ? v3 : v2;
  return dl & 2 ? hi : lo;
}

// Sums of a small table in LDS: lanes adding to one entry wait for each other, so
// tables of up to half as many entries as this get several copies, a lane adds to
// its own, until there are this many entries (8 KB).  Two views of 644 x 687 rays
// through 257 x 408 x 111 voxels, half a voxel a sample, 2 / 16 / 32 / 64 entries:
// 5.7 / 5.1 / 4.0 / 3.1 ms with one copy, 2.1 / 2.1 / 2.3 / 2.5 so; twice as many
// entries 2.3 at 64, but 64^3 at 96^2 205 against 185 us (occupancy).
constexpr int kTableEntries = 256;
constexpr int kAhead = 3;  // layers of windows kept ahead in registers
// A workgroup clears and writes out its table sums (32 bytes an entry) once for all
// its tiles.  With large tables that is a good part of a tile's time and of the
// memory a call takes, so views of many tiles give each workgroup several (RUN),
// as long as kRunBlocks workgroups remain: three 900^2 views of 64 x 60 x 70, 2048
// entries, 11.3 ms with one tile, 10.1, 9.4 and 9.5 with two, four and eight; of
// noise of 128 x 120 x 130 13.1 -> 12.0, of a smooth 256^3 cube 18.7 -> 19.2.  1024
// entries 6.5 -> 6.2 and 12.2 -> 12.8, 256 entries 5.9 -> 6.1: one tile each.
constexpr int kRunEntries = 2048, kRunBlocks = 3072, kRunMax = 4;

template <bool REPLAY, bool by, bool RUN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_bwd_ring(MarchArgs a, BwdArgs ba) {
  extern __shared__ double dsm[];
  const int M = a.M, L = ba.K;
  // table gradients [4][M][copies]: neighbouring entries in neighbouring banks (an
  // [M][4] layout makes entries 8 apart collide: 56 cycles per add against 33)
  const int csh = ba.copy_shift;
  double* s_gtf = dsm;
  float4* s_tf = reinterpret_cast<float4*>(dsm + (4 * M << csh));  // [M]
  const int slot = a.ring_slot;
  // The gradient windows hold doubles: on gfx950 one ds_add_f32 takes about
  // 195 cycles of a compute unit's LDS whatever its addresses (it retires
  // about a lane every three cycles), ds_add_f64 9 without conflicts and 28
  // with a tile's.
  double* s_grad = reinterpret_cast<double*>(s_tf + M);                          // [L + 1][slot]
  float* s_vox = reinterpret_cast<float*>(s_grad + (size_t)(L + 1) * slot);     // [L + 1][slot]
  int* s_boff = reinterpret_cast<int*>(s_vox + (size_t)(L + 1) * slot);         // [32] window offsets
  int* s_range = s_boff + 32;                                                   // [8] layer ranges
  double* s_T = reinterpret_cast<double*>(s_boff + 64);                         // REPLAY: [blocks][64]
  for (int i = threadIdx.x; i < M; i += blockDim.x) s_tf[i] = a.tf[i];
  for (int i = threadIdx.x; i < 4 * M << csh; i += blockDim.x) s_gtf[i] = 0.0;
  for (int e = threadIdx.x; e < (L + 1) * slot; e += blockDim.x) s_grad[e] = 0.0;

  // same tile order as the forward
  const int xcd = (int)(blockIdx.x & 7), per = (a.ntiles + 7) >> 3;
  const bool bands = ba.band[8] > 0;
  const int run = RUN ? ba.run : 1;
  const int tile0 = (bands ? ba.band[xcd] : xcd * per) + (int)(blockIdx.x >> 3) * run;
  const int tile_end = min(tile0 + run, bands ? ba.band[xcd + 1] : min((xcd + 1) * per, a.ntiles));
  int tile = tile0 < tile_end ? tile0 : a.ntiles;
  do {  // (one tile; the body keeps its indent)
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, dl = tid & 3;
  // a wavefront's 16 rays are every other pixel of the tile both ways: rays
  // next to each other would add to the same voxels (8 views 14.8 ms against
  // 13.1)
  const int ray = tid >> 2;
  const DevBrickView bvw = a.bv[0];
  const DevBrick br = a.bricks[0];
  const int tx = tile % bvw.tiles_x, ty = tile / bvw.tiles_x;
  const int lx = tx * 8 + ((ray & 3) << 1) + (wave & 1);
  const int ly = ty * 8 + ((ray >> 2 & 3) << 1) + (wave >> 1);
  const bool valid = tile < a.ntiles && lx < bvw.w && ly < bvw.h;
  const int u = bvw.x0 + min(lx, bvw.w - 1), v = bvw.y0 + min(ly, bvw.h - 1);
  const int pix = ly * bvw.w + lx;

  // ---- ray setup, frame and layer range: as the forward ring march
  const double* d = a.cam.e3;
  double o[3];
  pixel_origin(a.cam, u, v, o);
  int cnt = 0;
  double p0[3] = {0.0, 0.0, 0.0};
  const double sv[3] = {a.step * d[0], a.step * d[1], a.step * d[2]};
  double tin;
  int64_t n;
  if (valid && ray_lattice(o, d, a.hi, a.step, tin, n)) {
    int64_t k0, k1;
    brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0, k1);
    if (k1 > k0) {
      const double t0 = tin + ((double)k0 + 0.5) * a.step;
      for (int i = 0; i < 3; i++) p0[i] = o[i] + t0 * d[i] - (double)br.lo[i];
      cnt = (int)(k1 - k0);
    }
  }
  const float pb = (float)(by ? p0[1] : p0[2]), sb = (float)(a.step * (by ? d[1] : d[2]));
  const int cloB = by ? br.clo[1] : br.clo[2], chiB = by ? br.chi[1] : br.chi[2];
  const int cloG = by ? br.clo[2] : br.clo[1], chiG = by ? br.chi[2] : br.chi[1];
  const int cloF = br.clo[0], chiF = br.chi[0];
  const double db = by ? d[1] : d[2], dg = by ? d[2] : d[1];
  const bool up = db > 0.0;
  // cell layer of sample j, as the forward has it
  auto layer_of = [&](int j) {
    return (int)floorf(__builtin_amdgcn_fmed3f(fmaf((float)j, sb, pb), (float)cloB, (float)chiB));
  };
  // the tile's layers end with the last sample any of its rays took (rays that
  // stopped early leave the groups behind empty: 1024^2 rays of 256^3, stopped after
  // some 20 samples, 2.6 ms with them, 1.2 without)
  const int used = valid ? ba.nused[pix] : 0;
  int c_first = up ? 0x7fffffff : -0x7fffffff, c_last = up ? -0x7fffffff : 0x7fffffff;
  if (used > 0) {
    c_first = layer_of(0);
    c_last = layer_of(used - 1);
  }
  c_first = up ? wave_imin(c_first) : wave_imax(c_first);
  c_last = up ? wave_imax(c_last) : wave_imin(c_last);
  if (lane == 0) {
    s_range[wave] = c_first;
    s_range[4 + wave] = c_last;
  }
  __syncthreads();
  int Lbeg = s_range[0], Lend = s_range[4];
  for (int w = 1; w < 4; ++w) {
    Lbeg = up ? min(Lbeg, s_range[w]) : max(Lbeg, s_range[w]);
    Lend = up ? max(Lend, s_range[4 + w]) : min(Lend, s_range[4 + w]);
  }
  Lbeg = uni(Lbeg);
  Lend = uni(Lend);
  if (up ? Lbeg <= Lend : Lbeg >= Lend) {  // the same for the whole workgroup
    // groups are counted from the box's first layer in marching order: the
    // tile's start where the group of its first layer starts
    const int g0 = uni((up ? Lbeg - cloB : chiB - Lbeg) / L);
    Lbeg = up ? cloB + g0 * L : chiB - g0 * L;
    const int nlay = up ? Lend - Lbeg + 1 : Lbeg - Lend + 1;
    const int vstep = up ? 1 : -1;
    const int V0 = up ? Lbeg : Lbeg + 1;  // voxel layer V_k = V0 + k vstep
    // window geometry from the tile's corner rays (lanes 0..3)
    const double rfd = d[0] / db, rgd = dg / db;
    const float rf = (float)rfd, rg = (float)rgd;
    float Af, Ag;
    {
      const int cx = bvw.x0 + tx * 8, cy = bvw.y0 + ty * 8;
      const int ex = min(cx + 7, bvw.x0 + bvw.w - 1), ey = min(cy + 7, bvw.y0 + bvw.h - 1);
      const int cc = lane & 3;
      double oc[3];
      pixel_origin(a.cam, (cc & 1) ? ex : cx, (cc & 2) ? ey : cy, oc);
      const double ob = (by ? oc[1] : oc[2]) - (double)(by ? br.lo[1] : br.lo[2]);
      Af = (float)(oc[0] - (double)br.lo[0] - ob * rfd);
      Ag = (float)((by ? oc[2] : oc[1]) - (double)(by ? br.lo[2] : br.lo[1]) - ob * rgd);
    }
    const float Af_lo = unif(wmin4(Af)), Af_hi = unif(wmax4(Af));
    const float Ag_lo = unif(wmin4(Ag)), Ag_hi = unif(wmax4(Ag));
    const float arf = fabsf(rf), arg = fabsf(rg);
    const int NF = uni((int)floorf(Af_hi - Af_lo + 2.f * arf + 0.2f) + 3);
    const int pitch = (NF + 3) & ~3;
    int NG = uni((int)floorf(Ag_hi - Ag_lo + 2.f * arg + 0.2f) + 3);
    NG = min(NG, chiG + 2 - cloG);
    const int ysl = br.sy, zsl = br.sz;
    const int sB = by ? ysl : zsl, sG = by ? zsl : ysl;
    gfloat* gbase = (gfloat*)br.base;
    float* gvol = ba.gvol;  // whole volume: brick-local == global
    const bool inl = !(pitch > chiF + 2 - cloF || pitch * NG > slot || pitch > 256);
    auto window = [&](int V) {
      Window w;
      const float Pf = (float)V * rf, Pg = (float)V * rg;
      const int flo = max((int)floorf(Af_lo + Pf - arf - 0.05f), cloF);
      const int glo = max((int)floorf(Ag_lo + Pg - arg - 0.05f), cloG);
      w.f0 = uni(max(cloF, min(flo, chiF + 2 - pitch)));
      w.g0 = uni(max(cloG, min(glo, chiG + 2 - NG)));
      return w;
    };
    // element e of a window: row e / pitch, column e % pitch
    const float inv_pitch = 1.0f / (float)pitch;
    const int nwin = NG * pitch;

    // per-ray state of the backward walk
    float4 gf = valid ? ba.gout[pix] : make_float4(0.f, 0.f, 0.f, 0.f);
    const double dvs = (double)(M - 1) * ba.inv_range;  // du/dv inside the window
    double S = 0.0;
    const int ngrp = (nlay + L - 1) / L;
    const int npix = ba.npix;
    // first sample in cell layer k or a later one (marching order): the
    // forward's layers are monotone along a ray
    const float inv_sb = 1.f / sb;
    auto first_at = [&](int k) {
      const int c = up ? Lbeg + k : Lbeg - k;
      const float est = ((float)(up ? c : c + 1) - pb) * inv_sb;
      int j = min(max((int)ceilf(fminf(fmaxf(est, -1.f), 1e9f)), 0), cnt);
      while (j > 0 && (up ? layer_of(j - 1) >= c : layer_of(j - 1) <= c)) --j;
      while (j < cnt && !(up ? layer_of(j) >= c : layer_of(j) <= c)) ++j;
      return j;
    };
    // Voxel layer V_m lives in slot m % (L + 1) for every group, so the layer
    // two consecutive groups share (V_{k0} of a group, V_{k1} of the one
    // before it, which is taken next) keeps its voxel window and its gradient
    // window: it is neither reloaded nor cleared there, and flushed once,
    // with both groups' terms, by the group taken later.
    auto pslot = [&](int m) { return m % (L + 1); };
    // groups of this workgroup (relative to the tile's first): all, or those of
    // one part of the layers
    int gb = 0, ge = ngrp;
    if (ba.parts > 1) {
      const int q = ba.part_groups, k = (int)blockIdx.y;
      gb = max(0, k * q - g0);
      ge = min(ngrp, (k + 1) * q - g0);
    }
    int jn = cnt;  // first sample of the group taken before (behind) this one
    float Tn = valid && ge > gb ? ba.ckpt[(int64_t)(g0 + ge) * npix + pix] : 1.f;  // T behind the group
    float Tg = valid && ge > gb ? ba.ckpt[(int64_t)(g0 + ge - 1) * npix + pix] : 1.f;  // T before the group
    if (gb < ge && ge < ngrp) {
      // what the ray gathers behind the part, per unit of transmittance there: 1
      // minus the opacity gathered in front of it, or, where that difference has
      // lost its digits (opaque rays: it can be 0), the T stored there.  The sums'
      // own rounding, about 1e-16, is then divided by T here and multiplied by it
      // in every gradient; no transmittance left, nothing behind counts.
      jn = first_at(ge * L);
      if (jn > 0 && jn < used) {
        const double4 all = ba.sums[pix], f = ba.sums[(int64_t)((int)blockIdx.y + 1) * npix + pix];
        const double left = 1.0 - f.w, behind = left > 1e-8 ? left : (double)Tn;
        if (behind > 0.0)
          S = ((double)gf.x * (all.x - f.x) + (double)gf.y * (all.y - f.y) + (double)gf.z * (all.z - f.z) +
               (double)gf.w * (all.w - f.w)) / behind;
      }
    }
    // chunk (16 bytes) of a window this lane copies: row pr, column pc
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));
    auto chunk = [&](int V, const Window& w, int e) {
      const int r = (int)(((float)e + 0.5f) * inv_pitch), col = e - r * pitch;
      return (v4f) * (const v4u __attribute__((address_space(1)))*)(gbase + ((int64_t)V * sB + (int64_t)(w.g0 + r) * sG +
                                                                             w.f0 + col));
    };
    // windows of one chunk per lane: the next group's are loaded into registers
    // while this group's samples are taken
    const bool ahead = inl && nwin <= 1024 && L <= kAhead && ((int64_t)NG * sG + pitch) * 4 < ((int64_t)1 << 31);
    // byte offset of this lane's chunk from the window's first voxel
    const int pre_row = (int)(((float)(4 * tid) + 0.5f) * inv_pitch);
    unsigned pre_off = ahead ? (unsigned)(pre_row * sG + 4 * tid - pre_row * pitch) * 4u : 0u;
    v4f pre[kAhead];
    for (int g = ge - 1; g >= gb; --g) {
      const int k0 = g * L, k1 = min(nlay, k0 + L);  // cell layers k0 .. k1 - 1
      const int nv = k1 - k0 + 1;                     // voxel layers V_{k0} .. V_{k1}
      if (inl) {
        for (int i = 0; i < nv; ++i) {
          const int V = V0 + (k0 + i) * vstep;
          const Window w = window(V);
          const int ps = pslot(k0 + i);
          if (!(g + 1 < ge && i == nv - 1) && !(ahead && g + 1 < ge))  // (V_{k1} is kept from group g + 1)
            for (int e = 4 * tid; e < nwin; e += 1024) *reinterpret_cast<v4f*>(s_vox + ps * slot + e) = chunk(V, w, e);
          if (tid == 0) s_boff[i] = ps * slot - w.g0 * pitch - w.f0;
        }
        if (ahead && g + 1 < ge && 4 * tid < nwin)
#pragma unroll
          for (int i = 0; i < kAhead; ++i)
            if (i < L) *reinterpret_cast<v4f*>(s_vox + pslot(k0 + i) * slot + 4 * tid) = pre[i];
        __syncthreads();
        if (ahead && g > gb && 4 * tid < nwin)
#pragma unroll
          for (int i = 0; i < kAhead; ++i)
            if (i < L) {
              const int V = V0 + (k0 - L + i) * vstep;
              const Window w = window(V);
              asm volatile("" : "+v"(pre_off));  // (not hoisted as a 64-bit address per window)
              const char* wb = (const char*)unip(gbase + ((int64_t)V * sB + (int64_t)w.g0 * sG + w.f0));
              pre[i] = (v4f) * (const v4u __attribute__((address_space(1)))*)(wb + pre_off);
            }
      }
      float Tp_next = valid && g > gb ? ba.ckpt[(int64_t)(g0 + g - 1) * npix + pix] : 1.f;
      const int js = first_at(k0), je = min(jn, used);
      jn = js;
      // cell of sample j and its eight corners, from the windows when both of
      // its voxel layers are in the group's slots (always, up to rounding at
      // a layer boundary), else from global memory; lofs/uofs: LDS offsets of
      // the lower and upper corner rows, -1 for global
      auto corners = [&](int j, CellD& c, float (&vv)[8], int& lofs, int& uofs) {
        c = cell_d(j, p0, sv, br);
        lofs = uofs = -1;
        if (inl) {
          const int ib = by ? c.iy : c.iz, ig = by ? c.iz : c.iy;
          const int kc = up ? ib - Lbeg : Lbeg - ib;  // cell layer index
          const int sl = (up ? kc : kc + 1) - k0, su = (up ? kc + 1 : kc) - k0;
          if (sl >= 0 && sl < nv && su >= 0 && su < nv) {
            lofs = s_boff[sl] + __mul24(ig, pitch) + c.ix;
            uofs = s_boff[su] + __mul24(ig, pitch) + c.ix;
            const float* p = s_vox + lofs;
            const float* q = s_vox + uofs;
            if (by) {  // rows along z inside a window, layers along y
              vv[0] = p[0]; vv[1] = p[1]; vv[2] = q[0]; vv[3] = q[1];
              vv[4] = p[pitch]; vv[5] = p[pitch + 1]; vv[6] = q[pitch]; vv[7] = q[pitch + 1];
            } else {   // rows along y, layers along z
              vv[0] = p[0]; vv[1] = p[1]; vv[2] = p[pitch]; vv[3] = p[pitch + 1];
              vv[4] = q[0]; vv[5] = q[1]; vv[6] = q[pitch]; vv[7] = q[pitch + 1];
            }
            return;
          }
        }
        gfloat* p = gbase + (c.iz * zsl + c.iy * ysl + c.ix);
        vv[0] = p[0]; vv[1] = p[1]; vv[2] = p[ysl]; vv[3] = p[ysl + 1];
        vv[4] = p[zsl]; vv[5] = p[zsl + 1]; vv[6] = p[zsl + ysl]; vv[7] = p[zsl + ysl + 1];
      };
      int nblk = (max(je - js, 0) + 3) >> 2;  // blocks of four samples from js on
      if constexpr (REPLAY) {
        // T before every block; the plan bounds a ray's samples in one group by
        // smax (L layers at one step each): a group beyond it is flagged
        if (nblk > (ba.smax + 3) / 4) {
          atomicOr(ba.flag, 1);
          nblk = (ba.smax + 3) / 4;
        }
        double T = (double)Tg;
        for (int b = 0; b < nblk; ++b) {
          if (dl == 0) s_T[b * 64 + ray] = T;
          const int j = js + 4 * b + dl;
          CellD c;
          float vv[8];
          int lofs, uofs;
          corners(min(j, je - 1), c, vv, lofs, uofs);
          const Eval e = eval_d(vv, c, ba.vmin, ba.inv_range, M, s_tf);
          const double al = j < je ? e.a : 0.0;
          T = fma(-T, quad_bcast<0>(al), T);
          T = fma(-T, quad_bcast<1>(al), T);
          T = fma(-T, quad_bcast<2>(al), T);
          T = fma(-T, quad_bcast<3>(al), T);
        }
      }
      double Tend = (double)Tn;
      for (int b = nblk - 1; b >= 0; --b) {
        const int j = js + 4 * b + dl;
        const bool on = j < je;
        CellD c;
        float vv[8];
        int lofs, uofs;
        corners(min(j, je - 1), c, vv, lofs, uofs);
        const Eval e = eval_d(vv, c, ba.vmin, ba.inv_range, M, s_tf);
        asm volatile("" : "+v"(gf.x), "+v"(gf.y), "+v"(gf.z), "+v"(gf.w));  // (kept in single precision)
        const double gx = gf.x, gy = gf.y, gz = gf.z;
        const double h = fma(gx, e.r, fma(gy, e.g, fma(gz, e.b, (double)gf.w)));
        const double al = on ? e.a : 0.0;
        const double a0 = quad_bcast<0>(al), a1 = quad_bcast<1>(al), a2 = quad_bcast<2>(al), a3 = quad_bcast<3>(al);
        const double h0 = quad_bcast<0>(h), h1 = quad_bcast<1>(h), h2 = quad_bcast<2>(h), h3 = quad_bcast<3>(h);
        // T before this lane's sample
        const double e1 = 1.0 - a0, e2 = fma(-e1, a1, e1), e3 = fma(-e2, a2, e2);
        double Ts;
        if constexpr (REPLAY) {
          Ts = s_T[b * 64 + ray];
        } else {
          const double e4 = fma(-e3, a3, e3);
          // Tend / e4: the hardware's reciprocal and two Newton steps
          double r = __builtin_amdgcn_rcp(e4);
          r = fma(r, fma(-e4, r, 1.0), r);
          r = fma(r, fma(-e4, r, 1.0), r);
          Ts = Tend * r;
          Tend = Ts;
        }
        const double Tp = Ts * quad_pick(dl, 1.0, e1, e2, e3);
        // S behind this lane's sample
        const double S2 = fma(a3, h3 - S, S), S1 = fma(a2, h2 - S2, S2), S0 = fma(a1, h1 - S1, S1);
        const double Sk = quad_pick(dl, S0, S1, S2, S);
        S = fma(a0, h0 - S0, S0);
        if (!on) continue;
        const double ta = Tp * e.a;
        const double gr = gx * ta, gg = gy * ta, gb = gz * ta;
        const double ga = Tp * (h - Sk);
        const double w1 = e.w, w0 = 1.0 - e.w;
        double* q = s_gtf + ((e.i << csh) + (lane & ((1 << csh) - 1)));
        const int q1 = 1 << csh, qm = M << csh;  // to the next entry, channel
        atomicAdd(q, w0 * gr);
        atomicAdd(q + q1, w1 * gr);
        atomicAdd(q + qm, w0 * gg);
        atomicAdd(q + qm + q1, w1 * gg);
        atomicAdd(q + 2 * qm, w0 * gb);
        atomicAdd(q + 2 * qm + q1, w1 * gb);
        atomicAdd(q + 3 * qm, w0 * ga);
        atomicAdd(q + 3 * qm + q1, w1 * ga);
        if (gvol && e.sraw > 0.0 && e.sraw < 1.0) {
          const double du = gr * ((double)e.t1.x - (double)e.t0.x) + gg * ((double)e.t1.y - (double)e.t0.y) +
                            gb * ((double)e.t1.z - (double)e.t0.z) + ga * ((double)e.t1.w - (double)e.t0.w);
          const double gv = du * dvs;
          if (gv != 0.0) {
            const double x1 = e.wx * gv, x0 = gv - x1, y1 = e.wy, y0 = 1.0 - e.wy, z1 = e.wz, z0 = 1.0 - e.wz;
            const double yz00 = y0 * z0, yz10 = y1 * z0, yz01 = y0 * z1, yz11 = y1 * z1;
            if (lofs >= 0) {
              // rows of the lower and of the upper voxel layer: y selects the
              // layer and z the row, or z the layer and y the row
              double* lo = s_grad + lofs;
              double* hi = s_grad + uofs;
              const double l1 = by ? yz01 : yz10, u0 = by ? yz10 : yz01;
              atomicAdd(lo, x0 * yz00);
              atomicAdd(lo + 1, x1 * yz00);
              atomicAdd(lo + pitch, x0 * l1);
              atomicAdd(lo + pitch + 1, x1 * l1);
              atomicAdd(hi, x0 * u0);
              atomicAdd(hi + 1, x1 * u0);
              atomicAdd(hi + pitch, x0 * yz11);
              atomicAdd(hi + pitch + 1, x1 * yz11);
            } else {
              float* gq = gvol + (c.iz * zsl + c.iy * ysl + c.ix);
              unsafeAtomicAdd(gq, (float)(x0 * yz00));
              unsafeAtomicAdd(gq + 1, (float)(x1 * yz00));
              unsafeAtomicAdd(gq + ysl, (float)(x0 * yz10));
              unsafeAtomicAdd(gq + ysl + 1, (float)(x1 * yz10));
              unsafeAtomicAdd(gq + zsl, (float)(x0 * yz01));
              unsafeAtomicAdd(gq + zsl + 1, (float)(x1 * yz01));
              unsafeAtomicAdd(gq + zsl + ysl, (float)(x0 * yz11));
              unsafeAtomicAdd(gq + zsl + ysl + 1, (float)(x1 * yz11));
            }
          }
        }
      }
      // what the next group needs has arrived by now: taken here, no wait for
      // it comes after the atomics below (memory operations return in order,
      // and a wait for a load would wait for every atomic issued before it)
#pragma unroll
      for (int i = 0; i < kAhead; ++i) asm volatile("" : "+v"(pre[i]));
      asm volatile("" : "+v"(Tp_next));
      Tn = Tg;
      Tg = Tp_next;
      if (inl) {
        __syncthreads();  // every sample of the group is in the windows
        // add the finished gradient windows to the volume (rows contiguous
        // along axis 1) and clear them; V_{k0} goes on into group g - 1
        for (int i = g > gb ? 1 : 0; i < nv && gvol; ++i) {
          const int V = V0 + (k0 + i) * vstep;
          const Window w = window(V);
          float* gl = gvol + ((int64_t)V * sB + (int64_t)w.g0 * sG + w.f0);
          double* sg = s_grad + pslot(k0 + i) * slot;
          for (int e = tid; e < nwin; e += 256) {
            const float val = (float)sg[e];
            sg[e] = 0.0;
            if (val != 0.f) {
              const int r = (int)(((float)e + 0.5f) * inv_pitch), col = e - r * pitch;
              unsafeAtomicAdd(gl + ((int64_t)r * sG + col), val);
            }
          }
        }
      }
    }
  }
  __syncthreads();  // (the windows and the layer ranges are the next tile's)
  } while (RUN && ++tile < tile_end);
  double* part = ba.tf_part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * M * 4;
  for (int i = threadIdx.x; i < M * 4; i += blockDim.x) {
    double sum = 0.0;
    for (int c = 0; c < 1 << csh; ++c) sum += s_gtf[(((i & 3) * M + (i >> 2)) << csh) + c];
    part[i] = sum;
  }
}

}  // namespace

size_t bwd_ring_lds_bytes(int M, int L, int slot, int smax, bool replay) {
  return sizeof(double) * 4 * (size_t)M + sizeof(float4) * (size_t)M + sizeof(float) * tile_floats(L, slot, smax, replay);
}

int bwd_ring_run(int ntiles, int M) {
  return M < kRunEntries ? 1 : std::max(1, std::min(kRunMax, ntiles / kRunBlocks));
}

int bwd_ring_blocks(const MarchArgs& a, const BwdArgs& ba) {
  if (a.ntiles <= 0) return 0;
  const int parts = std::max(1, ba.parts);
  int widest = (a.ntiles + 7) / 8;
  if (ba.band[8] > 0) {
    widest = 0;
    for (int x = 0; x < 8; x++) widest = std::max(widest, ba.band[x + 1] - ba.band[x]);
  }
  return 8 * ((widest + ba.run - 1) / ba.run) * parts;
}

hipError_t launch_bwd_ring(const MarchArgs& a, const BwdArgs& ba, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  // (the offsets of L + 1 windows have 32 places)
  if (a.tile_w != 8 || a.ring_slot <= 0 || (a.ring_slot & 3) != 0 || a.cam.persp != 0 || ba.K < 1 || ba.K > 31 ||
      ba.smax < 1 || ba.run < 1)
    return hipErrorInvalidValue;
  size_t lds = bwd_ring_lds_bytes(a.M, ba.K, a.ring_slot, ba.smax, ba.replay != 0);
  BwdArgs bc = ba;
  // each doubling of the sums' copies adds as many bytes as they take so far
  while (bc.copy_shift < 6 && a.M << (bc.copy_shift + 1) <= kTableEntries &&
         lds + ((size_t)32 * a.M << bc.copy_shift) <= 160 * 1024) {
    lds += (size_t)32 * a.M << bc.copy_shift;
    bc.copy_shift++;
  }
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  const bool by = a.slab_axis == 1;
  using Kernel = void (*)(MarchArgs, BwdArgs);
  const Kernel one[2][2] = {{&k_bwd_ring<false, false, false>, &k_bwd_ring<false, true, false>},
                            {&k_bwd_ring<true, false, false>, &k_bwd_ring<true, true, false>}};
  const Kernel several[2][2] = {{&k_bwd_ring<false, false, true>, &k_bwd_ring<false, true, true>},
                                {&k_bwd_ring<true, false, true>, &k_bwd_ring<true, true, true>}};
  const Kernel f = (ba.run > 1 ? several : one)[ba.replay != 0][by];
  if (lds > 64 * 1024) {  // dynamic LDS beyond the default limit
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  if (ba.parts > 1 && (!ba.sums || ba.part_groups < 1)) return hipErrorInvalidValue;
  const int parts = std::max(1, ba.parts);
  const dim3 g(bwd_ring_blocks(a, ba) / parts, parts), b(256);
  hipLaunchKernelGGL(f, g, b, lds, s, a, bc);
  return hipGetLastError();
}

}  // namespace vr
