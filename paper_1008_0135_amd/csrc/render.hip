// render.hip -- forward ray-casting and over-composite kernels for gfx950.
//
// March (paper Sec. 2 and 2.4): one lane per pixel ray of a brick's
// rendering rectangle, wavefronts own TW x TH pixel tiles.  Each lane does
// the ray setup in double precision (whole-volume box test, lattice count,
// the brick's share [k0, k1) of the lattice), then marches its share in
// single precision with brick-local coordinates: trilinear reconstruction from
// four dword-pair loads, normalisation, a transfer-function lookup from LDS,
// front-to-back emission-absorption and the early-termination test.  The
// wavefront keeps issuing while any of its lanes is still marching.
//
// Composite (paper Sec. 2.5): one lane per output pixel walks the brick
// images front to back and applies the over operator where its pixel lies
// inside a brick's rectangle (the element-wise maximum for maximum intensity
// projection, which needs no order).
//
// Maximum intensity projection (paper Sec. 2.4): the march keeps the largest
// normalised sample value M of the ray and stops once M reaches 1; pixels are
// (M, M, M, M).
#include <type_traits>

#include "sample.h"
#include "vr_internal.h"

namespace vr {

namespace {

typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef const float __attribute__((address_space(1))) gfloat;

// two adjacent voxels with one 8-byte global load (dword alignment suffices)
__device__ __forceinline__ f2u ld_pair(gfloat* p) {
  return *reinterpret_cast<const f2u __attribute__((address_space(1)))*>(p);
}

// Blocks of 256 lanes (4 wavefronts, 4 consecutive tiles).  Consecutive
// hardware block ids go round-robin over the 8 XCDs; they are remapped so that
// each XCD takes runs of kXcdRun consecutive blocks (neighbouring tiles share
// its L2), dealt round robin: rays differ in length across the image, and one
// contiguous eighth each left the XCDs at the image's border idle (whole
// 201 x 187 x 333 volume 535 -> 395 us for two views; whole-ray termination
// over 64 bricks 4.4 -> 2.5 ms).
constexpr int kXcdRun = 8;
template <int RUN = kXcdRun>
__device__ __forceinline__ int xcd_block() {
  // which XCD takes which run of a round of eight moves on by three from round
  // to round: image rows of 8 or 16 runs would else give an XCD the same column
  // of the image in every row
  const int b = grid_block(), n = b / (8 * RUN), r = b - n * (8 * RUN);
  return b - r + ((r + 3 * (n >> 2)) & 7) * RUN + (r >> 3);
}

// Tile t of a grid of tiles numbered by blocks of 2 x 2 (blocks_x blocks a row):
// the four wavefronts of a workgroup share more lines than four tiles in a row.
__device__ __forceinline__ void block_tile(int t, int blocks_x, int& tx, int& ty) {
  const int q = t >> 2, by = q / blocks_x;
  tx = (q - by * blocks_x) * 2 + (t & 1);
  ty = by * 2 + (t >> 1 & 1);
}

// Rays through all bricks (a.bv front to back): the bricks whose rectangles meet a
// tile of w x h pixels at (x0, y0), 64 tested at a time, a lane each (the whole
// wavefront takes part); f(view) for each in order while more() holds.  One test
// after another had every wavefront wait for every brick: 32768 bricks, one 768^2
// view, 76 ms.
template <class More, class F>
__device__ __forceinline__ void bricks_of_tile(const MarchArgs& a, int x0, int y0, int w, int h, More more, F f) {
  const int lane = threadIdx.x & 63;
  for (int b0 = 0; b0 < a.nbv && more(); b0 += 64) {
    bool hit = false;
    if (b0 + lane < a.nbv) {
      const DevBrickView& v = a.bv[b0 + lane];
      hit = x0 < v.x0 + v.w && x0 + w > v.x0 && y0 < v.y0 + v.h && y0 + h > v.y0;
    }
    for (unsigned long long m = __ballot(hit); m != 0 && more(); m &= m - 1) f(a.bv[b0 + __builtin_ctzll(m)]);
  }
}

// Run of samples of a ray from sample j on whose cells lie in the macrocell
// holding sample j's: its length (1 to 1024, a chunk of the walk; 0.001 voxel of
// margin at the far planes against the rounding of sample positions) and whether that macrocell
// is clear, i.e. whether each of them would add exactly nothing.
__device__ __forceinline__ int macrocell_run(const MarchArgs& a, const DevBrick& br, int j, const float4& pos,
                                             const float4& dir, const float4& inv, float inv_mc, uint8_t& clear) {
  const SamplePos q = sample_pos(j, pos.x, pos.y, pos.z, dir.x, dir.y, dir.z);
  const Cell c = cell_of(q, br);
  // macrocell of a cell index i >= 0 (below kSkipIndex): floor((i + 1/2) / mc)
  const float fmc = (float)a.mc;
  const float mx = floorf(((float)(c.ix + br.lo[0]) + 0.5f) * inv_mc);
  const float my = floorf(((float)(c.iy + br.lo[1]) + 0.5f) * inv_mc);
  const float mz = floorf(((float)(c.iz + br.lo[2]) + 0.5f) * inv_mc);
  clear = a.mc_clear[((int64_t)(int)mz * a.mcn[1] + (int)my) * a.mcn[0] + (int)mx];
  // steps to the far plane; inv = 1 / dir, 1e9 for a component of 0.  The plane
  // is made brick-local first (whole numbers, exact): its margin would be lost in
  // the rounding of a coordinate of the whole axis, from 2^14 on
  auto steps = [&](float q1, float is, float m1, int lo) {
    const float edge = fmaf(m1, fmc, -(float)lo) + (is > 0.f ? fmc - 1e-3f : 1e-3f);
    return (edge - q1) * is;
  };
  const float n = fminf(fminf(steps(q.x, inv.x, mx, br.lo[0]), steps(q.y, inv.y, my, br.lo[1])),
                        steps(q.z, inv.z, mz, br.lo[2]));
  return 1 + (int)__builtin_amdgcn_fmed3f(floorf(n), 0.f, 1023.f);
}

// Empty-space skipping ray by ray (emission-absorption).  8 x 8 rays per
// wavefront, two phases per 1024 samples of the rays: every lane walks its own
// ray from macrocell to macrocell and marks the blocks of 16 samples that
// touch one that is not clear; then 16 lanes at a time take the marked blocks
// of a ray, 4 rays (2 x 2 pixels) side by side, as k_march<16> does.  Passed
// samples would add nothing and leave T as it is, so the images are those of
// the other marches.
// What a view costs follows its rays and marked samples, not the voxels of its
// bricks (two 1024^2 views of 1024 x 1024 x 768 with 95 % of the macrocells clear:
// 0.88 ms, 3.48 by a march that skips whole steps of a brick's layers).  Few
// wavefronts have many blocks, and one alone issues as fast as its SIMD does for
// one: a compute unit held 7.5 wavefronts on average while workgroups of four kept
// their LDS for the longest of theirs (VALU issue 41 %).  So a workgroup is one
// wavefront, up to tables of kSkipTable entries (its own copy of the table then
// leaves room for few: 256 entries 0.88 against 1.03 ms, 1024 0.99 and 1.00, 2048
// 1.52 and 1.07).  Two rods in step and blocks that add nothing to any of four
// rays left out: 1.13 -> 1.04 ms, four flags in flight 1 to 3 % more.
constexpr int kSkipTable = 1024;
template <int WAVES, bool MASK, bool THRU>
__global__ __launch_bounds__(64 * WAVES) void k_march_skip(MarchArgs a) {
  extern __shared__ float4 s_tf[];
  __shared__ float4 s_pos[WAVES][64], s_dir[WAVES][64], s_acc[WAVES][64];
  __shared__ unsigned long long s_blocks[WAVES][64];
  [[maybe_unused]] bool table = WAVES > 1;  // in LDS: one wavefront reads it when it finds its first block
  if constexpr (WAVES > 1) {
    for (int i = threadIdx.x; i < a.M; i += 64 * WAVES) s_tf[i] = a.tf[i];
    __syncthreads();
  }

  const int lb = xcd_block<kXcdRun * 4 / WAVES>();
  const int wave = WAVES > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0, lane = threadIdx.x & 63;
  const int tile = lb * WAVES + wave;
  if (tile >= a.ntiles) return;  // this wavefront only: no barrier follows
  int lo = 0, hi = THRU ? 0 : a.nbv - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (a.bv[mid].tile_begin <= tile) lo = mid;
    else hi = mid - 1;
  }
  const int rx = THRU ? 0 : a.bv[lo].x0, ry = THRU ? 0 : a.bv[lo].y0;
  const int rw = THRU ? a.cam.W : a.bv[lo].w, rh = THRU ? a.cam.H : a.bv[lo].h;
  const int t = THRU ? tile : tile - a.bv[lo].tile_begin;
  int tx, ty;
  block_tile(t, THRU ? (rw + 15) / 16 : a.bv[lo].tiles_x, tx, ty);
  // ray `lane` belongs to rod lane >> 2 (2 x 2 pixels, 4 x 4 rods)
  const int lx = tx * 8 + ((lane >> 2) & 3) * 2 + (lane & 1), ly = ty * 8 + (lane >> 4) * 2 + ((lane >> 1) & 1);
  const bool valid = lx < rw && ly < rh;
  const int u = rx + lx, v = ry + ly;
  float4* const dst =
      THRU || a.carry ? a.img + (int64_t)v * a.cam.W + u : a.img + a.bv[lo].img_off + (int64_t)ly * rw + lx;
  float4 acc = make_float4(0.f, 0.f, 0.f, 1.f);  // colour and transmittance
  if (!THRU && a.carry && valid) acc = *dst;
  bool live = valid && (THRU || !a.carry || 1.f - acc.w < a.tau);
  double o[3], d[3], tin = 0.0;
  int64_t n = 0;
  if (live) {
    pixel_ray(a.cam, u, v, o, d);
    live = ray_lattice(o, d, a.hi, a.step, tin, n);
  }
  s_acc[wave][lane] = acc;
  const float inv_mc = 1.f / (float)a.mc;
  const int dl = lane & 15;
  bool touched = false;
  auto march = [&](const DevBrickView& bvw) {
    const DevBrick br = a.bricks[bvw.brick];
    float4 pos = make_float4(0.f, 0.f, 0.f, 0.f), dir = pos;
    int cnt = 0;
    if (live) {
      int64_t k0, k1;
      brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0, k1);
      if (k1 > k0) {
        const double t0 = tin + ((double)k0 + 0.5) * a.step;
        pos.x = (float)(o[0] + t0 * d[0] - (double)br.lo[0]);
        pos.y = (float)(o[1] + t0 * d[1] - (double)br.lo[1]);
        pos.z = (float)(o[2] + t0 * d[2] - (double)br.lo[2]);
        dir = make_float4((float)(a.step * d[0]), (float)(a.step * d[1]), (float)(a.step * d[2]), 0.f);
        cnt = (int)(k1 - k0);
        touched = true;
      }
    }
    if (!__any(cnt > 0)) return;
    pos.w = __int_as_float(cnt);
    s_pos[wave][lane] = pos;
    s_dir[wave][lane] = dir;
    const float4 inv = make_float4(dir.x != 0.f ? 1.f / dir.x : 1e9f, dir.y != 0.f ? 1.f / dir.y : 1e9f,
                                   dir.z != 0.f ? 1.f / dir.z : 1e9f, 0.f);
    gfloat* base = (gfloat*)br.base;
    const int ys = br.sy, zs = br.sz;
    [[maybe_unused]] gfloat* mask = nullptr;
    if constexpr (MASK) mask = (gfloat*)(a.mask + br.lo[a.mask_axis]);
    for (int jc = 0; __any(jc < cnt); jc += 1024) {
      unsigned long long blocks = 0;
      const int jend = min(cnt, jc + 1024);
      // where a run ends does not depend on its flag: four flags in flight
      // (past the last sample positions stay in the brick's last cells)
      for (int j = jc; j < jend;) {
        int at[5];
        uint8_t clear[4];
        at[0] = j;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int run = macrocell_run(a, br, at[i], pos, dir, inv, inv_mc, clear[i]);
          at[i + 1] = min(at[i] + run, jend);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (at[i] < jend && !clear[i]) {
            const int b0 = (at[i] - jc) >> 4, b1 = (at[i + 1] - 1 - jc) >> 4;
            blocks |= (~0ull << b0) & (~0ull >> (63 - b1));
          }
        }
        j = at[4];
      }
      if (!__any(blocks != 0)) continue;
      if (!table) {
        for (int i = lane; i < a.M; i += 64) s_tf[i] = a.tf[i];
        table = true;
      }
      s_blocks[wave][lane] = blocks;
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      for (int q = 0; q < 16; q += 2) {
        // two rods in step: their loads and compositing chains overlap
        unsigned long long m[2];
        float4 rp[2], rd[2], c0[2];
        int rc[2], j[2];
        bool more[2];
        Cell c[2];
        f2u a00[2] = {}, a01[2] = {}, a10[2] = {}, a11[2] = {};
        [[maybe_unused]] f2u mw[2] = {};
#pragma unroll
        for (int i = 0; i < 2; ++i) m[i] = s_blocks[wave][4 * (q + i) + (lane >> 4)];
        if (!__any((m[0] | m[1]) != 0)) continue;
        // the corners of the next block are loaded while one is composited
        auto load = [&](int i) {
          j[i] = jc + 16 * __builtin_ctzll(m[i]) + dl;
          m[i] &= m[i] - 1;
          c[i] = cell_of(sample_pos(min(j[i], rc[i] - 1), rp[i].x, rp[i].y, rp[i].z, rd[i].x, rd[i].y, rd[i].z), br);
          gfloat* p = base + (c[i].iz * zs + c[i].iy * ys + c[i].ix);
          a00[i] = ld_pair(p);
          a01[i] = ld_pair(p + ys);
          a10[i] = ld_pair(p + zs);
          a11[i] = ld_pair(p + zs + ys);
          if constexpr (MASK) mw[i] = ld_pair(mask + (a.mask_axis == 2 ? c[i].iz : c[i].iy));
        };
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int ray = 4 * (q + i) + (lane >> 4);
          rp[i] = s_pos[wave][ray];
          rd[i] = s_dir[wave][ray];
          c0[i] = s_acc[wave][ray];
          rc[i] = __float_as_int(rp[i].w);
          j[i] = 0;
          c[i] = Cell{};
          more[i] = m[i] != 0 && !(1.f - c0[i].w >= a.tau);
          if (more[i]) load(i);
        }
        while (__any(more[0] || more[1])) {
          Classified k[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float val =
                trilerp(a00[i].x, a00[i].y, a01[i].x, a01[i].y, a10[i].x, a10[i].y, a11[i].x, a11[i].y, c[i]);
            k[i] = classify(val, a.vmin, a.inv_range, a.M, s_tf);
            if constexpr (MASK) k[i].a *= channel_weight(mw[i].x, mw[i].y, a.mask_axis, c[i]);
            // no block left, or past the ray's last sample: adds nothing
            if (!more[i] || j[i] >= rc[i]) k[i].a = 0.f;
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            more[i] = more[i] && m[i] != 0;
            if (more[i]) load(i);
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (__any(k[i].a != 0.f) && accumulate_group<16>(k[i], a.tau, c0[i].x, c0[i].y, c0[i].z, c0[i].w))
              more[i] = false;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (dl == 0) s_acc[wave][4 * (q + i) + (lane >> 4)] = c0[i];
      }
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (1.f - s_acc[wave][lane].w >= a.tau) {  // the ray has stopped
        live = false;
        cnt = 0;
      }
    }
  };
  if constexpr (THRU) bricks_of_tile(a, tx * 8, ty * 8, 8, 8, [&] { return __any(live) != 0; }, march);
  else march(a.bv[lo]);
  acc = s_acc[wave][lane];
  // carried state: only a ray with samples here owns its pixel in this wave
  if (!valid || (!THRU && a.carry && !touched)) return;
  *dst = make_float4(acc.x, acc.y, acc.z, !THRU && a.carry ? acc.w : 1.f - acc.w);
}

// D lanes of a wavefront share a ray and hold D consecutive samples of it
// (D = 1: one lane per ray); TW x 64 / (D TW) pixels per wavefront.  The lanes
// of a group read neighbouring voxels, so a load touches fewer cache lines,
// and a ray's chain of loads is D times shorter.  Bound by the L1's tag
// lookups (one a cycle and compute unit, 36 per load instruction at D = 4) and,
// in small views, by the chain.  64^3 at 128^2: 25 us a call with D = 16 (128
// by the cell march, 77 with D = 1); two 1024^2 views of 512 x 512 x 1024: 3.9
// ms with D = 4 or 16, 14.0 with D = 1 (2.4 by the cell march).
// THRU: tiles of the frame, every ray taken through all its bricks front to
// back (a.bv in that order) with one opacity test over the whole ray.
template <int D, int TW, bool MIP, bool MASK, bool THRU>
__global__ __launch_bounds__(256) void k_march(MarchArgs a) {
  static_assert(D == 1 || D == 4 || D == 16, "lane groups the cross-lane steps know");
  extern __shared__ float4 s_tf[];
  for (int i = threadIdx.x; i < a.M; i += 256) s_tf[i] = a.tf[i];
  __syncthreads();

  constexpr int TH = 64 / D / TW;
  const int nblk = (a.ntiles + 3) >> 2;
  // one lane per ray, tiles in rows: a contiguous eighth for each XCD (its tiles
  // have no shared corners to gain from short runs: 276 x 97 x 295 in perspective
  // at 665 x 349, tiles of 4 x 16, 434 us in runs of eight blocks, 336 so)
  const int per = (nblk + 7) >> 3, hw = grid_block();
  if (D == 1 && hw >= 8 * per) return;
  const int lb = D > 1 ? xcd_block() : (hw & 7) * per + (hw >> 3);
  if (lb >= nblk) return;
  int tile = __builtin_amdgcn_readfirstlane(lb * 4 + (int)(threadIdx.x >> 6));
  if (tile >= a.ntiles) return;

  // brick owning this tile: last entry with tile_begin <= tile
  int lo = 0, hi = THRU ? 0 : a.nbv - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (a.bv[mid].tile_begin <= tile) lo = mid;
    else hi = mid - 1;
  }
  const int rx = THRU ? 0 : a.bv[lo].x0, ry = THRU ? 0 : a.bv[lo].y0;
  const int rw = THRU ? a.cam.W : a.bv[lo].w, rh = THRU ? a.cam.H : a.bv[lo].h;
  const int t = THRU ? tile : tile - a.bv[lo].tile_begin;
  const int tiles_x = THRU ? (rw + 2 * TW - 1) / (2 * TW) : a.bv[lo].tiles_x;
  int tx, ty;
  if constexpr (D > 1) {
    block_tile(t, tiles_x, tx, ty);
  } else {
    tx = t % tiles_x;
    ty = t / tiles_x;
  }
  const int ray = (threadIdx.x & 63) / D, dl = threadIdx.x & (D - 1);
  const int lx = tx * TW + (ray % TW), ly = ty * TH + (ray / TW);
  const bool inside = lx < rw && ly < rh;
  if (!THRU && !inside) return;  // (THRU: every lane tests bricks)
  const int u = rx + lx, v = ry + ly;

  double o[3], d[3];
  pixel_ray(a.cam, u, v, o, d);
  float4* const dst = THRU || a.carry ? a.img + (int64_t)v * a.cam.W + u : a.img + a.bv[lo].img_off + (int64_t)ly * rw + lx;
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = 1.f, mx = 0.f;
  if (!THRU && a.carry) {
    const float4 s0 = *dst;
    if (1.f - s0.w >= a.tau) return;  // the ray stopped in a brick in front
    Cr = s0.x;
    Cg = s0.y;
    Cb = s0.z;
    T = s0.w;
  }
  double tin;
  int64_t n;
  bool touched = false;  // the ray has samples in this brick
  bool stopped = false;
  const bool meets = inside && ray_lattice(o, d, a.hi, a.step, tin, n);
  {
    const float sx = (float)(a.step * d[0]), sy = (float)(a.step * d[1]), sz = (float)(a.step * d[2]);
    auto march = [&](const DevBrickView& bvw) {
      // (a copy costs two masked 768^2 views of 512^3 in 64 bricks, four lanes per ray, 2.29 -> 2.48 ms)
      std::conditional_t<D == 1, const DevBrick, const DevBrick&> br = a.bricks[bvw.brick];
      int64_t k0, k1;
      brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0, k1);
      if (k1 <= k0) return;
      touched = true;
      const double t0 = tin + ((double)k0 + 0.5) * a.step;
      const float px = (float)(o[0] + t0 * d[0] - (double)br.lo[0]);
      const float py = (float)(o[1] + t0 * d[1] - (double)br.lo[1]);
      const float pz = (float)(o[2] + t0 * d[2] - (double)br.lo[2]);
      const int cnt = (int)(k1 - k0);
      gfloat* base = (gfloat*)br.base;
      const int ys = br.sy, zs = br.sz;
      [[maybe_unused]] gfloat* mask = nullptr;
      if constexpr (MASK) mask = (gfloat*)(a.mask + br.lo[a.mask_axis]);
      // the corners (and mask weights) of the next samples are loaded while
      // these are composited; loads return in order, so a load of its own in
      // the middle of a sample would wait for the next corners too.  One lane per
      // ray loads its sample where it takes it: a view of many rays is bound by
      // instructions, of which the copies were a quarter (the view above 336 -> 310)
      int j;
      Cell c;
      f2u a00, a01, a10, a11;
      [[maybe_unused]] f2u mw;
      auto load = [&](int jb) {
        j = jb + dl;
        c = cell_of(sample_pos(D == 1 ? j : min(j, cnt - 1), px, py, pz, sx, sy, sz), br);
        gfloat* p = base + (c.iz * zs + c.iy * ys + c.ix);
        a00 = ld_pair(p);
        a01 = ld_pair(p + ys);
        a10 = ld_pair(p + zs);
        a11 = ld_pair(p + zs + ys);
        if constexpr (MASK) mw = ld_pair(mask + (a.mask_axis == 2 ? c.iz : c.iy));
      };
      if constexpr (D > 1) load(0);
      for (int jb = 0;;) {
        if constexpr (D == 1) load(jb);
        const float val = trilerp(a00.x, a00.y, a01.x, a01.y, a10.x, a10.y, a11.x, a11.y, c);
        [[maybe_unused]] float w = 1.f;
        if constexpr (MASK) w = channel_weight(mw.x, mw.y, a.mask_axis, c);
        const bool past = D > 1 && j >= cnt;
        jb += D;
        const bool more = jb < cnt;
        if (D > 1 && more) load(jb);
        if (MIP) {
          float s = norm_value(val, a.vmin, a.inv_range);
          if constexpr (MASK) s *= w;
          mx = fmaxf(mx, s);
          stopped = mx >= 1.f;
        } else {
          Classified k = classify(val, a.vmin, a.inv_range, a.M, s_tf);
          if constexpr (MASK) k.a *= w;
          if constexpr (D == 1) {
            accumulate(k, Cr, Cg, Cb, T);
            stopped = 1.f - T >= a.tau;
          } else {
            if (past) k.a = 0.f;  // past the ray's last sample: adds nothing
            stopped = accumulate_group<D>(k, a.tau, Cr, Cg, Cb, T);
          }
        }
        if (stopped || !more) break;
      }
    };
    if constexpr (THRU)
      bricks_of_tile(a, tx * TW, ty * TH, TW, TH, [&] { return __any(meets && !stopped) != 0; },
                     [&](const DevBrickView& bvw) {
                       if (meets && !stopped) march(bvw);
                     });
    else if (meets) march(a.bv[lo]);
  }
  if (THRU && !inside) return;
  // carried state: only a ray with samples here owns its pixel in this wave
  // (another brick of the wave whose rectangle holds the pixel may update it)
  if (!THRU && a.carry && !touched) return;
  if constexpr (MIP && D > 1)
    for (int off = D >> 1; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if (dl == 0) *dst = MIP ? make_float4(mx, mx, mx, mx) : make_float4(Cr, Cg, Cb, !THRU && a.carry ? T : 1.f - T);
}

// v of the lane N before in the row of 16; 1 where there is none.
template <int N>
__device__ __forceinline__ double row_shr(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x110 + N, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0x3ff00000, __double2hiint(v), 0x110 + N, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// A sample as the adjoint evaluates it: opacity and colour in double precision at the
// double-precision position, trilinear over the corners a00 (y, z) .. a11 of cell c.
struct Sample64 {
  double a, r, g, b;
};
__device__ __forceinline__ Sample64 sample64(int j, const double (&p0)[3], const double (&sv)[3], const Cell& c,
                                             const f2u& a00, const f2u& a01, const f2u& a10, const f2u& a11,
                                             double vmin, double inv_range, int M, const float4* s_tf) {
  const double k = (double)j;
  const double wx = fma(k, sv[0], p0[0]) - (double)c.ix, wy = fma(k, sv[1], p0[1]) - (double)c.iy,
               wz = fma(k, sv[2], p0[2]) - (double)c.iz;
  auto lerp = [](double w, double x, double y) { return fma(w, y - x, x); };
  const double c0 = lerp(wy, lerp(wx, a00.x, a00.y), lerp(wx, a01.x, a01.y));
  const double c1 = lerp(wy, lerp(wx, a10.x, a10.y), lerp(wx, a11.x, a11.y));
  const double s = fmin(fmax((lerp(wz, c0, c1) - vmin) * inv_range, 0.0), 1.0), u = s * (double)(M - 1);
  const int i = min((int)u, M - 2);
  const double w = u - (double)i;
  const float4 t0 = s_tf[i], t1 = s_tf[i + 1];
  return Sample64{lerp(w, t0.w, t1.w), lerp(w, t0.x, t1.x), lerp(w, t0.y, t1.y), lerp(w, t0.z, t1.z)};
}

// Sum of v over the 16 lanes of a row, and over its lanes before lane dl.
__device__ __forceinline__ double row_sum(double v) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 16);
  return v;
}
__device__ __forceinline__ double row_before(double v, int dl) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const double w = __shfl_up(v, o, 16);
    v += dl >= o ? w : 0.0;
  }
  const double w = __shfl_up(v, 1, 16);
  return dl > 0 ? w : 0.0;
}

// The checkpointing forward by gathers: k_march<16, 2> over the whole volume
// that also stores T where a ray enters a group of sa.K cell layers along the
// slab axis, T at its end, and the number of its samples.  These, and the sums of
// parts, are made from each sample as the adjoint has it (double-precision position,
// value and table lookup over the same eight corners), beside the image's own
// single-precision chain: the adjoint divides by the samples' 1 - a between two
// stored T and starts parts behind the sums, and what the two evaluations differ by
// (a rounded position times the table's slope) would be in every gradient.  For small views,
// whose rays a wavefront of 64 rays would walk one sample at a time (100 x 92
// rays through 61 x 83 x 72 voxels: 135 us by windows of one ray per lane).
template <bool BY, bool PARTS>
__global__ __launch_bounds__(256) void k_march_save(MarchArgs a, SaveArgs sa) {
  constexpr int D = 16, TW = 2, TH = 2;
  extern __shared__ float4 s_tf[];
  for (int i = threadIdx.x; i < a.M; i += 256) s_tf[i] = a.tf[i];
  __syncthreads();
  const int tile = __builtin_amdgcn_readfirstlane(xcd_block() * 4 + (int)(threadIdx.x >> 6));
  if (tile >= a.ntiles) return;
  const int ray = (threadIdx.x & 63) / D, dl = threadIdx.x & (D - 1);
  int tx, ty;
  block_tile(tile, (a.cam.W + 2 * TW - 1) / (2 * TW), tx, ty);
  const int u = tx * TW + ray % TW, v = ty * TH + ray / TW;
  if (u >= a.cam.W || v >= a.cam.H) return;
  const int pix = v * a.cam.W + u;
  const DevBrick& br = a.bricks[0];
  double o[3], d[3], tin;
  pixel_ray(a.cam, u, v, o, d);
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = 1.f;
  int64_t n, k0 = 0, k1 = 0;
  if (ray_lattice(o, d, a.hi, a.step, tin, n)) brick_krange(o, d, tin, a.step, n, br.lo, br.hi, br.closed, k0, k1);
  int used = 0;
  if (k1 > k0) {
    const float sx = (float)(a.step * d[0]), sy = (float)(a.step * d[1]), sz = (float)(a.step * d[2]);
    const double t0 = tin + ((double)k0 + 0.5) * a.step;
    const double p0[3] = {o[0] + t0 * d[0] - (double)br.lo[0], o[1] + t0 * d[1] - (double)br.lo[1],
                          o[2] + t0 * d[2] - (double)br.lo[2]};
    const double sv[3] = {a.step * d[0], a.step * d[1], a.step * d[2]};
    const float px = (float)p0[0], py = (float)p0[1], pz = (float)p0[2];
    const int cnt = (int)(k1 - k0);
    const int ys = br.sy, zs = br.sz;
    gfloat* base = (gfloat*)br.base;
    // group of a cell, and of sample j
    const bool up = (BY ? d[1] : d[2]) > 0.0;
    const int clo = BY ? br.clo[1] : br.clo[2], chi = BY ? br.chi[1] : br.chi[2];
    auto group = [&](int ib) { return (up ? ib - clo : chi - ib) / sa.K; };
    auto group_at = [&](int j) {
      const Cell c = cell_of(sample_pos(j, px, py, pz, sx, sy, sz), br);
      return group(BY ? c.iy : c.iz);
    };
    int j;
    Cell c;
    f2u a00, a01, a10, a11;
    auto load = [&](int jb) {
      j = jb + dl;
      c = cell_of(sample_pos(min(j, cnt - 1), px, py, pz, sx, sy, sz), br);
      gfloat* p = base + (c.iz * zs + c.iy * ys + c.ix);
      a00 = ld_pair(p);
      a01 = ld_pair(p + ys);
      a10 = ld_pair(p + zs);
      a11 = ld_pair(p + zs + ys);
    };
    load(0);
    int last = -1;  // group of the sample before this block's first
    // what this lane's samples add to the ray (parts: summed over the 16 lanes
    // where a part begins and at the end)
    double4 own = make_double4(0.0, 0.0, 0.0, 0.0);
    double Td = 1.0;
    for (int jb = D;; jb += D) {
      const float val = trilerp(a00.x, a00.y, a01.x, a01.y, a10.x, a10.y, a11.x, a11.y, c);
      const int jc = j, gi = group(BY ? c.iy : c.iz);
      const Sample64 k64 = sample64(jc, p0, sv, c, a00, a01, a10, a11, sa.vmin, sa.inv_range, a.M, s_tf);
      const bool more = jb < cnt;
      if (more) load(jb);
      Classified k = classify(val, a.vmin, a.inv_range, a.M, s_tf);
      if (jc >= cnt) k.a = 0.f;  // past the ray's last sample: adds nothing
      const int gp = __shfl_up(gi, 1, D);
      int taken = 0;
      const bool stopped = accumulate_group<D>(k, a.tau, Cr, Cg, Cb, T, &taken);
      used = stopped ? jb - D + taken : min(jb, cnt);
      // T before this lane's sample: the product over the lanes before
      const double e = jc < used ? 1.0 - k64.a : 1.0;
      double q = e;
      q *= row_shr<1>(q);
      q *= row_shr<2>(q);
      q *= row_shr<4>(q);
      q *= row_shr<8>(q);
      const double Tb = Td * row_shr<1>(q);
      Td *= __shfl(q, D - 1, D);
      // groups this sample is the ray's first in or behind: its own, and those
      // since the last sample's (steps longer than a group leave some without a
      // sample; the group in front of such a one ends with the T stored there)
      const int before = dl == 0 ? last : gp;
      const bool begins = jc < used && gi != before;
      const int from = before < 0 ? gi : before + 1;
      if (begins)
        for (int g = from; g <= gi; ++g) sa.ckpt[(int64_t)g * sa.npix + pix] = (float)Tb;
      if constexpr (PARTS) {
        const double w = jc < used ? Tb * k64.a : 0.0;
        const double4 add = make_double4(w * k64.r, w * k64.g, w * k64.b, w);
        // the part that begins at one of these groups (the last, if several do)
        const int pg = gi - gi % sa.part_groups;
        const bool part = begins && pg >= from;
        if (__any(part)) {
          // all blocks before this one, and this block's lanes before this one
          const double4 f = make_double4(row_sum(own.x) + row_before(add.x, dl), row_sum(own.y) + row_before(add.y, dl),
                                         row_sum(own.z) + row_before(add.z, dl), row_sum(own.w) + row_before(add.w, dl));
          if (part)
            for (int g = pg; g >= from && g > 0; g -= sa.part_groups)
              sa.sums[(int64_t)(g / sa.part_groups) * sa.npix + pix] = f;
        }
        own.x += add.x;
        own.y += add.y;
        own.z += add.z;
        own.w += add.w;
      }
      last = __shfl(gi, D - 1, D);
      if (stopped || !more) break;
    }
    if (dl == 0) sa.ckpt[(int64_t)(group_at(used - 1) + 1) * sa.npix + pix] = (float)Td;
    if constexpr (PARTS) {
      const double4 all = make_double4(row_sum(own.x), row_sum(own.y), row_sum(own.z), row_sum(own.w));
      if (dl == 0) sa.sums[pix] = all;
    }
  }
  if (dl == 0) {
    sa.nused[pix] = used;
    a.img[a.bv[0].img_off + pix] = make_float4(Cr, Cg, Cb, 1.f - T);
  }
}

// Carried state over the frame: (C, T) = (0, 1) before the first brick, and
// (C, 1 - T) once the last has been marched.
__global__ __launch_bounds__(256) void k_carry_init(float4* img, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) img[i] = make_float4(0.f, 0.f, 0.f, 1.f);
}
// Cleared pixels (brick images of footprint-cell marches).
__global__ __launch_bounds__(256) void k_zero(float4* img, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) img[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}
__global__ __launch_bounds__(256) void k_carry_final(float4* img, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    const float4 s = img[i];
    img[i] = make_float4(s.x, s.y, s.z, 1.f - s.w);
  }
}

__global__ __launch_bounds__(256) void k_composite(CompArgs a) {
  const int x = blockIdx.x * 16 + (threadIdx.x & 15);
  const int y = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (x >= a.W || y >= a.H) return;
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, A = 0.f;
  for (int i = 0; i < a.n; ++i) {
    const CompLayer L = a.layers[i];
    const unsigned lx = (unsigned)(x - L.x0), ly = (unsigned)(y - L.y0);
    if (lx < (unsigned)L.w && ly < (unsigned)L.h) {
      const float4 c = L.rgba[(int64_t)ly * L.w + lx];
      if (a.mip) {
        Cr = fmaxf(Cr, c.x);
        Cg = fmaxf(Cg, c.y);
        Cb = fmaxf(Cb, c.z);
        A = fmaxf(A, c.w);
      } else {
        const float t = 1.f - A;
        Cr = fmaf(t, c.x, Cr);
        Cg = fmaf(t, c.y, Cg);
        Cb = fmaf(t, c.z, Cb);
        A = fmaf(t, c.w, A);
      }
    }
  }
  a.out[(int64_t)y * a.W + x] = make_float4(Cr, Cg, Cb, A);
}

}  // namespace

hipError_t launch_carry(float4* img, int64_t n, bool final, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t grid = (n + 255) / 256;
  if (final) hipLaunchKernelGGL(k_carry_final, dim3((unsigned)grid), dim3(256), 0, s, img, n);
  else hipLaunchKernelGGL(k_carry_init, dim3((unsigned)grid), dim3(256), 0, s, img, n);
  return hipGetLastError();
}

hipError_t launch_zero(float4* img, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t grid = (n + 255) / 256;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)grid), dim3(256), 0, s, img, n);
  return hipGetLastError();
}

hipError_t launch_march(const MarchArgs& a, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  const int nblk = (a.ntiles + 3) / 4;
  const int grid = (nblk + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun);
  const size_t lds = sizeof(float4) * (size_t)a.M;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid_rows(grid), dim3(256), lds, s, a); };
  const bool mask = a.mask != nullptr, mip = a.mip != 0;
  if (a.skip) {
    if (mip || a.mc < 2) return hipErrorInvalidValue;
    auto skip = [&](auto waves) {
      constexpr int N = decltype(waves)::value;
      const int round = 8 * kXcdRun * 4;
      const dim3 blocks = grid_rows(((int64_t)a.ntiles + round - 1) / round * round / N), threads(64 * N);
      if (a.thru && mask) hipLaunchKernelGGL((k_march_skip<N, true, true>), blocks, threads, lds, s, a);
      else if (a.thru) hipLaunchKernelGGL((k_march_skip<N, false, true>), blocks, threads, lds, s, a);
      else if (mask) hipLaunchKernelGGL((k_march_skip<N, true, false>), blocks, threads, lds, s, a);
      else hipLaunchKernelGGL((k_march_skip<N, false, false>), blocks, threads, lds, s, a);
    };
    if (a.M <= kSkipTable) skip(std::integral_constant<int, 1>{});
    else skip(std::integral_constant<int, 4>{});
  } else if (a.thru) {
    if (mip || (a.depth != 16 && a.depth != 4)) return hipErrorInvalidValue;
    // (4 lanes or 16)
    if (a.depth == 4 && mask) go(k_march<4, 4, false, true, true>);
    else if (a.depth == 4) go(k_march<4, 4, false, false, true>);
    else if (mask) go(k_march<16, 2, false, true, true>);
    else go(k_march<16, 2, false, false, true>);
  } else {
    auto shape = [&](auto d, auto tw) {
      constexpr int D = decltype(d)::value, TW = decltype(tw)::value;
      if (mask && mip) go(k_march<D, TW, true, true, false>);
      else if (mask) go(k_march<D, TW, false, true, false>);
      else if (mip) go(k_march<D, TW, true, false, false>);
      else go(k_march<D, TW, false, false, false>);
    };
    if (a.depth == 16) shape(std::integral_constant<int, 16>{}, std::integral_constant<int, 2>{});
    else if (a.depth == 4) shape(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
    else if (a.tile_w == 8) shape(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
    else if (a.tile_w == 16) shape(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
    else if (a.tile_w == 4) shape(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_march_save(const MarchArgs& a, const SaveArgs& sa, hipStream_t s) {
  if (a.ntiles <= 0) return hipSuccess;
  if (a.cam.persp || a.mip || a.mask || a.mc || a.carry || sa.K < 1 || (a.slab_axis != 1 && a.slab_axis != 2))
    return hipErrorInvalidValue;
  const int nblk = (a.ntiles + 3) / 4;
  const int grid = (nblk + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun);
  const size_t lds = sizeof(float4) * (size_t)a.M;
  if (sa.parts > 1 && (!sa.sums || sa.part_groups < 1)) return hipErrorInvalidValue;
  const bool by = a.slab_axis == 1;
  const auto f = sa.parts > 1 ? (by ? &k_march_save<true, true> : &k_march_save<false, true>)
                              : (by ? &k_march_save<true, false> : &k_march_save<false, false>);
  hipLaunchKernelGGL(f, grid_rows(grid), dim3(256), lds, s, a, sa);
  return hipGetLastError();
}

hipError_t launch_composite(const CompArgs& a, hipStream_t s) {
  dim3 grid((a.W + 15) / 16, (a.H + 15) / 16);
  hipLaunchKernelGGL(k_composite, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace vr
