// batch.hip -- batched rendering of many independent requests in one
// persistent launch (gfx950).
//
// Each request is a whole (unbricked) volume with its own view, transfer
// function, window and output image.  Work items are (request, pixel tile)
// pairs numbered in the host's order (requests with the most samples per tile
// first, so the longest items start first); a request's tile is 64 pixels,
// 4 x 16, 8 x 8, 16 x 4 or 32 x 2, as the autotuner chose for its size
// class.  A grid sized to the device pulls items from one atomic counter, one
// item per wavefront per
// pull, until the queue is empty: every wavefront reaches the exit test after
// each item, so the grid drains by itself.  A wavefront keeps the table of
// the request it is working on in its own LDS slot and reloads it only when
// the next item belongs to another request.  Four lanes share a ray and hold
// four consecutive samples of it (k_march<4> of the plain gather march), 16
// rays of the tile at a time; the rays are set up one per lane and passed
// through LDS.  The per-sample arithmetic is the one of every other march
// (sample.h).  64 requests: 2.43 ms with a lane per ray at its best grid (8
// wavefronts per compute unit), 1.81 so (16); 16 lanes per ray, 2.5, repeat
// the compositing steps too often.  Bound by the L1's tag lookups.
#include <mutex>

#include "runtime.h"
#include "sample.h"
#include "vr_internal.h"

namespace vr {

// Device scratch of the allocation-free batched entry point
// (vr_render_batch_noalloc): the descriptor table of at most
// kNoAllocMaxReq requests, then the work counter.  Each device holds its own
// copy for the life of the process; host code reaches it only through the
// address hipGetSymbolAddress returns for that device.
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int noalloc_init(int device) {
  if (device < 0 || device >= kMaxDevices) return fail(VR_EUNSUPPORTED, "device %d beyond %d", device, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[device]) return VR_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) {
    (void)hipGetLastError();
    return fail(VR_EHIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", device, hipGetErrorString(e));
  }
  g_scratch_ptr[device] = p;
  return VR_OK;
}

void* noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return g_scratch_ptr[device];
}

namespace {

typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef const float __attribute__((address_space(1))) gfloat;

__device__ __forceinline__ f2u ld_pair(gfloat* p) {
  return *reinterpret_cast<const f2u __attribute__((address_space(1)))*>(p);
}

__global__ void k_batch_reset(unsigned int* counter) { *counter = 0u; }

// Pixel of ray `lane` in a tile of 2^sh x 64 / 2^sh pixels: 4 consecutive
// lanes are 2 x 2 pixels, 16 are 4 x 4 (8 x 2 in 32 x 2 tiles).
__device__ __forceinline__ void tile_pixel(int lane, int sh, int& x, int& y) {
  const int b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1, hi = lane >> 4;
  if (sh == 5) {
    x = b0 | (lane >> 2 << 1);
    y = b1;
    return;
  }
  x = b0 | b2 << 1;
  y = b1 | b3 << 1;
  if (sh == 3) {
    x |= (hi & 1) << 2;
    y |= (hi >> 1) << 2;
  } else if (sh == 4) {
    x |= hi << 2;
  } else {
    y |= hi << 2;
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_batch(BatchArgs ba) {
  extern __shared__ float4 smem[];
  __shared__ float4 s_pos[4][64], s_dir[4][64];  // per ray: start and sample count, step and pixel
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float4* s_tf = smem + (size_t)wave * ba.max_M;
  int cur = -1;  // request whose table sits in this wavefront's slot
  for (;;) {
    unsigned int item = 0;
    if (lane == 0) item = atomicAdd(ba.counter, 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= (unsigned)ba.total_items) break;
    // request owning the item: last with item_begin <= item
    int lo = 0, hi = ba.nreq - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (ba.reqs[mid].item_begin <= (int)item) lo = mid;
      else hi = mid - 1;
    }
    const BatchReq& rq = ba.reqs[lo];
    if (lo != cur) {
      for (int i = lane; i < rq.M; i += 64) s_tf[i] = rq.tf[i];
      cur = lo;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    const int t = (int)item - rq.item_begin;
    const int tx = t % rq.tiles_x, ty = t / rq.tiles_x;
    // ---- ray setup, one ray per lane: ray `lane` belongs to rod lane >> 2
    // (2 x 2 pixels; the tile's rods in rows of tile width / 2)
    const int sh = rq.tile_shift;
    int px, py;
    tile_pixel(lane, sh, px, py);
    const int u = (tx << sh) + px, v = ty * (64 >> sh) + py;
    const bool valid = u < rq.cam.W && v < rq.cam.H;
    const DevBrick& br = rq.br;
    float4 pos = make_float4(0.f, 0.f, 0.f, 0.f), dir = pos;
    int cnt = 0;
    if (valid) {
      double o[3], d[3], tin;
      int64_t n;
      pixel_ray(rq.cam, u, v, o, d);
      if (ray_lattice(o, d, rq.hi, ba.step, tin, n)) {
        pos.x = (float)(o[0] + (tin + 0.5 * ba.step) * d[0]);
        pos.y = (float)(o[1] + (tin + 0.5 * ba.step) * d[1]);
        pos.z = (float)(o[2] + (tin + 0.5 * ba.step) * d[2]);
        dir = make_float4((float)(ba.step * d[0]), (float)(ba.step * d[1]), (float)(ba.step * d[2]), 0.f);
        cnt = (int)n;
      }
    }
    pos.w = __int_as_float(cnt);
    dir.w = __int_as_float(valid ? v * rq.cam.W + u : -1);
    s_pos[wave][lane] = pos;
    s_dir[wave][lane] = dir;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // ---- rods: 4 rays at a time, 16 lanes each holding consecutive samples
    gfloat* base = (gfloat*)br.base;
    const int ys = br.sy, zs = br.sz;
    const int dl = lane & (D - 1);
    for (int q = 0; q < D; ++q) {
      const int ray = q * (64 / D) + lane / D;
      const float4 rp = s_pos[wave][ray], rd = s_dir[wave][ray];
      const int rc = __float_as_int(rp.w);
      float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = 1.f;
      for (int jb = 0; jb < rc; jb += D) {
        const Cell c = cell_of(sample_pos(min(jb + dl, rc - 1), rp.x, rp.y, rp.z, rd.x, rd.y, rd.z), br);
        gfloat* p = base + (c.iz * zs + c.iy * ys + c.ix);
        const f2u a00 = ld_pair(p), a01 = ld_pair(p + ys), a10 = ld_pair(p + zs), a11 = ld_pair(p + zs + ys);
        const float val = trilerp(a00.x, a00.y, a01.x, a01.y, a10.x, a10.y, a11.x, a11.y, c);
        Classified k = classify(val, rq.vmin, rq.inv_range, rq.M, s_tf);
        if (jb + dl >= rc) k.a = 0.f;  // past the ray's last sample: adds nothing
        if (accumulate_group<D>(k, ba.tau, Cr, Cg, Cb, T)) break;
      }
      const int at = __float_as_int(rd.w);
      if (dl == 0 && at >= 0) rq.out[at] = make_float4(Cr, Cg, Cb, 1.f - T);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

}  // namespace

hipError_t launch_batch(const BatchArgs& a, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(1), 0, s, a.counter);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = sizeof(float4) * (size_t)a.max_M * 4;
  hipLaunchKernelGGL(k_batch<4>, dim3(blocks), dim3(256), lds, s, a);
  return hipGetLastError();
}

}  // namespace vr
