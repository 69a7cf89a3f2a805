// batch.hip -- batched rendering of many independent requests in one launch
// (gfx950).
//
// Each request is a whole (unbricked) volume with its own view, transfer
// function, window and output image.  Work items are (request, pixel tile)
// pairs numbered in the host's order (requests with the most samples per tile
// first, so the longest items start first); a request's tile is 64 pixels,
// 4 x 16, 8 x 8, 16 x 4 or 32 x 2, as the autotuner chose for its size
// class.  A workgroup takes one item, and the hardware hands items out as
// compute units come free (a grid that pulled them from one atomic counter paid
// 15 ns an item for that counter, 1.1 of 1.8 ms at 64 requests, and 60 us just
// to find it empty).  Where rays are close, four lanes share a ray and hold
// four consecutive samples of it, and the item is a tile; where they are
// sparse, or the batch is small, 16 lanes share a ray and the item is a quarter
// of a tile (BatchReq::lanes; as k_march of the plain gather march).  The
// per-sample arithmetic is the one of every other march (sample.h).  64
// requests of 32^3 to 256^3 voxels: 2.43 ms (a lane per ray, counter) -> 1.86
// (four lanes) -> 1.33.  Bound by the L1's tag
// lookups.
#include <algorithm>
#include <mutex>

#include "runtime.h"
#include "sample.h"
#include "vr_internal.h"

namespace vr {

// Device scratch of the allocation-free batched entry point
// (vr_render_batch_noalloc): the descriptor table of at most
// kNoAllocMaxReq requests.  Each device holds its own
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

// Workgroups of an XCD: runs of kRun consecutive ones (neighbouring tiles share
// its L2), dealt round robin, as in the gather march.
constexpr int kRun = 8;

// 64 / D rays of a tile from ray `first` on, D lanes each.
template <int D>
__device__ __forceinline__ void batch_rays(const BatchArgs& ba, const BatchReq& rq, const float4* s_tf, int tx, int ty,
                                           int first, int lane) {
  const int dl = lane & (D - 1), sh = rq.tile_shift;
  int px, py;
  tile_pixel(first + lane / D, sh, px, py);
  const int u = (tx << sh) + px, v = ty * (64 >> sh) + py;
  if (u >= rq.cam.W || v >= rq.cam.H) return;
  const DevBrick& br = rq.br;
  double o[3], d[3], tin;
  int64_t n;
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = 1.f;
  pixel_ray(rq.cam, u, v, o, d);
  if (ray_lattice(o, d, rq.hi, ba.step, tin, n)) {
    const float x = (float)(o[0] + (tin + 0.5 * ba.step) * d[0]);
    const float y = (float)(o[1] + (tin + 0.5 * ba.step) * d[1]);
    const float z = (float)(o[2] + (tin + 0.5 * ba.step) * d[2]);
    const float sx = (float)(ba.step * d[0]), sy = (float)(ba.step * d[1]), sz = (float)(ba.step * d[2]);
    const int cnt = (int)n;
    gfloat* base = (gfloat*)br.base;
    const int ys = br.sy, zs = br.sz;
    // the corners of the next samples are loaded while these are composited
    int j = 0;
    Cell c;
    f2u a00, a01, a10, a11;
    auto load = [&](int jb) {
      j = jb + dl;
      c = cell_of(sample_pos(min(j, cnt - 1), x, y, z, sx, sy, sz), br);
      gfloat* p = base + (c.iz * zs + c.iy * ys + c.ix);
      a00 = ld_pair(p);
      a01 = ld_pair(p + ys);
      a10 = ld_pair(p + zs);
      a11 = ld_pair(p + zs + ys);
    };
    if (cnt > 0) load(0);
    for (int jb = D; jb < cnt + D; jb += D) {
      const float val = trilerp(a00.x, a00.y, a01.x, a01.y, a10.x, a10.y, a11.x, a11.y, c);
      const bool past = j >= cnt;
      if (jb < cnt) load(jb);
      Classified k = classify(val, rq.vmin, rq.inv_range, rq.M, s_tf);
      if (past) k.a = 0.f;  // past the ray's last sample: adds nothing
      if (accumulate_group<D>(k, ba.tau, Cr, Cg, Cb, T)) break;
    }
  }
  if (dl == 0) rq.out[(int64_t)v * rq.cam.W + u] = make_float4(Cr, Cg, Cb, 1.f - T);
}

__global__ __launch_bounds__(256) void k_batch(BatchArgs ba) {
  extern __shared__ float4 s_tf[];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int b = grid_block(), round = b / (8 * kRun), r = b - round * (8 * kRun);
  const int item = b - r + ((r + 3 * (round >> 2)) & 7) * kRun + (r >> 3);
  if (item >= ba.total_items) return;  // the whole workgroup
  // request owning the item: last with item_begin <= item
  int lo = 0, hi = ba.nreq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ba.reqs[mid].item_begin <= item) lo = mid;
    else hi = mid - 1;
  }
  const BatchReq& rq = ba.reqs[lo];
  for (int i = threadIdx.x; i < rq.M; i += 256) s_tf[i] = rq.tf[i];
  __syncthreads();
  const int t = item - rq.item_begin;
  if (rq.lanes == 16) {  // a quarter of a tile per item, 4 rays per wavefront
    const int tile = t >> 2;
    batch_rays<16>(ba, rq, s_tf, tile % rq.tiles_x, tile / rq.tiles_x, (t & 3) * 16 + wave * 4, lane);
  } else {  // a tile per item, 16 rays per wavefront
    batch_rays<4>(ba, rq, s_tf, t % rq.tiles_x, t / rq.tiles_x, wave * 16, lane);
  }
}

}  // namespace

hipError_t launch_batch(const BatchArgs& a, int waves_per_cu, hipStream_t s) {
  if (a.total_items <= 0) return hipSuccess;
  const int64_t grid = ((int64_t)a.total_items + 8 * kRun - 1) / (8 * kRun) * (8 * kRun);
  // at most waves_per_cu wavefronts per compute unit (0, kBatchWaves: as many as
  // fit): LDS for one workgroup more than that would not fit
  size_t lds = sizeof(float4) * (size_t)a.max_M;
  if (waves_per_cu > 0 && waves_per_cu < kBatchWaves) lds = std::max(lds, 160 * 1024 / (size_t)(std::max(1, waves_per_cu / 4) + 1) + 1024);
  if (lds > 64 * 1024) {  // dynamic LDS beyond the default limit
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_batch), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_batch, grid_rows(grid), dim3(256), lds, s, a);
  return hipGetLastError();
}

}  // namespace vr
