// forward.h -- forward-path planning and launch sequence shared by the
// forward, differentiable and autotuning entry points.
#pragma once

#include <vector>

#include "runtime.h"

namespace vr {

struct ViewPlan {
  std::vector<DevBrickView> bv;       // rendered bricks, launch order
  std::vector<int32_t> layers_order;  // indices into bv, front to back
  int32_t ntiles = 0;
  int64_t pixels = 0;                 // brick-image pixels of this view
  // opacity tested over the whole ray: bv grouped into front-to-back waves,
  // wave w = bv[wave_begin[w] .. wave_begin[w + 1]) with tile_begin counted
  // from the wave's first brick and wave_tiles[w] tiles
  std::vector<int32_t> wave_begin, wave_tiles;
  // perspective views: bv grouped into classes, class c = bv[class_begin[c] ..
  // class_begin[c + 1]) with tile_begin counted from the class's first brick and
  // class_tiles[c] work items: bricks marched over footprint cells sized per
  // brick with slab axis class_axis[c] (1 or 2), then those marched by gathers
  // (class_axis 0); empty: one launch for the view
  std::vector<int32_t> class_begin, class_tiles, class_axis;
  // gather march: lanes per ray (1, 4 or 16; 0: another march), with macrocells
  // passed over ray by ray (skip), or every ray through all its bricks (thru;
  // bv front to back)
  int32_t deep = 0;
  bool skip = false, thru = false;
  // ring march over footprint cells (parallel rays): bv counts cells, not tiles
  bool foot = false;
  FootShape fs;
};

struct MarchTimes {
  double cells = 1e30, gather = 0.0;  // seconds
  double samples = 0.0, chain = 0.0;  // samples, and the part of cells that is a wavefront's chain
  double pitch = 0.0;                 // voxels between rays
};
// What the estimates need of the boxes a view marches, gathered in one pass over
// them (a volume may have 65536).
struct BoxSums {
  double samples = 0.0, bytes = 0.0;
  int64_t pixels = 0;           // of the rectangles
  double chord = 0.0;           // longest way along the view direction through a box, voxels
  int64_t most[3] = {0, 0, 0};  // largest extent along each axis, voxels
};
// Lanes per ray of a view's gathers: 4 x 4 rays of four consecutive samples
// touch fewer lines than 2 x 2 rays of sixteen where rays are less than 1.1
// voxels apart, sixteen lanes shorten the chain of a ray where there are few (two
// views of 201 x 187 x 333 at 0.8 voxels 405 us with 16, 330 with 4; 400^3 at
// 0.7 1.23 ms and 1.00, at 1.35 414 us and 484; 256^2 rays through 128^3 59
// and 59, fewer rays up to twice as slow with 4); otherwise whichever number is
// estimated faster, 1 among them.
int32_t gather_lanes(const Camera& cam, const BoxSums& boxes, double step, int32_t M);
void add_box(BoxSums& s, const Camera& cam, const Box& box, int64_t pixels, double step);
MarchTimes march_times(const Camera& cam, const BoxSums& boxes, const FootShape* fs, int views = 1);

// Footprint-cell shape of one parallel view of a volume of size n, as the
// forward picks it: plain = the plain march (no macrocell skipping, no mask),
// reg_on = register staging allowed, nslots = the ring-slot rule (0, 2 or 3),
// cells of about `rays` pixels with window rows of at most kmax 128-byte
// lines (+ pad floats), along slab axis `axis` (0: either).  False when the view has no suitable slab axis.
bool pick_foot(const Camera& cam, const int64_t n[3], int32_t M, bool plain, bool reg_on, int32_t nslots,
               double rays, int32_t pad, int32_t kmax, FootShape& fs, int32_t max_px = 0,
               int32_t axis = 0);

// Whether the rows of a brick (of the whole volume when it is not bricked) can be
// read `pitch` floats at a time: library storage has 64 floats of slack, a
// wrapped array none.
bool brick_rows_readable(const vr_volume* vol, int32_t brick, int32_t pitch);

// Launch arguments of the cell march with shape fs (wpb: wavefronts per
// workgroup), and the shape and place of a box's cells in its view entry;
// returns the number of cells.
void foot_args(const vr_ctx* ctx, const FootShape& fs, MarchArgs& a, int& wpb);
int32_t foot_brick(const Camera& cam, const FootShape& fs, const Box& box, DevBrickView& b);

void plan_bricked_view(const vr_volume* vol, const Camera& cam, const vr_params* p, int32_t tile_w,
                       const float* tf, int32_t M, double vmin, double vmax, ViewPlan& vp);
// The planned bricks regrouped by front-to-back wave.
void plan_waves(const vr_volume* vol, const Camera& cam, int32_t tile_w, ViewPlan& vp);
int render_forward(vr_ctx* ctx, vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p, float* out,
                   hipStream_t s);
int validate_render(vr_ctx* ctx, const vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p);
int render_with_state(vr_ctx* ctx, vr_volume* vol, const vr_view* views, int32_t nviews, const vr_params* p,
                      float* out, hipStream_t s, vr_state** save);

}  // namespace vr
