// Per-view render descriptor shared by the plain, batched and served paths.
#pragma once

#include "ls_internal.h"

// Everything one view needs, passed by value to the plain kernel and read
// from device memory (uniform, scalar loads) by the persistent kernel.
struct RenderArgs {
  const uint32_t* offsets;
  const uint64_t* records;
  const unsigned long long* occ;  // per 4^3 macro cell: mask of non-empty voxels
  // the same words grown by one voxel in every direction (neighbour mode; may be
  // null: the kernel forms them)
  const unsigned long long* grown;
  int32_t g[3];
  int32_t mg[3];                  // macro grid dims
  float inv_bins;
  const float* lut;
  const float* ao;
  const float* sh;
  float eye[3], fwd[3], right[3], up[3];
  int32_t ortho, W, H;
  float radius, r2, alpha_stop;
  int32_t mode, opaque, merge, shading;
  int32_t dist_alpha;             // opacity from the chord length inside the tube
  float inv_2r;                   // 1 / (2 radius)
  float ka, kd, ks, shin;
  float light[3];
  // shading 2 sources: ao_mode 0 grid / 1 hemisphere rays per fragment;
  // shadow_mode 0 grid / 1 cone per fragment / 2 representative-line ray
  int32_t ao_mode, shadow_mode, ao_rays, rep_level, n_levels;
  float ao_radius;
  const float* rho;               // density pyramid, levels flat
  const uint32_t* rep;            // representative lines, levels flat
  const uint16_t* ends;           // per-record endpoint attributes (or null)
  // opacity acceleration: switch at A >= accel_A0 (2: off), depth scale
  float accel_A0, accel_depth;
  const float* rgb;               // colour pyramid, levels flat, 3 floats per cell
  float* out;
  RenderCounters* counters;
  int32_t wx, wy;                 // tile = wx x wy waves of 8 x 8 pixels
  int32_t tiles_x, n_tiles, tiles_per_xcd;
  // plain launch order: the image's tiles in square rings around the tile
  // (spiral_x, spiral_y) out to ring spiral_r, or rows interleaved over the XCDs
  // when spiral_r < 0
  int32_t spiral_x, spiral_y, spiral_r;
  // the tiles of the first split_n spiral positions (the innermost rings)
  // are rendered by split_s workgroups each, on 64 / split_s of its pixels, so
  // the waves over the densest part of the image hold fewer rays
  int32_t split_n, split_s;
  // ordered frames: the first top_n launch positions (the longest measured
  // tiles) are split top_s ways (4, 8 or 16), before the split_n ones above
  int32_t top_n, top_s;
  // plain launch order by measured cost (tile_order): workgroup position p
  // renders tile order[p]; null: the ring order above. times (or null):
  // each workgroup adds its duration (10 ns ticks) to its tile's entry
  const int32_t* order;
  uint32_t* times;
};

// Tile queues of the persistent kernel: one contiguous range per XCD.
struct BatchQueues {
  int32_t begin[8];
  int32_t len[8];
};

struct BatchPlan {
  int32_t wx, wy;     // tile shape in waves
  int32_t blocks;     // persistent workgroups
};

// Plan of a batch that is neither tuned nor given one: single waves, which free
// their tile at once. With the queue counters in one cache line the pops of so
// many tiles held them back (24 mixed views: 3.12 ms against 2.58 with 2 x 2
// waves); a line each, they are the fastest: 2.42 against 2.57 ms (40 views of
// two sets 2.32 against 2.53; 4 small views the same).
constexpr BatchPlan kDefaultPlan{1, 1, 0};

// Tiles of an image of tx x ty tiles within the square rings 0 .. r around the
// tile (x, y).
__host__ __device__ inline int ring_tiles(int x, int y, int tx, int ty, int r) {
  const int x0 = x < r ? x : r, x1 = tx - 1 - x < r ? tx - 1 - x : r;
  const int y0 = y < r ? y : r, y1 = ty - 1 - y < r ? ty - 1 - y : r;
  return (x0 + x1 + 1) * (y0 + y1 + 1);
}

int make_render_args(const ls_lineset* s, const ls_camera* cam, const ls_render_params* p,
                     float* out, int wx, int wy, RenderCounters* dev_counters, RenderArgs* R);
int launch_render(const RenderArgs& R, hipStream_t st);
// True when the view needs the kernels' extended instance: it samples the
// pyramid or the representative lines per fragment (view-dependent
// illumination), or its set carries per-line endpoint attributes.
inline bool view_dependent(const RenderArgs& R) {
  return (R.shading == 2 && (R.ao_mode != 0 || R.shadow_mode != 0)) || R.ends != nullptr ||
         R.accel_A0 <= 1.f;
}
// What the views of a batch need of its kernel, which is compiled with and
// without: the extended instance (view_dependent), the neighbour mode.
struct BatchKind {
  bool vdi = false, nb = false;
};
BatchQueues make_queues(int total_tiles);
// Words of the queue counters: one per queue, a 128-byte line apart.
constexpr int kQueueStride = 32;
constexpr int kQueueWords = 8 * kQueueStride;
// dev_queue: kQueueWords words (zeroed before the launch), followed by a
// RenderCounters block when `count` is set.
int launch_render_batch(const RenderArgs* dev_views, const int32_t* dev_tile_start, int n_views,
                        const BatchQueues& q, unsigned* dev_queue, const BatchPlan& plan,
                        bool count, const BatchKind& kind, hipStream_t st);
int batch_blocks_per_cu(int wx, int wy, const BatchKind& kind, int* out);
int render_merge_slots();   // intervals in the per-ray curve-merge table
