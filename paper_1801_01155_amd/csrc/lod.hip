// Density pyramid (section "LoD construction") on gfx950.
//
// Level 0 over each voxel's contiguous line list:
//   count = #lines, len = sum |exit - entry|, rho = sum |exit - entry| * sigma
// (sigma = lut[attr].a, or 1 for opaque lines). Each coarser level averages
// the 2^3 children of the finer one (children beyond an odd side count as 0).
// The three fields are written as separate float arrays (structure of arrays)
// so the renderer and the cone tracer read only rho.
#include <algorithm>

#include "ls_internal.h"
#include "wave.h"

namespace {

constexpr int kBlock = 256;

__device__ inline void decode_point(uint32_t code, float inv_bins, float p[3]) {
  const int face = (int)(code & 7u);
  const int axis = face >> 1;
  const float side = (float)(face & 1);
  const float u = ((float)((code >> 3) & 63u) + 0.5f) * inv_bins;
  const float w = ((float)((code >> 9) & 63u) + 0.5f) * inv_bins;
  p[0] = axis == 0 ? side : u;
  p[1] = axis == 1 ? side : (axis == 0 ? u : w);
  p[2] = axis == 2 ? side : w;
}

// Level 0, a wave per 64 consecutive voxels. Their lists are one contiguous
// run of records, read 64 at a time by the whole wave (coalesced); each
// line's length goes through a segmented scan over the lanes holding its
// voxel's lines, and the voxel's lane collects its segment's total. A wave
// costs (lines of its voxels) / 64 steps instead of its longest list. The
// scans and the owners are DPP moves (wave.h): as chains of cross-lane reads
// (18 per step) level 0 took 122 us at 256^3 with 9.5M records, against about 60
// for its memory traffic; so 115.
// Sums of the wave's voxels: this lane's list is [lo, lo + n).
__device__ inline void lod_sums(const uint64_t* __restrict__ records, uint32_t lo, uint32_t n,
                                float inv_bins, const float* s_alpha, uint32_t* own, float& l,
                                float& r) {
  // this voxel's lines are the wave's lines [P, P + n), records lo0 + [P, P + n)
  uint32_t N;
  const uint32_t P = wave_excl_scan(n, N);
  const uint32_t lo0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
  l = r = 0.f;
  // the records of the next two steps are in flight while a step is summed
  uint64_t r0 = 0, r1 = 0;
  if ((uint32_t)wave_lane() < N) r0 = records[lo0 + (uint32_t)wave_lane()];
  if ((uint32_t)wave_lane() + 64u < N) r1 = records[lo0 + (uint32_t)wave_lane() + 64u];
  for (uint32_t base = 0; base < N; base += 64) {
    const uint32_t w = base + (uint32_t)wave_lane();
    const uint64_t rec = r0;
    r0 = r1;
    if (w + 128u < N) r1 = records[lo0 + w + 128u];
    const int o = chunk_owner(own, P, n, base);
    float L = 0.f, Ls = 0.f;
    if (w < N) {
      float a[3], b[3];
      decode_point((uint32_t)(rec & 0x7FFFu), inv_bins, a);
      decode_point((uint32_t)((rec >> 15) & 0x7FFFu), inv_bins, b);
      const float dx = b[0] - a[0], dy = b[1] - a[1], dz = b[2] - a[2];
      L = sqrtf(dx * dx + dy * dy + dz * dz);
      Ls = L * s_alpha[(rec >> 32) & 0xFF];
    }
    // lanes of one owner form a contiguous run
    const uint32_t po = (uint32_t)__shfl((int)P, o, 64);
    const int seg0 = po > base ? (int)(po - base) : 0;
    L = wave_seg_sum(L, seg0);
    Ls = wave_seg_sum(Ls, seg0);
    // this voxel's run in the chunk ends at lane min(P + n, base + 64) - 1
    // (all lanes shuffle; lanes without a run here discard the value)
    const bool here = n != 0 && P < base + 64u && P + n > base;
    const int end = here ? (int)((P + n < base + 64u ? P + n : base + 64u) - 1u - base) : 0;
    const float tl = __shfl(L, end, 64), tr = __shfl(Ls, end, 64);
    if (here) {
      l += tl;
      r += tr;
    }
  }
}

// The transfer function's opacities, staged once per block (a record's opacity
// is then not a global load that waits for the record).
__device__ inline void stage_alpha(const float* lut, int opaque, float* s_alpha) {
  static_assert(kBlock == 256, "one thread per transfer-function entry");
  s_alpha[threadIdx.x] = opaque ? 1.f : lut[4 * threadIdx.x + 3];
  __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_lod0(const uint32_t* __restrict__ offsets,
                                                 const uint64_t* __restrict__ records,
                                                 int64_t nvox, float inv_bins, const float* lut,
                                                 int opaque, float* __restrict__ count,
                                                 float* __restrict__ len, float* __restrict__ rho) {
  __shared__ float s_alpha[256];
  __shared__ uint32_t marks[kBlock];
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool in = v < nvox;
  const uint32_t lo = in ? offsets[v] : 0u, n = in ? offsets[v + 1] - lo : 0u;
  stage_alpha(lut, opaque, s_alpha);
  float l, r;
  lod_sums(records, lo, n, inv_bins, s_alpha, marks + (threadIdx.x & ~63u), l, r);
  if (!in) return;
  count[v] = (float)n;
  len[v] = l;
  rho[v] = r;
}

struct LodRows {
  int32_t g[3], p[3];   // level 0 and level 1 dims
  int64_t off1;         // level 1's first cell
  int32_t turn;         // log2 of the rows of blocks after which the columns turn
};

// Levels 0 and 1 together: a block takes 64 x 2 x 2 voxels, a wave per row along
// x, and averages its 32 level-1 cells from LDS (children in k_mip's order, so
// the same bits), instead of reading the three fields of level 0 again. 256^3,
// 9.5M records: 171 us for both as two kernels, 121 so; its traffic takes 75, what
// is left is the latency of a block's few serial stages.
// Blocks go to the XCDs, and within one to its shader engines, in turn along x
// first. With two or four blocks to a row each XCD would see the same columns of
// the grid only, and half of them the partly empty last one (80^3, 6.3M records
// 92.8 us, 200^3, 16M 178), so the columns turn, every eight blocks of an XCD (70
// to 90 and 118; every block: 93 and 182, as that keeps to the same engines).
constexpr int kTurnRows = 3;   // log2 of an XCD's blocks between turns

// Where that is faster than k_lod0 and k_mip (whole density pyramids, us, two
// kernels against this one; "few" and "many": 10k and 300k curves of 100
// vertices). One block per row, cubes: 24^3 few 33 and 20, 32^3 28 and 19, many
// 212 and 112, 64^3 28 and 24, 80 and 78; in 400 x 400 rows of 24 53 and 56, of 40
// 71 and 61. Else the lanes beyond the last row end idle: 80^3 (3/8 idle) few 32
// and 29, many 74 and 90, 95^3 (1/4) 37 and 30, 82 and 83, 193^3 (1/4) 71 and 66,
// 125 and 109, 208^3 (3/16) 82 and 72, 148 and 131. Beyond 2^23.5 voxels memory
// counts: 104 x 400 x 400 (3/16) 151 and 154, 156 and 167, 257^3 (1/5) 166 and
// 182, 264^3 (7/40) 182 and 184, 184 and 193, 272^3 (3/20) 200 and 183, 260 and
// 227.
constexpr int kRowMin = 32;
constexpr int64_t kRowLarge = int64_t(3) << 22;

bool rows_together(const ls_lineset* s) {
  const int64_t g = s->grid[0], lanes = (g + 63) / 64 * 64;
  if (s->n_levels < 2 || g < kRowMin) return false;
  return lanes == 64 || (s->nvox <= kRowLarge ? 4 * g >= 3 * lanes : 6 * g >= 5 * lanes);
}

__global__ __launch_bounds__(kBlock) void k_lod01(const uint32_t* __restrict__ offsets,
                                                  const uint64_t* __restrict__ records,
                                                  LodRows g, float inv_bins, const float* lut,
                                                  int opaque, float* __restrict__ count,
                                                  float* __restrict__ len,
                                                  float* __restrict__ rho) {
  __shared__ float s_alpha[256];
  __shared__ uint32_t marks[kBlock];
  __shared__ float s_row[3][kBlock];
  const int lane = wave_lane(), wave = (int)(threadIdx.x >> 6);
  const uint32_t row = blockIdx.y + gridDim.y * blockIdx.z;
  const int bx = (int)((blockIdx.x + (row >> g.turn)) % gridDim.x);
  const int x = 64 * bx + lane, y = 2 * (int)blockIdx.y + (wave & 1),
            z = 2 * (int)blockIdx.z + (wave >> 1);
  const bool in = x < g.g[0] && y < g.g[1] && z < g.g[2];
  const int64_t v = x + (int64_t)g.g[0] * (y + (int64_t)g.g[1] * z);
  const uint32_t lo = in ? offsets[v] : 0u, n = in ? offsets[v + 1] - lo : 0u;
  stage_alpha(lut, opaque, s_alpha);
  float l, r;
  lod_sums(records, lo, n, inv_bins, s_alpha, marks + (threadIdx.x & ~63u), l, r);
  if (in) {
    count[v] = (float)n;
    len[v] = l;
    rho[v] = r;
  }
  // rows and voxels outside the grid hold 0
  s_row[0][threadIdx.x] = (float)n;
  s_row[1][threadIdx.x] = l;
  s_row[2][threadIdx.x] = r;
  __syncthreads();
  const int c = wave, i = lane;   // field, cell
  const int px = 32 * bx + i;
  if (c >= 3 || i >= 32 || px >= g.p[0]) return;
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k)   // x fastest, then y, then z
    sum += s_row[c][64 * (k >> 1) + 2 * i + (k & 1)];
  float* out = c == 0 ? count : (c == 1 ? len : rho);
  out[g.off1 + px + (int64_t)g.p[0] * ((int)blockIdx.y + (int64_t)g.p[1] * (int)blockIdx.z)] =
      sum * 0.125f;
}

struct MipArgs {
  int32_t cx, cy, cz;  // child dims
  int32_t px, py, pz;  // parent dims
};

__global__ __launch_bounds__(kBlock) void k_mip(const float* __restrict__ c_count,
                                                const float* __restrict__ c_len,
                                                const float* __restrict__ c_rho, float* p_count,
                                                float* p_len, float* p_rho, MipArgs m) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  int64_t n = (int64_t)m.px * m.py * m.pz;
  if (i >= n) return;
  int32_t x = (int32_t)(i % m.px), y = (int32_t)((i / m.px) % m.py),
          z = (int32_t)(i / ((int64_t)m.px * m.py));
  float sc = 0.f, sl = 0.f, sr = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    int32_t ax = 2 * x + (k & 1), ay = 2 * y + ((k >> 1) & 1), az = 2 * z + (k >> 2);
    if (ax < m.cx && ay < m.cy && az < m.cz) {
      int64_t ci = ax + (int64_t)m.cx * (ay + (int64_t)m.cy * az);
      sc += c_count[ci];
      sl += c_len[ci];
      sr += c_rho[ci];
    }
  }
  p_count[i] = sc * 0.125f;
  p_len[i] = sl * 0.125f;
  p_rho[i] = sr * 0.125f;
}

// Small levels, up to kBrickLevels per launch: each
// workgroup takes an 8^3 brick of the first level it writes and reduces it
// to one voxel through LDS (8^3 -> 4^3 -> 2^3 -> 1), so a small level costs
// a few LDS passes instead of a launch. Sums run over the children in the
// same order as k_mip, so every level is bit-identical to one k_mip per level.
// Levels larger than kBrickMaxVoxels keep one k_mip launch each: a brick's
// few loads in flight per thread read a big level slower than a thread per
// voxel does (measured at 512^3: 128^3 bricked 1.31 ms for the pyramid,
// 1.27 ms with k_mip).
constexpr int kBrick = 8;
constexpr int kBrickLevels = 4;
constexpr int64_t kBrickMaxVoxels = 1 << 18;

struct BrickArgs {
  int32_t dims[kBrickLevels + 1][3];   // level L (children) .. L + nl
  int64_t off[kBrickLevels + 1];       // their element offsets in the pyramid
  int32_t nl;                          // levels written, 1..kBrickLevels
  int32_t bx, by;                      // bricks along x and y of level L + 1
};

__global__ __launch_bounds__(kBlock) void k_mip_brick(float* count, float* len, float* rho,
                                                      BrickArgs a) {
  // level L + j of the brick (side kBrick >> (j - 1)) at lds[c][base[j] + v]
  __shared__ float lds[3][512 + 64 + 8];
  const int base[4] = {0, 0, 512, 576};
  const int b = blockIdx.x;
  const int ox = b % a.bx, oy = (b / a.bx) % a.by, oz = b / (a.bx * a.by);
  float* const ch[3] = {count, len, rho};
  for (int j = 1; j <= a.nl; ++j) {
    const int side = kBrick >> (j - 1);
    const int32_t* cd = a.dims[j - 1];
    const int32_t* pd = a.dims[j];
    const int32_t gx0 = ox * side, gy0 = oy * side, gz0 = oz * side;
    for (int v = threadIdx.x; v < side * side * side; v += kBlock) {
      const int x = v % side, y = (v / side) % side, z = v / (side * side);
      const int32_t gx = gx0 + x, gy = gy0 + y, gz = gz0 + z;
      if (gx >= pd[0] || gy >= pd[1] || gz >= pd[2]) continue;
      float sum[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int kx = k & 1, ky = (k >> 1) & 1, kz = k >> 2;
        const int32_t ax = 2 * gx + kx, ay = 2 * gy + ky, az = 2 * gz + kz;
        if (ax < cd[0] && ay < cd[1] && az < cd[2]) {
          if (j == 1) {
            const int64_t ci = a.off[0] + ax + (int64_t)cd[0] * (ay + (int64_t)cd[1] * az);
#pragma unroll
            for (int c = 0; c < 3; ++c) sum[c] += ch[c][ci];
          } else {
            const int s2 = 2 * side;
            const int li = base[j - 1] + (2 * x + kx) + s2 * ((2 * y + ky) + s2 * (2 * z + kz));
#pragma unroll
            for (int c = 0; c < 3; ++c) sum[c] += lds[c][li];
          }
        }
      }
      const int64_t pi = a.off[j] + gx + (int64_t)pd[0] * (gy + (int64_t)pd[1] * gz);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float m = sum[c] * 0.125f;
        ch[c][pi] = m;
        if (j < a.nl) lds[c][base[j] + v] = m;
      }
    }
    __syncthreads();
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Colour beside the density for opacity acceleration: per voxel the sum over
// its lines of length * sigma * (transfer-function colour), three floats
// interleaved; a thread per voxel walks its list.
__global__ __launch_bounds__(kBlock) void k_lodc0(const uint32_t* offsets, const uint64_t* records,
                                                  int64_t nvox, float inv_bins, const float* lut,
                                                  int opaque, float* rgb) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= nvox) return;
  float c[3] = {0.f, 0.f, 0.f};
  for (uint32_t k = offsets[v]; k < offsets[v + 1]; ++k) {
    const uint64_t rec = records[k];
    float a[3], b[3];
    decode_point((uint32_t)(rec & 0x7FFFu), inv_bins, a);
    decode_point((uint32_t)((rec >> 15) & 0x7FFFu), inv_bins, b);
    const float dx = b[0] - a[0], dy = b[1] - a[1], dz = b[2] - a[2];
    const float L = sqrtf(dx * dx + dy * dy + dz * dz);
    const float* l = lut + 4 * ((rec >> 32) & 0xFF);
    const float w = L * (opaque ? 1.f : l[3]);
    c[0] += w * l[0];
    c[1] += w * l[1];
    c[2] += w * l[2];
  }
  rgb[3 * v + 0] = c[0];
  rgb[3 * v + 1] = c[1];
  rgb[3 * v + 2] = c[2];
}

// One coarser colour level: parent cell v averages its 8 children (x fastest,
// missing children beyond an odd side count as 0).
__device__ inline void mipc_cell(const float* child, float* parent, const MipArgs& m, int64_t v) {
  const int32_t x = (int32_t)(v % m.px), y = (int32_t)((v / m.px) % m.py),
                z = (int32_t)(v / ((int64_t)m.px * m.py));
  float s[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int32_t cx = 2 * x + (k & 1), cy = 2 * y + ((k >> 1) & 1), cz = 2 * z + (k >> 2);
    if (cx >= m.cx || cy >= m.cy || cz >= m.cz) continue;
    const int64_t ci = cx + (int64_t)m.cx * (cy + (int64_t)m.cy * cz);
    s[0] += child[3 * ci + 0];
    s[1] += child[3 * ci + 1];
    s[2] += child[3 * ci + 2];
  }
  parent[3 * v + 0] = s[0] * 0.125f;
  parent[3 * v + 1] = s[1] * 0.125f;
  parent[3 * v + 2] = s[2] * 0.125f;
}

__global__ __launch_bounds__(kBlock) void k_mipc(const float* __restrict__ child,
                                                 float* __restrict__ parent, MipArgs m) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v < (int64_t)m.px * m.py * m.pz) mipc_cell(child, parent, m, v);
}

// The small top levels (up to kTailCells each) in one workgroup, level by level,
// instead of a launch each.
constexpr int64_t kTailCells = 1024;
constexpr int kTailThreads = 1024;
struct ColorTail {
  int32_t n;              // levels written
  int32_t dim[14][3];     // the level below them, then them
  int64_t off[14];
};

__global__ __launch_bounds__(kTailThreads) void k_mipc_tail(ColorTail t, float* rgb) {
  for (int l = 1; l <= t.n; ++l) {
    const MipArgs m{t.dim[l - 1][0], t.dim[l - 1][1], t.dim[l - 1][2],
                    t.dim[l][0],     t.dim[l][1],     t.dim[l][2]};
    const int64_t n = (int64_t)m.px * m.py * m.pz;
    for (int64_t v = threadIdx.x; v < n; v += kTailThreads)
      mipc_cell(rgb + 3 * t.off[l - 1], rgb + 3 * t.off[l], m, v);
    __syncthreads();
  }
}

}  // namespace

int lod_color_build(ls_lineset* s, const float* lut, int opaque, hipStream_t st) {
  int rc;
  if (!s->lod_rgb) {
    if ((rc = ls_alloc(s, (void**)&s->lod_rgb,
                       3 * sizeof(float) * (size_t)s->level_off[s->n_levels])))
      return rc;
  }
  if (s->nvox > 0) {
    hipLaunchKernelGGL(k_lodc0, dim3(blocks_for(s->nvox)), dim3(kBlock), 0, st, s->offsets,
                       s->records, s->nvox, 1.0f / (float)s->bins, lut, opaque, s->lod_rgb);
    LS_HIP(hipGetLastError());
  }
  int L = 0;
  for (; L + 1 < s->n_levels; ++L) {
    const int64_t n = s->level_off[L + 2] - s->level_off[L + 1];
    if (n <= kTailCells) break;
    MipArgs m{s->level_dims[L][0],     s->level_dims[L][1],     s->level_dims[L][2],
              s->level_dims[L + 1][0], s->level_dims[L + 1][1], s->level_dims[L + 1][2]};
    hipLaunchKernelGGL(k_mipc, dim3(blocks_for(n)), dim3(kBlock), 0, st,
                       s->lod_rgb + 3 * s->level_off[L], s->lod_rgb + 3 * s->level_off[L + 1], m);
    LS_HIP(hipGetLastError());
  }
  if (L + 1 < s->n_levels) {
    ColorTail t{};
    t.n = s->n_levels - 1 - L;   // at most 11 levels in all: sides up to 1024
    for (int k = 0; k <= t.n; ++k) {
      for (int a = 0; a < 3; ++a) t.dim[k][a] = s->level_dims[L + k][a];
      t.off[k] = s->level_off[L + k];
    }
    hipLaunchKernelGGL(k_mipc_tail, dim3(1), dim3(kTailThreads), 0, st, t, s->lod_rgb);
    LS_HIP(hipGetLastError());
  }
  return LS_OK;
}

void lod_plan(const int32_t grid[3], int32_t* n_levels, int32_t dims[][3], int64_t* level_off) {
  int n = 0;
  int32_t cur[3] = {grid[0], grid[1], grid[2]};
  level_off[0] = 0;
  for (;;) {
    for (int a = 0; a < 3; ++a) dims[n][a] = cur[a];
    level_off[n + 1] = level_off[n] + (int64_t)cur[0] * cur[1] * cur[2];
    ++n;
    if ((cur[0] == 1 && cur[1] == 1 && cur[2] == 1) || n == LS_MAX_LEVELS) break;
    for (int a = 0; a < 3; ++a) cur[a] = (cur[a] + 1) / 2;
  }
  *n_levels = n;
}

int lod_build(ls_lineset* s, const float* lut, int opaque, hipStream_t st) {
  int rc;
  if (!s->lod_rho) {
    lod_plan(s->grid, &s->n_levels, s->level_dims, s->level_off);
    size_t bytes = sizeof(float) * (size_t)s->level_off[s->n_levels];
    if ((rc = ls_alloc(s, (void**)&s->lod_count, bytes)) ||
        (rc = ls_alloc(s, (void**)&s->lod_len, bytes)) || (rc = ls_alloc(s, (void**)&s->lod_rho, bytes)))
      return rc;
  }
  int L = 0;
  if (rows_together(s)) {
    LodRows g{};
    for (int a = 0; a < 3; ++a) {
      g.g[a] = s->level_dims[0][a];
      g.p[a] = s->level_dims[1][a];
    }
    g.off1 = s->level_off[1];
    const int nx = (g.g[0] + 63) / 64;
    // nx blocks to a row: a column is back on its XCD after 8 / gcd(nx, 8) rows
    g.turn = 3;
    while (g.turn > 0 && nx % (16 >> g.turn) == 0) --g.turn;
    g.turn += kTurnRows;
    hipLaunchKernelGGL(k_lod01, dim3(nx, g.p[1], g.p[2]), dim3(kBlock), 0, st,
                       s->offsets, s->records, g, 1.0f / (float)s->bins, lut, opaque,
                       s->lod_count, s->lod_len, s->lod_rho);
    LS_HIP(hipGetLastError());
    L = 1;
  } else if (s->nvox > 0) {
    hipLaunchKernelGGL(k_lod0, dim3(blocks_for(s->nvox)), dim3(kBlock), 0, st, s->offsets,
                       s->records, s->nvox, 1.0f / (float)s->bins, lut, opaque, s->lod_count,
                       s->lod_len, s->lod_rho);
    LS_HIP(hipGetLastError());
  }
  // large levels stream their children at full occupancy (a thread per
  // voxel); the small rest goes kBrickLevels levels per launch through LDS
  for (; L + 1 < s->n_levels; ++L) {
    const int64_t p0 = s->level_off[L + 1];
    const int64_t n = s->level_off[L + 2] - p0;
    if (n <= kBrickMaxVoxels) break;
    const int64_t c0 = s->level_off[L];
    MipArgs m{s->level_dims[L][0],     s->level_dims[L][1],     s->level_dims[L][2],
              s->level_dims[L + 1][0], s->level_dims[L + 1][1], s->level_dims[L + 1][2]};
    hipLaunchKernelGGL(k_mip, dim3(blocks_for(n)), dim3(kBlock), 0, st, s->lod_count + c0,
                       s->lod_len + c0, s->lod_rho + c0, s->lod_count + p0, s->lod_len + p0,
                       s->lod_rho + p0, m);
    LS_HIP(hipGetLastError());
  }
  for (; L + 1 < s->n_levels; L += kBrickLevels) {
    BrickArgs a{};
    a.nl = std::min(kBrickLevels, s->n_levels - 1 - L);
    for (int j = 0; j <= a.nl; ++j) {
      for (int c = 0; c < 3; ++c) a.dims[j][c] = s->level_dims[L + j][c];
      a.off[j] = s->level_off[L + j];
    }
    a.bx = (a.dims[1][0] + kBrick - 1) / kBrick;
    a.by = (a.dims[1][1] + kBrick - 1) / kBrick;
    const int64_t bz = (a.dims[1][2] + kBrick - 1) / kBrick;
    const int64_t blocks = (int64_t)a.bx * a.by * bz;
    hipLaunchKernelGGL(k_mip_brick, dim3((unsigned)blocks), dim3(kBlock), 0, st, s->lod_count,
                       s->lod_len, s->lod_rho, a);
    LS_HIP(hipGetLastError());
  }
  return LS_OK;
}
