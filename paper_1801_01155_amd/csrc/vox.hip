// Voxelization of curves into per-voxel quantized line lists (CSR) on gfx950.
//
// Sections "Curve voxelization", "Line quantization" and "GPU
// implementation". The paper's GPU construction appends per-curve lines
// tagged with voxel ids, sorts by voxel and prefix-sums the counts. Here the
// append is replaced by a count pass that sizes every curve's output range
// exactly (so the emit pass writes without global atomics on a cursor), the
// sort by a histogram + scan + scatter, and determinism inside a voxel by a
// rank pass:
//   k_count   wave per curve: upper bound of the curve's lines (plane
//             crossings - 1); validates the input
//   scan      curve ranges
//   k_emit    wave per curve, lane per segment: exact integer clipping,
//             quantization and packing; a wave prefix sum numbers the events
//             along the curve, so lanes write their lines to consecutive slots
//             (coalesced) in curve order, each taking its rank in its voxel
//             with one atomic on the histogram
//   scan      voxel offsets (CSR)
//   k_scatter thread per emitted line: index into its voxel's range
//   k_rank    thread per CSR slot: ranks the voxel's lines by emission order
//             and gathers the record, so each list is in (curve, position
//             along curve) order regardless of atomic order
// Larger grids go by bricks of 8^3 voxels instead of by atomics and scattered
// writes per line (see "Lists by bricks" below): a curve stays in a brick for
// several lines, so what is counted, placed and read per brick are runs.
// All arithmetic deciding a line's voxel, faces and bins is exact integer
// arithmetic on the 1/256-voxel lattice.
#include "ls_internal.h"
#include "wave.h"

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>
#include <vector>

namespace {

constexpr int kBlock = 256;

struct GridArgs {
  int32_t g[3];
  int32_t bins;
  int32_t bin_shift;  // log2(256 / bins)
};

// Grid set-up (section "Curve voxelization"): fp64 without contraction, the
// same expression as documented in lineset.h.
__device__ inline int32_t snap_coord(float x, double lo, double scale) {
  double y = __dmul_rn(__dadd_rn((double)x, -lo), scale);
  y = __dadd_rn(y, 0.5);
  return (int32_t)floor(y) + 256;
}

template <bool kFloatIn>
__device__ inline void load_vertex(const float* xyz, const int32_t* lat, int64_t v,
                                   const SnapArgs& sa, int32_t q[3]) {
  if (kFloatIn) {
    const float* p = xyz + 3 * v;
    q[0] = snap_coord(p[0], sa.lo[0], sa.scale);
    q[1] = snap_coord(p[1], sa.lo[1], sa.scale);
    q[2] = snap_coord(p[2], sa.lo[2], sa.scale);
  } else {
    const int32_t* p = lat + 3 * v;
    q[0] = p[0];
    q[1] = p[1];
    q[2] = p[2];
  }
}

__device__ inline bool in_range(const int32_t q[3], const GridArgs& ga) {
  return q[0] >= 0 && q[1] >= 0 && q[2] >= 0 && q[0] < 256 * ga.g[0] && q[1] < 256 * ga.g[1] &&
         q[2] < 256 * ga.g[2];
}

// error codes written to err[0]
constexpr int kErrOffsets = 1;
constexpr int kErrRange = 2;
constexpr int kErrNonFinite = 4;

// Lattice scale 256 (G_a - 2) / extent_a, minimised over the axes with a
// positive extent (0 if none): the grid set-up of section "Curve
// voxelization", the same expression on the host and the device.
__host__ __device__ inline double lattice_scale(const double lo[3], const double hi[3],
                                                const int32_t grid[3]) {
  double s = INFINITY;
  for (int a = 0; a < 3; ++a) {
    const double ext = hi[a] - lo[a];
    if (ext > 0) {
      const double cand = (256.0 * (double)(grid[a] - 2)) / ext;
      if (cand < s) s = cand;
    }
  }
  return s == INFINITY ? 0.0 : s;
}

// Low 32 bits of a * b for a, b below 2^24: one full-rate 24-bit multiply
// (written out because the operands' range is not visible to instruction
// selection across basic blocks, which then picks the quarter-rate 32-bit one).
__device__ inline uint32_t mul_lo24(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// floor(num / den) for 0 <= num <= 256 den, 0 < den < 2^18 (quotient at
// most 256): an fp32 estimate (relative error below 1e-6, so off by at most
// one) corrected by one exact step either way; 24-bit products.
__device__ inline int32_t floor_div_small(int32_t num, int32_t den) {
  __builtin_assume(den > 0 && den < (1 << 18));
  int32_t q = (int32_t)((float)num * __builtin_amdgcn_rcpf((float)den));
  __builtin_assume(q >= 0 && q <= 512);
  if ((int32_t)mul_lo24((uint32_t)q, (uint32_t)den) > num) --q;
  else if ((int32_t)mul_lo24((uint32_t)(q + 1), (uint32_t)den) <= num) ++q;
  return q;
}

// Low 32 bits of the exact event point times den: P0 den + nf d, with
// lattice coordinates and den below 2^18 (24-bit products, wrapping sum).
__device__ inline void event_low(const int32_t P0[3], const int32_t d[3], int32_t den, int32_t nf,
                                 uint32_t xl[3]) {
#pragma unroll
  for (int b = 0; b < 3; ++b)
    xl[b] = mul_lo24((uint32_t)P0[b], (uint32_t)den) + (uint32_t)__mul24(nf, d[b]);
}

// In-face bins of an event point on voxel `cell`, face normal `axis`.
// xl = low 32 bits of (event point * den); the local coordinate
// xn - 256 cell den lies in [0, 256 den] (below 2^26), so it is exact in
// wrapping 32-bit arithmetic.
__device__ inline uint32_t face_code(int axis, int side, const uint32_t xl[3], int32_t den,
                                     const int32_t cell[3], const GridArgs& ga) {
  const uint32_t x_u = axis == 0 ? xl[1] : xl[0];
  const uint32_t x_w = axis == 2 ? xl[1] : xl[2];
  const int32_t c_u = axis == 0 ? cell[1] : cell[0];
  const int32_t c_w = axis == 2 ? cell[1] : cell[2];
  const int32_t lu = (int32_t)(x_u - mul_lo24((uint32_t)(c_u << 8), (uint32_t)den));
  const int32_t lw = (int32_t)(x_w - mul_lo24((uint32_t)(c_w << 8), (uint32_t)den));
  // bin = floor(l / (den 256 / N)) = floor(floor(l / 2^sh) / den), 256 / N = 2^sh
  int32_t bu = floor_div_small(lu >> ga.bin_shift, den);
  int32_t bw = floor_div_small(lw >> ga.bin_shift, den);
  bu = bu < ga.bins - 1 ? bu : ga.bins - 1;
  bw = bw < ga.bins - 1 ? bw : ga.bins - 1;
  return (uint32_t)(2 * axis + side) | ((uint32_t)bu << 3) | ((uint32_t)bw << 9);
}

// Brick index of voxel (x, y, z): brick << 9 | voxel in its brick (8^3 voxels, x
// fastest). Bricks are numbered in blocks of 4 x 4 x 2 (x fastest), the blocks
// row by row (nbx along x, nbxy in a layer): the bricks a curve visits in turn
// then mostly share a 128-byte line of an array of words per brick, and
// atomics of a wave that meet in one line travel as one request.
__device__ inline uint32_t brick_index(uint32_t x, uint32_t y, uint32_t z, uint32_t nbx,
                                       uint32_t nbxy) {
  return (((x >> 5) + nbx * (y >> 5) + nbxy * (z >> 4)) << 14) |
         ((x & 7u) | (y & 7u) << 3 | (z & 7u) << 6 | (x >> 3 & 3u) << 9 | (y >> 3 & 3u) << 11 |
          (z >> 3 & 1u) << 13);
}

constexpr int kRunShift = 9;   // of the voxel in its brick

// Words of the line sample, and the word of a brick: its own up to kSampleWords
// bricks, a hashed one beyond (also of the indices that vertices outside the grid
// give).
constexpr uint32_t kSampleWords = 1u << 12;
__host__ __device__ inline uint32_t sample_slot(uint32_t brick) {
  return (brick ^ (brick >> 12) * 0x9E5u) & (kSampleWords - 1);
}

// One wave per curve; lane l of the wave handles segment s0 + l, 64 segments
// at a time, so vertex loads and record writes are contiguous across lanes.
constexpr int kWavesPerBlock = kBlock / 64;

// Line sample: thread i takes the i-th of kSamples even parts of the vertices and in
// it a hashed vertex and its successor, and adds the crossings between them, at
// most 8, to the word of the brick that holds a hashed point of that segment. (A
// curve's last vertex gives a segment to the next curve, as crowded as the curves
// are; the limit keeps its weight near the others'.)
constexpr int kSamples = 4096;
constexpr int kSampleBlocks = kSamples / kBlock;

template <bool kFloatIn>
__device__ inline void sample_line(int i, const float* xyz, const int32_t* lat, int64_t n_vertices,
                                   const SnapArgs& sa, uint32_t nbx, uint32_t nbxy,
                                   uint32_t* sample) {
  if (n_vertices < 2) return;
  uint32_t x = (uint32_t)i * 0x9E3779B1u;
  x = (x ^ x >> 15) * 0xC2B2AE3Du;
  x ^= x >> 13;
  const int64_t v0 = (n_vertices - 1) * i / kSamples, v1 = (n_vertices - 1) * (i + 1) / kSamples;
  const int64_t v = v0 + (int64_t)((uint64_t)x * (uint64_t)(v1 - v0) >> 32);
  int32_t p[3], q[3];
  load_vertex<kFloatIn>(xyz, lat, v, sa, p);
  load_vertex<kFloatIn>(xyz, lat, v + 1, sa, q);
  const uint32_t f = (x * 0x165667B1u) >> 20;   // 12 bits: place on the segment
  uint32_t n = 0, c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    n += (uint32_t)abs((q[a] >> 8) - (p[a] >> 8));
    c[a] = (uint32_t)((p[a] + ((int32_t)((uint32_t)(q[a] - p[a]) * f) >> 12)) >> 8);
  }
  // (vertices outside the grid give some word: the call fails later)
  if (n != 0u)
    atomicAdd(sample + sample_slot(brick_index(c[0], c[1], c[2], nbx, nbxy) >> kRunShift),
              min(n, 8u));
}

// Per-curve count of line slots: plane crossings - 1 (an upper bound of the
// lines; simultaneous crossings merge into one event). Validates the input.
// Bound by reading the vertices and by the snap's fp64 instructions, so each is
// loaded and snapped once and its neighbour comes by a DPP move: 20M vertices
// 73 -> 54 us, 100M 441 -> 352 us. (In the emission, whose own work hides the
// loads, the same made no difference.)
// sample (or null): the first kSampleBlocks workgroups take the line sample.
template <bool kFloatIn>
__global__ __launch_bounds__(kBlock) void k_count(const float* xyz, const int32_t* lat,
                                                  const int64_t* curve_off, int64_t n_curves,
                                                  int64_t n_vertices, const SnapArgs* sap,
                                                  GridArgs ga, uint64_t* slots, int* err,
                                                  uint32_t* sample, uint32_t nbx,
                                                  uint32_t nbxy) {
  const int lane = threadIdx.x & 63;
  const SnapArgs sa = kFloatIn ? *sap : SnapArgs{};
  int64_t b = blockIdx.x;
  if (sample) {
    if (b < kSampleBlocks) {
      sample_line<kFloatIn>((int)(b * kBlock + threadIdx.x), xyz, lat, n_vertices, sa, nbx, nbxy,
                            sample);
      return;
    }
    b -= kSampleBlocks;
  }
  const int64_t c = b * kWavesPerBlock + (threadIdx.x >> 6);
  if (c >= n_curves) return;  // wave-uniform
  const int64_t v0 = curve_off[c], v1 = curve_off[c + 1];
  if (v0 < 0 || v1 < v0 || v1 > n_vertices || (c == 0 && v0 != 0)) {
    if (lane == 0) {
      atomicOr(err, kErrOffsets);
      slots[c] = 0;
    }
    return;
  }
  unsigned long long crossings = 0;
  bool bad = false;
  // 128 vertices per pass, loaded and snapped once, the next one's read from
  // the next lane; the pass's last vertex is the next pass's first. Indices are
  // clamped to the curve's last vertex (v1 > v0 inside the loop), so the loads
  // need no branch, and a repeated vertex adds nothing.
  for (int64_t s0 = v0; s0 + 1 < v1 || (s0 == v0 && v0 < v1); s0 += 127) {
    int32_t q[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t v = s0 + 64 * h + lane;
      load_vertex<kFloatIn>(xyz, lat, v < v1 ? v : v1 - 1, sa, q[h]);
    }
    uint32_t n = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bad |= !in_range(q[h], ga);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int32_t k = q[h][a] >> 8;
        const int32_t last = h == 0 ? __builtin_amdgcn_readfirstlane(q[1][a] >> 8) : k;
        n += (uint32_t)abs(wave_next(k, last) - k);
      }
    }
    crossings += n;
  }
  if (bad) atomicOr(err, kErrRange);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) crossings += __shfl_xor(crossings, d, 64);
  if (lane == 0) slots[c] = crossings > 0 ? crossings - 1 : 0;
}

// An event: the curve crosses from `cell` into the next voxel at the exact
// segment parameter nf / den (den = |d| of the face axis, nf the numerator on
// that axis), i.e. at the point xn / den with xn = P0 den + nf d.
struct Ev {
  int32_t den, nf;
  uint32_t exit_code, entry_code;   // set when face codes are requested
  int fa, exit_side;                // face axis, side of the exited voxel's face
  int planes;                       // planes crossed at this event (1 to 3)
  int32_t ncell[3];                 // the entered voxel
  uint32_t xl[3];                   // low 32 bits of the point times den (face codes requested)
};

// a * b for a, b below 2^24: two full-rate 24-bit multiplies.
__device__ inline uint64_t mul_wide24(uint32_t a, uint32_t b) {
  return (uint64_t)(a & 0xFFFFFFu) * (b & 0xFFFFFFu);
}

// Enumerates the events of segment P0 -> P1 in order: crossings of the
// planes x_a = 256 k (up iff P0_a < 256k <= P1_a, down iff P1_a < 256k <=
// P0_a), ordered by their exact parameter; equal parameters are one event
// whose face is the lowest axis's. f(ev, cell_before) per event.
template <bool kCodes, typename F>
__device__ inline void for_each_event(const int32_t P0[3], const int32_t P1[3], const GridArgs& ga,
                                      F&& f) {
  // lattice coordinates are below 2^18 (grid sides <= 1024): differences,
  // plane offsets and the numerators num_a = distance from P0 to the next
  // plane along a (below 2^19) fit 24 bits, their cross products 48
  int32_t d[3], dn[3], num[3], left[3], cell[3], sg[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    d[a] = P1[a] - P0[a];
    const int32_t c0 = P0[a] >> 8, c1 = P1[a] >> 8;
    cell[a] = c0;
    sg[a] = d[a] > 0 ? 1 : (d[a] < 0 ? -1 : 0);
    dn[a] = d[a] > 0 ? d[a] : -d[a];
    num[a] = d[a] > 0 ? 256 * (c0 + 1) - P0[a] : P0[a] - 256 * c0;
    left[a] = abs(c1 - c0);
  }
  while (left[0] + left[1] + left[2] > 0) {
    // next crossing parameter of axis a: num_a / dn_a; compared exactly by
    // cross products. grp: the axes whose next crossing is the earliest
    // (several at once make one event; its face is the lowest axis's).
    const uint64_t a01 = mul_wide24(num[0], dn[1]), a10 = mul_wide24(num[1], dn[0]);
    const uint64_t a02 = mul_wide24(num[0], dn[2]), a20 = mul_wide24(num[2], dn[0]);
    const uint64_t a12 = mul_wide24(num[1], dn[2]), a21 = mul_wide24(num[2], dn[1]);
    const bool n0 = left[0] == 0, n1 = left[1] == 0, n2 = left[2] == 0;
    bool grp[3];
    grp[0] = !n0 && (n1 || a01 <= a10) && (n2 || a02 <= a20);
    grp[1] = !n1 && (n0 || a10 <= a01) && (n2 || a12 <= a21);
    grp[2] = !n2 && (n0 || a20 <= a02) && (n1 || a21 <= a12);
    const int fa = grp[0] ? 0 : (grp[1] ? 1 : 2);
    int32_t ncell[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ncell[a] = cell[a] + (grp[a] ? sg[a] : 0);
    Ev ev;
    ev.den = fa == 0 ? dn[0] : (fa == 1 ? dn[1] : dn[2]);
    ev.nf = fa == 0 ? num[0] : (fa == 1 ? num[1] : num[2]);
    const int exit_side = (fa == 0 ? sg[0] : (fa == 1 ? sg[1] : sg[2])) > 0 ? 1 : 0;
    ev.fa = fa;
    ev.exit_side = exit_side;
    ev.planes = (int)grp[0] + (int)grp[1] + (int)grp[2];
#pragma unroll
    for (int b = 0; b < 3; ++b) ev.ncell[b] = ncell[b];
    if (kCodes) {
      uint32_t* xl = ev.xl;
      event_low(P0, d, ev.den, ev.nf, xl);
      ev.exit_code = face_code(fa, exit_side, xl, ev.den, cell, ga);
      // one plane crossed: the entered voxel has the same in-face cells, so
      // the entry face has the exit face's bins and the other side
      ev.entry_code = ev.planes == 1 ? ev.exit_code ^ 1u
                                     : face_code(fa, 1 - exit_side, xl, ev.den, ncell, ga);
    }
    f(ev, cell);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cell[a] = ncell[a];
      if (grp[a]) {
        --left[a];
        num[a] += 256;
      }
    }
  }
}

// The last event of the lanes before this one (or of earlier chunks): its point
// is voxel corner + l / den in the voxel it enters (l in [0, 256 den], below
// 2^26, so 32 bits hold it exactly); den = 0: none.
struct Last {
  uint32_t den, l[3];
  uint32_t entry;
  uint32_t attr;   // vertex attribute interpolated to the event (attribute input)
};

template <bool kAttr>
__device__ inline Last shfl_last(const Last& v, int src) {
  Last o;
  o.den = (uint32_t)__shfl((int)v.den, src, 64);
#pragma unroll
  for (int b = 0; b < 3; ++b) o.l[b] = (uint32_t)__shfl((int)v.l[b], src, 64);
  o.entry = (uint32_t)__shfl((int)v.entry, src, 64);
  o.attr = kAttr ? (uint32_t)__shfl((int)v.attr, src, 64) : 0u;
  return o;
}

// Lane `src`'s (wave-uniform) event to all lanes.
template <bool kAttr>
__device__ inline Last read_last(const Last& v, int src) {
  Last o;
  o.den = (uint32_t)__builtin_amdgcn_readlane((int)v.den, src);
#pragma unroll
  for (int b = 0; b < 3; ++b) o.l[b] = (uint32_t)__builtin_amdgcn_readlane((int)v.l[b], src);
  o.entry = (uint32_t)__builtin_amdgcn_readlane((int)v.entry, src);
  o.attr = kAttr ? (uint32_t)__builtin_amdgcn_readlane((int)v.attr, src) : 0u;
  return o;
}

// Section "Curve voxelization": a line attribute interpolated to the face
// crossing at parameter num / den of the segment whose vertices carry a0 and
// a1, rounded to the nearest integer (halves up), exactly.
__device__ inline unsigned event_attr(unsigned a0, unsigned a1, long long num, long long den) {
  const long long s = 2 * ((long long)a0 * den + ((long long)a1 - (long long)a0) * num) + den;
  return (unsigned)(s / (2 * den));
}

// Plane crossings of segment P0 -> P1 and its last event, without walking
// the events: the last event is the crossing of the largest parameter
// (exact cross-multiplied comparison; on a tie the lowest axis, the face the
// walk in for_each_event gives a simultaneous event), and it enters the
// segment's final voxel.
// (kAttr: also the vertex attribute a0 -> a1 interpolated to that event.)
template <bool kAttr>
__device__ inline uint32_t last_event(const int32_t P0[3], const int32_t P1[3],
                                      const GridArgs& ga, Last& out, unsigned a0 = 0,
                                      unsigned a1 = 0) {
  // lattice coordinates are below 2^18, so everything here is below 2^24 and
  // the cross products are exact in two 24-bit multiplies
  int32_t d[3], num[3], dn[3];
  int32_t c1[3];
  uint32_t cross = 0;
  bool has[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    d[a] = P1[a] - P0[a];
    const int32_t c0 = P0[a] >> 8;
    c1[a] = P1[a] >> 8;
    const uint32_t n = (uint32_t)abs(c1[a] - c0);
    cross += n;
    has[a] = n != 0;
    num[a] = d[a] > 0 ? 256 * c1[a] - P0[a] : P0[a] - 256 * (c1[a] + 1);
    dn[a] = d[a] > 0 ? d[a] : -d[a];
  }
  if (cross == 0) return 0;
  int fa = has[0] ? 0 : (has[1] ? 1 : 2);
  int32_t nf = num[0], den = dn[0], df = d[0];
  if (!has[0]) {
    nf = has[1] ? num[1] : num[2];
    den = has[1] ? dn[1] : dn[2];
    df = has[1] ? d[1] : d[2];
  }
#pragma unroll
  for (int a = 1; a < 3; ++a) {
    if (has[a] && mul_wide24((uint32_t)num[a], (uint32_t)den) >
                      mul_wide24((uint32_t)nf, (uint32_t)dn[a])) {
      fa = a;
      nf = num[a];
      den = dn[a];
      df = d[a];
    }
  }
  uint32_t xl[3];
  event_low(P0, d, den, nf, xl);
  out.den = (uint32_t)den;
#pragma unroll
  for (int b = 0; b < 3; ++b) out.l[b] = xl[b] - mul_lo24((uint32_t)(c1[b] << 8), (uint32_t)den);
  out.entry = face_code(fa, df > 0 ? 0 : 1, xl, den, c1, ga);
  out.attr = kAttr ? event_attr(a0, a1, nf, den) : 0u;
  return cross;
}

// Segments with events wait in a per-wave ring in LDS until 64 of them
// (or the curve's last ones) can be walked together, so the event walk runs
// on full waves instead of on the lanes of each 64-segment chunk that happen
// to cross a plane. An entry holds what the walk needs: the segment's
// lattice end points, the curve's crossings before it and the event before
// it (entry code and exact point; den = 0: none).
constexpr int kEmitRing = 128;   // >= 2 * 64 - 1 pending entries
struct EmitRing {
  int32_t p[6][kEmitRing];
  uint32_t g[kEmitRing];
  uint32_t entry[kEmitRing];
  uint32_t den[kEmitRing];
  uint32_t l[3][kEmitRing];
};

struct EmitRingAttr : EmitRing {
  uint32_t va[kEmitRing];   // a0 | a1 << 8 | (attribute at the event before) << 16
};

// LDS of a k_emit workgroup that takes ranks: a quarter of a CU's 160 KB, so four
// waves run per SIMD. Its returning atomics are what it waits for, and from six
// waves on (what its rings leave room for) they hold each other up. Whole call with
// 6, 5, 4, 3 waves: 14.2M lines in 64^3 1505, 1420, 1267, 1202 us; 19.8M in 160^3
// 1844, 1665, 1581, 1597; few lines in large grids are a little faster with more
// (3.9M in 512^3 1099, 1102, 1106, 1116).
constexpr size_t kEmitRankLds = 40960;
constexpr uint64_t kEmitFew = 1u << 19;

// Lines of every curve in curve order: the line inside a voxel runs from
// one event's entry point to the next event's exit point; it is dropped if
// the two exact points or the two quantized endpoints coincide. The line
// ending at an event goes to slot slot_off[c] + (plane crossings of the curve
// before that event) - 1; slots no line takes (dropped lines, and the extra
// numbers of an event of several planes) get the invalid mark. kRank: each
// line takes its rank in its voxel with one atomic on the histogram, and
// vox_out is the row-major voxel; else vox_out is the voxel's brick index.
// With per-vertex attributes (kAttr) every event carries the
// attribute interpolated to it; a line writes its two endpoint attributes to
// ends_out and their mean (rounded down) as its record's attribute byte.
//
// Bound by vector instructions: two exact events per segment, and a walk per
// event. Event points are therefore kept relative to their voxel, in 32 bits
// (the grid position would need 64-bit products on both sides of every
// comparison), the numbering is a DPP scan and the carried event a readlane; 81
// instead of 104 registers and 24.5 KB of LDS leave five waves per SIMD instead
// of four. At 256^3, 9.5M lines (100k x 200 curves): 360 -> 264 us.
template <bool kFloatIn, bool kAttr, bool kRank>
__global__ __launch_bounds__(kBlock, 4) void k_emit(const float* xyz, const int32_t* lat,
                                                 const int64_t* curve_off, const uint8_t* attr,
                                                 const uint8_t* vattr,
                                                 int64_t n_curves, int64_t curve_base,
                                                 const SnapArgs* sap,
                                                 GridArgs ga, const uint64_t* slot_off,
                                                 uint64_t* rec_out, uint16_t* ends_out,
                                                 uint32_t* vox_out, uint32_t* rank_out,
                                                 uint32_t* hist, uint32_t nbx,
                                                 uint32_t nbxy) {
  using Ring = std::conditional_t<kAttr, EmitRingAttr, EmitRing>;
  __shared__ Ring rings[kWavesPerBlock];
  const int lane = threadIdx.x & 63;
  const SnapArgs sa = kFloatIn ? *sap : SnapArgs{};
  const int64_t c = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (c >= n_curves) return;  // wave-uniform
  Ring& Q = rings[threadIdx.x >> 6];
  const int64_t v0 = curve_off[c], v1 = curve_off[c + 1];
  const uint64_t w0 = slot_off[c], w_end = slot_off[c + 1];
  const uint64_t hi_bits =
      ((uint64_t)(attr ? attr[c] : 255) << 32) | ((uint64_t)((curve_base + c) & 0xFFFFFF) << 40);
  const int64_t gx = ga.g[0], gxy = (int64_t)ga.g[0] * ga.g[1];
  const unsigned long long below = (1ull << lane) - 1ull;

  // walks the first `count` ring entries from `head`, one per lane
  auto walk = [&](uint32_t head, uint32_t count) {
    // ring writes by other lanes of this wave precede these reads (LDS
    // operations of a wave complete in order; the fence keeps the compiler
    // from moving them)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if ((uint32_t)lane >= count) return;
    const uint32_t k = (head + (uint32_t)lane) & (kEmitRing - 1);
    const int32_t P0[3] = {Q.p[0][k], Q.p[1][k], Q.p[2][k]};
    const int32_t P1[3] = {Q.p[3][k], Q.p[4][k], Q.p[5][k]};
    const uint32_t bden = Q.den[k];
    const uint32_t bl[3] = {Q.l[0][k], Q.l[1][k], Q.l[2][k]};
    uint64_t g = Q.g[k];
    bool has_prev = bden != 0, first = true;
    uint32_t prev_entry = Q.entry[k];
    uint32_t va = 0u;
    if constexpr (kAttr) va = Q.va[k];
    uint32_t prev_attr = va >> 16;
    for_each_event<true>(P0, P1, ga, [&](const Ev& ev, const int32_t* cell) {
      const uint32_t ea = kAttr ? event_attr(va & 0xFFu, (va >> 8) & 0xFFu, ev.nf, ev.den) : 0u;
      const uint64_t w = w0 + (g - 1);
      for (int k = 1; k < ev.planes; ++k)
        if (w + k < w_end) vox_out[w + k] = LS_INVALID_VOXEL;
      if (has_prev) {
        if (w < w_end) {
          // events of one segment have distinct parameters, so only its
          // first event can coincide with the event before it
          bool same = false;
          if (first) {
            // both points relative to this voxel: equal iff l / den agree on
            // every axis; the low halves of the cross products settle almost
            // every case
            const uint32_t den = (uint32_t)ev.den;
            uint32_t el[3], diff = 0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
              el[b] = ev.xl[b] - mul_lo24((uint32_t)(cell[b] << 8), den);
              diff |= bl[b] * den ^ el[b] * bden;
            }
            if (diff == 0u) {
              same = true;
#pragma unroll
              for (int b = 0; b < 3; ++b)
                same = same && (uint64_t)bl[b] * den == (uint64_t)el[b] * bden;
            }
          }
          if (same || prev_entry == ev.exit_code) {
            vox_out[w] = LS_INVALID_VOXEL;
          } else {
            uint64_t hb = hi_bits;
            if (kAttr) {
              hb = (hb & ~(0xFFull << 32)) | ((uint64_t)((prev_attr + ea) >> 1) << 32);
              ends_out[w] = (uint16_t)(prev_attr | (ea << 8));
            }
            rec_out[w] = (uint64_t)prev_entry | ((uint64_t)ev.exit_code << 15) | hb;
            if (kRank) {
              const uint32_t vid = (uint32_t)(cell[0] + gx * cell[1] + gxy * cell[2]);
              vox_out[w] = vid;
              rank_out[w] = atomicAdd(hist + vid, 1u);
            } else {
              vox_out[w] = brick_index(cell[0], cell[1], cell[2], nbx, nbxy);
            }
          }
        }
      }
      has_prev = true;
      first = false;
      prev_entry = ev.entry_code;
      prev_attr = ea;
      g += (uint64_t)ev.planes;
    });
  };

  Last carry{};
  uint64_t g0 = 0;       // crossings of the curve before this chunk
  uint32_t q_head = 0, q_n = 0;   // ring state (wave-uniform)
  for (int64_t s0 = v0; s0 + 1 < v1; s0 += 64) {
    const int64_t i = s0 + lane;
    const bool valid = i + 1 < v1;
    int32_t P0[3] = {0, 0, 0}, P1[3] = {0, 0, 0};
    if (valid) {
      load_vertex<kFloatIn>(xyz, lat, i, sa, P0);
      load_vertex<kFloatIn>(xyz, lat, i + 1, sa, P1);
    }
    // plane crossings and the last event. Lines are numbered by crossings
    // (an event of k simultaneous planes uses k numbers), so the numbering
    // needs no walk; the unused numbers stay invalid slots.
    uint32_t e = 0;
    Last mine{};
    uint32_t a01 = 0;
    if (kAttr && valid) a01 = (uint32_t)vattr[i] | ((uint32_t)vattr[i + 1] << 8);
    if (valid) e = last_event<kAttr>(P0, P1, ga, mine, a01 & 0xFFu, a01 >> 8);
    // exclusive prefix sum of the crossing counts
    uint32_t total;
    const uint32_t base = wave_excl_scan(e, total);
    // the last event strictly before this lane: that of the highest lane below
    // it with one
    const unsigned long long em = __ballot(mine.den != 0u);
    const unsigned long long eb = em & below;
    const int prev_src = eb ? 63 - __clzll((long long)eb) : -1;
    Last before = shfl_last<kAttr>(mine, prev_src >= 0 ? prev_src : 0);
    if (prev_src < 0) before = carry;
    // queue the segments with events
    const bool act = valid && e > 0;
    const unsigned long long am = __ballot(act);
    if (act) {
      const uint32_t k = (q_head + q_n + (uint32_t)__popcll(am & below)) & (kEmitRing - 1);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        Q.p[a][k] = P0[a];
        Q.p[3 + a][k] = P1[a];
      }
      Q.g[k] = (uint32_t)(g0 + base);
      Q.entry[k] = before.entry;
      Q.den[k] = before.den;
#pragma unroll
      for (int b = 0; b < 3; ++b) Q.l[b][k] = before.l[b];
      if constexpr (kAttr) Q.va[k] = a01 | (before.attr << 16);
    }
    q_n += (uint32_t)__popcll(am);
    // carry the chunk's last event
    if (em) carry = read_last<kAttr>(mine, 63 - __builtin_clzll(em));
    g0 += total;
    if (q_n >= 64) {
      walk(q_head, 64);
      q_head = (q_head + 64) & (kEmitRing - 1);
      q_n -= 64;
    }
  }
  if (q_n > 0) walk(q_head, q_n);
}

// Each emitted line e of voxel v goes to slot offsets[v] + rank[e] of its
// voxel's range, as the pair (v, e): one 8-byte write, so the rank pass reads
// the voxel with the index instead of gathering it.
__global__ __launch_bounds__(kBlock) void k_scatter(const uint32_t* vox, const uint32_t* rank,
                                                    int64_t n_slots, const uint32_t* offsets,
                                                    uint64_t* idx) {
  int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n_slots) return;
  uint32_t v = vox[e];
  if (v == LS_INVALID_VOXEL) return;
  idx[offsets[v] + rank[e]] = ((uint64_t)v << 32) | (uint32_t)e;
}

// Each CSR slot p holds some emitted line e of voxel v; its final position is
// offsets[v] + (number of lines of v emitted before e). A block handles 256
// consecutive slots; the lists overlapping them (slots are grouped by voxel,
// so they span [lo of the first slot's voxel, hi of the last's)) are staged
// in LDS when they fit, else counted from memory.
constexpr int kRankLds = 4096;

__global__ __launch_bounds__(kBlock) void k_rank(const uint64_t* idx, const uint64_t* rec,
                                                 const uint16_t* ends_in, int64_t n_records,
                                                 const uint32_t* offsets, uint64_t* records,
                                                 uint16_t* ends) {
  __shared__ uint32_t s_idx[kRankLds];
  __shared__ uint32_t s_range[2];
  const int64_t p0 = (int64_t)blockIdx.x * kBlock;
  const int64_t p = p0 + threadIdx.x;
  const int64_t n_here = n_records - p0 < kBlock ? n_records - p0 : kBlock;
  uint32_t e = 0, lo = 0, hi = 0;
  if (p < n_records) {
    const uint64_t ve = idx[p];
    e = (uint32_t)ve;
    const uint32_t v = (uint32_t)(ve >> 32);
    lo = offsets[v];
    hi = offsets[v + 1];
  }
  if (threadIdx.x == 0) s_range[0] = lo;
  if ((int64_t)threadIdx.x == n_here - 1) s_range[1] = hi;
  __syncthreads();
  const uint32_t blo = s_range[0], bhi = s_range[1];
  const bool staged = bhi - blo <= (uint32_t)kRankLds;   // block-uniform
  if (staged)
    for (uint32_t q = blo + threadIdx.x; q < bhi; q += kBlock) s_idx[q - blo] = (uint32_t)idx[q];
  __syncthreads();
  if (p >= n_records) return;
  uint32_t r = 0;
  if (staged) {
    for (uint32_t q = lo; q < hi; ++q) r += s_idx[q - blo] < e;
  } else {
    for (uint32_t q = lo; q < hi; ++q) r += (uint32_t)idx[q] < e;
  }
  records[lo + r] = rec[e];
  if (ends) ends[lo + r] = ends_in[e];
}

// Occupancy mask per 4^3 macro cell: bit (x & 3) + 4 (y & 3) + 16 (z & 3) of
// the cell's 64-bit word is set when that voxel's list is not empty. One
// load tells the ray caster which voxels of the macro cell it can skip
// (a zero word: the whole macro cell). The same pass counts the non-empty
// voxels and the longest list (wave and block reduction, one atomic each per
// workgroup; these, at some 10 ns each on one line, bound it from 128^3 on, so
// more lanes per cell only lose there: 128^3 106 -> 112 us for the whole call
// with four). Grids of up to kOccFew cells leave the chip idle with a lane per
// cell: four lanes share one (64^3: 123 -> 118 us for the whole call). Rows
// that end at a side that is no multiple of 4 are five clamped loads issued
// together (201x97x130: 178 -> 170 us, against a test and two loads per voxel).
constexpr int64_t kOccFew = 8192;

template <int kLanes>
__global__ __launch_bounds__(kBlock) void k_occupancy(const uint32_t* offsets, GridArgs ga,
                                                      int32_t mx, int32_t my, int32_t mz,
                                                      unsigned long long* occ,
                                                      unsigned long long* nonempty,
                                                      unsigned int* max_list) {
  __shared__ unsigned long long s_ne[kBlock / 64];
  __shared__ unsigned s_mx[kBlock / 64];
  constexpr int kCells = 64 / kLanes, kRows = 16 / kLanes;   // per wave, per lane
  const int lane = threadIdx.x & 63, part = lane / kCells;
  const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int64_t m = wave * kCells + (lane & (kCells - 1));
  const int64_t nm = (int64_t)mx * my * mz;
  unsigned long long bits = 0;
  unsigned mxl = 0;
  if (m < nm) {
    const int32_t bx = (int32_t)(m % mx), by = (int32_t)((m / mx) % my),
                  bz = (int32_t)(m / ((int64_t)mx * my));
    const int w = ga.g[0] - 4 * bx;   // voxels of the cell's rows below the side
#pragma unroll 4
    for (int k = 0; k < kRows; ++k) {
      const int r = part * kRows + k;
      const int32_t y = 4 * by + (r & 3), z = 4 * bz + (r >> 2);
      if (y >= ga.g[1] || z >= ga.g[2]) continue;
      const int64_t v = 4 * (int64_t)bx + (int64_t)ga.g[0] * (y + (int64_t)ga.g[1] * z);
      uint32_t o[5];
      if ((ga.g[0] & 3) == 0) {
        // whole macro cells along x: the row of 4 voxels is one aligned
        // 16-byte load of their offsets plus the next row start
        const uint4 a = *reinterpret_cast<const uint4*>(offsets + v);
        o[0] = a.x;
        o[1] = a.y;
        o[2] = a.z;
        o[3] = a.w;
        o[4] = offsets[v + 4];
      } else {
#pragma unroll
        for (int c = 0; c < 5; ++c) o[c] = offsets[v + (c < w ? c : w)];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const unsigned n = o[c + 1] - o[c];
        if (n > 0) bits |= 1ull << (4 * r + c);
        mxl = n > mxl ? n : mxl;
      }
    }
  }
  unsigned long long ne = (unsigned long long)__popcll(bits);
#pragma unroll
  for (int d = kCells; d < 64; d <<= 1) bits |= __shfl_xor(bits, d, 64);
  if (part == 0 && m < nm) occ[m] = bits;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    ne += __shfl_xor(ne, d, 64);
    const unsigned o = __shfl_xor(mxl, d, 64);
    mxl = o > mxl ? o : mxl;
  }
  if ((threadIdx.x & 63) == 0) {
    s_ne[threadIdx.x >> 6] = ne;
    s_mx[threadIdx.x >> 6] = mxl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) {
      ne += s_ne[w];
      mxl = s_mx[w] > mxl ? s_mx[w] : mxl;
    }
    if (ne) atomicAdd(nonempty, ne);
    if (mxl) atomicMax(max_list, mxl);
  }
}


// ---------------------------------------------------------------------------
// Lists by bricks. The emitted lines lie in slot order (curve by curve), and
// consecutive slots of a curve mostly share a brick of 8^3 voxels. A run is a
// maximal sequence of consecutive slots of one brick within 64 slots.
//   k_runs<false>  counts runs per brick (one atomic per run), in kReps copies
//                  of the counters: workgroup b counts in copy b mod kReps, so
//                  a busy brick's counter is not one address for the chip
//   scan           run offsets, copy by copy
//   k_runs<true>   writes each run (first slot, length) to its brick's list,
//                  one list per copy
//   k_brick_count  workgroup per 4 bricks along x: voxel histogram in LDS,
//                  written to the offsets array (counts), with the occupancy
//                  words and list statistics of its macro cells; lists the
//                  bricks too large for k_brick_fill as (brick, voxel range),
//                  their voxels of many lines by themselves (k_long_rank)
//   scan           voxel offsets (CSR)
//   k_brick_fill   workgroup per brick (k_brick_items: per listed range):
//                  places the slots of its lines by voxel in LDS, ranks each
//                  voxel's slots and gathers the records into the CSR, whose
//                  rows of 8 voxels it fills by itself
// One atomic and one scattered write per run (11 lines at 512^3) replace, per
// line, the rank atomic, the scattered 8-byte pair, its reading back and the
// scattered gather. The fills are bound by the latency of a brick's serial
// stages (offsets, runs, slots, records), so each keeps kAhead loads per lane
// in flight; the figures stand at kBrickMinVoxels.
constexpr uint32_t kBrickVox = 1u << kRunShift;

struct BrickGrid {
  int32_t g[3];          // voxel grid (row-major ids)
  int32_t m[3];          // macro-cell grid (4^3 voxels)
  uint32_t nk[3];        // blocks of 4 x 4 x 2 bricks
  uint32_t n;            // bricks, those of partial blocks included
  // room for items and for the long voxels after them (pointers of their own made
  // every workgroup of k_brick_count wait for its arguments: 548 -> 580 us at 512^3)
  uint32_t item_max, long_max;
  // coordinates of brick b
  __device__ inline void brick(uint32_t b, uint32_t c[3]) const {
    const uint32_t k = b >> 5;
    c[0] = 4 * (k % nk[0]) + (b & 3u);
    c[1] = 4 * ((k / nk[0]) % nk[1]) + (b >> 2 & 3u);
    c[2] = 2 * (k / (nk[0] * nk[1])) + (b >> 4 & 1u);
  }
};

constexpr uint32_t kReps = 32;   // a power of two, at most 64

template <bool kPlace>
__global__ __launch_bounds__(kBlock) void k_runs(const uint32_t* __restrict__ vox, int64_t n_slots,
                                                 uint32_t n_bricks, uint32_t* brick,
                                                 uint32_t* cursor, unsigned long long* runs) {
  const int lane = threadIdx.x & 63;
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t v = e < n_slots ? vox[e] : LS_INVALID_VOXEL;
  const bool ok = v != LS_INVALID_VOXEL;
  const uint32_t b = ok ? v >> kRunShift : LS_INVALID_VOXEL;
  const uint32_t p = __shfl_up(b, 1, 64);
  const bool start = ok && (lane == 0 || p != b);
  // a run ends before the next start or the next invalid slot
  const unsigned long long stop = __ballot(start || !ok);
  if (!start) return;
  const unsigned long long rest = lane < 63 ? stop >> (lane + 1) : 0ull;
  const uint32_t len = rest ? (uint32_t)__builtin_ctzll(rest) + 1u : 64u - (uint32_t)lane;
  const size_t c = (size_t)(blockIdx.x % kReps) * n_bricks + b;
  if (kPlace) {
    const uint32_t pos = brick[c] + atomicAdd(cursor + c, 1u);
    runs[pos] = (unsigned long long)len << 32 | (uint32_t)e;
  } else {
    atomicAdd(brick + c, 1u);
  }
}

// Lines of a brick that k_brick_fill places in LDS (18 KB with the voxel
// tables: 8 workgroups per CU), and that one listed range may hold.
constexpr uint32_t kFillCap = 2048;
constexpr uint32_t kItemCap = 8192;
constexpr uint32_t kLongMin = 1024;   // lines of a voxel that goes by itself (k_long_rank)
constexpr int kGroupBricks = 4;      // bricks per k_brick_count workgroup, along x
constexpr int kCountThreads = 512;
constexpr int kItemThreads = 1024;

// A range [v0, v1) of the voxels of a brick.
struct BrickItem {
  uint32_t brick;
  uint16_t v0, v1;
};

// The run lists of bricks [b, b + nb) (consecutive): one segment of
// `runs` per copy of the counters.
struct RunLists {
  uint32_t pre[kReps + 1];   // runs before each segment
  uint32_t at[kReps];        // the segment's first run
};

// Filled by the workgroup's first threads; a barrier follows in the caller.
__device__ inline void run_lists(const uint32_t* __restrict__ brick, uint32_t n_bricks, uint32_t b,
                                 uint32_t nb, RunLists& L) {
  if (threadIdx.x < 64) {
    const uint32_t k = threadIdx.x;
    const uint32_t lo = k < kReps ? brick[(size_t)k * n_bricks + b] : 0u;
    const uint32_t hi = k < kReps ? brick[(size_t)k * n_bricks + b + nb] : 0u;
    const uint32_t inc = wave_incl_sum(hi - lo);
    if (k < kReps) {
      L.pre[k + 1] = inc;
      L.at[k] = lo;
    }
    if (k == 0) L.pre[0] = 0u;
  }
}

// Visits the lines of L's runs: f(slot, brick index of its voxel). A wave
// takes up to 64 runs at a time, numbers their lines by a prefix sum and deals
// them to its lanes, kAhead x 64 lines' loads in flight. own: 64 words of LDS
// for this wave.
constexpr int kAhead = 4;

template <int kThreads, typename F>
__device__ inline void for_each_line(const unsigned long long* __restrict__ runs,
                                     const RunLists& L, const uint32_t* __restrict__ vox,
                                     uint32_t* own, F&& f) {
  constexpr uint32_t kWaves = kThreads / 64;
  const uint32_t lane = (uint32_t)wave_lane();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.pre[kReps]);
  const uint32_t take = min(64u, (n + kWaves - 1) / kWaves);
  for (uint32_t r0 = wave * take; r0 < n; r0 += kWaves * take) {
    unsigned long long run = 0;
    if (lane < take && r0 + lane < n) {
      const uint32_t r = r0 + lane;
      uint32_t k = 0;   // last segment with pre <= r
#pragma unroll
      for (uint32_t j = kReps / 2; j >= 1; j >>= 1)
        if (L.pre[k + j] <= r) k += j;
      run = runs[L.at[k] + (r - L.pre[k])];
    }
    const uint32_t len = (uint32_t)(run >> 32);
    uint32_t total;
    const uint32_t P = wave_excl_scan(len, total);
    const uint32_t rel = (uint32_t)run - P;   // slot of line w: w + rel of its run
    for (uint32_t base = 0; base < total; base += 64 * kAhead) {
      uint32_t e[kAhead], v[kAhead];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        const uint32_t w0 = base + 64 * j;
        e[j] = v[j] = LS_INVALID_VOXEL;
        if (w0 < total) {   // wave-uniform
          const int o = chunk_owner(own, P, len, w0);
          const uint32_t s = w0 + lane + (uint32_t)__shfl((int)rel, o, 64);
          if (w0 + lane < total) {
            e[j] = s;
            v[j] = vox[s];
          }
        }
      }
#pragma unroll
      for (int j = 0; j < kAhead; ++j)
        if (v[j] != LS_INVALID_VOXEL) f(e[j], v[j]);
    }
  }
}

__global__ __launch_bounds__(kCountThreads) void k_brick_count(
    const uint32_t* __restrict__ brick, const unsigned long long* __restrict__ runs,
    const uint32_t* __restrict__ vox, BrickGrid bg, uint32_t* counts, unsigned long long* occ,
    unsigned long long* part, uint32_t* n_items, BrickItem* items) {
  __shared__ uint32_t hist[kGroupBricks * kBrickVox];
  __shared__ uint32_t s_ne, s_mx, own[kCountThreads], s_lines[kGroupBricks];
  __shared__ RunLists lists;
  const uint32_t b0 = blockIdx.x * kGroupBricks;
  constexpr uint32_t nb = kGroupBricks;
  uint32_t bc[3];
  bg.brick(b0, bc);
  const uint32_t bx0 = bc[0], by = bc[1], bz = bc[2];
  if (8 * bx0 >= (uint32_t)bg.g[0] || 8 * by >= (uint32_t)bg.g[1] || 8 * bz >= (uint32_t)bg.g[2]) {
    if (threadIdx.x == 0) part[blockIdx.x] = 0ull;
    return;   // a partial block's bricks outside the grid
  }
  for (uint32_t i = threadIdx.x; i < kGroupBricks * kBrickVox; i += kCountThreads) hist[i] = 0u;
  if (threadIdx.x == 0) s_ne = s_mx = 0u;
  if (threadIdx.x < kGroupBricks) s_lines[threadIdx.x] = 0u;
  run_lists(brick, bg.n, b0, nb, lists);
  __syncthreads();
  const uint32_t base = b0 << kRunShift;
  for_each_line<kCountThreads>(runs, lists, vox, own + (threadIdx.x & ~63u),
                               [&](uint32_t, uint32_t v) { atomicAdd(hist + (v - base), 1u); });
  __syncthreads();
  // counts, in rows of up to 32 voxels
  for (uint32_t i = threadIdx.x; i < kGroupBricks * kBrickVox; i += kCountThreads) {
    const uint32_t xx = i & 31u, row = i >> 5, y = 8 * by + (row & 7u), z = 8 * bz + (row >> 3);
    const uint32_t x = 8 * bx0 + xx;
    if (x < (uint32_t)bg.g[0] && y < (uint32_t)bg.g[1] && z < (uint32_t)bg.g[2])
      counts[x + (int64_t)bg.g[0] * (y + (int64_t)bg.g[1] * z)] =
          hist[(xx >> 3) << kRunShift | (xx & 7u) | row << 3];
  }
  // a wave per macro cell: lane = voxel, the ballot is its occupancy word
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t ne = 0, mx = 0;
  for (uint32_t q = threadIdx.x >> 6; q < 8 * nb; q += kCountThreads / 64) {
    const uint32_t lx = (lane & 3u) | (q & 1u) << 2, ly = (lane >> 2 & 3u) | (q & 2u) << 1,
                   lz = (lane >> 4) | (q & 4u);
    const uint32_t n = hist[(q >> 3) << kRunShift | lx | ly << 3 | lz << 6];
    const unsigned long long w = __ballot(n != 0u);
    const uint32_t cx = 2 * (bx0 + (q >> 3)) + (q & 1u), cy = 2 * by + (q >> 1 & 1u),
                   cz = 2 * bz + (q >> 2 & 1u);
    if (lane == 0 && cx < (uint32_t)bg.m[0] && cy < (uint32_t)bg.m[1] && cz < (uint32_t)bg.m[2])
      occ[cx + (int64_t)bg.m[0] * (cy + (int64_t)bg.m[1] * cz)] = w;
    ne += (uint32_t)__popcll(w);
    mx = max(mx, n);
    const uint32_t lines = wave_incl_sum(n);
    if (lane == 63 && lines) atomicAdd(s_lines + (q >> 3), lines);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) mx = max(mx, (uint32_t)__shfl_xor(mx, d, 64));
  if (lane == 0 && ne) {
    atomicAdd(&s_ne, ne);
    atomicMax(&s_mx, mx);
  }
  __syncthreads();
  // bricks beyond k_brick_fill's room, cut into voxel ranges of at most kItemCap
  // lines; voxels of more than kLongMin are listed by themselves
  if (threadIdx.x < nb) {
    const uint32_t b = b0 + threadIdx.x, n = s_lines[threadIdx.x];
    if (n > kFillCap && n <= kItemCap && s_mx <= kLongMin) {
      items[atomicAdd(n_items, 1u)] = BrickItem{b, 0, (uint16_t)kBrickVox};
    } else if (n > kFillCap) {
      const uint32_t* h = hist + threadIdx.x * kBrickVox;
      uint32_t v0 = 0, sum = 0, n_long = 0;
      auto cut = [&](uint32_t v) {
        if (sum > 0) items[atomicAdd(n_items, 1u)] = BrickItem{b, (uint16_t)v0, (uint16_t)v};
        v0 = v;
        sum = 0;
      };
      // one lane's chain, at the end of the kernel: eight voxels at a time (one by one,
      // 100k x 200 curves in 256^3 94 us for the kernel, so 69)
      for (uint32_t v8 = 0; v8 < kBrickVox; v8 += 8) {
        uint32_t all = 0, most = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          all += h[v8 + j];
          most = max(most, h[v8 + j]);
        }
        if (most <= kLongMin && sum + all <= kItemCap) {
          sum += all;
          continue;
        }
#pragma unroll 1
        for (uint32_t v = v8; v < v8 + 8; ++v) {
          const uint32_t c = h[v];
          if (c > kLongMin || sum + c > kItemCap) cut(v);
          if (c > kLongMin) {
            items[bg.item_max + atomicAdd(n_items + 1, 1u)] =
                BrickItem{b, (uint16_t)v, (uint16_t)(v + 1)};
            ++n_long;
            v0 = v + 1;
          } else {
            sum += c;
          }
        }
      }
      cut(kBrickVox);
      if (n_long)
        reinterpret_cast<uint32_t*>(items + bg.item_max + bg.long_max)[atomicAdd(n_items + 2, 1u)] =
            b;
    }
  }
  if (threadIdx.x == 0)
    part[blockIdx.x] = (unsigned long long)s_mx << 32 | s_ne;
}

// What the host reads once the lists are counted.
struct ListHeader {
  unsigned long long nonempty, max_list;
  uint32_t n_records, n_items, n_longs, n_long_bricks;
};

// Sums k_brick_count's list statistics (non-empty voxels, longest list; the two
// words after the occupancy words) and gathers the header.
__global__ __launch_bounds__(1024) void k_list_stats(const unsigned long long* __restrict__ part,
                                                     int64_t n, const uint32_t* n_records,
                                                     const uint32_t* n_items,
                                                     unsigned long long* stats, ListHeader* out) {
  __shared__ unsigned long long s_ne;
  __shared__ unsigned s_mx;
  if (threadIdx.x == 0) {
    s_ne = 0ull;
    s_mx = 0u;
  }
  __syncthreads();
  unsigned long long ne = 0;
  unsigned mx = 0;
  for (int64_t i = threadIdx.x; i < n; i += 1024) {
    const unsigned long long p = part[i];
    ne += (uint32_t)p;
    mx = max(mx, (unsigned)(p >> 32));
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    ne += __shfl_xor(ne, d, 64);
    mx = max(mx, (unsigned)__shfl_xor(mx, d, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&s_ne, ne);
    atomicMax(&s_mx, mx);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    stats[0] = s_ne;
    stats[1] = s_mx;
    *out = ListHeader{s_ne, s_mx, *n_records, n_items[0], n_items[1], n_items[2]};
  }
}

// The lines of voxels [v0, v1) of brick b, at most kCap: slots placed by
// voxel in LDS, ranked within the voxel by slot (= emission order), records
// gathered into the CSR. lds: kCap slots, kCap voxels (16 bit).
template <int kThreads, uint32_t kCap>
__device__ inline void brick_fill(const unsigned long long* __restrict__ runs,
                                  const uint32_t* __restrict__ vox,
                                  const uint64_t* __restrict__ rec,
                                  const uint16_t* __restrict__ ends_in, const BrickGrid& bg,
                                  const uint32_t* __restrict__ offsets, uint32_t b, uint32_t v0,
                                  uint32_t v1, uint32_t* s_e, uint16_t* s_v, uint32_t* s_off,
                                  uint32_t* s_lo, uint32_t* s_cur, uint32_t* own,
                                  RunLists& lists, uint64_t* __restrict__ records,
                                  uint16_t* __restrict__ ends) {
  static_assert(kThreads >= 64 && kBrickVox % 64 == 0, "scan by one wave");
  uint32_t bc[3];
  bg.brick(b, bc);
  for (uint32_t i = threadIdx.x; i < kBrickVox; i += kThreads) {
    const uint32_t x = 8 * bc[0] + (i & 7u), y = 8 * bc[1] + (i >> 3 & 7u), z = 8 * bc[2] + (i >> 6);
    uint32_t lo = 0, n = 0;
    if (i >= v0 && i < v1 && x < (uint32_t)bg.g[0] && y < (uint32_t)bg.g[1] &&
        z < (uint32_t)bg.g[2]) {
      const int64_t v = x + (int64_t)bg.g[0] * (y + (int64_t)bg.g[1] * z);
      lo = offsets[v];
      n = offsets[v + 1] - lo;
    }
    s_off[i] = lo;
    s_lo[i] = n;
    s_cur[i] = 0u;
  }
  __syncthreads();
  // exclusive scan of the counts: the first wave, 8 voxels per lane
  if (threadIdx.x < 64) {
    constexpr int kPer = kBrickVox / 64;
    uint32_t c[kPer], sum = 0, total;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      c[k] = s_lo[threadIdx.x * kPer + k];
      sum += c[k];
    }
    uint32_t pre = wave_excl_scan(sum, total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      s_lo[threadIdx.x * kPer + k] = pre;
      pre += c[k];
    }
    if (threadIdx.x == 0) s_lo[kBrickVox] = total;
  }
  __syncthreads();
  const uint32_t n = s_lo[kBrickVox];
  if (n > kCap) return;   // a listed brick
  for_each_line<kThreads>(runs, lists, vox, own, [&](uint32_t e, uint32_t bv) {
    const uint32_t v = bv & (kBrickVox - 1);
    if (v < v0 || v >= v1) return;
    const uint32_t p = s_lo[v] + atomicAdd(s_cur + v, 1u);
    s_e[p] = e;
    s_v[p] = (uint16_t)v;
  });
  __syncthreads();
  // kAhead lines per thread: their ranks, then their loads, then their writes
  for (uint32_t p0 = threadIdx.x; p0 < n; p0 += kAhead * kThreads) {
    uint32_t e[kAhead], w[kAhead];
    uint64_t r[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const uint32_t p = p0 + j * kThreads;
      if (p < n) {
        const uint32_t v = s_v[p], hi = s_lo[v + 1];
        e[j] = s_e[p];
        w[j] = s_off[v];
        r[j] = rec[e[j]];
        for (uint32_t q = s_lo[v]; q < hi; ++q) w[j] += s_e[q] < e[j];
      }
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      if (p0 + j * kThreads < n) {
        records[w[j]] = r[j];
        if (ends) ends[w[j]] = ends_in[e[j]];
      }
    }
  }
}

// Bricks of up to kFillCap lines, a workgroup each; XCD x (= block mod 8) takes
// a contiguous run of bricks, so the rows that neighbouring bricks fill meet in
// one L2.
__global__ __launch_bounds__(kBlock) void k_brick_fill(
    const uint32_t* __restrict__ brick, const unsigned long long* __restrict__ runs,
    const uint32_t* __restrict__ vox, const uint64_t* __restrict__ rec,
    const uint16_t* __restrict__ ends_in, BrickGrid bg, const uint32_t* __restrict__ offsets,
    uint64_t* records, uint16_t* ends) {
  __shared__ uint32_t s_e[kFillCap], s_off[kBrickVox], s_lo[kBrickVox + 1], s_cur[kBrickVox];
  __shared__ uint16_t s_v[kFillCap];
  __shared__ uint32_t own[kBlock];
  __shared__ RunLists lists;
  const uint32_t per = (bg.n + 7u) / 8u, b = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= per || b >= bg.n) return;
  run_lists(brick, bg.n, b, 1u, lists);
  __syncthreads();
  if (lists.pre[kReps] == 0u) return;
  brick_fill<kBlock, kFillCap>(runs, vox, rec, ends_in, bg, offsets, b, 0u, kBrickVox, s_e, s_v,
                               s_off, s_lo, s_cur, own + (threadIdx.x & ~63u), lists, records,
                               ends);
}

// The listed voxel ranges of larger bricks, dealt over the grid.
constexpr size_t kItemLds = kItemCap * (sizeof(uint32_t) + sizeof(uint16_t));

__global__ __launch_bounds__(kItemThreads) void k_brick_items(
    const uint32_t* __restrict__ brick, const unsigned long long* __restrict__ runs,
    const uint32_t* __restrict__ vox, const uint64_t* __restrict__ rec,
    const uint16_t* __restrict__ ends_in, BrickGrid bg, const uint32_t* __restrict__ offsets,
    const uint32_t* __restrict__ n_items, const BrickItem* __restrict__ items, uint64_t* records,
    uint16_t* ends) {
  extern __shared__ uint32_t item_lds[];
  __shared__ uint32_t s_off[kBrickVox], s_lo[kBrickVox + 1], s_cur[kBrickVox];
  __shared__ uint32_t own[kItemThreads];
  __shared__ RunLists lists;
  uint16_t* s_v = reinterpret_cast<uint16_t*>(item_lds + kItemCap);
  const uint32_t n = *n_items;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const BrickItem it = items[i];
    run_lists(brick, bg.n, it.brick, 1u, lists);
    brick_fill<kItemThreads, kItemCap>(runs, vox, rec, ends_in, bg, offsets, it.brick, it.v0,
                                       it.v1, item_lds, s_v, s_off, s_lo, s_cur,
                                       own + (threadIdx.x & ~63u), lists, records, ends);
    __syncthreads();
  }
}

// Voxels of more than kLongMin lines: a workgroup per brick collects their slots in
// the order it meets them (idx, at the voxel's places in the CSR), then a thread per
// line counts the lines of smaller slots, from LDS, over the whole device where
// k_brick_items would compare them in one workgroup. Whole calls without bricks and
// with them, in us: 26.5M lines in 256^3 with 4 voxels of 9000 3094 and 1414, 44M
// with 4 of 60k 10123 and 2858; 9000 curves from one point, 10M lines (voxels of up
// to 1600) 1012 and, with kLongMin 512, 1024, 2048, 8192, 815, 852, 1132, 1083; 400
// seeds on a line of 1500 curves, 66M 6257 and 5510, 5388, 5351, 5382.
constexpr uint32_t kLongTile = 4096;
constexpr uint32_t kLongLaunch = 32768;   // voxels per launch (grid limit)

// The voxel of a long item and its lines [lo, lo + n).
__device__ inline void long_voxel(const BrickGrid& bg, const BrickItem& it,
                                  const uint32_t* __restrict__ offsets, uint32_t& lo, uint32_t& n) {
  uint32_t bc[3];
  bg.brick(it.brick, bc);
  const uint32_t i = it.v0, x = 8 * bc[0] + (i & 7u), y = 8 * bc[1] + (i >> 3 & 7u),
                 z = 8 * bc[2] + (i >> 6);
  const int64_t v = x + (int64_t)bg.g[0] * (y + (int64_t)bg.g[1] * z);
  lo = offsets[v];
  n = offsets[v + 1] - lo;
}

__global__ __launch_bounds__(kItemThreads) void k_long_gather(
    const uint32_t* __restrict__ brick, const unsigned long long* __restrict__ runs,
    const uint32_t* __restrict__ vox, BrickGrid bg, const uint32_t* __restrict__ offsets,
    const uint32_t* __restrict__ long_bricks, uint32_t* __restrict__ idx) {
  __shared__ uint32_t own[kItemThreads], next[kBrickVox];   // next place; none: not long
  __shared__ RunLists lists;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const uint32_t b = long_bricks[blockIdx.x];
  uint32_t bc[3];
  bg.brick(b, bc);
  for (uint32_t i = threadIdx.x; i < kBrickVox; i += kItemThreads) {
    const uint32_t x = 8 * bc[0] + (i & 7u), y = 8 * bc[1] + (i >> 3 & 7u), z = 8 * bc[2] + (i >> 6);
    next[i] = kNone;
    if (x < (uint32_t)bg.g[0] && y < (uint32_t)bg.g[1] && z < (uint32_t)bg.g[2]) {
      const int64_t v = x + (int64_t)bg.g[0] * (y + (int64_t)bg.g[1] * z);
      const uint32_t lo = offsets[v];
      if (offsets[v + 1] - lo > kLongMin) next[i] = lo;
    }
  }
  run_lists(brick, bg.n, b, 1u, lists);
  __syncthreads();
  for_each_line<kItemThreads>(runs, lists, vox, own + (threadIdx.x & ~63u),
                              [&](uint32_t e, uint32_t bv) {
                                const uint32_t v = bv & (kBrickVox - 1);
                                if (next[v] != kNone) idx[atomicAdd(next + v, 1u)] = e;
                              });
}

__global__ __launch_bounds__(kBlock) void k_long_rank(
    const uint32_t* __restrict__ idx, const uint64_t* __restrict__ rec,
    const uint16_t* __restrict__ ends_in, BrickGrid bg, const uint32_t* __restrict__ offsets,
    const BrickItem* __restrict__ longs, uint64_t* __restrict__ records,
    uint16_t* __restrict__ ends) {
  __shared__ uint4 tile[kLongTile / 4];
  uint32_t lo, n;
  long_voxel(bg, longs[blockIdx.y], offsets, lo, n);
  for (uint64_t p0 = (uint64_t)blockIdx.x * kBlock; p0 < n; p0 += (uint64_t)gridDim.x * kBlock) {
    const bool in = p0 + threadIdx.x < n;
    const uint32_t e = in ? idx[lo + p0 + threadIdx.x] : 0u;
    uint32_t r = 0;
    for (uint64_t q0 = 0; q0 < n; q0 += kLongTile) {
      __syncthreads();
      for (uint32_t q = threadIdx.x; q < kLongTile; q += kBlock)
        reinterpret_cast<uint32_t*>(tile)[q] = q0 + q < n ? idx[lo + q0 + q] : 0xFFFFFFFFu;
      __syncthreads();
      const uint32_t m = (uint32_t)min((uint64_t)kLongTile, n - q0);
      for (uint32_t q = 0; q < (m + 3) / 4; q += 8)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint4 t = tile[q + j];   // the same for all lanes
          r += (t.x < e ? 1u : 0u) + (t.y < e ? 1u : 0u) + (t.z < e ? 1u : 0u) + (t.w < e ? 1u : 0u);
        }
    }
    if (in) {
      records[lo + r] = rec[e];
      if (ends) ends[lo + r] = ends_in[e];
    }
  }
}

// Per-block bounds of the vertices (min and max are exact in fp32; widened
// to fp64 for the set-up). kVec: xyz 16-byte aligned, read as three float4
// per 4 vertices.
template <bool kVec>
__global__ __launch_bounds__(kBlock) void k_bbox(const float* xyz, int64_t nv, double* part,
                                                 int* bad) {
  __shared__ double s[6][kBlock];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool fin = true;
  auto take = [&](int a, float x) {
    fin &= isfinite(x);
    lo[a] = fminf(lo[a], x);
    hi[a] = fmaxf(hi[a], x);
  };
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  int64_t v_tail = 0;
  if (kVec) {
    const float4* g4 = reinterpret_cast<const float4*>(xyz);
    const int64_t ng = nv / 4;
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < ng; g += stride) {
      const float4 a = g4[3 * g], b = g4[3 * g + 1], c = g4[3 * g + 2];
      take(0, a.x); take(1, a.y); take(2, a.z);
      take(0, a.w); take(1, b.x); take(2, b.y);
      take(0, b.z); take(1, b.w); take(2, c.x);
      take(0, c.y); take(1, c.z); take(2, c.w);
    }
    v_tail = 4 * ng;
  }
  for (int64_t v = v_tail + (int64_t)blockIdx.x * kBlock + threadIdx.x; v < nv; v += stride) {
#pragma unroll
    for (int a = 0; a < 3; ++a) take(a, xyz[3 * v + a]);
  }
  if (!fin) *bad = 1;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    s[a][threadIdx.x] = (double)lo[a];
    s[3 + a][threadIdx.x] = (double)hi[a];
  }
  __syncthreads();
  for (int st = kBlock / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s[a][threadIdx.x] = fmin(s[a][threadIdx.x], s[a][threadIdx.x + st]);
        s[3 + a][threadIdx.x] = fmax(s[3 + a][threadIdx.x], s[3 + a][threadIdx.x + st]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int a = 0; a < 6; ++a) part[6 * blockIdx.x + a] = s[a][0];
}

// Reduces k_bbox's per-block bounds and writes the lattice set-up; flags
// non-finite input (bad, from k_bbox) in err.
__global__ __launch_bounds__(kBlock) void k_lattice(const double* part, int blocks, int64_t nv,
                                                    GridArgs ga, const int* bad, SnapArgs* out,
                                                    int* err) {
  __shared__ double s[6][kBlock];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int b = threadIdx.x; b < blocks; b += kBlock) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fmin(lo[a], part[6 * b + a]);
      hi[a] = fmax(hi[a], part[6 * b + 3 + a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    s[a][threadIdx.x] = lo[a];
    s[3 + a][threadIdx.x] = hi[a];
  }
  __syncthreads();
  for (int st = kBlock / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s[a][threadIdx.x] = fmin(s[a][threadIdx.x], s[a][threadIdx.x + st]);
        s[3 + a][threadIdx.x] = fmax(s[3 + a][threadIdx.x], s[3 + a][threadIdx.x + st]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double l[3], h[3];
    for (int a = 0; a < 3; ++a) {
      l[a] = nv > 0 ? s[a][0] : 0.0;
      h[a] = nv > 0 ? s[3 + a][0] : 0.0;
    }
    SnapArgs r;
    for (int a = 0; a < 3; ++a) r.lo[a] = l[a];
    r.scale = lattice_scale(l, h, ga.g);
    *out = r;
    if (*bad) atomicOr(err, kErrNonFinite);
  }
}

__global__ __launch_bounds__(kBlock) void k_snap(const float* xyz, int64_t nv, SnapArgs sa,
                                                 int32_t* lat) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= 3 * nv) return;
  int a = (int)(i % 3);
  lat[i] = snap_coord(xyz[i], sa.lo[a], sa.scale);
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// How the lists are formed: by bricks, or by one rank atomic per line in k_emit,
// k_scatter and k_rank. Whole calls, atomics against bricks, in us:
//  - kBrickMinSlots: few lines cost less than the brick passes' launches. In 128^3
//    0.55M lines 131 and 133, 1.1M 184 and 155, 2.2M 266 and 181; in 160^3 0.55M
//    141 and 149, 1.1M 183 and 165.
//  - kBrickMinMean: each brick costs its workgroups, so a grid with few lines per
//    brick loses. Even at 1.6M lines in 256^3 (49 a brick), 7.2M in 400^3 (53),
//    13M in 512^3 (50), 21M in 640^3 (40), 30M in 1000x1000x400 (37); 10M in 640^3
//    (19) 2341 and 3011, 17.7M in 512^3 (68) 2308 and 2011.
//  - kMaxShare, kMinSpread: a workgroup counts four bricks and ranges of a large
//    brick each read all its lines, so sets crowded into few bricks lose. All
//    lines in 16^3 voxels (8 bricks) of 256^3, 9.4M: 3370 and 7250; 32^3 (64 bricks)
//    1205 and 1710, 40^3 (125) 1112 and 1121, 48^3 (216) 965 and 842; 29M in 40^3
//    4000 and 4685, 48^3 3045 and 3170, 56^3 (343) 2880 and 2450. One crowded
//    brick among others: 1/41 of 24M lines in 256^3 2165 and 2510, 1/93 1965 and
//    1746.
// At 256^3, 9.5M lines (100k x 200 curves): 1169 -> 1080 us for the whole call; at
// 512^3, 140.6M lines (1M x 100): 14.63 -> 8.23 ms, of it the emission 4.66 ->
// 2.77 ms without the rank atomics, and scatter + rank + occupancy + histogram
// copy 7.96 -> 3.45 ms as runs (0.50 + 0.75), counts 0.55, fills 0.51 + 1.16
// (with counting, emission and scans as they are now 860 us and 7.35 ms).
// Run atomics are bound by requests per 128-byte line: one copy of the counters
// in plain brick order took 1.0 + 1.2 ms at 512^3 and 0.13 + 0.15 ms at 256^3,
// 4 x 4 x 2 blocks and 32 copies take 0.50 + 0.75 and 0.04 + 0.04.
constexpr int64_t kBrickMinVoxels = int64_t(1) << 20;
constexpr int64_t kBrickMinSlots = int64_t(1) << 20;
constexpr int64_t kBrickMinMean = 48;
constexpr uint64_t kMaxShare = 64;    // the fullest brick holds at most 1/64 of the lines
constexpr uint64_t kMinSpread = 192;  // sum over bricks of share^2 at most 1/192

// The line sample: lines, of the fullest word, and the sum of the words' squares.
struct Sample {
  uint32_t total, most;
  unsigned long long squares;
};

bool by_bricks(int64_t nvox, int64_t n_slots, int64_t n_bricks, const Sample& m) {
  return nvox >= kBrickMinVoxels && n_slots >= kBrickMinSlots &&
         n_slots >= kBrickMinMean * n_bricks && kMaxShare * m.most <= m.total &&
         kMinSpread * m.squares <= (unsigned long long)m.total * m.total;
}

// Writes what the host reads after k_count to pinned memory: `words` words from
// src, then the line sample's sums if the slot count (src's first 64 bits) makes
// bricks possible.
__global__ __launch_bounds__(kBlock) void k_read_counts(const uint32_t* __restrict__ src, int words,
                                                      const uint32_t* __restrict__ sample,
                                                      uint32_t* dst) {
  __shared__ uint32_t s_total, s_most;
  __shared__ unsigned long long s_sq;
  if (threadIdx.x < (unsigned)words) dst[threadIdx.x] = src[threadIdx.x];
  if (*reinterpret_cast<const uint64_t*>(src) < (uint64_t)kBrickMinSlots) return;   // uniform
  if (threadIdx.x == 0) {
    s_total = s_most = 0u;
    s_sq = 0ull;
  }
  __syncthreads();
  constexpr int kPer = (int)kSampleWords / (4 * kBlock);
  uint4 q[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    q[k] = reinterpret_cast<const uint4*>(sample)[k * kBlock + threadIdx.x];
  uint32_t total = 0, most = 0;
  unsigned long long sq = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t w[4] = {q[k].x, q[k].y, q[k].z, q[k].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      total += w[j];
      most = max(most, w[j]);
      sq += (unsigned long long)w[j] * w[j];
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    total += (uint32_t)__shfl_xor((int)total, d, 64);
    most = max(most, (uint32_t)__shfl_xor((int)most, d, 64));
    sq += __shfl_xor(sq, d, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&s_total, total);
    atomicMax(&s_most, most);
    atomicAdd(&s_sq, sq);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    dst[words] = s_total;
    dst[words + 1] = s_most;
    dst[words + 2] = (uint32_t)s_sq;
    dst[words + 3] = (uint32_t)(s_sq >> 32);
  }
}

inline unsigned curve_blocks(int64_t n) {
  return (unsigned)((n + kWavesPerBlock - 1) / kWavesPerBlock);
}

// Temporary device buffers from the memory cache; released after the stream
// they were used on has drained (one wait for all of them).
struct Drain {
  hipStream_t st;
  bool idle = false;   // the stream was waited for after the last use
  explicit Drain(hipStream_t s) : st(s) {}
  void wait() {
    if (!idle) (void)hipStreamSynchronize(st);
    idle = true;
  }
};

struct DeviceBuf {
  void* p = nullptr;
  Drain& d;
  explicit DeviceBuf(Drain& drain) : d(drain) {}
  DeviceBuf(const DeviceBuf&) = delete;
  DeviceBuf& operator=(const DeviceBuf&) = delete;
  ~DeviceBuf() {
    if (p) {
      d.wait();
      pool_free(p);
    }
  }
  int alloc(size_t bytes) { return pool_alloc(bytes, &p, nullptr); }
  template <typename T>
  T* as() { return static_cast<T*>(p); }
};

}  // namespace

int vox_bbox(const float* xyz, int64_t nv, double lo[3], double hi[3], hipStream_t st) {
  for (int a = 0; a < 3; ++a) {
    lo[a] = 0.0;
    hi[a] = 0.0;
  }
  if (nv <= 0) return LS_OK;
  int64_t blocks = (nv + kBlock - 1) / kBlock;
  if (blocks > 1024) blocks = 1024;
  Drain drain(st);
  DeviceBuf part(drain), bad(drain);
  int rc;
  if ((rc = part.alloc(sizeof(double) * 6 * blocks)) || (rc = bad.alloc(sizeof(int)))) return rc;
  LS_HIP(hipMemsetAsync(bad.p, 0, sizeof(int), st));
  if ((reinterpret_cast<uintptr_t>(xyz) & 15) == 0)
    hipLaunchKernelGGL(k_bbox<true>, dim3((unsigned)blocks), dim3(kBlock), 0, st, xyz, nv,
                       part.as<double>(), bad.as<int>());
  else
    hipLaunchKernelGGL(k_bbox<false>, dim3((unsigned)blocks), dim3(kBlock), 0, st, xyz, nv,
                       part.as<double>(), bad.as<int>());
  LS_HIP(hipGetLastError());
  std::vector<double> h(6 * blocks);
  int hbad = 0;
  LS_HIP(hipMemcpyAsync(h.data(), part.p, sizeof(double) * 6 * blocks, hipMemcpyDeviceToHost, st));
  LS_HIP(hipMemcpyAsync(&hbad, bad.p, sizeof(int), hipMemcpyDeviceToHost, st));
  LS_HIP(hipStreamSynchronize(st));
  if (hbad) {
    ls_set_error("non-finite vertex coordinate");
    return LS_EINVAL;
  }
  for (int a = 0; a < 3; ++a) {
    lo[a] = INFINITY;
    hi[a] = -INFINITY;
  }
  for (int64_t b = 0; b < blocks; ++b)
    for (int a = 0; a < 3; ++a) {
      lo[a] = std::fmin(lo[a], h[6 * b + a]);
      hi[a] = std::fmax(hi[a], h[6 * b + 3 + a]);
    }
  return LS_OK;
}

double vox_scale(const double lo[3], const double hi[3], const int32_t grid[3]) {
  return lattice_scale(lo, hi, grid);
}

int vox_snap(const float* xyz, int64_t nv, SnapArgs sa, int32_t* lat, hipStream_t st) {
  if (nv <= 0) return LS_OK;
  hipLaunchKernelGGL(k_snap, dim3(blocks_for(3 * nv)), dim3(kBlock), 0, st, xyz, nv, sa, lat);
  LS_HIP(hipGetLastError());
  return LS_OK;
}

// The macro grid and its occupancy words (with the two statistics words).
static int occupancy_alloc(ls_lineset* s) {
  for (int a = 0; a < 3; ++a) s->macro[a] = (s->grid[a] + 3) / 4;
  const int64_t nm = (int64_t)s->macro[0] * s->macro[1] * s->macro[2];
  return ls_alloc(s, (void**)&s->occupancy, sizeof(uint64_t) * (nm + 2));
}

int vox_build(ls_lineset* s, const float* xyz, const int32_t* lat, const int64_t* curve_off,
              const uint8_t* attr, const uint8_t* vattr, hipStream_t st, bool lists_only) {
  GridArgs ga;
  for (int a = 0; a < 3; ++a) ga.g[a] = s->grid[a];
  ga.bins = s->bins;
  int sh = 0;
  while ((256 >> sh) > s->bins) ++sh;
  ga.bin_shift = sh;  // 256 / bins = 2^sh
  const int64_t C = s->n_curves;
  const bool float_in = xyz != nullptr;
  int rc;

  // 0. float input: grid set-up on the device (bounds, then the lattice
  //    scale), read back with the slot count below
  const int64_t nv = s->n_vertices;
  const int bb_blocks = (int)std::min<int64_t>(std::max<int64_t>((nv + kBlock - 1) / kBlock, 1), 1024);
  // The slot counts [C + 1] (the scan leaves their total at [C]) are
  // followed in the same buffer by the grid set-up and the error flags, so
  // one copy reads all three back.
  struct Header {
    uint64_t n_slots;
    SnapArgs sa;
    int err[2];
    Sample sample;   // from k_read_counts
  };
  constexpr int kCounts = (int)(offsetof(Header, sample) / sizeof(uint32_t));
  static_assert(4 * kCounts == sizeof(uint64_t) + sizeof(SnapArgs) + 2 * sizeof(int) &&
                    sizeof(Header) == 4 * kCounts + sizeof(Sample),
                "header layout");
  const size_t slot_bytes = sizeof(uint64_t) * (C + 1);
  Drain drain(st);
  DeviceBuf slots(drain), sums64(drain), lattice(drain), sample(drain);
  if ((rc = slots.alloc(slot_bytes + sizeof(SnapArgs) + 2 * sizeof(int))) ||
      (rc = sums64.alloc(sizeof(uint64_t) * scan_block_sums_len(C))) ||
      (rc = lattice.alloc(sizeof(double) * 6 * bb_blocks)))
    return rc;
  SnapArgs* sad = reinterpret_cast<SnapArgs*>(slots.as<char>() + slot_bytes);
  int* errp = reinterpret_cast<int*>(sad + 1);
  // the offsets array and, where the lists cannot go by bricks, the words that
  // start at zero: one launch clears them with the error flags
  if ((rc = ls_alloc(s, (void**)&s->offsets, sizeof(uint32_t) * (s->nvox + 1)))) return rc;
  const bool small = s->nvox < kBrickMinVoxels;
  BrickGrid bg{};
  for (int a = 0; a < 3; ++a) {
    bg.g[a] = s->grid[a];
    bg.m[a] = (s->grid[a] + 3) / 4;
    bg.nk[a] = (uint32_t)(s->grid[a] + (a < 2 ? 31 : 15)) / (a < 2 ? 32 : 16);
  }
  bg.n = 32 * bg.nk[0] * bg.nk[1] * bg.nk[2];
  if (!small && (rc = sample.alloc(sizeof(uint32_t) * kSampleWords))) return rc;
  if (small) {
    if ((rc = occupancy_alloc(s))) return rc;
    const int64_t nm = (int64_t)s->macro[0] * s->macro[1] * s->macro[2];
    if ((rc = clear_u32(reinterpret_cast<uint32_t*>(errp), 2, s->offsets, s->nvox + 1,
                        reinterpret_cast<uint32_t*>(s->occupancy + nm), 4, st)))
      return rc;
  } else if ((rc = clear_u32(reinterpret_cast<uint32_t*>(errp), 2, sample.as<uint32_t>(),
                             kSampleWords, nullptr, 0, st))) {
    return rc;
  }
  if (float_in) {
    double* part = lattice.as<double>();
    if ((reinterpret_cast<uintptr_t>(xyz) & 15) == 0)
      hipLaunchKernelGGL(k_bbox<true>, dim3((unsigned)bb_blocks), dim3(kBlock), 0, st, xyz, nv,
                         part, errp + 1);
    else
      hipLaunchKernelGGL(k_bbox<false>, dim3((unsigned)bb_blocks), dim3(kBlock), 0, st, xyz, nv,
                         part, errp + 1);
    hipLaunchKernelGGL(k_lattice, dim3(1), dim3(kBlock), 0, st, part, bb_blocks, nv, ga,
                       errp + 1, sad, errp);
    LS_HIP(hipGetLastError());
  }
  // 1. per-curve slot counts + validation
  if (C > 0) {
    const unsigned count_blocks = curve_blocks(C) + (small ? 0 : kSampleBlocks);
    if (float_in)
      hipLaunchKernelGGL((k_count<true>), dim3(count_blocks), dim3(kBlock), 0, st, xyz, lat,
                         curve_off, C, s->n_vertices, sad, ga, slots.as<uint64_t>(), errp,
                         sample.as<uint32_t>(), bg.nk[0], bg.nk[0] * bg.nk[1]);
    else
      hipLaunchKernelGGL((k_count<false>), dim3(count_blocks), dim3(kBlock), 0, st, xyz, lat,
                         curve_off, C, s->n_vertices, sad, ga, slots.as<uint64_t>(), errp,
                         sample.as<uint32_t>(), bg.nk[0], bg.nk[0] * bg.nk[1]);
    LS_HIP(hipGetLastError());
  }
  if ((rc = exclusive_scan_u64(slots.as<uint64_t>(), slots.as<uint64_t>(), C, sums64.as<uint64_t>(),
                               st)))
    return rc;
  Header hh{};
  if (small) {
    if ((rc = read_words(slots.as<uint64_t>() + C, &hh, 4 * kCounts, st))) return rc;
  } else if ((rc = read_pinned(&hh, sizeof(Header), st, [&](uint32_t* dst) {
               hipLaunchKernelGGL(k_read_counts, dim3(1), dim3(kBlock), 0, st,
                                  reinterpret_cast<const uint32_t*>(slots.as<uint64_t>() + C),
                                  kCounts, sample.as<uint32_t>(), dst);
             }))) {
    return rc;
  }
  const uint64_t n_slots = hh.n_slots;
  const int herr = hh.err[0];
  const SnapArgs hsa = hh.sa;
  if (herr & kErrNonFinite) {
    ls_set_error("non-finite vertex coordinate");
    return LS_EINVAL;
  }
  if (float_in) {
    for (int a = 0; a < 3; ++a) s->lo_scale[a] = hsa.lo[a];
    s->lo_scale[3] = hsa.scale;
  }
  if (herr & kErrOffsets) {
    ls_set_error("curve_off must start at 0, be non-decreasing and end at most at n_vertices");
    return LS_EINVAL;
  }
  if (herr & kErrRange) {
    ls_set_error("a vertex lies outside [0, 256 * grid) in lattice units");
    return LS_EINVAL;
  }
  if (n_slots >= 0xFFFFFFFFull) {
    ls_set_error("too many per-voxel lines (%llu slots >= 2^32 - 1)", (unsigned long long)n_slots);
    return LS_ENOMEM;
  }
  s->n_slots = (int64_t)n_slots;

  // 2. the way the lists are formed
  const bool bricks = by_bricks(s->nvox, s->n_slots, bg.n, hh.sample);

  // 3. emit
  DeviceBuf rec(drain), vox(drain), rank(drain), sums32(drain), ends_slots(drain);
  if ((rc = rec.alloc(sizeof(uint64_t) * n_slots)) || (rc = vox.alloc(sizeof(uint32_t) * n_slots)) ||
      (rc = sums32.alloc(sizeof(uint32_t) * scan_block_sums_len(s->nvox))))
    return rc;
  if (!bricks) {
    // the offsets array doubles as the histogram
    if ((rc = rank.alloc(sizeof(uint32_t) * n_slots))) return rc;
    if (!small) {
      if (!lists_only && (rc = occupancy_alloc(s))) return rc;
      const int64_t nm = (int64_t)s->macro[0] * s->macro[1] * s->macro[2];
      if ((rc = clear_u32(s->offsets, s->nvox + 1,
                          lists_only ? nullptr : reinterpret_cast<uint32_t*>(s->occupancy + nm), 4,
                          nullptr, 0, st)))
        return rc;
    }
  }
  if (vattr && (rc = ends_slots.alloc(sizeof(uint16_t) * (n_slots ? n_slots : 1)))) return rc;
  uint16_t* eo = vattr ? ends_slots.as<uint16_t>() : nullptr;
  if (C > 0) {
    using Emit = decltype(&k_emit<true, true, true>);
    static const Emit kernels[2][2][2] = {
        {{k_emit<false, false, false>, k_emit<false, false, true>},
         {k_emit<false, true, false>, k_emit<false, true, true>}},
        {{k_emit<true, false, false>, k_emit<true, false, true>},
         {k_emit<true, true, false>, k_emit<true, true, true>}}};
    // (few lines do not, and then more waves hide more: 70k lines 22.4 and 24.1 us)
    const bool few = n_slots < kEmitFew;
    const size_t rings = kWavesPerBlock * (vattr ? sizeof(EmitRingAttr) : sizeof(EmitRing));
    static_assert(kWavesPerBlock * sizeof(EmitRingAttr) <= kEmitRankLds, "rings fit");
    hipLaunchKernelGGL(kernels[float_in][vattr != nullptr][!bricks], dim3(curve_blocks(C)),
                       dim3(kBlock), bricks || few ? 0 : kEmitRankLds - rings, st, xyz, lat, curve_off, attr, vattr, C, s->curve_base, sad,
                       ga, slots.as<uint64_t>(), rec.as<uint64_t>(), eo, vox.as<uint32_t>(),
                       rank.as<uint32_t>(), s->offsets, bg.nk[0], bg.nk[0] * bg.nk[1]);
    LS_HIP(hipGetLastError());
  }

  // 4. counts -> offsets (in place)
  DeviceBuf brick(drain), runs(drain), items(drain), part(drain), sums_b(drain);
  int64_t n_groups = 0;
  // items (a long voxel may cut one in two), long voxels, bricks with some
  bg.long_max = (uint32_t)(n_slots / kLongMin) + 1;
  bg.item_max = 3 * (uint32_t)(n_slots / kFillCap) + bg.long_max;
  uint32_t* n_items = nullptr;
  BrickItem* longs = nullptr;
  uint32_t* long_bricks = nullptr;
  uint32_t* cursor = nullptr;
  if (bricks) {
    // run counts (kReps copies, one past the last), run cursors, item counts
    n_groups = bg.n / kGroupBricks;
    const int64_t nc = (int64_t)kReps * bg.n;
    const size_t words = 2 * (size_t)nc + 4;
    if ((rc = brick.alloc(sizeof(uint32_t) * words)) ||
        (rc = sums_b.alloc(sizeof(uint32_t) * scan_block_sums_len(nc))) ||
        (rc = runs.alloc(sizeof(uint64_t) * (n_slots ? n_slots : 1))) ||
        (rc = items.alloc(sizeof(BrickItem) * ((size_t)bg.item_max + bg.long_max) +
                          sizeof(uint32_t) * bg.long_max)) ||
        (rc = part.alloc(sizeof(ListHeader) + sizeof(uint64_t) * n_groups)) ||
        (rc = occupancy_alloc(s)))
      return rc;
    uint32_t* bc = brick.as<uint32_t>();
    cursor = bc + nc + 1;
    n_items = cursor + nc;
    longs = items.as<BrickItem>() + bg.item_max;
    long_bricks = reinterpret_cast<uint32_t*>(longs + bg.long_max);
    if ((rc = fill_u32(bc, 0u, (int64_t)words, st))) return rc;
    if (n_slots > 0) {
      hipLaunchKernelGGL(k_runs<false>, dim3(blocks_for((int64_t)n_slots)), dim3(kBlock), 0, st,
                         vox.as<uint32_t>(), (int64_t)n_slots, bg.n, bc, cursor,
                         runs.as<unsigned long long>());
      LS_HIP(hipGetLastError());
    }
    if ((rc = exclusive_scan_u32(bc, bc, nc, sums_b.as<uint32_t>(), st))) return rc;
    if (n_slots > 0) {
      hipLaunchKernelGGL(k_runs<true>, dim3(blocks_for((int64_t)n_slots)), dim3(kBlock), 0, st,
                         vox.as<uint32_t>(), (int64_t)n_slots, bg.n, bc, cursor,
                         runs.as<unsigned long long>());
      LS_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_brick_count, dim3((unsigned)n_groups), dim3(kCountThreads), 0, st, bc,
                       runs.as<unsigned long long>(), vox.as<uint32_t>(), bg, s->offsets,
                       reinterpret_cast<unsigned long long*>(s->occupancy),
                       reinterpret_cast<unsigned long long*>(part.as<ListHeader>() + 1), n_items,
                       items.as<BrickItem>());
    LS_HIP(hipGetLastError());
  }
  if ((rc = exclusive_scan_u32(s->offsets, s->offsets, s->nvox, sums32.as<uint32_t>(), st)))
    return rc;
  ListHeader lh{};
  if (bricks) {
    const int64_t nm = (int64_t)s->macro[0] * s->macro[1] * s->macro[2];
    ListHeader* d_lh = part.as<ListHeader>();
    hipLaunchKernelGGL(k_list_stats, dim3(1), dim3(1024), 0, st,
                       reinterpret_cast<unsigned long long*>(d_lh + 1), n_groups,
                       s->offsets + s->nvox, n_items,
                       reinterpret_cast<unsigned long long*>(s->occupancy + nm), d_lh);
    LS_HIP(hipGetLastError());
    if ((rc = read_words(d_lh, &lh, sizeof(lh), st))) return rc;
  } else if ((rc = read_words(s->offsets + s->nvox, &lh.n_records, sizeof(uint32_t), st))) {
    return rc;
  }
  const uint32_t n_rec = lh.n_records, h_items = lh.n_items;
  s->n_records = n_rec;
  if (bricks) {
    s->nonempty = (int64_t)lh.nonempty;
    s->max_list = (int64_t)lh.max_list;
    s->stats_pending = false;
  }

  // 5. the records, list by list
  if ((rc = ls_alloc(s, (void**)&s->records, sizeof(uint64_t) * (n_rec ? n_rec : 1)))) return rc;
  if (vattr && (rc = ls_alloc(s, (void**)&s->ends, sizeof(uint16_t) * (n_rec ? n_rec : 1))))
    return rc;
  uint16_t* ends = vattr ? s->ends : nullptr;
  DeviceBuf idx(drain);
  if (bricks) {
    if (n_rec > 0) {
      hipLaunchKernelGGL(k_brick_fill, dim3(8 * ((bg.n + 7) / 8)), dim3(kBlock), 0, st,
                         brick.as<uint32_t>(), runs.as<unsigned long long>(),
                         vox.as<uint32_t>(), rec.as<uint64_t>(), eo, bg, s->offsets, s->records,
                         ends);
      if (h_items > 0)
        hipLaunchKernelGGL(k_brick_items, dim3(h_items), dim3(kItemThreads), kItemLds, st,
                           brick.as<uint32_t>(), runs.as<unsigned long long>(),
                           vox.as<uint32_t>(), rec.as<uint64_t>(), eo, bg, s->offsets, n_items,
                           items.as<BrickItem>(), s->records, ends);
      if (lh.n_longs > 0) {
        if ((rc = idx.alloc(sizeof(uint32_t) * (size_t)n_rec))) return rc;
        hipLaunchKernelGGL(k_long_gather, dim3(lh.n_long_bricks), dim3(kItemThreads), 0, st,
                           brick.as<uint32_t>(), runs.as<unsigned long long>(),
                           vox.as<uint32_t>(), bg, s->offsets, long_bricks, idx.as<uint32_t>());
        // the longest voxel's lines at once, unless the voxels fill the device
        const unsigned across =
            std::min(blocks_for(s->max_list), std::max(16u, 65536u / lh.n_longs));
        for (uint32_t k = 0; k < lh.n_longs; k += kLongLaunch)
          hipLaunchKernelGGL(k_long_rank, dim3(across, std::min(kLongLaunch, lh.n_longs - k)),
                             dim3(kBlock), 0, st, idx.as<uint32_t>(), rec.as<uint64_t>(), eo, bg,
                             s->offsets, longs + k, s->records, ends);
      }
      LS_HIP(hipGetLastError());
    }
  } else {
    if ((rc = idx.alloc(sizeof(uint64_t) * (n_rec ? n_rec : 1)))) return rc;
    if (n_slots > 0) {
      hipLaunchKernelGGL(k_scatter, dim3(blocks_for((int64_t)n_slots)), dim3(kBlock), 0, st,
                         vox.as<uint32_t>(), rank.as<uint32_t>(), (int64_t)n_slots, s->offsets,
                         idx.as<uint64_t>());
      LS_HIP(hipGetLastError());
    }
    if (n_rec > 0) {
      hipLaunchKernelGGL(k_rank, dim3(blocks_for(n_rec)), dim3(kBlock), 0, st, idx.as<uint64_t>(),
                         rec.as<uint64_t>(), eo, (int64_t)n_rec, s->offsets, s->records, ends);
      LS_HIP(hipGetLastError());
    }
  }

  // 6. macro-cell occupancy and list statistics (k_brick_count's by now)
  if (!bricks && !lists_only && (rc = vox_occupancy(s, st, true))) return rc;
  LS_HIP(hipStreamSynchronize(st));
  drain.idle = true;
  return LS_OK;
}

// Macro-cell occupancy words and list statistics of s->offsets; the
// statistics stay on the device after the occupancy words until
// lineset_info asks for them.
int vox_occupancy(ls_lineset* s, hipStream_t st, bool cleared) {
  GridArgs ga;
  for (int a = 0; a < 3; ++a) ga.g[a] = s->grid[a];
  ga.bins = s->bins;
  ga.bin_shift = 0;
  int rc;
  if (!s->occupancy && (rc = occupancy_alloc(s))) return rc;
  const int64_t nm = (int64_t)s->macro[0] * s->macro[1] * s->macro[2];
  char* stats = reinterpret_cast<char*>(s->occupancy + nm);
  if (!cleared && (rc = fill_u32(reinterpret_cast<uint32_t*>(stats), 0u, 4, st))) return rc;
  auto launch = [&](auto kernel, int lanes) {
    hipLaunchKernelGGL(kernel, dim3(blocks_for(nm * lanes)), dim3(kBlock), 0, st, s->offsets, ga,
                       s->macro[0], s->macro[1], s->macro[2], (unsigned long long*)s->occupancy,
                       reinterpret_cast<unsigned long long*>(stats),
                       reinterpret_cast<unsigned int*>(stats + 8));
  };
  if (nm <= kOccFew)
    launch(k_occupancy<4>, 4);
  else
    launch(k_occupancy<1>, 1);
  LS_HIP(hipGetLastError());
  s->stats_pending = true;
  return LS_OK;
}
