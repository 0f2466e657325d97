// Restricted geodesic Voronoi pass (Eq. 1), snapped centroid update (Sec. 3.1
// "Centroids"; Sec. 3.2.3) and the fixed-iteration Lloyd loop (Algorithm 1).
//
// Voronoi pass.  The regions of Eq. 1 with ties to the lower id are computed by
// one of two schedules with the same result (lsrvt_set_vt_engine): by default
// the brick relaxation, which is described where its kernels begin (BRArgs), and
// on request the level search, which comes first in this file.
//
// Level search: a breadth-first search restricted to same-band face edges, run
// level by level over the whole volume.  Level 0 holds the sites; at level L every
// voxel not reached yet that has a same-band neighbour reached at level L - 1
// takes the smallest site id among those neighbours.  By induction a voxel
// at hop distance L from its nearest sites receives exactly the smallest of
// their ids: each such site reaches it through a neighbour at distance L - 1
// whose own id is no larger, and every neighbour's id names a site within
// distance L.  Each level is one launch, so the ids of level L - 1 are final
// when level L reads them and the result does not depend on scheduling.
//
// The volume is cut into 16^3 bricks (by both schedules).  Per brick row (16
// voxels along x) the search keeps 16-bit masks in global memory: the same-band
// edges in each direction (built once per call, since bands do not change), the
// voxels reached so far and the frontier of the last two levels, plus the
// frontier's brick faces packed into a few words for the neighbours to read.
// A level launch has one wave per brick; a brick works only if it was marked
// for the level (a brick that reached anything marks itself and its six
// neighbours for the next one, with plain stores of the level number).
// Frontier words of bricks that reached nothing at a level are stale, but
// only hold voxels whose neighbours were all reached one level after them,
// so they are masked off by the reached mask, and a voxel that is new at
// some level has no such stale neighbour.  Each voxel is written once per
// pass.
//
// Update.  Per site, M = sum w and S_a = sum w a are exact uint64 sums
// (per-brick or per-tile LDS aggregation, then one set of global atomics per
// distinct cell).  The nearest lattice point to S/M with ties
// rounded down, q_a = floor((2 S_a + M - 1) / (2 M)), is the answer whenever
// it lies in the cell (it then minimises the distance over all lattice
// points, and among tied points the all-lower corner has the smallest linear
// index).  Otherwise cubes of growing half-width r around q are searched, by a
// wave and then, where that is not enough, by a workgroup; voxels outside the
// cube are at least r + 1/2 from the centroid,
// so the search stops once 4 D_best < (M (2 r + 1))^2, comparing
// D = sum_a (M a - S_a)^2 exactly in 128 bits.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <utility>
#include <vector>

#include "common.h"

namespace lsrvt {

namespace {

constexpr int BX = 16, BY = 16, BZ = 16;
constexpr int kRows = BY * BZ;  // a brick is 256 rows of 16 voxels along x
constexpr int kVTThreads = 256;
constexpr int kHistLen = 8192;  // per-level record of which levels reached anything

struct VTGrid {
  int32_t nbx, nby, nbz;
  int64_t nbricks;
};

// Global level-synchronous BFS state.  Brick b, row r (y = r & 15,
// z = r >> 4) holds 16 voxels along x as the low 16 bits of a word.
struct BFSArgs {
  Geom g;
  VTGrid bg;
  const uint32_t *eq;  // [nbricks][256][3]: (x- | x+ << 16), (y- | y+ << 16), (z- | z+ << 16) same-band bits
  uint16_t *fr;        // [2][nbricks][256] voxels reached at the level of that parity
  uint16_t *vis;       // [nbricks][256] voxels reached so far
  unsigned long long *xf;  // [2][nbricks][8] x = 0 face (words 0..3), x = 15 face (4..7) of the frontier;
                           // bit t of word k is row (t & 15) + 16 (4 (t >> 4) + k)
  uint16_t *yf;        // [2][nbricks][32] y = 0 face rows (0..15), y = 15 face rows (16..31) of the frontier, by z
  uint32_t *cell;      // [nbricks][4096] site id of every reached voxel, brick-major (x + 16 y + 256 z in the brick)
  uint32_t *dist;      // [nbricks][4096] level at which each voxel was reached (its hop distance), brick-major
  uint32_t *act;       // [2][nbricks]: act[L & 1][b] == L when brick b takes part in level L
  uint32_t *alive;     // [3]: alive[L % 3] != 0 when some brick takes part in level L
  uint32_t *hist;      // [kHistLen] alive flag of every level
  uint32_t *err;
  // incremental passes only
  uint16_t *inv;       // [nbricks][256] voxels whose site moved in the last update
  uint32_t *bnd;       // [nbricks][4096] kept voxels next to an invalid one: dist << 12 | x + 16 row
  uint32_t *bcnt;      // [nbricks] entries of bnd
  uint32_t *wake;      // [nbricks] next level at which the brick injects kept voxels (NONE: none)
  unsigned long long *dbg;  // diagnostics (LSRVT_DEBUG_LEVELS only): brick visits, candidates, ...
};

// Entries of the kept-voxel lists hold the level in 20 bits; a pass whose
// lists would need more runs as a full pass.
constexpr uint32_t kMaxBndLevel = (1u << 20) - 1;

__device__ __forceinline__ int64_t brick_row_base(const Geom &g, int x0, int y, int z) {
  return x0 + (int64_t)g.nx * (y + (int64_t)g.ny * z);
}

// Marks brick (bx, by, bz) and its six face neighbours for level L (plain
// stores: every writer stores the same tag).
__device__ __forceinline__ void mark_brick(const BFSArgs &A, int bx, int by, int bz, int k, uint32_t L) {
  const int qx = bx + (k == 1 ? -1 : k == 2 ? 1 : 0);
  const int qy = by + (k == 3 ? -1 : k == 4 ? 1 : 0);
  const int qz = bz + (k == 5 ? -1 : k == 6 ? 1 : 0);
  if (qx >= 0 && qy >= 0 && qz >= 0 && qx < A.bg.nbx && qy < A.bg.nby && qz < A.bg.nbz)
    A.act[(size_t)(L & 1) * A.bg.nbricks + (size_t)(qx + A.bg.nbx * (qy + A.bg.nby * qz))] = L;
}

// Same-band masks of every row toward its six neighbours (across brick faces
// too); voxels outside the volume have no edges.  One voxel per lane, so a
// wave covers four rows of a brick and the band reads are coalesced.  Bands
// do not change during a Lloyd loop, so this runs once per call.
__global__ __launch_bounds__(kVTThreads) void k_vt_eq(const uint8_t *__restrict__ band, Geom g, VTGrid bg,
                                                      uint32_t *__restrict__ eq) {
  const int64_t slots = bg.nbricks * kRows * BX;
  const int lane = lane_id();
  const int64_t sy = g.nx, sz = (int64_t)g.nx * g.ny;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i - lane < slots;
       i += (int64_t)gridDim.x * blockDim.x) {
    bool p[6] = {false, false, false, false, false, false};
    const int64_t row = i >> 4;  // brick * 256 + (ly + 16 lz)
    if (i < slots) {
      const int64_t b = row / kRows;
      const int t = (int)(row % kRows);
      const int bx = (int)(b % bg.nbx), by = (int)((b / bg.nbx) % bg.nby), bz = (int)(b / ((int64_t)bg.nbx * bg.nby));
      const int x = bx * BX + (int)(i & 15), y = by * BY + (t & 15), z = bz * BZ + (t >> 4);
      if (x < g.nx && y < g.ny && z < g.nz) {
        const int64_t v = x + sy * y + sz * z;
        const uint8_t bv = band[v];
        p[0] = x > 0 && band[v - 1] == bv;
        p[1] = x + 1 < g.nx && band[v + 1] == bv;
        p[2] = y > 0 && band[v - sy] == bv;
        p[3] = y + 1 < g.ny && band[v + sy] == bv;
        p[4] = z > 0 && band[v - sz] == bv;
        p[5] = z + 1 < g.nz && band[v + sz] == bv;
      }
    }
    uint64_t m[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) m[k] = __ballot(p[k]);
    if (i < slots && (lane & 15) == 0) {
      const int sh = lane;  // this lane's row occupies ballot bits sh .. sh + 15
      uint32_t *dst = eq + row * 3;
      dst[0] = (uint32_t)((m[0] >> sh) & 0xFFFFu) | ((uint32_t)((m[1] >> sh) & 0xFFFFu) << 16);
      dst[1] = (uint32_t)((m[2] >> sh) & 0xFFFFu) | ((uint32_t)((m[3] >> sh) & 0xFFFFu) << 16);
      dst[2] = (uint32_t)((m[4] >> sh) & 0xFFFFu) | ((uint32_t)((m[5] >> sh) & 0xFFFFu) << 16);
    }
  }
}
// The same edges for the brick relaxation, one word per line of a brick:
// words [0, 256) the x lines by row (ly, lz), [256, 512) the y lines (lx, lz),
// [512, 768) the z lines (lx, ly), the first coordinate fastest.  Bit i, 1 to
// 15: edge between the line's voxels i - 1 and i; bit 0: edge of voxel 0 across
// the brick's face; bit 16: that of voxel 15.  One workgroup per brick: thread
// (lx, ly) reads its z line (16 voxels of x a run), the other two axes are
// compared from LDS, so each band is read once and the lines a thread sweeps
// need no transposition in the rounds.
__device__ __forceinline__ void d_br_masks(const uint8_t *__restrict__ band, Geom g, VTGrid bg,
                                           uint32_t *__restrict__ eq) {
  constexpr uint32_t kOut = 256u;  // no band: outside the volume
  __shared__ uint16_t B[kRows * (BX + 2)];  // by row, padded against bank conflicts
  const int t = threadIdx.x, lo = t & 15, hi = t >> 4;
  for (int64_t b = blockIdx.x; b < bg.nbricks; b += gridDim.x) {
    const int x0 = (int)(b % bg.nbx) * BX, y0 = (int)((b / bg.nbx) % bg.nby) * BY,
              z0 = (int)(b / ((int64_t)bg.nbx * bg.nby)) * BZ;
    auto at = [&](int x, int y, int z) -> uint32_t {
      const bool in = x >= 0 && y >= 0 && z >= 0 && x < g.nx && y < g.ny && z < g.nz;
      return in ? (uint32_t)band[x + (int64_t)g.nx * (y + (int64_t)g.ny * z)] : kOut;
    };
    // the word of the line with voxels v(-1) .. v(16)
    auto word = [&](auto v) {
      uint32_t m = 0, last = v(-1);
#pragma unroll
      for (int i = 0; i <= BX; ++i) {
        const uint32_t c = v(i);
        m |= (uint32_t)(c == last && c != kOut) << i;
        last = c;
      }
      return m;
    };
    uint32_t v[BZ + 2];
#pragma unroll
    for (int i = 0; i < BZ + 2; ++i) v[i] = at(x0 + lo, y0 + hi, z0 + i - 1);
    const uint32_t xm = at(x0 - 1, y0 + lo, z0 + hi), xp = at(x0 + BX, y0 + lo, z0 + hi);
    const uint32_t ym = at(x0 + lo, y0 - 1, z0 + hi), yp = at(x0 + lo, y0 + BY, z0 + hi);
#pragma unroll
    for (int i = 0; i < BZ; ++i) B[(hi + BY * i) * (BX + 2) + lo] = (uint16_t)v[i + 1];
    __syncthreads();
    uint32_t *dst = eq + (size_t)b * kRows * 3;
    dst[t] = word([&](int i) -> uint32_t { return i < 0 ? xm : i == BX ? xp : B[t * (BX + 2) + i]; });
    dst[kRows + t] =
        word([&](int i) -> uint32_t { return i < 0 ? ym : i == BY ? yp : B[(i + BY * hi) * (BX + 2) + lo]; });
    dst[2 * kRows + t] = word([&](int i) -> uint32_t { return v[i + 1]; });
    __syncthreads();
  }
}
__global__ __launch_bounds__(kVTThreads) void k_br_masks(const uint8_t *__restrict__ band, Geom g, VTGrid bg,
                                                         uint32_t *__restrict__ eq) { d_br_masks(band, g, bg, eq); }

struct BrickPos {
  uint32_t b, row, lx;
  int bx, by, bz;
  size_t bi;  // brick-major index: b * 4096 + lx + 16 * row
};

__device__ __forceinline__ BrickPos brick_pos(const BFSArgs &A, uint32_t v) {
  const uint32_t x = v % (uint32_t)A.g.nx, r = v / (uint32_t)A.g.nx;
  const uint32_t y = r % (uint32_t)A.g.ny, z = r / (uint32_t)A.g.ny;
  BrickPos p;
  p.bx = (int)(x / BX);
  p.by = (int)(y / BY);
  p.bz = (int)(z / BZ);
  p.b = (uint32_t)p.bx + (uint32_t)A.bg.nbx * ((uint32_t)p.by + (uint32_t)A.bg.nby * (uint32_t)p.bz);
  p.row = (y % BY) + BY * (z % BZ);
  p.lx = x % BX;
  p.bi = (size_t)p.b * (kRows * BX) + p.lx + BX * p.row;
  return p;
}

// Bit of voxel (row, lx) of brick b in a 16-bit row array, read through the
// 32-bit word that holds it.
__device__ __forceinline__ bool row_bit(const uint16_t *rows, const BrickPos &p) {
  return (rows[(size_t)p.b * kRows + p.row] >> p.lx) & 1u;
}

__device__ __forceinline__ void or_row_bit(uint16_t *rows, const BrickPos &p) {
  const size_t w = ((size_t)p.b * kRows + p.row) >> 1;
  atomicOr(reinterpret_cast<uint32_t *>(rows) + w, (1u << p.lx) << ((p.row & 1u) * 16u));
}

// Puts a voxel into the frontier of level 0 (rows and packed faces) and
// marks its brick and the six neighbours for level 1.
__device__ void frontier0(const BFSArgs &A, const BrickPos &p) {
  or_row_bit(A.fr, p);
  const uint32_t ly = p.row & 15u, lz = p.row >> 4;
  if (p.lx == 0 || p.lx == BX - 1) {
    const uint32_t lane = ly + 16u * (lz >> 2), k = lz & 3u;
    atomicOr(&A.xf[(size_t)p.b * 8 + (p.lx ? 4 : 0) + k], 1ull << lane);
  }
  if (ly == 0 || ly == BY - 1) {
    const size_t yi = (size_t)p.b * 32 + (ly ? 16 : 0) + lz;
    atomicOr(reinterpret_cast<uint32_t *>(A.yf) + (yi >> 1), (1u << p.lx) << ((yi & 1u) * 16u));
  }
  // the brick, and the face neighbours whose shared face the voxel lies on
  const uint32_t lz2 = p.row >> 4, ly2 = p.row & 15u;
  const bool on[7] = {true, p.lx == 0, p.lx == BX - 1, ly2 == 0, ly2 == BY - 1, lz2 == 0, lz2 == BZ - 1};
#pragma unroll
  for (int k = 0; k < 7; ++k)
    if (on[k]) mark_brick(A, p.bx, p.by, p.bz, k, 1u);
  A.alive[1] = 1u;
}

// Level 0: every site reaches its own voxel; co-located sites keep the lowest id.
__global__ void k_bfs_init(const uint32_t *__restrict__ sites, uint32_t S, BFSArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  uint32_t v = sites[s];
  if ((int64_t)v >= A.g.n) {
    atomicOr(A.err, 1u);
    return;
  }
  const BrickPos p = brick_pos(A, v);
  atomicMin(&A.cell[p.bi], s);
  A.dist[p.bi] = 0u;
  or_row_bit(A.vis, p);
  frontier0(A, p);
}

// ----------------------------------------------------------------------------
// Incremental passes.  After an update only the sites that moved can change
// the regions.  A voxel whose site did not move keeps a key (distance, id)
// that is still the best over the sites that did not move, so the new key is
// the better of that one and the best over the moved sites; voxels whose site
// moved ("invalid") know neither.  The pass is the same level-synchronous
// search, restricted: its frontier at level L holds the voxels changed at
// level L - 1 and the kept voxels of distance L - 1 that touch an invalid
// voxel ("boundary", injected from per-brick lists at their level).  An
// invalid voxel reached at level L takes the smallest id of its frontier
// neighbours, as in a full pass: every neighbour at distance L - 1 is in the
// frontier (it changed, or it was kept and touches this invalid voxel).  A
// kept voxel reached at level L takes (L, id) only when that key is smaller
// than its own: a kept neighbour at distance L - 1 offers a key it already
// beats, so leaving such neighbours out of the frontier changes nothing.  A
// kept voxel that changes joins the frontier, so changes spread as far as
// they reach, and the result is the full pass's.

// Invalid rows: voxels whose site moved.  One voxel per lane, ballots per row
// (the slot index is the brick-major index of the cells).
__global__ __launch_bounds__(kVTThreads) void k_inc_reset(const uint32_t *__restrict__ cellb,
                                                          const uint8_t *__restrict__ moved, Geom g, VTGrid bg,
                                                          uint16_t *__restrict__ inv) {
  const int64_t slots = bg.nbricks * kRows * BX;
  const int lane = lane_id();
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i - lane < slots;
       i += (int64_t)gridDim.x * blockDim.x) {
    bool p = false;
    const int64_t row = i >> 4;
    if (i < slots) {
      const int64_t b = row / kRows;
      const int t = (int)(row % kRows);
      const int bx = (int)(b % bg.nbx), by = (int)((b / bg.nbx) % bg.nby), bz = (int)(b / ((int64_t)bg.nbx * bg.nby));
      const int x = bx * BX + (int)(i & 15), y = by * BY + (t & 15), z = bz * BZ + (t >> 4);
      if (x < g.nx && y < g.ny && z < g.nz) {
        const uint32_t c = cellb[i];
        p = c != kNone && moved[c] != 0;
      }
    }
    const uint64_t m = __ballot(p);
    if (i < slots && (lane & 15) == 0) inv[row] = (uint16_t)((m >> lane) & 0xFFFFu);
  }
}

// Level 0 of an incremental pass, step 1: a site voxel changes when it is
// invalid or holds a larger key than (0, s); such voxels are cleared and
// flagged as changed (every writer stores the same values).
__global__ void k_inc_site_a(const uint32_t *__restrict__ sites, uint32_t S, BFSArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint32_t v = sites[s];
  if ((int64_t)v >= A.g.n) {
    atomicOr(A.err, 1u);
    return;
  }
  const BrickPos p = brick_pos(A, v);
  if (row_bit(A.inv, p) || A.dist[p.bi] != 0u || A.cell[p.bi] > s) {
    A.cell[p.bi] = kNone;
    A.dist[p.bi] = 0u;
    or_row_bit(A.vis, p);
  }
}

// Step 2: every site on a changed voxel takes part in the minimum; changed
// site voxels form the frontier of level 0.
__global__ void k_inc_site_b(const uint32_t *__restrict__ sites, uint32_t S, BFSArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint32_t v = sites[s];
  if ((int64_t)v >= A.g.n) return;
  const BrickPos p = brick_pos(A, v);
  if (!row_bit(A.vis, p)) return;
  atomicMin(&A.cell[p.bi], s);
  frontier0(A, p);
}

constexpr int kLvlThreads = 64;  // one wave per brick
constexpr int kNewCap = 1024;    // new voxels per brick and level shared out through LDS

// Ids of the six face neighbours of new voxel (lx, row) of brick b, the
// sources among them flagged by a0..a5 (x-, x+, y-, y+, z-, z+; at least one
// is set), read from the brick-major cell array.  A source across a brick
// face lies in the neighbour brick (which exists: edges join voxels of the
// volume only).  All six loads are issued unconditionally so that they are in
// flight together; a direction that is not a source reads the first source
// again, which hits the line that load brings in.
__device__ __forceinline__ void gather6(const uint32_t *cell, size_t b, uint32_t lx, uint32_t row, size_t bsy,
                                        size_t bsz, uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t a4,
                                        uint32_t a5, uint32_t g[6]) {
  constexpr size_t kB = (size_t)kRows * BX;
  const uint32_t ly = row & 15u, lz = row >> 4;
  const size_t v = b * kB + lx + BX * row;
  const size_t n0 = lx > 0 ? v - 1 : (b - 1) * kB + 15 + BX * row;
  const size_t n1 = lx < 15 ? v + 1 : (b + 1) * kB + BX * row;
  const size_t n2 = ly > 0 ? v - 16 : (b - bsy) * kB + lx + 16 * 15 + 256 * lz;
  const size_t n3 = ly < 15 ? v + 16 : (b + bsy) * kB + lx + 256 * lz;
  const size_t n4 = lz > 0 ? v - 256 : (b - bsz) * kB + lx + 16 * ly + 256 * 15;
  const size_t n5 = lz < 15 ? v + 256 : (b + bsz) * kB + lx + 16 * ly;
  size_t f = a5 ? n5 : v;
  f = a4 ? n4 : f;
  f = a3 ? n3 : f;
  f = a2 ? n2 : f;
  f = a1 ? n1 : f;
  f = a0 ? n0 : f;
  g[0] = cell[a0 ? n0 : f];
  g[1] = cell[a1 ? n1 : f];
  g[2] = cell[a2 ? n2 : f];
  g[3] = cell[a3 ? n3 : f];
  g[4] = cell[a4 ? n4 : f];
  g[5] = cell[a5 ? n5 : f];
}

__device__ __forceinline__ uint32_t min_id6(const uint32_t m0, const uint32_t m1, const uint32_t m2, const uint32_t g[6]) {
  uint32_t id = (m0 & 1u) ? g[0] : kNone;
  id = min(id, ((m0 >> 16) & 1u) ? g[1] : kNone);
  id = min(id, (m1 & 1u) ? g[2] : kNone);
  id = min(id, ((m1 >> 16) & 1u) ? g[3] : kNone);
  id = min(id, (m2 & 1u) ? g[4] : kNone);
  id = min(id, ((m2 >> 16) & 1u) ? g[5] : kNone);
  return id;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = min(v, (uint32_t)__shfl_xor(v, o, kWave));
  return v;
}

// LDS of one level workgroup (one wave).
struct LvlLds {
  uint16_t lst[kNewCap];   // listed candidates: x | row << 4
  uint32_t dmp[3 * kRows]; // per row: source directions of its candidates
  uint32_t inv[kRows];     // incremental: invalid voxels of candidate rows
  uint32_t acc[kRows];     // incremental: candidates that took a new key
  uint32_t inj[kRows];     // incremental: kept voxels injected at this level
};

// Level L: a candidate is a voxel that has not changed yet in this pass and
// has a same-band face neighbour in the frontier of level L - 1; its key
// would be (L, smallest id among those neighbours).  In a full pass every
// voxel is invalid and every candidate takes its key (Eq. 1 with ties to the
// lower id).  In an incremental pass a kept candidate takes it only when it
// is smaller than its own (distance, id).  One wave per brick: lane t owns
// the four rows ly = t & 15, lz = 4 (t >> 4) + k (k = 0..3), so the y- and
// z-neighbour rows inside the brick come from other lanes' registers, and
// the rows beyond the brick's faces from the neighbours' packed face words;
// every load of the brick's masks is issued at once.  Candidates are listed
// in LDS and shared out one per lane, whatever row they are in.  The
// frontier the brick writes for level L holds its changed voxels and, in an
// incremental pass, its kept voxels of distance L that touch an invalid one;
// when it is not empty the brick marks itself and its six neighbours for
// level L + 1.
template <bool INC>
__device__ void bfs_brick(const BFSArgs &A, uint32_t L, uint32_t b, LvlLds &S) {
  const int t = threadIdx.x;
  const int ly = t & 15, g4 = (t >> 4) * 4;
  const size_t pin = (size_t)((L - 1) & 1), pout = (size_t)(L & 1);
  const size_t nbk = (size_t)A.bg.nbricks;
  const uint16_t *fin = A.fr + pin * nbk * kRows;
  uint16_t *fout = A.fr + pout * nbk * kRows;
  const unsigned long long *xin = A.xf + pin * nbk * 8;
  unsigned long long *xout = A.xf + pout * nbk * 8;
  const uint16_t *yin = A.yf + pin * nbk * 32;
  uint16_t *yout = A.yf + pout * nbk * 32;
  const int64_t bsy = A.bg.nbx, bsz = (int64_t)A.bg.nbx * A.bg.nby;
  const int lm1 = (t + kWave - 1) & (kWave - 1), lp1 = (t + 1) & (kWave - 1);
  const int lm16 = (t + kWave - 16) & (kWave - 1), lp16 = (t + 16) & (kWave - 1);
  const int bx = (int)(b % A.bg.nbx), by = (int)((b / A.bg.nbx) % A.bg.nby), bz = (int)(b / ((uint32_t)A.bg.nbx * A.bg.nby));
  const int64_t rb = (int64_t)b * kRows;
  const bool hym = ly == 0 && by > 0, hyp = ly == BY - 1 && by < A.bg.nby - 1;
  uint32_t F[4], V[4], I[4], XM[4], XP[4], YM[4], YP[4], E[4][3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ly + 16 * (g4 + k);
#pragma unroll
    for (int j = 0; j < 3; ++j) E[k][j] = A.eq[(rb + r) * 3 + j];
    F[k] = fin[rb + r];
    V[k] = A.vis[rb + r];
    I[k] = INC ? (uint32_t)A.inv[rb + r] : 0xFFFFu;
    const unsigned long long xm = bx > 0 ? xin[(size_t)(b - 1) * 8 + 4 + k] : 0ull;
    const unsigned long long xp = bx < A.bg.nbx - 1 ? xin[(size_t)(b + 1) * 8 + k] : 0ull;
    XM[k] = (uint32_t)(xm >> t) & 1u;
    XP[k] = (uint32_t)(xp >> t) & 1u;
    YM[k] = hym ? yin[(size_t)(b - bsy) * 32 + 16 + g4 + k] : 0u;
    YP[k] = hyp ? yin[(size_t)(b + bsy) * 32 + g4 + k] : 0u;
  }
  const uint32_t ZM = (g4 == 0 && bz > 0) ? fin[(b - bsz) * kRows + 240 + ly] : 0u;
  const uint32_t ZP = (g4 == 12 && bz < A.bg.nbz - 1) ? fin[(b + bsz) * kRows + ly] : 0u;
  const uint32_t zlo = __shfl(F[3], lm16, kWave), zhi = __shfl(F[0], lp16, kWave);
  uint32_t cand[4], c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ly + 16 * (g4 + k);
    const uint32_t up = __shfl(F[k], lm1, kWave), dn = __shfl(F[k], lp1, kWave);
    const uint32_t fym = ly > 0 ? up : YM[k];
    const uint32_t fyp = ly < BY - 1 ? dn : YP[k];
    const uint32_t fzm = k > 0 ? F[k - 1] : (g4 > 0 ? zlo : ZM);
    const uint32_t fzp = k < 3 ? F[k + 1] : (g4 < 12 ? zhi : ZP);
    const uint32_t sxm = (F[k] << 1) | XM[k];
    const uint32_t sxp = (F[k] >> 1) | (XP[k] << 15);
    // reached from each direction: frontier neighbour with a same-band edge
    const uint32_t d0 = sxm & E[k][0] & 0xFFFFu, d1 = sxp & (E[k][0] >> 16);
    const uint32_t d2 = fym & E[k][1] & 0xFFFFu, d3 = fyp & (E[k][1] >> 16);
    const uint32_t d4 = fzm & E[k][2] & 0xFFFFu, d5 = fzp & (E[k][2] >> 16);
    cand[k] = (d0 | d1 | d2 | d3 | d4 | d5) & ~V[k] & 0xFFFFu;
    if (cand[k]) {
      S.dmp[r] = d0 | (d1 << 16);
      S.dmp[kRows + r] = d2 | (d3 << 16);
      S.dmp[2 * kRows + r] = d4 | (d5 << 16);
      if (INC) S.inv[r] = I[k];
    }
    c += (uint32_t)__popc(cand[k]);
  }
  // kept voxels of distance L that touch an invalid voxel join the frontier
  uint32_t inj[4] = {0u, 0u, 0u, 0u};
  if (INC && __builtin_amdgcn_readfirstlane(A.wake[b]) == L) {
#pragma unroll
    for (int k = 0; k < 4; ++k) S.inj[ly + 16 * (g4 + k)] = 0u;
    __syncthreads();
    const uint32_t cnt = A.bcnt[b];
    const uint32_t *list = A.bnd + (size_t)b * (kRows * BX);
    uint32_t nxt = kNone;
    for (uint32_t i = t; i < cnt; i += kWave) {
      const uint32_t e = list[i], d = e >> 12;
      if (d == L)
        atomicOr(&S.inj[(e & 0xFFFu) >> 4], 1u << (e & 15u));
      else if (d > L)
        nxt = min(nxt, d);
    }
    nxt = wave_min_u32(nxt);
    if (t == 0) A.wake[b] = nxt;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) inj[k] = S.inj[ly + 16 * (g4 + k)] & ~V[k];
  }
  uint32_t inc = c;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, kWave);
    if (t >= o) inc += v;
  }
  const uint32_t total = __shfl(inc, kWave - 1, kWave);
  const size_t vb = (size_t)b * (kRows * BX);  // the brick's first cell (brick-major arrays)
  uint32_t nw[4] = {0u, 0u, 0u, 0u};
  if (A.dbg && t == 0) {
    atomicAdd(reinterpret_cast<uint32_t *>(A.dbg + 8) + (L % kHistLen), 1u);
    atomicAdd(&A.dbg[0], 1ull);
    atomicAdd(&A.dbg[1], (unsigned long long)total);
    if (total > (uint32_t)kNewCap) {
      atomicAdd(&A.dbg[2], 1ull);
      atomicAdd(&A.dbg[3], (unsigned long long)total);
    }
  }
  if (total > 0 && total <= (uint32_t)kNewCap) {
    uint32_t p = inc - c;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t bits = cand[k];
      const uint32_t r = (uint32_t)(ly + 16 * (g4 + k));
      if (INC) S.acc[r] = 0u;
      while (bits) {
        const uint32_t x = (uint32_t)(__ffs(bits) - 1);
        bits &= bits - 1;
        S.lst[p++] = (uint16_t)(x | (r << 4));
      }
    }
    __syncthreads();
    // keys of the listed voxels, two per lane at a time
    for (uint32_t e = t; e < total; e += 2 * kWave) {
      size_t v[2];
      uint32_t g[2][6], m[2][3], ob[2], od[2], oc[2], ri[2], xi[2];
      bool have[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t ee = e + (uint32_t)u * kWave;
        have[u] = ee < total;
        const uint32_t idx = S.lst[have[u] ? ee : 0u];
        const uint32_t r = idx >> 4, x = idx & 15u;
        ri[u] = r;
        xi[u] = x;
        v[u] = vb + x + BX * r;
        m[u][0] = S.dmp[r] >> x;
        m[u][1] = S.dmp[kRows + r] >> x;
        m[u][2] = S.dmp[2 * kRows + r] >> x;
        gather6(A.cell, b, x, r, (size_t)bsy, (size_t)bsz, m[u][0] & 1u, (m[u][0] >> 16) & 1u, m[u][1] & 1u,
                (m[u][1] >> 16) & 1u, m[u][2] & 1u, (m[u][2] >> 16) & 1u, g[u]);
        ob[u] = INC ? (S.inv[r] >> x) & 1u : 1u;
        od[u] = 0u;
        oc[u] = 0u;
        if (!ob[u]) {  // a kept voxel: its own key
          od[u] = A.dist[v[u]];
          oc[u] = A.cell[v[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t id = min_id6(m[u][0], m[u][1], m[u][2], g[u]);
        const bool ok = ob[u] || L < od[u] || (L == od[u] && id < oc[u]);
        if (have[u] && ok) {
          A.cell[v[u]] = id;
          A.dist[v[u]] = L;
          if (INC) atomicOr(&S.acc[ri[u]], 1u << xi[u]);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) nw[k] = INC ? S.acc[ly + 16 * (g4 + k)] : cand[k];
  } else if (total > 0) {
    // more candidates than the list holds: each lane takes its own rows
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t bits = cand[k];
      const int r = ly + 16 * (g4 + k);
      const size_t base = vb + BX * (size_t)r;
      const uint32_t m0 = S.dmp[r], m1 = S.dmp[kRows + r], m2 = S.dmp[2 * kRows + r];
      while (bits) {
        const int x = __ffs(bits) - 1;
        bits &= bits - 1;
        const size_t v = base + x;
        uint32_t gg[6];
        gather6(A.cell, b, (uint32_t)x, (uint32_t)r, (size_t)bsy, (size_t)bsz, (m0 >> x) & 1u, (m0 >> (16 + x)) & 1u,
                (m1 >> x) & 1u, (m1 >> (16 + x)) & 1u, (m2 >> x) & 1u, (m2 >> (16 + x)) & 1u, gg);
        const uint32_t id = min_id6(m0 >> x, m1 >> x, m2 >> x, gg);
        bool ok = true;
        if (INC && !((I[k] >> x) & 1u)) {
          const uint32_t od = A.dist[v], oc = A.cell[v];
          ok = L < od || (L == od && id < oc);
        }
        if (ok) {
          A.cell[v] = id;
          A.dist[v] = L;
          nw[k] |= 1u << x;
        }
      }
    }
  }
  uint32_t out[4], any = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    out[k] = nw[k] | inj[k];
    any |= out[k];
  }
  if (A.dbg) {
    uint32_t na = 0, ni = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      na += (uint32_t)__popc(nw[k]);
      ni += (uint32_t)__popc(inj[k]);
    }
    na = wave_sum_u32(na);
    ni = wave_sum_u32(ni);
    if (t == 0) {
      atomicAdd(&A.dbg[4], (unsigned long long)na);
      atomicAdd(&A.dbg[5], (unsigned long long)ni);
    }
  }
  // nothing reached or injected: the frontier words of this parity stay
  // stale, which is harmless (see above)
  if (__ballot(any != 0u) == 0ull) return;
  // the brick works at level L + 1, and so does each face neighbour whose
  // shared face the frontier touches (only through it can the frontier
  // reach that neighbour's voxels)
  uint32_t fxm = 0, fxp = 0, fym = 0, fyp = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    fxm |= out[k] & 1u;
    fxp |= (out[k] >> 15) & 1u;
    fym |= ly == 0 ? out[k] : 0u;
    fyp |= ly == BY - 1 ? out[k] : 0u;
  }
  const uint32_t fzm = g4 == 0 ? out[0] : 0u, fzp = g4 == 12 ? out[3] : 0u;
  const uint32_t mk = 1u | (__ballot(fxm != 0u) ? 2u : 0u) | (__ballot(fxp != 0u) ? 4u : 0u) |
                      (__ballot(fym != 0u) ? 8u : 0u) | (__ballot(fyp != 0u) ? 16u : 0u) |
                      (__ballot(fzm != 0u) ? 32u : 0u) | (__ballot(fzp != 0u) ? 64u : 0u);
  if (t < 7 && ((mk >> t) & 1u)) mark_brick(A, bx, by, bz, t, L + 1);
  if (t == 0) A.alive[(L + 1) % 3] = 1u;
  // this level's frontier: rows, and the packed faces the neighbours read
  unsigned long long xw = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ly + 16 * (g4 + k);
    if (nw[k]) A.vis[rb + r] = (uint16_t)(V[k] | nw[k]);
    fout[rb + r] = (uint16_t)out[k];
    const unsigned long long lo_k = __ballot(out[k] & 1u), hi_k = __ballot((out[k] >> 15) & 1u);
    if (t == k) xw = lo_k;
    if (t == 4 + k) xw = hi_k;
    if (ly == 0) yout[(size_t)b * 32 + g4 + k] = (uint16_t)out[k];
    if (ly == BY - 1) yout[(size_t)b * 32 + 16 + g4 + k] = (uint16_t)out[k];
  }
  if (t < 8) xout[(size_t)b * 8 + t] = xw;
  __syncthreads();  // the LDS lists and masks are reused by the next brick
}

// One BFS level per launch over the bricks marked for it (and, in an
// incremental pass, the bricks that inject kept voxels at this level).
// Workgroup 0 records whether level L is alive and clears the flag of level
// L + 2 (level L + 1 sets it), so launches may be enqueued past the last
// level: they find no marked brick and return.
template <bool INC>
__global__ __launch_bounds__(kLvlThreads) void k_bfs_level(BFSArgs A, uint32_t L) {
  __shared__ LvlLds S;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    A.hist[L % kHistLen] = A.alive[L % 3];
    A.alive[(L + 2) % 3] = 0u;
  }
  const uint32_t *act = A.act + (size_t)(L & 1) * A.bg.nbricks;
  // workgroups are dealt to the eight XCDs in turn (the grid is a multiple of
  // 8): XCD i % 8 takes the i-th eighth of the bricks, neighbours included
  const int64_t per = (A.bg.nbricks + 7) / 8;
  for (int64_t i = blockIdx.x; i < 8 * per; i += gridDim.x) {
    const int64_t b = (i & 7) * per + (i >> 3);
    if (b >= A.bg.nbricks) continue;
    bool go = __builtin_amdgcn_readfirstlane(act[b]) == L;
    if (INC && !go) go = __builtin_amdgcn_readfirstlane(A.wake[b]) == L;
    if (!go) continue;
    bfs_brick<INC>(A, L, (uint32_t)b, S);
  }
}

// Incremental pass set-up: per brick, the kept voxels (not invalid, not yet
// changed) with a same-band face neighbour that is invalid.  Those of
// distance 0 (sites) go into the frontier of level 0 at once; the others are
// listed as (distance << 12 | x + 16 row), and the brick's wake level is
// their smallest distance.  One wave per brick, rows as in the level kernel.
__global__ __launch_bounds__(kLvlThreads) void k_bnd_build(BFSArgs A) {
  __shared__ uint16_t lst[kRows * BX];
  __shared__ uint32_t cnt_s;
  const int t = threadIdx.x;
  const int ly = t & 15, g4 = (t >> 4) * 4;
  const int lm1 = (t + kWave - 1) & (kWave - 1), lp1 = (t + 1) & (kWave - 1);
  const int lm16 = (t + kWave - 16) & (kWave - 1), lp16 = (t + 16) & (kWave - 1);
  const int64_t bsy = A.bg.nbx, bsz = (int64_t)A.bg.nbx * A.bg.nby;
  for (int64_t b = blockIdx.x; b < A.bg.nbricks; b += gridDim.x) {
    const int bx = (int)(b % A.bg.nbx), by = (int)((b / A.bg.nbx) % A.bg.nby),
              bz = (int)(b / ((int64_t)A.bg.nbx * A.bg.nby));
    const int64_t rb = b * kRows;
    const bool hym = ly == 0 && by > 0, hyp = ly == BY - 1 && by < A.bg.nby - 1;
    uint32_t I[4], V[4], XM[4], XP[4], YM[4], YP[4], E[4][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = ly + 16 * (g4 + k);
#pragma unroll
      for (int j = 0; j < 3; ++j) E[k][j] = A.eq[(rb + r) * 3 + j];
      I[k] = A.inv[rb + r];
      V[k] = A.vis[rb + r];
      XM[k] = bx > 0 ? ((uint32_t)A.inv[(b - 1) * kRows + r] >> 15) & 1u : 0u;
      XP[k] = bx < A.bg.nbx - 1 ? (uint32_t)A.inv[(b + 1) * kRows + r] & 1u : 0u;
      YM[k] = hym ? A.inv[(b - bsy) * kRows + 15 + 16 * (g4 + k)] : 0u;
      YP[k] = hyp ? A.inv[(b + bsy) * kRows + 16 * (g4 + k)] : 0u;
    }
    const uint32_t ZM = (g4 == 0 && bz > 0) ? A.inv[(b - bsz) * kRows + 240 + ly] : 0u;
    const uint32_t ZP = (g4 == 12 && bz < A.bg.nbz - 1) ? A.inv[(b + bsz) * kRows + ly] : 0u;
    const uint32_t zlo = __shfl(I[3], lm16, kWave), zhi = __shfl(I[0], lp16, kWave);
    uint32_t bm[4], c = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t up = __shfl(I[k], lm1, kWave), dn = __shfl(I[k], lp1, kWave);
      const uint32_t fym = ly > 0 ? up : YM[k];
      const uint32_t fyp = ly < BY - 1 ? dn : YP[k];
      const uint32_t fzm = k > 0 ? I[k - 1] : (g4 > 0 ? zlo : ZM);
      const uint32_t fzp = k < 3 ? I[k + 1] : (g4 < 12 ? zhi : ZP);
      const uint32_t sxm = (I[k] << 1) | XM[k];
      const uint32_t sxp = (I[k] >> 1) | (XP[k] << 15);
      const uint32_t adj = (sxm & E[k][0] & 0xFFFFu) | (sxp & (E[k][0] >> 16)) | (fym & E[k][1] & 0xFFFFu) |
                           (fyp & (E[k][1] >> 16)) | (fzm & E[k][2] & 0xFFFFu) | (fzp & (E[k][2] >> 16));
      bm[k] = adj & ~I[k] & ~V[k] & 0xFFFFu;
      c += (uint32_t)__popc(bm[k]);
    }
    uint32_t inc = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t v = __shfl_up(inc, o, kWave);
      if (t >= o) inc += v;
    }
    const uint32_t total = __shfl(inc, kWave - 1, kWave);
    if (total == 0) {
      if (t == 0) {
        A.bcnt[b] = 0u;
        A.wake[b] = kNone;
      }
      continue;
    }
    uint32_t p = inc - c;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t bits = bm[k];
      const uint32_t r = (uint32_t)(ly + 16 * (g4 + k));
      while (bits) {
        const uint32_t x = (uint32_t)(__ffs(bits) - 1);
        bits &= bits - 1;
        lst[p++] = (uint16_t)(x | (r << 4));
      }
    }
    if (t == 0) cnt_s = 0u;
    __syncthreads();
    const size_t vb = (size_t)b * (kRows * BX);
    uint32_t *list = A.bnd + (size_t)b * (kRows * BX);
    uint32_t nxt = kNone;
    for (uint32_t e = t; e < total; e += kWave) {
      const uint32_t idx = lst[e];
      const uint32_t r = idx >> 4, x = idx & 15u;
      const uint32_t d = A.dist[vb + x + BX * r];
      if (d == 0u) {
        BrickPos q;
        q.b = (uint32_t)b;
        q.row = r;
        q.lx = x;
        q.bx = bx;
        q.by = by;
        q.bz = bz;
        frontier0(A, q);
      } else if (d > kMaxBndLevel) {
        atomicOr(A.err, 4u);
      } else {
        list[atomicAdd(&cnt_s, 1u)] = (d << 12) | idx;
        nxt = min(nxt, d);
      }
    }
    nxt = wave_min_u32(nxt);
    __syncthreads();
    if (t == 0) {
      A.bcnt[b] = cnt_s;
      A.wake[b] = nxt;
    }
    __syncthreads();
  }
}

// Smallest wake level over all bricks (the next level at which some brick
// injects kept voxels), atomically into *out, which holds NONE beforehand.
__global__ __launch_bounds__(256) void k_wake_min(const uint32_t *__restrict__ wake, int64_t nb, uint32_t *out) {
  uint32_t m = kNone;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += (int64_t)gridDim.x * blockDim.x)
    m = min(m, wake[i]);
  m = wave_min_u32(m);
  if (lane_id() == 0 && m != kNone) atomicMin(out, m);
}

// ----------------------------------------------------------------------------
// Brick relaxation engine (the default schedule).
//
// The regions of Eq. 1 with ties to the lower id are the unique fixed point
// of key(v) = min(key(v), min over same-band face neighbours w of
// key(w) + (1, 0)), keys (distance, id) compared lexicographically and
// packed as distance << 32 | id, started from (0, s) at the sites and
// "unreached" elsewhere.  Any order of such relaxations that starts from
// keys that are lengths of real paths (upper bounds) and stops when nothing
// changes reaches that fixed point, so the result is the level search's, bit
// for bit.  Here a round is one launch over the bricks marked for it: a
// workgroup loads a brick's keys into LDS, takes the offers of the six face
// neighbours (their stored keys plus one hop), relaxes the brick to its own
// fixed point by line sweeps along x, y and z (forward and backward, with the
// same-band edge masks) until a sweep round changes nothing, stores the keys
// that changed, and marks for the next round each face neighbour whose shared
// face changed.  Neighbours never work in the same round (br_first), and a
// neighbour that lowers a face key after the read marks the brick again, so the
// rounds end exactly at the fixed point.  An incremental pass starts from the
// previous keys with the voxels of moved sites set to unreached.  That reset is
// done either by its own kernel (which marks the bricks that hold such voxels),
// or fused into the bricks' first rounds, in which every brick works: each key
// that is not yet reset (the brick's own; in round 1 the neighbours' faces too)
// is taken as unreached when its site moved, unless it is the site's own new
// voxel, and the whole brick is stored.
//
// Keys come in two widths.  Wide keys are 64 bits, distance << 32 | id.
// Narrow keys are 32 bits, distance << b | id with b the bits the site ids
// need (at most 24 by default); one hop adds 1 << b with unsigned
// saturation, so a key that would pass 2^32 - 1 stays "unreached" (all
// ones), which is never an offer.  Every key of a voxel whose true
// distance is below D = 2^(32 - b) - 2 is then exact (its shortest path
// never saturates), and a voxel farther away has a voxel at distance
// exactly D on its shortest path.  So a round that stores a key of
// distance D or more flags the pass, and the host repeats the pass (and
// runs the rest of the call) with wide keys; a pass that ends unflagged
// has every distance below D and is exact.
constexpr int kBRThreads = 256;
constexpr int kBRRow = BX + 1;  // LDS row stride (keys): padding against bank conflicts

struct BRArgs {
  Geom g;
  VTGrid bg;
  const uint32_t *eq;              // [nbricks][3][256] same-band edge words of the bricks' lines (d_br_masks)
  void *key;                       // [nbricks][4096] brick-major keys (narrow or wide), all ones = unreached
  void *xface;                     // [nbricks][2][256] keys of the x = 0 and x = 15 voxels of every row
  uint32_t hop32;                  // narrow keys: one hop (1 << b)
  uint32_t idmask;                 // the id bits of a key (0xFFFFFFFF for wide keys)
  uint32_t lim32;                  // narrow keys: the smallest key whose distance is D (flagged when stored)
  uint32_t *mark;                  // [2][nbricks]: mark[r & 1][b] == r when brick b works in round r
  uint32_t *list;                  // [nbricks] bricks of the current round (large volumes)
  uint32_t *cnt;                   // [2] length of round r's list at r & 1
  uint32_t *ctl;                   // [1] moved sites, [2] reset fused into the first rounds, [3] error bits, [12] bricks worked on (if counted), [13] last round
  const uint8_t *moved;            // the sites the last update moved (fused reset)
  const uint32_t *fsites;          // the sites' voxels (fused reset)
  uint32_t *alive;                 // [3] round alive flags (by r % 3); shared by the jobs of a batch
  uint32_t *hist;                  // [kHistLen] bricks that worked in each round
  unsigned long long *dbg;         // diagnostics (LSRVT_DEBUG_LEVELS only): processings, sweep rounds
};

// The two key widths: unreached value, one hop, and key + hop, which stays
// unreached from unreached (a wide key tests for it, a narrow one
// saturates).
template <class KT>
struct BRKey;
template <>
struct BRKey<unsigned long long> {
  static constexpr unsigned long long inf = ~0ull;
  __device__ static unsigned long long hop(const BRArgs &) { return 1ull << 32; }
  __device__ static unsigned long long add(unsigned long long k, unsigned long long h) {
    return k == inf ? inf : k + h;
  }
  // the hop over an edge (cut = 0) or none (cut = all ones), and the offer over it
  __device__ static unsigned long long edge(unsigned long long, unsigned long long cut) { return cut; }
  __device__ static unsigned long long over(unsigned long long k, unsigned long long h, unsigned long long e) {
    return add(k, h) | e;
  }
};
template <>
struct BRKey<uint32_t> {
  static constexpr uint32_t inf = ~0u;
  __device__ static uint32_t hop(const BRArgs &A) { return A.hop32; }
  __device__ static uint32_t add(uint32_t k, uint32_t h) { return __builtin_elementwise_add_sat(k, h); }
  __device__ static uint32_t edge(uint32_t h, uint32_t cut) { return h | cut; }
  __device__ static uint32_t over(uint32_t k, uint32_t, uint32_t e) { return __builtin_elementwise_add_sat(k, e); }
};

// A key of the previous pass as the fused reset sees it at voxel v:
// unreached when its site moved, unless it is that site's new voxel
// (distance 0 at the site's voxel).
template <class KT>
__device__ __forceinline__ KT br_filter(const BRArgs &A, KT k, KT hop, uint32_t v) {
  if (k == BRKey<KT>::inf) return k;
  const uint32_t id = (uint32_t)k & A.idmask;
  if (!A.moved[id] || (k < hop && A.fsites[id] == v)) return k;
  return BRKey<KT>::inf;
}

// *p = min(*p, k) with the stored value taken through the fused reset's
// filter; returns whether k was stored.
template <class KT>
__device__ __forceinline__ bool br_cas_min(const BRArgs &A, KT *p, KT k, KT hop, uint32_t v) {
  KT old = __atomic_load_n(p, __ATOMIC_RELAXED);
  for (;;) {
    if (k >= br_filter<KT>(A, old, hop, v)) return false;
    const KT prev = atomicCAS(p, old, k);
    if (prev == old) return true;
    old = prev;
  }
}

__device__ __forceinline__ void br_mark(const BRArgs &A, int bx, int by, int bz, int k, uint32_t r) {
  const int qx = bx + (k == 1 ? -1 : k == 2 ? 1 : 0);
  const int qy = by + (k == 3 ? -1 : k == 4 ? 1 : 0);
  const int qz = bz + (k == 5 ? -1 : k == 6 ? 1 : 0);
  if (qx >= 0 && qy >= 0 && qz >= 0 && qx < A.bg.nbx && qy < A.bg.nby && qz < A.bg.nbz)
    A.mark[(size_t)(r & 1) * A.bg.nbricks + (size_t)(qx + A.bg.nbx * (qy + A.bg.nby * qz))] = r;
}

__device__ __forceinline__ void br_coords(const BRArgs &A, int64_t b, int &bx, int &by, int &bz) {
  const uint32_t row = (uint32_t)b / (uint32_t)A.bg.nbx;
  bx = (int)((uint32_t)b - row * (uint32_t)A.bg.nbx);
  by = (int)(row % (uint32_t)A.bg.nby);
  bz = (int)(row / (uint32_t)A.bg.nby);
}

// The round in which a brick works first: the bricks of even coordinate sum work
// in odd rounds and the others in even ones (a brick marks its face neighbours,
// which are of the other kind, for the next round, so this holds by itself
// once the first marks are set so).  No two neighbours work in one round, and
// the second kind already sees what the first found: 114.6 ms for the flame step
// (1024 x 512 x 512, 30 updates) and 122.3 with all kinds in every round, 14.6
// and 16.0 for 379 x 251 x 147 with 20 updates, 37.0 and 38.5 for sixteen jobs of
// 32^3 to 192^3, the same for one pass of 192 x 96 x 96.
__device__ __forceinline__ uint32_t br_first(int bx, int by, int bz) { return 1u + (uint32_t)((bx + by + bz) & 1); }

// Marks neighbour k of a brick (0: itself) for its first round.
__device__ __forceinline__ void br_mark_first(const BRArgs &A, int bx, int by, int bz, int k) {
  const uint32_t r = br_first(bx, by, bz);
  br_mark(A, bx, by, bz, k, k ? 3u - r : r);
  A.alive[k ? 3u - r : r] = 1u;
}

// Site keys of a pass: (0, s) wherever it is smaller than the stored key
// (every voxel of a full pass is unreached); a site voxel that changes
// marks its brick, and the face neighbours whose face it lies on, for their
// first rounds (its packed x-face copy follows).
template <class KT>
__device__ __forceinline__ void d_br_sites(const uint32_t *__restrict__ sites, uint32_t S, BRArgs A) {
  KT *key = static_cast<KT *>(A.key), *xface = static_cast<KT *>(A.xface);
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint32_t v = sites[s];
  if ((int64_t)v >= A.g.n) {
    atomicOr(&A.ctl[3], 1u);
    return;
  }
  const uint32_t x = v % (uint32_t)A.g.nx, rr = v / (uint32_t)A.g.nx;
  const uint32_t y = rr % (uint32_t)A.g.ny, z = rr / (uint32_t)A.g.ny;
  const int bx = (int)(x / BX), by = (int)(y / BY), bz = (int)(z / BZ);
  const size_t b = (size_t)bx + (size_t)A.bg.nbx * ((size_t)by + (size_t)A.bg.nby * (size_t)bz);
  const uint32_t lx = x % BX, ly = y % BY, lz = z % BZ;
  const uint32_t row = ly + BY * lz;
  const KT k = (KT)s;
  if (A.ctl[2] == 0u) {
    const KT old = atomicMin(&key[b * (kRows * BX) + lx + BX * row], k);
    if (k >= old) return;
    if (lx == 0) atomicMin(&xface[b * 512 + row], k);
    if (lx == BX - 1) atomicMin(&xface[b * 512 + 256 + row], k);
  } else {  // previous keys, seen through the fused reset's filter
    const KT hop = BRKey<KT>::hop(A);
    if (!br_cas_min<KT>(A, &key[b * (kRows * BX) + lx + BX * row], k, hop, v)) return;
    if (lx == 0) br_cas_min<KT>(A, &xface[b * 512 + row], k, hop, v);
    if (lx == BX - 1) br_cas_min<KT>(A, &xface[b * 512 + 256 + row], k, hop, v);
  }
  const bool on[7] = {true, lx == 0, lx == BX - 1, ly == 0, ly == BY - 1, lz == 0, lz == BZ - 1};
#pragma unroll
  for (int q = 0; q < 7; ++q)
    if (on[q]) br_mark_first(A, bx, by, bz, q);
}
template <class KT>
__global__ void k_br_sites(const uint32_t *__restrict__ sites, uint32_t S, BRArgs A) { d_br_sites<KT>(sites, S, A); }


// Incremental pass set-up: voxels whose site moved become unreached (keys
// and packed faces), and their bricks are marked for their first rounds.  One thread
// per voxel slot (the slot index is the brick-major index).
template <class KT>
__device__ __forceinline__ void d_br_reset(const uint8_t *__restrict__ moved, BRArgs A) {
  constexpr KT kInf = BRKey<KT>::inf;
  KT *key = static_cast<KT *>(A.key), *xface = static_cast<KT *>(A.xface);
  const int64_t slots = A.bg.nbricks * kRows * BX;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int lane = lane_id();
  constexpr int kU = 8;  // slots per thread and step: their loads are issued together
  // A wave's 64 slots of a step lie in one brick (bricks are 4096 slots,
  // waves and the stride multiples of 64), so the loop bounds are the same
  // for the whole wave and one lane marks the brick.
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < slots; i0 += kU * stride) {
    KT k[kU];
    uint8_t mv[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int64_t i = i0 + j * stride;
      k[j] = i < slots ? key[i] : kInf;
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) mv[j] = k[j] != kInf ? moved[(uint32_t)k[j] & A.idmask] : (uint8_t)0;
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int64_t i = i0 + j * stride;
      if (mv[j]) {
        key[i] = kInf;
        const int64_t b = i / (kRows * BX);
        const int loc = (int)(i % (kRows * BX));
        const int lx = loc & 15, row = loc >> 4;
        if (lx == 0) xface[b * 512 + row] = kInf;
        if (lx == BX - 1) xface[b * 512 + 256 + row] = kInf;
      }
      const uint64_t any = __ballot(mv[j] != 0);
      if (any && lane == __builtin_ctzll(any)) {
        int bx, by, bz;
        br_coords(A, i / (kRows * BX), bx, by, bz);
        br_mark_first(A, bx, by, bz, 0);
      }
    }
  }
}
// Sites the last update moved, counted into *out (zeroed before).
__device__ __forceinline__ void d_count_moved(const uint8_t *__restrict__ moved, uint32_t S, uint32_t *out) {
  uint32_t c = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < S; i += gridDim.x * blockDim.x) c += moved[i] != 0;
  for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
  if (lane_id() == 0 && c) atomicAdd(out, c);
}
__global__ __launch_bounds__(256) void k_count_moved(const uint8_t *__restrict__ moved, uint32_t S, uint32_t *out) {
  d_count_moved(moved, S, out);
}

// Set-up of an incremental pass of lsrvt_cvt: with more than fuse_min
// sites moved (the count in ctl[1]; mode 0), or always (mode 2), the reset
// is fused into the first rounds (ctl[2] set, every brick marked for its own);
// otherwise (or always, mode 1) the voxels of moved sites are reset here.
template <class KT>
__device__ __forceinline__ void d_br_reset_or_fuse(const uint8_t *__restrict__ moved, const BRArgs &A,
                                                   uint32_t fuse_min, int32_t mode) {
  if (mode == 2 || (mode == 0 && A.ctl[1] > fuse_min)) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0) A.ctl[2] = 1u;
    for (int64_t b = i0; b < A.bg.nbricks; b += (int64_t)gridDim.x * blockDim.x) {
      int bx, by, bz;
      br_coords(A, b, bx, by, bz);
      br_mark_first(A, bx, by, bz, 0);
    }
    return;
  }
  d_br_reset<KT>(moved, A);
}
template <class KT>
__global__ __launch_bounds__(256) void k_br_reset_or_fuse(const uint8_t *__restrict__ moved, BRArgs A,
                                                          uint32_t fuse_min, int32_t mode) {
  d_br_reset_or_fuse<KT>(moved, A, fuse_min, mode);
}

// How the workgroups of a round find its marked bricks.  Up to kDirectBricks
// bricks there is one workgroup for each, which looks at its brick's mark and
// ends if it is not set.  Larger volumes have the marks listed by a launch
// before the round (k_br_list) and the round's workgroups stride over the
// list, so that a round with few bricks does not start a workgroup for every
// brick.  Loops listed and direct (all kinds of bricks in every round): 256 x 128 x 128 voxels (1024 bricks) with
// 20 updates 10.1 and 9.3 ms, 256^3 (4096) with 20 updates 16.9 and 16.3,
// 512 x 256 x 256 (8192) with 10 updates 8.59 and 8.45, 512 x 512 x 256
// (16384) with 10 updates 12.45 and 12.41, 512^3 (32768) 19.6 and 20.7.
// (Rounds that list the next round's bricks themselves, one counter atomic a
// brick, take 542 us instead of 204 for 16000 bricks: the atomics on one word
// queue up.)
// A set round grid (LSRVT_TUNE_BR_GRID) below the number of bricks asks for
// striding workgroups; one that covers them is a workgroup for every brick.
constexpr int64_t kDirectBricks = 16384;
bool direct_rounds(int64_t bricks) {
  const int64_t tg = tuning(LSRVT_TUNE_BR_GRID);
  return bricks <= (tg > 0 ? std::min(tg, kDirectBricks) : kDirectBricks);
}

// The bricks marked for round r, listed (one counter atomic per block).
__device__ __forceinline__ void d_br_list(const BRArgs &A, uint32_t r) {
  __shared__ uint32_t base_s;
  __shared__ uint32_t wcount[256 / kWave];
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const uint32_t *mk = A.mark + (size_t)(r & 1) * A.bg.nbricks;
  for (int64_t b0 = (int64_t)blockIdx.x * 256; b0 < A.bg.nbricks; b0 += (int64_t)gridDim.x * 256) {
    const int64_t b = b0 + t;
    const bool on = b < A.bg.nbricks && mk[b] == r;
    const uint64_t bal = __ballot(on);
    if (lane == 0) wcount[w] = (uint32_t)__popcll(bal);
    __syncthreads();
    if (t == 0) {
      uint32_t tot = 0;
      for (int q = 0; q < 256 / kWave; ++q) tot += wcount[q];
      base_s = tot ? atomicAdd(&A.cnt[r & 1], tot) : 0u;
    }
    __syncthreads();
    uint32_t off = base_s;
    for (int q = 0; q < w; ++q) off += wcount[q];
    if (on) A.list[off + (uint32_t)__popcll(bal & lanemask_lt())] = (uint32_t)b;
    __syncthreads();
  }
}
__global__ __launch_bounds__(256) void k_br_list(BRArgs A, uint32_t r) { d_br_list(A, r); }

__device__ __forceinline__ int br_at(int lx, int row) { return row * kBRRow + lx; }

// One line of 16 voxels at K[base + i * st] relaxed forward and backward
// along its same-band edges (mask bit i: edge between voxels i - 1 and i).
// Returns the bits of the voxels whose key dropped; the line is written back
// only then.  The calling thread owns the line for the whole stage.
// Branch-free, and one word serves both directions: a missing edge is a hop of
// all ones, which a narrow key's saturating addition turns into "unreached"
// (a wide key's offer is set to it), so a step is an addition and a minimum
// and what dropped is found by comparing once at the end.  The mask passes
// through an empty asm statement so that the per-voxel edge tests are made
// here, from one register, rather than hoisted out of the caller's sweep loop.
template <class KT>
__device__ __forceinline__ uint32_t br_sweep(KT *K, int base, int st, uint32_t mask, KT hop) {
  using KO = BRKey<KT>;
  uint32_t nm = ~mask;
  asm volatile("" : "+v"(nm));
  KT k[16], old[16], h[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) old[i] = k[i] = K[base + i * st];
#pragma unroll
  for (int i = 1; i < 16; ++i) h[i] = KO::edge(hop, (KT)(int64_t)((int32_t)(nm << (31 - i)) >> 31));
#pragma unroll
  for (int i = 1; i < 16; ++i) {
    const KT o = KO::over(k[i - 1], hop, h[i]);
    k[i] = o < k[i] ? o : k[i];
  }
#pragma unroll
  for (int i = 14; i >= 0; --i) {
    const KT o = KO::over(k[i + 1], hop, h[i + 1]);
    k[i] = o < k[i] ? o : k[i];
  }
  uint32_t c = 0;
#pragma unroll
  for (int i = 15; i >= 0; --i) c = c + c + (uint32_t)(k[i] != old[i]);
  if (c) {
#pragma unroll
    for (int i = 0; i < 16; ++i) K[base + i * st] = k[i];
  }
  return c;
}

// LDS of one brick processing: the keys (rows padded against bank
// conflicts), by row the voxels whose key changed in this processing and
// those among them that changed since the row's last x sweep, and the y and z
// lines to sweep: bit lx of yl[lz] and of zl[ly].
template <class KT>
struct BRLds {
  KT K[kRows * kBRRow];
  uint32_t chg[kRows];
  uint32_t pend[kRows];
  uint32_t yl[BZ], zl[BY];
  uint32_t more;
};

// The changed voxels of a wave's 64 lines along y (or z), bits c by place on
// the line; lane l holds line (lx, q) = (l & 15, l >> 4) of the wave's four.
// Ballot i holds the rows at place i, 16 bits for each q, and lane i takes
// it: no lane loops over its voxels.  row(i, q) is the row's index, lines[i]
// the summary of the other axis.
template <class Row>
__device__ __forceinline__ void br_spread(uint32_t c, uint32_t *pend, uint32_t *lines, uint32_t *more, uint32_t it,
                                          Row row) {
  if (__ballot(c != 0u) == 0ull) return;
  const int lane = lane_id();
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint64_t bal = __ballot(c >> i & 1u);
    lo = lane == i ? (uint32_t)bal : lo;
    hi = lane == i ? (uint32_t)(bal >> 32) : hi;
  }
  if (lane < 16) {
    const uint32_t part[4] = {lo & 0xFFFFu, lo >> 16, hi & 0xFFFFu, hi >> 16};
    // the rows of this wave's lines are no other wave's in this stage
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (part[q]) pend[row(lane, q)] |= part[q];
    const uint32_t any = part[0] | part[1] | part[2] | part[3];
    if (any) atomicOr(&lines[lane], any);
    if (lane == 0) *more = it;
  }
}

// One processing of brick b in round r (all threads of the workgroup).
// Thread t owns three lines of the brick for the whole processing: row t along
// x (ly, lz) = (t & 15, t >> 4), the y line (lx, lz) and the z line (lx, ly),
// the first coordinate t & 15 and the second t >> 4; their edge words stay in
// registers.
//
// Bound by the sweeps' vector operations and, in the rounds of few bricks, by
// the chain of LDS accesses and barriers between the axes.  Flame loop
// (1024 x 512 x 512, 30 updates): 78 ms, the rounds 1.9 ms a pass; 110 ms and
// 2.6 ms before neighbours took turns and the site update was cut, and 142 ms
// and 3.3 ms with a changed-voxel loop per lane, edge masks transposed from
// rows per processing, changes counted at every step of a sweep and 2048
// workgroups a round.  At the 110 ms form, 10 updates: six waves a SIMD 48.9 ms,
// 49.7 with five, 52.2 with seven and 59.7 with eight (spills); 2048 workgroups
// 53.3 instead of 48.9 with 8192, because the bricks' work is uneven.
template <class KT>
__device__ __forceinline__ void br_process(const BRArgs &A, int64_t b, uint32_t r, BRLds<KT> &L) {
  using KO = BRKey<KT>;
  constexpr KT kInf = KO::inf;
  const KT hop = KO::hop(A);
  KT *key = static_cast<KT *>(A.key), *xface = static_cast<KT *>(A.xface);
  KT *K = L.K;
  uint32_t *chg = L.chg;
  // the thread index passes through an empty asm statement so that what is
  // derived from it (LDS and global offsets) is recomputed per processing
  // instead of being kept live across a round's processings
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  const int lo4 = t & 15, hi4 = t >> 4;
  const size_t kB = (size_t)kRows * BX;
  const int64_t bsy = A.bg.nbx, bsz = (int64_t)A.bg.nbx * A.bg.nby;
  {
    const int bx = (int)(b % A.bg.nbx), by = (int)((b / A.bg.nbx) % A.bg.nby),
              bz = (int)(b / ((int64_t)A.bg.nbx * A.bg.nby));
    const bool hxm = bx > 0, hxp = bx < A.bg.nbx - 1, hym = by > 0, hyp = by < A.bg.nby - 1, hzm = bz > 0,
               hzp = bz < A.bg.nbz - 1;
    // every global read of the processing, issued together: the brick's keys
    // (16 per thread, coalesced), its edge words and the six faces of the
    // neighbours (a missing neighbour reads the brick itself, unused)
    KT kv[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) kv[i] = key[(size_t)b * kB + i * kBRThreads + t];
    const uint32_t *eq = A.eq + (size_t)b * kRows * 3 + t;
    const uint32_t mx = eq[0], my = eq[kRows], mz = eq[2 * kRows];
    KT fxm = xface[(size_t)(hxm ? b - 1 : b) * 512 + 256 + t];
    KT fxp = xface[(size_t)(hxp ? b + 1 : b) * 512 + t];
    KT fym = key[(size_t)(hym ? b - bsy : b) * kB + lo4 + 16 * 15 + 256 * hi4];
    KT fyp = key[(size_t)(hyp ? b + bsy : b) * kB + lo4 + 256 * hi4];
    KT fzm = key[(size_t)(hzm ? b - bsz : b) * kB + lo4 + 16 * hi4 + 256 * 15];
    KT fzp = key[(size_t)(hzp ? b + bsz : b) * kB + lo4 + 16 * hi4];
    // the brick's first round in an incremental pass with the reset fused in;
    // in round 2 its neighbours are through with theirs
    const bool fuse = r <= 2 && A.ctl[2] != 0u;
    if (fuse) {
      const uint32_t nx = (uint32_t)A.g.nx, nxy = (uint32_t)A.g.nx * (uint32_t)A.g.ny;
      const uint32_t x0 = (uint32_t)bx * BX, y0 = (uint32_t)by * BY, z0 = (uint32_t)bz * BZ;
      // thread t's voxel i is (x0 + lo4, y0 + hi4, z0 + i)
      const uint32_t v0 = x0 + lo4 + nx * (y0 + hi4) + nxy * z0;
#pragma unroll
      for (int i = 0; i < 16; ++i) kv[i] = br_filter<KT>(A, kv[i], hop, v0 + nxy * (uint32_t)i);
      // the face voxels' own coordinates (unused where the neighbour is missing)
      if (r == 1) {
        fxm = br_filter<KT>(A, fxm, hop, x0 - 1 + nx * (y0 + lo4) + nxy * (z0 + hi4));
        fxp = br_filter<KT>(A, fxp, hop, x0 + BX + nx * (y0 + lo4) + nxy * (z0 + hi4));
        fym = br_filter<KT>(A, fym, hop, x0 + lo4 + nx * (y0 - 1) + nxy * (z0 + hi4));
        fyp = br_filter<KT>(A, fyp, hop, x0 + lo4 + nx * (y0 + BY) + nxy * (z0 + hi4));
        fzm = br_filter<KT>(A, fzm, hop, x0 + lo4 + nx * (y0 + hi4) + nxy * (z0 - 1));
        fzp = br_filter<KT>(A, fzp, hop, x0 + lo4 + nx * (y0 + hi4) + nxy * (z0 + BZ));
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int loc = i * kBRThreads + t;
      K[br_at(loc & 15, loc >> 4)] = kv[i];
    }
    chg[t] = 0u;
    L.pend[t] = 0u;
    if (t < BZ) L.yl[t] = 0u;
    if (t < BY) L.zl[t] = 0u;
    if (t == 0) L.more = 0u;
    __syncthreads();
    // offers of the six face neighbours: their keys plus one hop
    {
      auto offer = [&](bool has, bool edge, KT h, int lx, int row) {
        const KT o = KO::add(h, hop);
        if (has && edge && h != kInf && atomicMin(&K[br_at(lx, row)], o) > o) {
          atomicOr(&L.pend[row], 1u << lx);
          atomicOr(&L.yl[row >> 4], 1u << lx);
          atomicOr(&L.zl[row & 15], 1u << lx);
        }
      };
      offer(hxm, mx & 1u, fxm, 0, t);
      offer(hxp, (mx >> 16) & 1u, fxp, 15, t);
      offer(hym, my & 1u, fym, lo4, 16 * hi4);
      offer(hyp, (my >> 16) & 1u, fyp, lo4, 15 + 16 * hi4);
      offer(hzm, mz & 1u, fzm, lo4, hi4);
      offer(hzp, (mz >> 16) & 1u, fzp, lo4, hi4 + 16 * 15);
    }
    __syncthreads();
    // The brick's own fixed point: line sweeps along x, y and z.  In its first round
    // every line is swept (sites were set, keys reset or the pass starts from
    // nothing).  Later a brick's keys are a fixed point of its own relaxation
    // (its last processing ended at one, or the previous pass's result is
    // one), so only the lines through voxels that a neighbour's offer lowered
    // can change; and a line is swept again along its axis only after another
    // axis changed a voxel on it.  The loop ends with an iteration whose y and
    // z sweeps change nothing: an x sweep's changes are swept along y and z in
    // the same iteration, a y sweep's along z.  (`more` is written in the y and
    // z stages only, and read before the x stage's barrier.)
    for (uint32_t it = 1;; ++it) {
      const bool all = r <= 2 && it == 1;  // (the brick's first round)
      {  // row t = (ly, lz)
        const uint32_t pd = L.pend[t];
        if (all || pd) {
          const uint32_t c = br_sweep<KT>(K, t * kBRRow, 1, mx, hop);
          L.pend[t] = 0u;
          chg[t] |= pd | c;  // only this thread touches row t's words in this stage
          if (c) {
            atomicOr(&L.yl[hi4], c);
            atomicOr(&L.zl[lo4], c);
          }
        }
      }
      __syncthreads();
      {  // y line (lx, lz) = (lo4, hi4); yl[lz] is this wave's alone here
        const uint32_t yl = L.yl[hi4];
        if (lo4 == 0) L.yl[hi4] = 0u;
        uint32_t c = 0;
        if (all || (yl >> lo4 & 1u)) c = br_sweep<KT>(K, 16 * kBRRow * hi4 + lo4, kBRRow, my, hop);
        br_spread(c, L.pend, L.zl, &L.more, it, [&](int y, int q) { return y + 16 * ((hi4 & ~3) + q); });
      }
      __syncthreads();
      {  // z line (lx, ly) = (lo4, hi4)
        const uint32_t zl = L.zl[hi4];
        if (lo4 == 0) L.zl[hi4] = 0u;
        uint32_t c = 0;
        if (all || (zl >> lo4 & 1u)) c = br_sweep<KT>(K, hi4 * kBRRow + lo4, 16 * kBRRow, mz, hop);
        br_spread(c, L.pend, L.yl, &L.more, it, [&](int z, int q) { return (hi4 & ~3) + q + 16 * z; });
      }
      __syncthreads();
      if (L.more != it) {
        if (A.dbg && t == 0) {
          atomicAdd(&A.dbg[0], 1ull);
          atomicAdd(&A.dbg[1], (unsigned long long)it);
        }
        break;
      }
    }
    // Which neighbours work in round r + 1: a face voxel that changed, has a
    // same-band edge across the face and whose key plus one hop beats the
    // neighbour's voxel across it as read at the top.  Keys only decrease
    // within a pass, so a neighbour whose key already was no larger can never
    // take the offer.  Thread t checks the face voxels it offered to above, and
    // each wave marks for itself (every writer stores the same tag).
    {
      auto gain = [&](bool has, bool edge, int lx, int row, KT nbk) {
        if (!has || !edge || !((chg[row] >> lx) & 1u)) return false;
        const KT k = K[br_at(lx, row)];
        return KO::add(k, hop) < nbk;
      };
      uint32_t f = 0;
      f |= __ballot(gain(hxm, mx & 1u, 0, t, fxm)) ? 2u : 0u;
      f |= __ballot(gain(hxp, (mx >> 16) & 1u, 15, t, fxp)) ? 4u : 0u;
      f |= __ballot(gain(hym, my & 1u, lo4, 16 * hi4, fym)) ? 8u : 0u;
      f |= __ballot(gain(hyp, (my >> 16) & 1u, lo4, 15 + 16 * hi4, fyp)) ? 16u : 0u;
      f |= __ballot(gain(hzm, mz & 1u, lo4, hi4, fzm)) ? 32u : 0u;
      f |= __ballot(gain(hzp, (mz >> 16) & 1u, lo4, hi4 + 16 * 15, fzp)) ? 64u : 0u;
      const int lane = lane_id();
      if (lane < 7 && (f >> lane & 1u)) br_mark(A, bx, by, bz, lane, r + 1);
      if (f && lane == 0) A.alive[(r + 1) % 3] = 1u;
    }
    // store what changed.  The thread index is passed through an empty asm
    // statement so that the store addresses are recomputed here instead of
    // being kept live (in registers) from the loads at the top across the
    // sweeps.
    // A narrow key of distance D or more flags the pass (all ones is
    // unreached: stored by the fused reset, it flags nothing).
    int tt = t;
    asm volatile("" : "+v"(tt));
    uint32_t top = 0;  // the largest stored key plus one (0 for unreached)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int lx = tt & 15, row = (tt >> 4) + 16 * i;
      if (fuse || ((chg[row] >> lx) & 1u)) {
        const KT k = K[br_at(lx, row)];
        if (sizeof(KT) == 4) top = max(top, (uint32_t)k + 1u);
        key[(size_t)b * kB + i * kBRThreads + tt] = k;
        if (lx == 0) xface[(size_t)b * 512 + row] = k;
        if (lx == BX - 1) xface[(size_t)b * 512 + 256 + row] = k;
      }
    }
    if (sizeof(KT) == 4 && top > A.lim32) atomicOr(&A.ctl[3], 4u);
    __syncthreads();
  }
}

template <class KT>
__global__ __launch_bounds__(kBRThreads, sizeof(KT) == 4 ? 6 : 4) void k_br_round(BRArgs A, uint32_t r) {
  __shared__ BRLds<KT> L;
  const uint32_t count = A.cnt[r & 1];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    A.alive[(r + 2) % 3] = 0u;  // round r + 1 sets it
    A.cnt[(r + 1) & 1] = 0u;    // the list of round r + 1 counts in it
    A.hist[r % kHistLen] = count;
    if (count) A.ctl[13] = r;   // the last round that had work
    A.ctl[12] += count;
  }
  for (uint32_t item = blockIdx.x; item < count; item += gridDim.x) br_process<KT>(A, A.list[item], r, L);
}

// The same round with one workgroup for every brick.  Tally: the bricks that work
// are counted, from every 32nd of them (one counter for all would queue up; loops of
// 1104 bricks take 1 % longer with it).
template <class KT, bool Tally>
__global__ __launch_bounds__(kBRThreads, sizeof(KT) == 4 ? 6 : 4) void k_br_round_all(BRArgs A, uint32_t r) {
  __shared__ BRLds<KT> L;
  if (blockIdx.x == 0 && threadIdx.x == 0) A.alive[(r + 2) % 3] = 0u;  // round r + 1 sets it
  if (A.mark[(size_t)(r & 1) * A.bg.nbricks + blockIdx.x] != r) return;
  if (threadIdx.x == 0) A.ctl[13] = r;  // the last round that had work
  if (Tally && threadIdx.x == 0 && (blockIdx.x * 2654435761u) >> 27 == 0u) atomicAdd(&A.ctl[12], 32u);
  br_process<KT>(A, blockIdx.x, r, L);
}

// ----------------------------------------------------------------------------
// update

// Per site: mass, mass-weighted x, y and z (M, S_x, S_y, S_z together, so that
// the four additions for a cell fall into one 32-byte sector).
struct Sums {
  unsigned long long *p;  // [S][4]
  __device__ __forceinline__ void add(uint32_t c, unsigned long long M, unsigned long long X, unsigned long long Y,
                                      unsigned long long Z) const {
    atomicAdd(&p[4 * (size_t)c], M);
    atomicAdd(&p[4 * (size_t)c + 1], X);
    atomicAdd(&p[4 * (size_t)c + 2], Y);
    atomicAdd(&p[4 * (size_t)c + 3], Z);
  }
};

// Cells as the update reads them: the caller's C-order array, or the search's
// own brick-major keys (inside the Lloyd loop the C-order cells are written by
// the last pass only).
struct CellView {
  const uint32_t *cell;
  int32_t nx, ny;
  __device__ __forceinline__ uint32_t id(int32_t x, int32_t y, int32_t z) const {
    return cell[x + (int64_t)nx * (y + (int64_t)ny * z)];
  }
};
template <class KT>
struct KeyView {
  const KT *key;
  VTGrid bg;
  uint32_t idmask;  // all ones for the level search's cells
  __device__ __forceinline__ uint32_t id(int32_t x_, int32_t y_, int32_t z_) const {
    const uint32_t x = (uint32_t)x_, y = (uint32_t)y_, z = (uint32_t)z_;
    const uint32_t b = x / BX + (uint32_t)bg.nbx * (y / BY + (uint32_t)bg.nby * (z / BZ));
    const KT k = key[(size_t)b * (kRows * BX) + x % BX + BX * (y % BY) + BX * BY * (z % BZ)];
    return k == (KT)~(KT)0 ? kNone : (uint32_t)k & idmask;
  }
};

// The centroid sums of the update (Sec. 3.1: mass and mass-weighted
// position of every cell, exact uint64 integers, so their order does not
// matter) taken at the end of the Voronoi pass that produces the cells, from
// the search's own brick-major keys.  Partial sums go into an LDS table keyed by
// cell id (global atomics where a cell finds no place), flushed with one set
// of global atomics per distinct cell of the workgroup's part.  Two forms:
//  - wide cells: one workgroup per slab of four bricks with running sums per
//    lane (d_br_finish_slabs): 0.39 ms for 2^28 voxels (0.56 with the C-order
//    cells written too);
//  - narrow cells (fewer than kSlabSites voxels per site): one workgroup per
//    brick, whose table has room for the hundreds of cells of a brick
//    (d_brick_sums).  Thread t takes voxel t, t + 256, ... of the brick, so the
//    16 lanes of each quarter wave hold one row along x, and a segmented scan
//    over those 16 lanes (DPP row shifts) sums (w, w * (x - x0)) over every run
//    of equal cell id, whose last lane adds it into the table.  All sums are
//    relative to the brick's corner and so below 2^32: five words a cell.
constexpr int64_t kSlabSites = 512;
struct Fuse {
  const uint16_t *w;  // weights (C order) or null for unit weights
  uint32_t S;
  Sums sums;          // zeroed before the pass
};

constexpr int kFinTab = 256;
struct FinTab {
  uint32_t tkey[kFinTab];
  unsigned long long tM[kFinTab], tX[kFinTab], tY[kFinTab], tZ[kFinTab];
};
constexpr int kBrickTab = 1024;
constexpr int kProbes = 16;
struct BrickTab {
  uint32_t key[kBrickTab], v[4][kBrickTab];
};

__device__ __forceinline__ void fin_clear(FinTab &T) {
  for (int i = threadIdx.x; i < kFinTab; i += blockDim.x) {
    T.tkey[i] = kNone;
    T.tM[i] = T.tX[i] = T.tY[i] = T.tZ[i] = 0ull;
  }
}

// v moved right by CTRL's shift within each row of 16 lanes; 0 where the
// source lane lies outside the row.
template <int CTRL>
__device__ __forceinline__ uint32_t row_shift(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// One voxel per lane, 16 lanes per row (lane & 15 = x - x0, every lane of
// the wave active): adds the runs of equal cell id of the wave's four rows
// (ly, lz) of the brick into the table.  c = kNone for voxels outside the
// volume (weight 0).
__device__ __forceinline__ void brick_row_runs(BrickTab &T, const Fuse &F, uint32_t c, uint32_t wv, uint32_t x0,
                                               uint32_t y0, uint32_t z0, uint32_t ly, uint32_t lz) {
  const uint32_t lx = threadIdx.x & 15;
  const uint32_t cl = (uint32_t)__builtin_amdgcn_update_dpp((int)kNone, (int)c, 0x111, 0xF, 0xF, false);  // row_shr:1
  const uint32_t cr = (uint32_t)__builtin_amdgcn_update_dpp((int)kNone, (int)c, 0x101, 0xF, 0xF, false);  // row_shl:1
  uint32_t m = wv, sx = wv * lx;  // sum of w * (x - x0) over a run: below 2^24
  uint32_t f = (lx == 0 || cl != c) ? 1u : 0u;  // a run starts within the lanes summed so far
#define LSRVT_SEG_STEP(CTRL)                                        \
  {                                                                 \
    const uint32_t mo = row_shift<CTRL>(m), so = row_shift<CTRL>(sx), fo = row_shift<CTRL>(f); \
    if (!f) {                                                       \
      m += mo;                                                      \
      sx += so;                                                     \
      f = fo;                                                       \
    }                                                               \
  }
  LSRVT_SEG_STEP(0x111)  // row_shr:1
  LSRVT_SEG_STEP(0x112)  // row_shr:2
  LSRVT_SEG_STEP(0x114)  // row_shr:4
  LSRVT_SEG_STEP(0x118)  // row_shr:8
#undef LSRVT_SEG_STEP
  const bool tail = lx == 15 || cr != c;
  if (tail && c < F.S && m) {
    const int sl = lds_slot<kBrickTab, kProbes>(T.key, c);
    if (sl >= 0) {
      atomicAdd(&T.v[0][sl], m);
      if (sx) atomicAdd(&T.v[1][sl], sx);
      if (ly) atomicAdd(&T.v[2][sl], m * ly);
      if (lz) atomicAdd(&T.v[3][sl], m * lz);
    } else {
      F.sums.add(c, m, (unsigned long long)m * x0 + sx, (unsigned long long)m * (y0 + ly),
                 (unsigned long long)m * (z0 + lz));
    }
  }
}

// Cell ids of a brick's voxels at the end of a pass: the relaxation's keys,
// or the level search's cells, where a voxel not reached (in an incremental
// pass: an invalid one not reached again) is set to NONE on the way.
template <class KT>
struct KeySource {
  const KT *key;
  uint32_t idmask;
  __device__ __forceinline__ uint32_t id(int64_t b, int loc) const {
    const KT k = key[b * (kRows * BX) + loc];
    return k == (KT)~(KT)0 ? kNone : (uint32_t)k & idmask;
  }
};
template <bool INC>
struct LevelSource {
  const uint16_t *vis, *inv;
  uint32_t *cellb;
  __device__ __forceinline__ uint32_t id(int64_t b, int loc) const {
    const int64_t rr = b * kRows + (loc >> 4);
    bool miss = !((vis[rr] >> (loc & 15)) & 1u);
    if (INC) miss = miss && ((inv[rr] >> (loc & 15)) & 1u);
    const size_t bi = (size_t)b * (kRows * BX) + loc;
    if (miss) cellb[bi] = kNone;
    return miss ? kNone : cellb[bi];
  }
};

// One workgroup per brick.  Workgroups are dealt to the eight XCDs in turn:
// XCD i % 8 takes the i-th eighth of the bricks, so that x-adjacent bricks,
// which share the 128-byte lines of the weights, meet in one L2.
//
// Bound by the row scans and the LDS table.  379 x 251 x 147 voxels in 77192
// cells take 52 us; slabs with a table of 256 cells, which a slab's thousands
// overflow, 207 us, and a full table searched to its end before the global
// atomics (249 us for one 64^3 volume in 12627 cells; now 18).
template <class Src>
__device__ __forceinline__ void d_brick_sums(const Src &src, Geom g, VTGrid bg, const Fuse &F, BrickTab &T) {
  const int t = threadIdx.x;
  const int64_t per = (bg.nbricks + 7) / 8;
  for (int64_t i = blockIdx.x; i < 8 * per; i += gridDim.x) {
    const int64_t b = (i & 7) * per + (i >> 3);
    if (b >= bg.nbricks) continue;
    const int x0 = (int)(b % bg.nbx) * BX, y0 = (int)((b / bg.nbx) % bg.nby) * BY,
              z0 = (int)(b / ((int64_t)bg.nbx * bg.nby)) * BZ;
    for (int k = t; k < kBrickTab; k += kVTThreads) {
      T.key[k] = kNone;
      T.v[0][k] = T.v[1][k] = T.v[2][k] = T.v[3][k] = 0u;
    }
    __syncthreads();
    const int x = x0 + (t & 15), y = y0 + (t >> 4);
    const bool xy = x < g.nx && y < g.ny;
    constexpr int kAhead = 4;  // voxels whose loads are issued together
    for (int z1 = 0; z1 < BZ; z1 += kAhead) {
      uint32_t c[kAhead], wt[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const bool in = xy && z0 + z1 + u < g.nz;
        c[u] = in ? src.id(b, (z1 + u) * kVTThreads + t) : kNone;
        wt[u] = !in ? 0u : F.w ? (uint32_t)F.w[x + (int64_t)g.nx * (y + (int64_t)g.ny * (z0 + z1 + u))] : 1u;
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        brick_row_runs(T, F, c[u], wt[u], (uint32_t)x0, (uint32_t)y0, (uint32_t)z0, (uint32_t)t >> 4,
                       (uint32_t)(z1 + u));
    }
    __syncthreads();
    // four lanes a cell, one sum each
    const uint32_t org = (t & 3) == 1 ? (uint32_t)x0 : (t & 3) == 2 ? (uint32_t)y0 : (uint32_t)z0;
    for (int k = t; k < 4 * kBrickTab; k += kVTThreads) {
      const uint32_t c = T.key[k >> 2], m = T.v[0][k >> 2];
      if (c == kNone || m == 0u) continue;
      const unsigned long long v =
          (k & 3) == 0 ? (unsigned long long)m : (unsigned long long)m * org + T.v[k & 3][k >> 2];
      atomicAdd(&F.sums.p[4 * (size_t)c + (k & 3)], v);
    }
    __syncthreads();
  }
}

// After the brick's rows (and a barrier): the table to global memory.  Ends
// with a barrier.
__device__ __forceinline__ void fin_flush(FinTab &T, const Fuse &F) {
  for (int i = threadIdx.x; i < kFinTab; i += blockDim.x) {
    const uint32_t c = T.tkey[i];
    if (c != kNone && T.tM[i]) F.sums.add(c, T.tM[i], T.tX[i], T.tY[i], T.tZ[i]);
  }
  __syncthreads();
}

// End of a relaxation pass: the keys to C-order cells (kNone where
// unreached) or, with SUMS, the centroid sums of the update that follows.
// One workgroup per slab of four x-adjacent bricks (64 x 16 x 16 voxels);
// lane l of every wave owns x = 64 sx + l, so a row's cells (256 B) and
// weights (128 B) are contiguous and each brick's 16 keys of the row are
// one 64 B run.  Wave w takes the slab's rows with z - z0 in [4w, 4w + 4),
// y fastest, eight rows per step with their loads issued together.  For
// the sums a lane keeps running totals (w, w (y - y0), w (z - z0)) of the
// cell it is in and adds them into the LDS table when its cell changes
// (w x = x times the mass, x being fixed per lane); the table goes to global
// memory once per slab.
constexpr int kFinRows = 8;
template <class KT, bool SUMS>
__device__ __forceinline__ void d_br_finish_slabs(const KT *__restrict__ key, Geom g, VTGrid bg, uint32_t idmask,
                                                  uint32_t *__restrict__ cell, const Fuse &F, FinTab *T) {
  const int t = threadIdx.x, lane = t & (kWave - 1), wv_id = t / kWave;
  const int nsx = (bg.nbx + 3) / 4;
  const int64_t nslabs = (int64_t)nsx * bg.nby * bg.nbz;
  for (int64_t sl = blockIdx.x; sl < nslabs; sl += gridDim.x) {
    const int sx = (int)(sl % nsx), by = (int)((sl / nsx) % bg.nby), bz = (int)(sl / ((int64_t)nsx * bg.nby));
    if constexpr (SUMS) {
      fin_clear(*T);
      __syncthreads();
    }
    const int bx = sx * 4 + (lane >> 4);
    const int x = bx * BX + (lane & 15);
    const bool has = bx < bg.nbx;  // the lane's brick exists
    const bool xin = x < g.nx;
    const int64_t b = (int64_t)(has ? bx : bg.nbx - 1) + (int64_t)bg.nbx * (by + (int64_t)bg.nby * bz);
    const KT *kb = key + (size_t)b * (kRows * BX) + (lane & 15);
    const int y0 = by * BY, z0 = bz * BZ;
    uint32_t cur = kNone, m = 0, sy = 0, sz = 0;  // the lane's running sums (below 2^26 over 64 rows)
    auto flush = [&]() {
      if (cur < F.S && m) {
        const unsigned long long M = m, X = (unsigned long long)m * (uint32_t)x,
                                 Y = (unsigned long long)m * (uint32_t)y0 + sy,
                                 Z = (unsigned long long)m * (uint32_t)z0 + sz;
        const int slot = lds_slot<kFinTab, kProbes>(T->tkey, cur);
        if (slot >= 0) {
          atomicAdd(&T->tM[slot], M);
          atomicAdd(&T->tX[slot], X);
          atomicAdd(&T->tY[slot], Y);
          atomicAdd(&T->tZ[slot], Z);
        } else {
          F.sums.add(cur, M, X, Y, Z);
        }
      }
    };
    for (int j0 = 0; j0 < kRows / (kVTThreads / kWave); j0 += kFinRows) {
      KT k[kFinRows];
      uint32_t wt[kFinRows];
#pragma unroll
      for (int u = 0; u < kFinRows; ++u) {
        const int r = (kRows / (kVTThreads / kWave)) * wv_id + j0 + u;  // (ly, lz) = (r & 15, r >> 4)
        const bool rin = y0 + (r & 15) < g.ny && z0 + (r >> 4) < g.nz;
        k[u] = has && rin ? kb[r * BX] : BRKey<KT>::inf;
        if constexpr (SUMS) {
          const int64_t v = (int64_t)g.nx * ((y0 + (r & 15)) + (int64_t)g.ny * (z0 + (r >> 4))) + x;
          wt[u] = xin && rin ? (F.w ? (uint32_t)F.w[v] : 1u) : 0u;
        }
      }
#pragma unroll
      for (int u = 0; u < kFinRows; ++u) {
        const int r = (kRows / (kVTThreads / kWave)) * wv_id + j0 + u;
        const int ly = r & 15, lz = r >> 4;
        const bool in = xin && y0 + ly < g.ny && z0 + lz < g.nz;
        const uint32_t c = k[u] == BRKey<KT>::inf ? kNone : (uint32_t)k[u] & idmask;
        if constexpr (!SUMS) {
          if (in) cell[(int64_t)g.nx * ((y0 + ly) + (int64_t)g.ny * (z0 + lz)) + x] = c;
        } else {
          const uint32_t cc = in ? c : kNone;
          if (cc != cur) {
            flush();
            cur = cc;
            m = sy = sz = 0;
          }
          m += wt[u];
          sy += wt[u] * (uint32_t)ly;
          sz += wt[u] * (uint32_t)lz;
        }
      }
    }
    if constexpr (SUMS) {
      flush();
      __syncthreads();
      fin_flush(*T, F);
    }
  }
}

template <class KT>
__global__ __launch_bounds__(kVTThreads) void k_br_finish_sums(const KT *__restrict__ key, Geom g, VTGrid bg,
                                                               uint32_t idmask, Fuse F) {
  __shared__ FinTab T;
  d_br_finish_slabs<KT, true>(key, g, bg, idmask, nullptr, F, &T);
}
template <class Src>
__global__ __launch_bounds__(kVTThreads) void k_brick_sums(Src src, Geom g, VTGrid bg, Fuse F) {
  __shared__ BrickTab T;
  d_brick_sums(src, g, bg, F, T);
}
template <class KT>
__global__ __launch_bounds__(kVTThreads) void k_br_finish(const KT *__restrict__ key, Geom g, VTGrid bg,
                                                          uint32_t idmask, uint32_t *__restrict__ cell) {
  d_br_finish_slabs<KT, false>(key, g, bg, idmask, cell, Fuse{}, nullptr);
}

// One workgroup per 64x8x8 tile; each wave takes rows of the tile with one
// lane per voxel (coalesced loads).  A segmented scan over the lanes sums
// (w, w x) over each run of equal cell id; the last lane of a run adds the
// run into an LDS hash table keyed by cell id, and the table is flushed with
// one set of global atomics per distinct cell in the tile.  Along a row y
// and z are fixed, so S_y = M y and S_z = M z per run.
//
// Where a few cells fill the volume, the atomics of all tiles on their sums
// queue up: with one lane adding a cell's four sums in turn 256^3 voxels in 7
// cells take 208 us and with 300 scattered cells 782, with four lanes adding
// them at once (one request to the line that holds them) 124 and 256.
constexpr int TX = 64, TY = 8, TZ = 8;
constexpr int kTabCap = 512;

__global__ __launch_bounds__(256) void k_centroid(const uint32_t *__restrict__ cell, const uint16_t *__restrict__ w,
                                                  Geom g, uint32_t S, Sums sums) {
  __shared__ uint32_t tkey[kTabCap];
  __shared__ unsigned long long tv[4][kTabCap];  // M, X, Y, Z
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY, ntz = (g.nz + TZ - 1) / TZ;
  const int64_t ntiles = (int64_t)ntx * nty * ntz;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    for (int i = t; i < kTabCap; i += 256) {
      tkey[i] = kNone;
      tv[0][i] = tv[1][i] = tv[2][i] = tv[3][i] = 0ull;
    }
    __syncthreads();
    const int tx = (int)(tile % ntx), ty = (int)((tile / ntx) % nty), tz = (int)(tile / ((int64_t)ntx * nty));
    const int x = tx * TX + lane;
    for (int r = wid; r < TY * TZ; r += 256 / kWave) {
      const int y = ty * TY + (r & 7), z = tz * TZ + (r >> 3);
      if (y >= g.ny || z >= g.nz) continue;  // uniform across the wave
      const bool in = x < g.nx;
      const int64_t v = x + (int64_t)g.nx * (y + (int64_t)g.ny * z);
      const uint32_t c = in ? cell[v] : kNone;
      const uint32_t wv = in ? (w ? (uint32_t)w[v] : 1u) : 0u;
      // segmented inclusive scan over runs of equal c
      const uint32_t cl = __shfl_up(c, 1, kWave), cr = __shfl_down(c, 1, kWave);
      const bool head = lane == 0 || cl != c;
      const bool tail = lane == kWave - 1 || cr != c;
      uint32_t m = wv;
      uint64_t sx = (uint64_t)wv * (uint64_t)x;
      bool seg = head;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t mo = __shfl_up(m, d, kWave);
        const uint64_t so = __shfl_up(sx, d, kWave);
        const bool fo = __shfl_up(seg ? 1 : 0, d, kWave) != 0;
        if (lane >= d && !seg) {
          m += mo;
          sx += so;
          seg = fo;
        }
      }
      if (tail && c < S && m) {
        const int sl = lds_slot<kTabCap, kProbes>(tkey, c);
        if (sl >= 0) {
          atomicAdd(&tv[0][sl], (unsigned long long)m);
          atomicAdd(&tv[1][sl], (unsigned long long)sx);
          atomicAdd(&tv[2][sl], (unsigned long long)m * (uint64_t)y);
          atomicAdd(&tv[3][sl], (unsigned long long)m * (uint64_t)z);
        } else {
          sums.add(c, m, sx, (unsigned long long)m * (uint64_t)y, (unsigned long long)m * (uint64_t)z);
        }
      }
    }
    __syncthreads();
    // four lanes a cell, one sum each: one request to the line that holds them
    for (int i = t; i < 4 * kTabCap; i += 256) {
      const uint32_t c = tkey[i >> 2];
      if (c != kNone && tv[0][i >> 2]) atomicAdd(&sums.p[4 * (size_t)c + (i & 3)], tv[i & 3][i >> 2]);
    }
    __syncthreads();
  }
}


struct U128 {
  uint64_t hi, lo;
};
__device__ __forceinline__ U128 sq64(uint64_t a) { return U128{__umul64hi(a, a), a * a}; }
__device__ __forceinline__ U128 add128(U128 a, U128 b) {
  uint64_t lo = a.lo + b.lo;
  return U128{a.hi + b.hi + (lo < a.lo ? 1ull : 0ull), lo};
}
__device__ __forceinline__ bool lt128(U128 a, U128 b) { return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo); }
__device__ __forceinline__ U128 shl2(U128 a) { return U128{(a.hi << 2) | (a.lo >> 62), a.lo << 2}; }
__device__ __forceinline__ uint64_t absdiff(uint64_t a, uint64_t b) { return a > b ? a - b : b - a; }

__device__ __forceinline__ uint64_t round_half_down(uint64_t S, uint64_t M) { return (2 * S + M - 1) / (2 * M); }

__device__ __forceinline__ double move_len(uint32_t a, uint32_t b, Geom g) {
  int64_t ax = a % (uint32_t)g.nx, ar = a / (uint32_t)g.nx, ay = ar % (uint32_t)g.ny, az = ar / (uint32_t)g.ny;
  int64_t bx = b % (uint32_t)g.nx, br = b / (uint32_t)g.nx, by = br % (uint32_t)g.ny, bz = br / (uint32_t)g.ny;
  double dx = (double)(ax - bx), dy = (double)(ay - by), dz = (double)(az - bz);
  return sqrt(dx * dx + dy * dy + dz * dz);
}

// moved[s] records whether site s moved (the next Voronoi pass is
// incremental over the moved sites).
template <class View>
__device__ __forceinline__ void d_snap(const View &cell, Geom g, uint32_t S, Sums sums, uint32_t *sites, double *ds,
                                       uint8_t *moved, uint32_t *fb_list, uint32_t *fb_cnt) {
  __shared__ uint32_t cnt_s, base_s;
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  bool out = false;  // the rounded centroid lies outside the site's cell
  if (s < S) {
    const unsigned long long *sm = sums.p + 4 * (size_t)s;
    const uint64_t M = sm[0];
    uint32_t old = sites[s];
    moved[s] = 0;
    if (M == 0) {
      if (ds) ds[s] = 0.0;
    } else {
      const uint64_t qx = round_half_down(sm[1], M), qy = round_half_down(sm[2], M), qz = round_half_down(sm[3], M);
      const uint32_t q = (uint32_t)(qx + (uint64_t)g.nx * (qy + (uint64_t)g.ny * qz));
      out = cell.id((int32_t)qx, (int32_t)qy, (int32_t)qz) != s;
      if (!out) {
        sites[s] = q;
        moved[s] = q != old;
        if (ds) ds[s] = move_len(old, q, g);
      }
    }
  }
  // one atomic on the list's length for each workgroup: they queue up (27 ns each)
  if (threadIdx.x == 0) cnt_s = 0u;
  __syncthreads();
  const uint64_t m = __ballot(out);
  uint32_t pos = 0;
  if (m && lane_id() == 0) pos = atomicAdd(&cnt_s, (uint32_t)__popcll(m));
  pos = __shfl(pos, 0, kWave) + (uint32_t)__popcll(m & lanemask_lt());
  __syncthreads();
  if (threadIdx.x == 0 && cnt_s) base_s = atomicAdd(fb_cnt, cnt_s);
  __syncthreads();
  if (out) fb_list[base_s + pos] = s;
}
template <class View>
__global__ void k_snap(View cell, Geom g, uint32_t S, Sums sums, uint32_t *sites, double *ds, uint8_t *moved,
                       uint32_t *fb_list, uint32_t *fb_cnt) {
  d_snap(cell, g, S, sums, sites, ds, moved, fb_list, fb_cnt);
}

// Exact nearest in-cell voxel by growing cubes around the centroid: half-widths
// up to kSnapNear by one wave (W = 1), from 2 kSnapNear on by a team of W waves.
// The site's own voxel, if it lies in the cell, is a first candidate, and a
// voxel farther from the centroid than the best one so far is left out without
// being read, in float64 with a margin far above its rounding.  What is read is
// compared exactly, so the answer is that of the whole search.  The team's waves
// take planes of the cube, 16, 32 or 64 lanes a row of it (by its width), eight
// rows in flight.  Returns false when the search has to go on beyond kSnapNear.
//
// Flat: volumes of at most kFlatEdge voxels along an axis, where a cube of that
// half-width holds little and one plane (or row) of it would be all that a team
// has to share.  The near search goes to the half-width that holds about a
// thousand voxels (flat_near), and the team's lanes take the voxels of the box
// one after the other.  One update in this and the other form (nx x ny x nz):
// 1 x 256 x 256 with 512 voxels a site 71 and 83 us, 256 x 256 x 1 with 4096 47
// and 53; cells of 400 consecutive voxels, of which many are broken at a row's
// end: 2048 x 1 x 2048 12.1 and 21.0 ms, 1024 x 1024 x 2 2.9 and 15.6,
// 512 x 512 x 6 1.48 and 1.81, 512 x 8 x 512 0.56 and 0.37.  (Rows of the box
// over the lanes instead of its voxels leave most lanes idle where x is short:
// 8.5 ms for 1 x 1024 x 1024 and such cells of 209 voxels, now 1.7.)
constexpr int32_t kSnapNear = 4;
constexpr int32_t kFlatEdge = 6;
__device__ __forceinline__ int32_t flat_near(Geom g) {
  const int32_t t = min(g.nx, min(g.ny, g.nz));
  return t == 1 ? 16 : t == 2 ? 12 : t == 3 ? 9 : 6;
}
struct SnapLds {
  uint64_t hi[16], lo[16];
  uint32_t v[16];
};
template <int W, bool Flat, class View>
__device__ __forceinline__ bool snap_search(const View &cell, Geom g, const unsigned long long *sm, uint32_t s,
                                            uint32_t old, int w, SnapLds *L, uint32_t &bestv) {
  constexpr int kRowsAhead = 8;
  const int lane = lane_id();
  const uint64_t M = sm[0];
  const uint64_t Sa[3] = {sm[1], sm[2], sm[3]};
  const int32_t q[3] = {(int32_t)round_half_down(Sa[0], M), (int32_t)round_half_down(Sa[1], M),
                        (int32_t)round_half_down(Sa[2], M)};
  const int32_t ext[3] = {g.nx, g.ny, g.nz};
  const double dM = (double)M;
  const double cx = (double)Sa[0] / dM, cy = (double)Sa[1] / dM, cz = (double)Sa[2] / dM;
  auto dist = [&](int32_t x, int32_t y, int32_t z) {  // (M |v - c|)^2
    U128 D = sq64(absdiff(M * (uint64_t)x, Sa[0]));
    D = add128(D, sq64(absdiff(M * (uint64_t)y, Sa[1])));
    return add128(D, sq64(absdiff(M * (uint64_t)z, Sa[2])));
  };
  U128 best{~0ull, ~0ull};
  bestv = kNone;
  auto take = [&](U128 D, uint32_t v) {
    if (lt128(D, best) || (D.hi == best.hi && D.lo == best.lo && v < bestv)) {
      best = D;
      bestv = v;
    }
  };
  if ((int64_t)old < g.n) {  // (lsrvt_update takes any value as a site to be moved)
    const int32_t ox = (int32_t)(old % (uint32_t)g.nx), oy = (int32_t)(old / (uint32_t)g.nx % (uint32_t)g.ny),
                  oz = (int32_t)(old / (uint32_t)g.nx / (uint32_t)g.ny);
    if (cell.id(ox, oy, oz) == s) take(dist(ox, oy, oz), old);
  }
  // squared distance of the best voxel so far
  auto reach = [&]() {
    return bestv == kNone ? __builtin_inf()
                          : ((double)best.hi * 0x1p64 + (double)best.lo) / (dM * dM) * (1.0 + 1e-9) + 1e-3;
  };
  auto wave_best = [&](uint32_t before) {  // the best of the wave's lanes, unless none found a new one
    if (__ballot(bestv != before) == 0ull) return;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t h = __shfl_xor(best.hi, o, kWave), l = __shfl_xor(best.lo, o, kWave);
      const uint32_t v = __shfl_xor(bestv, o, kWave);
      take(U128{h, l}, v);
    }
  };
  auto done = [&](int32_t r) {
    bool whole = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) whole = whole && q[a] - r <= 0 && q[a] + r >= ext[a] - 1;
    return whole || (bestv != kNone && lt128(shl2(best), sq64(M * (uint64_t)(2 * (int64_t)r + 1))));
  };
  if constexpr (W == 1) {
    // cubes of fixed size, their voxels over the lanes
    auto cube = [&](auto half) {
      constexpr int R = decltype(half)::value, kSide = 2 * R + 1, kAll = kSide * kSide * kSide;
      constexpr int kAhead = kAll < 8 * kWave ? (kAll + kWave - 1) / kWave : 6;
      const double rho2 = reach();
      const uint32_t before = bestv;
      for (int i0 = lane; i0 < kAll + lane; i0 += kAhead * kWave) {
        uint32_t id[kAhead];
        int32_t x[kAhead], y[kAhead], z[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int i = i0 + u * kWave;
          x[u] = q[0] - R + i % kSide;
          y[u] = q[1] - R + i / kSide % kSide;
          z[u] = q[2] - R + i / (kSide * kSide);
          const double ex = x[u] - cx, ey = y[u] - cy, ez = z[u] - cz;
          const bool in = i < kAll && x[u] >= 0 && y[u] >= 0 && z[u] >= 0 && x[u] < ext[0] && y[u] < ext[1] &&
                          z[u] < ext[2] && ex * ex + ey * ey + ez * ez <= rho2;
          id[u] = in ? cell.id(x[u], y[u], z[u]) : kNone;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if (id[u] == s) take(dist(x[u], y[u], z[u]), (uint32_t)(x[u] + (int64_t)g.nx * (y[u] + (int64_t)g.ny * z[u])));
      }
      wave_best(before);
      return done(R);
    };
    auto box = [&](int32_t r) {  // the same for any half-width, the part in the volume only
      constexpr int kAhead = 5;
      uint32_t lo[3], len[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = (uint32_t)max(q[a] - r, 0);
        len[a] = (uint32_t)min(q[a] + r, ext[a] - 1) + 1u - lo[a];
      }
      const uint32_t all = len[0] * len[1] * len[2];
      const double rho2 = reach();
      const uint32_t before = bestv;
      for (uint32_t i0 = (uint32_t)lane; i0 < all + lane; i0 += kAhead * kWave) {
        uint32_t id[kAhead];
        int32_t x[kAhead], y[kAhead], z[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const uint32_t i = i0 + u * kWave, row = i / len[0];
          x[u] = (int32_t)(lo[0] + i - row * len[0]);
          y[u] = (int32_t)(lo[1] + row % len[1]);
          z[u] = (int32_t)(lo[2] + row / len[1]);
          const double ex = x[u] - cx, ey = y[u] - cy, ez = z[u] - cz;
          id[u] = i < all && ex * ex + ey * ey + ez * ez <= rho2 ? cell.id(x[u], y[u], z[u]) : kNone;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if (id[u] == s) take(dist(x[u], y[u], z[u]), (uint32_t)(x[u] + (int64_t)g.nx * (y[u] + (int64_t)g.ny * z[u])));
      }
      wave_best(before);
      return done(r);
    };
    if constexpr (Flat) {
      const int32_t near = flat_near(g);
      return box(near / 3) || box(near);
    }
    if (cube(std::integral_constant<int, kSnapNear / 2>{})) return true;
    return cube(std::integral_constant<int, kSnapNear>{});
  }
  for (int32_t r = 2 * (Flat ? flat_near(g) : kSnapNear);; r *= 2) {
    int32_t lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = q[a] - r < 0 ? 0 : q[a] - r;
      hi[a] = q[a] + r > ext[a] - 1 ? ext[a] - 1 : q[a] + r;
    }
    const double rho2 = reach();
    const uint32_t before = bestv;
    const int32_t width = hi[0] - lo[0] + 1;
    const int32_t XL = width <= 16 ? 16 : width <= 32 ? 32 : kWave;  // lanes of a row
    const int32_t per = kWave / XL;
    if constexpr (Flat) {
      constexpr int kFlatAhead = 4;
      const uint32_t nx = (uint32_t)width, ny = (uint32_t)(hi[1] - lo[1] + 1);
      const uint32_t all = nx * ny * (uint32_t)(hi[2] - lo[2] + 1);
      for (uint32_t i0 = (uint32_t)(w * kWave); i0 < all; i0 += (uint32_t)(W * kFlatAhead * kWave)) {
        uint32_t id[kFlatAhead];
        int32_t x[kFlatAhead], y[kFlatAhead], z[kFlatAhead];
#pragma unroll
        for (int u = 0; u < kFlatAhead; ++u) {
          const uint32_t i = i0 + (uint32_t)(u * W * kWave + lane), row = i / nx;
          x[u] = lo[0] + (int32_t)(i - row * nx);
          y[u] = lo[1] + (int32_t)(row % ny);
          z[u] = lo[2] + (int32_t)(row / ny);
          const double ex = x[u] - cx, ey = y[u] - cy, ez = z[u] - cz;
          id[u] = i < all && ex * ex + ey * ey + ez * ez <= rho2 ? cell.id(x[u], y[u], z[u]) : kNone;
        }
#pragma unroll
        for (int u = 0; u < kFlatAhead; ++u)
          if (id[u] == s) take(dist(x[u], y[u], z[u]), (uint32_t)(x[u] + (int64_t)g.nx * (y[u] + (int64_t)g.ny * z[u])));
      }
    } else {
      for (int32_t z = lo[2] + w; z <= hi[2]; z += W) {
        const double ez2 = (z - cz) * (z - cz);
        if (ez2 > rho2) continue;
        // the rows and the part of them within reach of the plane
        int32_t y0 = lo[1], y1 = hi[1], x0 = lo[0], x1 = hi[0];
        if (rho2 < 1e12) {
          const double half = sqrt(rho2 - ez2) + 1.0;
          y0 = max(y0, (int32_t)(cy - half));
          y1 = min(y1, (int32_t)(cy + half) + 1);
          x0 = max(x0, (int32_t)(cx - half));
          x1 = min(x1, (int32_t)(cx + half) + 1);
        }
        for (int32_t xc = x0; xc <= x1; xc += XL)
          for (int32_t yc = y0; yc <= y1; yc += kRowsAhead * per) {
            const int32_t x = xc + lane % XL;
            const double ex2 = (x - cx) * (x - cx) + ez2;
            uint32_t id[kRowsAhead];
#pragma unroll
            for (int u = 0; u < kRowsAhead; ++u) {
              const int32_t y = yc + u * per + lane / XL;
              const double ey = y - cy;
              id[u] = x <= x1 && y <= y1 && ex2 + ey * ey <= rho2 ? cell.id(x, y, z) : kNone;
            }
#pragma unroll
            for (int u = 0; u < kRowsAhead; ++u) {
              if (id[u] != s) continue;
              const int32_t y = yc + u * per + lane / XL;
              take(dist(x, y, z), (uint32_t)(x + (int64_t)g.nx * (y + (int64_t)g.ny * z)));
            }
          }
      }
    }
    wave_best(before);
    if (lane == 0) {
      L->hi[w] = best.hi;
      L->lo[w] = best.lo;
      L->v[w] = bestv;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < W; ++i) take(U128{L->hi[i], L->lo[i]}, L->v[i]);
    __syncthreads();
    if (done(r)) return true;
  }
}

__device__ __forceinline__ void snap_store(Geom g, uint32_t s, uint32_t old, uint32_t v, uint32_t *sites, double *ds,
                                           uint8_t *moved) {
  if (v != kNone) {
    sites[s] = v;
    moved[s] = v != old;
    if (ds) ds[s] = move_len(old, v, g);
  } else if (ds) {
    ds[s] = 0.0;
  }
}

// The sites whose rounded centroid lies outside their cell, in two steps: one
// wave a site looks within kSnapNear voxels, which is enough for almost all of
// them, and takes the finished ones off the list (kNone); the rest get a
// workgroup of sixteen waves each.
//
// Bound by the latency of the reads: 379 x 251 x 147 voxels in 77192 cells take
// 32 us an update (42 us with one workgroup of four waves for every site, one
// cube after another and all of it read), the flame loop (1024 x 512 x 512),
// whose few far sites are searched over cubes of 65^3 voxels and more, 110 us
// (326 us, with a 64-bit division per voxel).
constexpr int kSnapFarThreads = 1024;
template <bool Flat, class View>
__device__ __forceinline__ void d_snap_near(const View &cell, Geom g, Sums sums, uint32_t *sites, double *ds,
                                            uint8_t *moved, uint32_t *fb_list, const uint32_t *fb_cnt) {
  const uint32_t count = *fb_cnt;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  for (uint32_t item = blockIdx.x * (256 / kWave) + w; item < count; item += gridDim.x * (256 / kWave)) {
    const uint32_t s = fb_list[item];
    const uint32_t old = sites[s];
    uint32_t v;
    if (!snap_search<1, Flat>(cell, g, sums.p + 4 * (size_t)s, s, old, 0, nullptr, v)) continue;
    if (lane_id() == 0) {
      snap_store(g, s, old, v, sites, ds, moved);
      fb_list[item] = kNone;
    }
  }
}
template <bool Flat, class View>
__device__ __forceinline__ void d_snap_far(const View &cell, Geom g, Sums sums, uint32_t *sites, double *ds,
                                           uint8_t *moved, const uint32_t *fb_list, const uint32_t *fb_cnt) {
  __shared__ SnapLds L;
  const uint32_t count = *fb_cnt;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  for (uint32_t item = blockIdx.x; item < count; item += gridDim.x) {
    const uint32_t s = fb_list[item];
    if (s == kNone) continue;  // uniform
    const uint32_t old = sites[s];
    uint32_t v;
    snap_search<kSnapFarThreads / kWave, Flat>(cell, g, sums.p + 4 * (size_t)s, s, old, w, &L, v);
    __syncthreads();  // every wave has read the site
    if (threadIdx.x == 0) snap_store(g, s, old, v, sites, ds, moved);
  }
}
template <bool Flat, class View>
__global__ __launch_bounds__(256) void k_snap_near(View cell, Geom g, Sums sums, uint32_t *sites, double *ds,
                                                   uint8_t *moved, uint32_t *fb_list, const uint32_t *fb_cnt) {
  d_snap_near<Flat>(cell, g, sums, sites, ds, moved, fb_list, fb_cnt);
}
template <bool Flat, class View>
__global__ __launch_bounds__(kSnapFarThreads) void k_snap_far(View cell, Geom g, Sums sums, uint32_t *sites,
                                                              double *ds, uint8_t *moved, const uint32_t *fb_list,
                                                              const uint32_t *fb_cnt) {
  d_snap_far<Flat>(cell, g, sums, sites, ds, moved, fb_list, fb_cnt);
}


// Mean of ds[0..S) in a fixed order: 256 contiguous chunks summed by 256
// workgroups, then the chunk sums in order by one workgroup.
constexpr int kMeanParts = 256;
__global__ __launch_bounds__(256) void k_mean_ds_part(const double *ds, uint32_t S, double *part) {
  __shared__ double red[256];
  const uint32_t chunk = (S + kMeanParts - 1) / kMeanParts;
  const uint32_t b0 = blockIdx.x * chunk;
  const uint32_t b1 = b0 + chunk < S ? b0 + chunk : S;
  double acc = 0.0;
  for (uint32_t i = b0 + threadIdx.x; i < b1; i += 256) acc += ds[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_mean_ds(const double *part, uint32_t S, double *out) {
  __shared__ double red[256];
  red[threadIdx.x] = part[threadIdx.x];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = S ? red[0] / (double)S : 0.0;
}

__device__ __forceinline__ void d_init_sites(const uint32_t *__restrict__ seeds, uint32_t S, const uint32_t *__restrict__ comp, Geom g,
                             uint32_t *sites, uint32_t *site_comp, uint32_t *err) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  uint32_t v = seeds[s];
  if ((int64_t)v >= g.n) {
    atomicOr(err, 1u);
    v = 0;  // keep later kernels in bounds; the call reports EINVAL
  }
  sites[s] = v;
  site_comp[s] = comp[v];
}
__global__ void k_init_sites(const uint32_t *__restrict__ seeds, uint32_t S, const uint32_t *__restrict__ comp, Geom g,
                             uint32_t *sites, uint32_t *site_comp, uint32_t *err) { d_init_sites(seeds, S, comp, g, sites, site_comp, err); }


// ----------------------------------------------------------------------------
// host side

struct CvtWork {
  uint32_t *eq;
  uint16_t *fr, *vis, *yf;
  unsigned long long *xf;
  uint32_t *act, *ctl;  // brick marks; ctl[0..2] level alive flags, ctl[3] error bits, ctl[4] next wake level
  uint32_t *fb_list, *fb_cnt, *err;
  uint32_t *hist;
  uint32_t *cellb;           // [nbricks][4096] cells, brick-major (the search's own copy)
  uint32_t *dist;            // [nbricks][4096] hop distance of every reached voxel, brick-major
  uint16_t *inv;             // [nbricks][256] invalid voxels (incremental passes)
  uint32_t *bnd, *bcnt, *wake;  // kept-voxel lists per brick, their counts and wake levels
  uint8_t *moved;            // [S] site moved in the last update
  unsigned long long *xface; // [nbricks][2][256] packed x faces of the brick relaxation keys
  uint32_t *brlist;          // [nbricks] bricks of a relaxation round
  unsigned long long *sums;  // 4 x S
  double *ds, *mean, *mean_part;
};

VTGrid vt_grid(const Geom &g) {
  VTGrid bg;
  bg.nbx = (g.nx + BX - 1) / BX;
  bg.nby = (g.ny + BY - 1) / BY;
  bg.nbz = (g.nz + BZ - 1) / BZ;
  bg.nbricks = (int64_t)bg.nbx * bg.nby * bg.nbz;
  return bg;
}

template <class A>
void cvt_layout(A &a, const Geom &g, uint32_t S, int32_t iters, CvtWork *W) {
  VTGrid bg = vt_grid(g);
  int64_t nb = bg.nbricks;
  size_t s1 = S ? S : 1;
  const bool inc = iters > 0;  // incremental passes follow the first one
  auto eq = a.template take<uint32_t>(nb * kRows * 3);
  // the search state of a pass, cleared together (clear_pass, run_br_k)
  auto fr = a.template take<uint16_t>(2 * nb * kRows);
  auto vis = a.template take<uint16_t>(nb * kRows);
  auto xf = a.template take<unsigned long long>(2 * nb * 8);
  auto yf = a.template take<uint16_t>(2 * nb * 32);
  auto act = a.template take<uint32_t>(2 * nb);
  auto ctl = a.template take<uint32_t>(8 + 2 * 8 + kHistLen);  // flags, diagnostic counters, visits per level
  auto fbl = a.template take<uint32_t>(s1);
  auto fbc = a.template take<uint32_t>(4);
  auto sums = a.template take<unsigned long long>(4 * s1);
  auto ds = a.template take<double>(s1);
  auto mean = a.template take<double>(iters > 0 ? iters : 1);
  auto mpart = a.template take<double>(kMeanParts);
  auto hist = a.template take<uint32_t>(kHistLen);
  auto cellb = a.template take<uint32_t>(nb * kRows * BX);
  auto dist = a.template take<uint32_t>(nb * kRows * BX);
  auto moved = a.template take<uint8_t>(s1);
  auto xface = a.template take<unsigned long long>(nb * 512);
  auto brlist = a.template take<uint32_t>(nb);
  auto inv = a.template take<uint16_t>(inc ? nb * kRows : 1);
  auto bnd = a.template take<uint32_t>(inc ? nb * kRows * BX : 1);
  auto bcnt = a.template take<uint32_t>(inc ? nb : 1);
  auto wake = a.template take<uint32_t>(inc ? nb : 1);
  if (W) {
    W->eq = eq;
    W->fr = fr;
    W->vis = vis;
    W->xf = xf;
    W->yf = yf;
    W->act = act;
    W->ctl = ctl;
    W->err = ctl + 3;
    W->fb_list = fbl;
    W->fb_cnt = fbc;
    W->sums = sums;
    W->ds = ds;
    W->mean = mean;
    W->mean_part = mpart;
    W->hist = hist;
    W->cellb = cellb;
    W->dist = dist;
    W->moved = moved;
    W->xface = xface;
    W->brlist = brlist;
    W->inv = inc ? inv : nullptr;
    W->bnd = inc ? bnd : nullptr;
    W->bcnt = inc ? bcnt : nullptr;
    W->wake = inc ? wake : nullptr;
  }
}

struct SizerT : Sizer {
  template <class T>
  T *take(size_t c) {
    Sizer::take<T>(c);
    return nullptr;
  }
};

size_t cvt_workspace(const Geom &g, uint32_t S, int32_t iters) {
  SizerT z;
  cvt_layout(z, g, S, iters, nullptr);
  return z.off + 256;
}

int32_t carve_cvt(void *d_work, size_t bytes, const Geom &g, uint32_t S, int32_t iters, CvtWork &W) {
  Carve cv(d_work, bytes);
  cvt_layout(cv, g, S, iters, &W);
  return cv.ok ? LSRVT_OK : LSRVT_EWORKSPACE;
}

// Driver state of one Lloyd run: the levels or rounds of the previous
// passes, which size the first batch of launches of the next one.
struct VTState {
  uint32_t levels = 0;      // levels of the last full pass
  uint32_t inc_levels = 0;  // levels of the first run of the last incremental pass
  uint32_t br_rounds = 0;   // rounds of the last full brick relaxation pass
  uint32_t br_rounds_inc = 0;  // rounds of the last incremental one
  bool bricks = false;      // passes by brick relaxation (else by level search)
  bool keys_set = false;    // the key width of the brick relaxation is chosen at its first pass
  uint32_t id_bits = 0;     // narrow keys: the id field's bits; 0: wide keys
  uint32_t br_work = 0;     // bricks relaxed by a pass that outgrew its narrow keys (0: not counted)
  const uint8_t *band = nullptr;  // the bands of the call
};

// Which schedule computes the Voronoi passes: the level-synchronous search
// or the brick relaxation (both give the same regions bit for bit).  The
// choice is made per host thread (lsrvt_set_vt_engine); by default the brick
// relaxation, which was the faster one for every volume and cell width tried with
// sites drawn by lsrvt_seed (and see levels_after_bricks).
// Levels against bricks: 8^3 with a site for every voxel or two, 10 updates,
// 1.52 and 1.18 ms; 25^3 with a site a voxel, one pass, 0.165 and 0.138; 64^3,
// 1.6 voxels a site, 10 updates, 1.80 and 1.41; one pass of 192 x 96 x 96 1.6
// and 0.67; 379 x 251 x 147 with 20 updates 27.3 and 12.3; 512 x 256 x 256
// flame block with 10 updates 52.9 and 8.4.  Thin volumes too, although their
// bricks are mostly empty (10 updates, 64 voxels a site): 2048 x 2048 x 1 in each
// of its three orientations 14.4 to 18.2 and 6.4 to 8.5, 2 x 1448 x 1448 8.1 and
// 6.0 (the closest of 19 shapes of one to 16 voxels along an axis, with 64, 512 and
// 4096 voxels a site: 1.3 to 6.3 times), 32767 x 1 x 1 2.4 and 1.4.
enum class VTEngine { Auto = 0, Levels = 1, Bricks = 2 };

thread_local VTEngine t_engine = VTEngine::Auto;

VTEngine vt_engine() {
  VTEngine e = t_engine;
  if (e == VTEngine::Auto) {
    static const char *env = getenv("LSRVT_VT_ENGINE");
    e = env && env[0] == 'l' ? VTEngine::Levels : VTEngine::Bricks;
  }
  return e;
}

// Benchmark timing of the Voronoi passes' dominant kernel (levels or
// relaxation rounds): while enabled, an event pair on the launch stream
// around every batch of launches; read back by lsrvt_timing_read.
struct KernelTimer {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending, pool;
  double ms = 0.0;
  uint64_t launches = 0;
  uint64_t passes = 0;
  int64_t voxels_per_pass = 0;
  int32_t engines = 0;  // bit 0: level passes recorded, bit 1: relaxation passes
};
// one timer per host thread: calls issued from different threads (streams)
// never share instrumentation state
KernelTimer &timer() {
  thread_local KernelTimer t;
  return t;
}

int32_t timed_begin(hipStream_t s, std::pair<hipEvent_t, hipEvent_t> &ev) {
  KernelTimer &T = timer();
  std::lock_guard<std::mutex> lk(T.mu);
  if (T.pool.empty()) {
    hipEvent_t a, b;
    LSRVT_HIP(hipEventCreate(&a));
    LSRVT_HIP(hipEventCreate(&b));
    T.pool.push_back({a, b});
  }
  ev = T.pool.back();
  T.pool.pop_back();
  LSRVT_HIP(hipEventRecord(ev.first, s));
  return LSRVT_OK;
}

int32_t timed_end(hipStream_t s, const std::pair<hipEvent_t, hipEvent_t> &ev, uint64_t launches) {
  KernelTimer &T = timer();
  LSRVT_HIP(hipEventRecord(ev.second, s));
  std::lock_guard<std::mutex> lk(T.mu);
  T.pending.push_back(ev);
  T.launches += launches;
  return LSRVT_OK;
}

// End of a pass: the brick-major cells are written to the caller's C-order
// cell array, row by row (16 contiguous voxels), with LSRVT_NONE for voxels
// never reached: in a full pass those of components without a site; in an
// incremental pass the invalid voxels not reached again (none: a moved site
// stays in its component), whose brick-major entry is set to NONE as well.
template <bool INC>
__global__ __launch_bounds__(kVTThreads) void k_vt_finish(const uint16_t *__restrict__ vis,
                                                          const uint16_t *__restrict__ inv, Geom g, VTGrid bg,
                                                          uint32_t *__restrict__ cellb, uint32_t *__restrict__ cell) {
  const int t = threadIdx.x;
  const int lx = t & 15;
  for (int64_t rr = (int64_t)blockIdx.x * (kVTThreads / BX) + (t >> 4); rr < bg.nbricks * kRows;
       rr += (int64_t)gridDim.x * (kVTThreads / BX)) {
    const int64_t b = rr / kRows;
    const int row = (int)(rr % kRows);
    const int bx = (int)(b % bg.nbx), by = (int)((b / bg.nbx) % bg.nby), bz = (int)(b / ((int64_t)bg.nbx * bg.nby));
    const int x = bx * BX + lx, y = by * BY + (row & 15), z = bz * BZ + (row >> 4);
    if (x >= g.nx || y >= g.ny || z >= g.nz) continue;
    const size_t bi = (size_t)rr * BX + lx;
    bool miss = !((vis[rr] >> lx) & 1u);
    if (INC) miss = miss && ((inv[rr] >> lx) & 1u);
    uint32_t c = cellb[bi];
    if (miss) {
      c = kNone;
      cellb[bi] = kNone;
    }
    cell[x + (int64_t)g.nx * (y + (int64_t)g.ny * z)] = c;
  }
}

// Site voxels cleared before level 0 of a full pass (brick-major cells).
__global__ void k_sites_clear(const uint32_t *__restrict__ sites, uint32_t S, BFSArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < S && (int64_t)sites[s] < A.g.n) A.cell[brick_pos(A, sites[s]).bi] = kNone;
}

unsigned brick_grid(const VTGrid &bg) { return (unsigned)std::min<int64_t>(bg.nbricks, 65535); }
// workgroups of d_brick_sums (a multiple of 8)
unsigned sums_grid(const VTGrid &bg) { return (unsigned)std::min<int64_t>((bg.nbricks + 7) / 8 * 8, 65528); }

// Workgroups of the relaxation's finish: one per slab of four x-adjacent bricks.
int64_t br_slabs(const VTGrid &bg) { return (int64_t)((bg.nbx + 3) / 4) * bg.nby * bg.nbz; }
unsigned slab_grid(const VTGrid &bg) { return (unsigned)std::min<int64_t>(br_slabs(bg), 65535); }

unsigned finish_grid(const VTGrid &bg) {
  const int64_t g = (bg.nbricks * kRows + kVTThreads / BX - 1) / (kVTThreads / BX);
  return (unsigned)(g < 65535 ? g : 65535);
}

// The edge masks of the bands in the form of the call's schedule.
int32_t vt_masks(const Geom &g, CvtWork &W, const VTState &st, hipStream_t s) {
  VTGrid bg = vt_grid(g);
  if (st.bricks) {
    hipLaunchKernelGGL(k_br_masks, dim3(brick_grid(bg)), dim3(kVTThreads), 0, s, st.band, g, bg, W.eq);
    LSRVT_LAUNCHED();
    return LSRVT_OK;
  }
  const int64_t slots = bg.nbricks * kRows * BX;
  const unsigned grid = (unsigned)std::min<int64_t>((slots + kVTThreads - 1) / kVTThreads, 65535);
  hipLaunchKernelGGL(k_vt_eq, dim3(grid), dim3(kVTThreads), 0, s, st.band, g, bg, W.eq);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}

// The schedule of the call's passes and its masks.
int32_t vt_prepare(const uint8_t *band, const Geom &g, CvtWork &W, VTState &st, hipStream_t s) {
  st.band = band;
  st.bricks = vt_engine() == VTEngine::Bricks;
  return vt_masks(g, W, st, s);
}

// Whether a call goes on by levels (by the library's choice only) where its narrow
// keys ran out of distance, or where its sites outnumber their 24 bits and the first
// pass has not ended after kLongPass rounds; work: the bricks relaxed in all rounds
// until then.  Where sites are many, narrow keys hold a few hundred hops, and a pass
// that needs more has long winding paths among them: noise with a site for every
// component, near the fraction at which a band's largest component reaches through
// the volume.  Its bricks are relaxed some twenty times, where a level touches only
// what it reaches.  By levels and with wide keys, one pass over three random bands:
// 256^3 voxels (7.4 a site, 6.7 relaxations a brick so far) 12.4 and 19.2 ms, 300^3
// 17.5 and 38.8, 360^3 (3.1 so far) 24.6 and 57.9, 512^3 59 and 113.  Long straight paths
// past many sites relax few bricks: 512 x 512 x 128 (8 a site, 0.9 so far) 12.8 and
// 1.7 ms.  With fewer than four voxels a site most components are a few voxels:
// 256^3 in six noisy bands (2.9 a site, 4.1 so far) 9.7 and 7.2.  (With sites drawn
// by lsrvt_seed passes over such volumes end within 20 rounds and far from the limit,
// and the relaxation takes 0.4 to 0.9 of the levels' time.)
constexpr uint32_t kLongPass = 24;
bool levels_after_bricks(const Geom &g, uint32_t S, uint32_t work) {
  const int64_t per = g.n / (int64_t)std::max<uint32_t>(S, 1u);
  return t_engine == VTEngine::Auto && tuning(LSRVT_TUNE_KEY_BITS) == 0 && per >= 4 && per < 1024 &&
         (int64_t)work >= 2 * vt_grid(g).nbricks;
}

BFSArgs bfs_args(const Geom &g, CvtWork &W) {
  BFSArgs A;
  A.g = g;
  A.bg = vt_grid(g);
  A.eq = W.eq;
  A.fr = W.fr;
  A.vis = W.vis;
  A.xf = W.xf;
  A.yf = W.yf;
  A.cell = W.cellb;
  A.dist = W.dist;
  A.act = W.act;
  A.alive = W.ctl;
  A.hist = W.hist;
  A.err = W.err;
  A.inv = W.inv;
  A.bnd = W.bnd;
  A.bcnt = W.bcnt;
  A.wake = W.wake;
  static const bool debug_levels = getenv("LSRVT_DEBUG_LEVELS") != nullptr;
  A.dbg = debug_levels ? reinterpret_cast<unsigned long long *>(W.ctl + 8) : nullptr;
  return A;
}

// Clears the per-pass search state (frontiers, reached rows, marks, flags).
int32_t clear_pass(CvtWork &W, hipStream_t s) {
  // fr, vis, xf, yf, act and ctl follow each other in the workspace (cvt_layout),
  // the last up to its level flags ctl[0 .. 2]: one launch
  uint32_t *from = reinterpret_cast<uint32_t *>(W.fr);
  return fill<uint32_t>(from, W.ctl + 3 - from, 0u, s);
}

// Launches of the level kernel from level 1 on, enqueued in batches (the
// first one sized by the previous pass of the same kind, since sites move
// little between passes); after each batch the host reads the flags.  An
// incremental pass whose frontier dies out before every brick has injected
// its kept voxels continues at the smallest pending wake level.  Sets *redo
// when a kept-voxel list could not hold a level (the caller then runs a full
// pass).
template <bool INC>
int32_t run_levels(const Geom &g, const BFSArgs &A, CvtWork &W, VTState &st, hipStream_t s, bool *redo) {
  const VTGrid &bg = A.bg;
  const int64_t max_level = g.n + 2;
  const unsigned lgrid = (unsigned)std::min<int64_t>(8 * ((bg.nbricks + 7) / 8), 65528);
  const unsigned wgrid = (unsigned)std::min<int64_t>((bg.nbricks + 255) / 256, 1024);
  uint32_t L = 0;  // levels enqueued
  uint32_t run_end = 0;  // last level of the first run of consecutive launches
  bool jumped = false;
  int batch = INC ? (int)std::max<uint32_t>(8, st.inc_levels + 2) : (st.levels ? (int)st.levels + 4 : 16);
  int32_t rc;
  uint32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  while (true) {
    // one event pair around a batch of back-to-back level launches (while
    // timing is on): the launches of a batch run without gaps
    const bool timed = timer().on;
    std::pair<hipEvent_t, hipEvent_t> ev;
    if (timed && (rc = timed_begin(s, ev))) return rc;
    for (int i = 0; i < batch; ++i) {
      ++L;
      hipLaunchKernelGGL(k_bfs_level<INC>, dim3(lgrid), dim3(kLvlThreads), 0, s, A, L);
      LSRVT_LAUNCHED();
    }
    if (timed && (rc = timed_end(s, ev, (uint64_t)batch))) return rc;
    if (INC) {
      if ((rc = fill<uint32_t>(W.ctl + 4, 1, kNone, s))) return rc;
      hipLaunchKernelGGL(k_wake_min, dim3(wgrid), dim3(256), 0, s, W.wake, bg.nbricks, W.ctl + 4);
      LSRVT_LAUNCHED();
    }
    if ((rc = read_words(W.ctl, 8, c, s))) return rc;
    const uint32_t e = c[3];
    if (INC && (e & 4u)) {
      *redo = true;
      return LSRVT_OK;
    }
    if (e & 1u) return LSRVT_EINVAL;
    if (e) return LSRVT_EDEVICE;
    if (!jumped) run_end = L;
    if (c[(L + 1) % 3] == 0) {  // no brick marked for the next level
      if (!INC || c[4] == kNone) break;
      // nothing marked until the next wake level: go there
      if ((rc = fill<uint32_t>(W.ctl, 3, 0u, s))) return rc;
      L = c[4] - 1;
      jumped = true;
    }
    if ((int64_t)L > max_level) return LSRVT_EDEVICE;
    batch = 8;
  }
  // the length of the first run of alive levels sizes the first batch of
  // the next pass of the same kind
  const uint32_t nl = std::min<uint32_t>(run_end + 1, kHistLen);
  std::vector<uint32_t> h(nl, 0);
  if (nl > 1) {
    LSRVT_HIP(hipMemcpyAsync(h.data(), W.hist, sizeof(uint32_t) * nl, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
  }
  uint32_t levels = 0;
  while (levels + 1 < nl && h[levels + 1]) ++levels;
  (INC ? st.inc_levels : st.levels) = levels;
  static const bool debug_levels = getenv("LSRVT_DEBUG_LEVELS") != nullptr;
  if (debug_levels) {
    unsigned long long d[8];
    LSRVT_HIP(hipMemcpyAsync(d, W.ctl + 8, sizeof(d), hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
    fprintf(stderr, "[lsrvt] vt %s levels=%u last=%u visits=%llu cand=%llu big=%llu bigcand=%llu new=%llu inj=%llu\n",
            INC ? "inc" : "full", levels, L, d[0], d[1], d[2], d[3], d[4], d[5]);
    std::vector<uint32_t> pv(std::min<uint32_t>(L + 1, kHistLen));
    LSRVT_HIP(hipMemcpyAsync(pv.data(), W.ctl + 24, pv.size() * 4, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
    fprintf(stderr, "[lsrvt]   visits per level:");
    for (size_t i = 1; i < pv.size(); ++i) fprintf(stderr, " %u", pv[i]);
    fprintf(stderr, "\n");
    if ((rc = fill<uint32_t>(W.ctl + 8, 2 * 8 + kHistLen, 0u, s))) return rc;
  }
  return LSRVT_OK;
}

// One restricted Voronoi pass over every voxel: level 0 at the sites, then
// the level launches until the device reports an empty level.
int32_t run_vt(const Geom &g, const uint32_t *sites, uint32_t S, uint32_t *cell, CvtWork &W, VTState &st,
               hipStream_t s, const Fuse *fz = nullptr) {
  VTGrid bg = vt_grid(g);
  int32_t rc;
  if ((rc = clear_pass(W, s))) return rc;
  BFSArgs A = bfs_args(g, W);
  if (S) {
    hipLaunchKernelGGL(k_sites_clear, dim3((S + 255) / 256), dim3(256), 0, s, sites, S, A);
    hipLaunchKernelGGL(k_bfs_init, dim3((S + 255) / 256), dim3(256), 0, s, sites, S, A);
    LSRVT_LAUNCHED();
    bool redo = false;
    if ((rc = run_levels<false>(g, A, W, st, s, &redo))) return rc;
  }
  if (fz)
    hipLaunchKernelGGL(k_brick_sums<LevelSource<false>>, dim3(sums_grid(bg)), dim3(kVTThreads), 0, s,
                       (LevelSource<false>{W.vis, W.inv, W.cellb}), g, bg, *fz);
  else
    hipLaunchKernelGGL(k_vt_finish<false>, dim3(finish_grid(bg)), dim3(kVTThreads), 0, s, W.vis, W.inv, g, bg,
                       W.cellb, cell);
  LSRVT_LAUNCHED();
  if (timer().on) {
    std::lock_guard<std::mutex> lk(timer().mu);
    timer().passes += 1;
    timer().engines |= 1;
    timer().voxels_per_pass = g.n;
  }
  return LSRVT_OK;
}

// One incremental pass after an update: cell and dist hold the previous
// pass's keys and W.moved flags the sites that moved.  The result is that of
// a full pass with the new sites (see the incremental-pass notes above).
int32_t run_vt_inc(const Geom &g, const uint32_t *sites, uint32_t S, uint32_t *cell, CvtWork &W, VTState &st,
                   hipStream_t s, const Fuse *fz = nullptr) {
  if (!W.inv || S == 0) return run_vt(g, sites, S, cell, W, st, s, fz);
  VTGrid bg = vt_grid(g);
  int32_t rc;
  if ((rc = clear_pass(W, s))) return rc;
  BFSArgs A = bfs_args(g, W);
  const int64_t slots = bg.nbricks * kRows * BX;
  const unsigned rgrid = (unsigned)std::min<int64_t>((slots + kVTThreads - 1) / kVTThreads, 65535);
  hipLaunchKernelGGL(k_inc_reset, dim3(rgrid), dim3(kVTThreads), 0, s, W.cellb, W.moved, g, bg, W.inv);
  hipLaunchKernelGGL(k_inc_site_a, dim3((S + 255) / 256), dim3(256), 0, s, sites, S, A);
  hipLaunchKernelGGL(k_inc_site_b, dim3((S + 255) / 256), dim3(256), 0, s, sites, S, A);
  hipLaunchKernelGGL(k_bnd_build, dim3((unsigned)std::min<int64_t>(bg.nbricks, 65535)), dim3(kLvlThreads), 0, s, A);
  LSRVT_LAUNCHED();
  bool redo = false;
  if ((rc = run_levels<true>(g, A, W, st, s, &redo))) return rc;
  if (redo) {
    if ((rc = fill<uint32_t>(W.err, 1, 0u, s))) return rc;
    return run_vt(g, sites, S, cell, W, st, s, fz);
  }
  if (fz)
    hipLaunchKernelGGL(k_brick_sums<LevelSource<true>>, dim3(sums_grid(bg)), dim3(kVTThreads), 0, s,
                       (LevelSource<true>{W.vis, W.inv, W.cellb}), g, bg, *fz);
  else
    hipLaunchKernelGGL(k_vt_finish<true>, dim3(finish_grid(bg)), dim3(kVTThreads), 0, s, W.vis, W.inv, g, bg,
                       W.cellb, cell);
  LSRVT_LAUNCHED();
  static const bool debug_levels = getenv("LSRVT_DEBUG_LEVELS") != nullptr;
  if (debug_levels) {  // sizes of the pass: moved sites, invalid and changed voxels, listed kept voxels
    std::vector<uint8_t> mv(S);
    std::vector<uint16_t> iv(bg.nbricks * kRows), vs(bg.nbricks * kRows);
    std::vector<uint32_t> bc(bg.nbricks);
    LSRVT_HIP(hipMemcpyAsync(mv.data(), W.moved, S, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipMemcpyAsync(iv.data(), W.inv, iv.size() * 2, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipMemcpyAsync(vs.data(), W.vis, vs.size() * 2, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipMemcpyAsync(bc.data(), W.bcnt, bc.size() * 4, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
    uint64_t nm = 0, ni = 0, nv = 0, nbd = 0, nbk = 0;
    for (uint8_t m : mv) nm += m != 0;
    for (size_t i = 0; i < iv.size(); ++i) {
      ni += __builtin_popcount(iv[i]);
      nv += __builtin_popcount(vs[i]);
    }
    for (uint32_t c : bc) {
      nbd += c;
      nbk += c != 0;
    }
    fprintf(stderr, "[lsrvt]   moved=%llu invalid=%llu changed=%llu kept-listed=%llu in %llu bricks\n",
            (unsigned long long)nm, (unsigned long long)ni, (unsigned long long)nv, (unsigned long long)nbd,
            (unsigned long long)nbk);
  }
  if (timer().on) {
    std::lock_guard<std::mutex> lk(timer().mu);
    timer().engines |= 1;
    timer().passes += 1;
    timer().voxels_per_pass = g.n;
  }
  return LSRVT_OK;
}

// The id bits of narrow relaxation keys for S sites, or 0 for wide keys.
// Narrow keys need the ids 0 .. S - 1 in b bits and, by default, keep at
// least 8 distance bits (b <= 24).  LSRVT_TUNE_KEY_BITS = 64 asks for wide
// keys; 1 .. 30 for narrow keys with an id field of at least that many bits.
uint32_t narrow_id_bits(uint32_t S) {
  const int32_t kb = tuning(LSRVT_TUNE_KEY_BITS);
  if (kb == 64) return 0;
  uint32_t b = 1;
  while (b < 32 && ((uint64_t)1 << b) < (uint64_t)S) ++b;
  if (kb > 0 && (uint32_t)kb > b) b = (uint32_t)kb;
  return b <= (kb > 0 ? 30u : 24u) ? b : 0u;
}

// Relaxation arguments over the workspace; id_bits: narrow keys with that
// id field, 0: wide keys.
BRArgs br_args(const Geom &g, CvtWork &W, uint32_t id_bits) {
  BRArgs A;
  A.moved = nullptr;
  A.fsites = nullptr;
  A.hop32 = id_bits ? 1u << id_bits : 0u;
  A.idmask = id_bits ? (1u << id_bits) - 1u : 0xFFFFFFFFu;
  A.lim32 = id_bits ? (uint32_t)(((uint64_t)1 << 32) - ((uint64_t)2 << id_bits)) : 0u;
  A.g = g;
  A.bg = vt_grid(g);
  A.eq = W.eq;
  A.key = W.cellb;  // spans the cell and distance arrays (room for wide keys)
  A.xface = W.xface;
  A.mark = W.act;
  A.list = W.brlist;
  A.cnt = W.ctl + 14;
  A.ctl = W.ctl;
  A.alive = W.ctl + 4;
  A.hist = W.hist;
  static const bool debug_levels = getenv("LSRVT_DEBUG_LEVELS") != nullptr;
  A.dbg = debug_levels ? reinterpret_cast<unsigned long long *>(W.ctl + 8) : nullptr;
  return A;
}

// One Voronoi pass by brick relaxation with keys KT: a full pass from the
// sites, or (inc) an incremental one from the previous keys after the
// update that set W.moved.  Rounds are enqueued in batches (the first sized
// by the previous pass); after each batch the host reads whether any brick
// is marked.  With narrow keys, a round that stored a key of the largest
// exact distance sets *far and the pass stops unfinished, as with wide keys (where
// far is given) a long pass does that levels_after_bricks hands to the levels.
// Moved sites above which the reset is fused into the first rounds
// (k_br_reset_or_fuse).
// The separate reset reads every key and lets only the bricks that hold reset
// voxels work first; the fused one works on every brick and reads the keys
// once.  Always fusing takes 108.8 ms for the flame
// loop (1024 x 512 x 512, 30 updates), never 113.9, and 1.6 ms less than
// with 1.25 % of the sites as the limit, so the limit lies lower: a cube
// of the mean cell volume n / S overlaps about (edge / 16 + 1)^3 bricks,
// the bricks beside them work too, and 32 times that count over 80 % of
// the bricks is 0.3 % of the sites there.
uint32_t fuse_limit(const Geom &g, uint32_t S) {
  const double edge = std::cbrt((double)g.n / std::max<uint32_t>(S, 1u));
  const double overlap = 32.0 * std::pow(edge / BX + 1.0, 3.0);
  return (uint32_t)std::min(0.8 * (double)vt_grid(g).nbricks / overlap, 4294967295.0);
}

// Workgroups of the reset: each thread takes eight slots a step.  A grid that
// covers the slots once leaves seven of the eight loads idle and costs a fused
// pass of 379 x 251 x 147 voxels 15 us to start and end instead of 3.4, and the
// passes of sixteen jobs of 32^3 to 192^3 135 us instead of 21.
unsigned reset_grid(int64_t nkeys) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((nkeys + 2047) / 2048, 4096));
}

template <class KT>
int32_t run_br_k(const Geom &g, const uint32_t *sites, uint32_t S, uint32_t *cell, CvtWork &W, VTState &st,
                 bool inc, hipStream_t s, const Fuse *fz, bool *far) {
  const VTGrid bg = vt_grid(g);
  BRArgs A = br_args(g, W, sizeof(KT) == 4 ? st.id_bits : 0u);
  A.moved = W.moved;
  A.fsites = sites;
  constexpr KT kInf = BRKey<KT>::inf;
  int32_t rc;
  const int64_t nkeys = bg.nbricks * kRows * BX;
  // marks (act and ctl follow each other), flags, the last round and the list lengths
  if ((rc = fill<uint32_t>(W.act, W.ctl + 3 - W.act, 0u, s))) return rc;
  if ((rc = fill<uint32_t>(W.ctl + 4, 12, 0u, s))) return rc;
  if (!inc) {
    if ((rc = fill<KT>(static_cast<KT *>(A.key), nkeys, kInf, s))) return rc;
    if ((rc = fill<KT>(static_cast<KT *>(A.xface), bg.nbricks * 512, kInf, s))) return rc;
  } else {
    hipLaunchKernelGGL(k_count_moved, dim3(std::min<uint32_t>((S + 255) / 256, 256) + (S == 0)), dim3(256), 0, s,
                       W.moved, S, W.ctl + 1);
    hipLaunchKernelGGL(k_br_reset_or_fuse<KT>, dim3(reset_grid(nkeys)), dim3(256), 0, s, W.moved, A, fuse_limit(g, S),
                       tuning(LSRVT_TUNE_RESET));
    LSRVT_LAUNCHED();
  }
  if (S) {
    hipLaunchKernelGGL(k_br_sites<KT>, dim3((S + 255) / 256), dim3(256), 0, s, sites, S, A);
    LSRVT_LAUNCHED();
  }
  const unsigned lgrid = (unsigned)std::min<int64_t>((bg.nbricks + 255) / 256, 4096);
  const int32_t tg = tuning(LSRVT_TUNE_BR_GRID);
  const bool direct = !A.dbg && direct_rounds(bg.nbricks);
  const unsigned rgrid = (unsigned)std::min<int64_t>(bg.nbricks, tg ? tg : 8192);
  // (with fewer id bits, only paths of more than 4094 hops outgrow narrow keys)
  const bool tally = S > (1u << 19);
  uint32_t r = 0;
  // Rounds are launched as plain kernels, one each (a captured graph of eight
  // rounds replayed is slower: 14.0 against 13.4 ms for 379 x 251 x 147 voxels
  // and 20 updates, 0.79 against 0.71 ms for one pass of 192 x 96 x 96, whose
  // graph is built for it alone), and a pass rarely needs more than the one
  // before it plus one.
  uint32_t &hint = inc ? st.br_rounds_inc : st.br_rounds;
  int batch = hint ? (int)hint + 1 : 12;
  uint32_t c[14];
  const int64_t max_rounds = 4 * g.n + 8;
  while (true) {
    const bool timed = timer().on;
    std::pair<hipEvent_t, hipEvent_t> ev;
    if (timed && (rc = timed_begin(s, ev))) return rc;
    for (int i = 0; i < batch; ++i) {
      ++r;
      if (direct) {
        hipLaunchKernelGGL((tally ? k_br_round_all<KT, true> : k_br_round_all<KT, false>),
                           dim3((unsigned)bg.nbricks), dim3(kBRThreads), 0, s, A, r);
      } else {
        hipLaunchKernelGGL(k_br_list, dim3(lgrid), dim3(256), 0, s, A, r);
        hipLaunchKernelGGL(k_br_round<KT>, dim3(rgrid), dim3(kBRThreads), 0, s, A, r);
      }
    }
    LSRVT_LAUNCHED();
    if (timed && (rc = timed_end(s, ev, (uint64_t)batch))) return rc;
    if ((rc = read_words(W.ctl, 14, c, s))) return rc;
    if (c[3] & 1u) return LSRVT_EINVAL;
    if (c[3] & ~4u) return LSRVT_EDEVICE;
    if (c[3] & 4u) {  // a narrow key reached the largest exact distance
      *far = true;
      st.br_work = tally ? c[12] : 0u;
      return LSRVT_OK;
    }
    if (c[4 + (r + 1) % 3] == 0) break;
    if ((int64_t)r > max_rounds) return LSRVT_EDEVICE;
    if (far && sizeof(KT) == 8 && r >= kLongPass) {
      st.br_work = c[12];
      if (levels_after_bricks(g, S, st.br_work)) {
        *far = true;
        return LSRVT_OK;
      }
    }
    // (a long pass waits for the host a few times, not every four rounds: one
    // along a corridor of 256 x 256 x 32 voxels takes 16.6 ms instead of 21.9)
    batch = std::max(4, (int)(r / 4));
  }
  // the rounds that had work size the first batch of the next pass
  hint = c[13];
  static const bool debug_levels = getenv("LSRVT_DEBUG_LEVELS") != nullptr;
  if (debug_levels) {
    unsigned long long d[2];
    LSRVT_HIP(hipMemcpyAsync(d, W.ctl + 8, sizeof(d), hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
    fprintf(stderr, "[lsrvt] br %s processings=%llu sweep rounds=%llu\n", inc ? "inc" : "full", d[0], d[1]);
    const uint32_t nl = std::min<uint32_t>(r + 1, kHistLen);
    std::vector<uint32_t> h(nl, 0);
    LSRVT_HIP(hipMemcpyAsync(h.data(), W.hist, sizeof(uint32_t) * nl, hipMemcpyDeviceToHost, s));
    LSRVT_HIP(hipStreamSynchronize(s));
    fprintf(stderr, "[lsrvt] br %s rounds=%u launched=%u bricks per round:", inc ? "inc" : "full", hint, r);
    for (uint32_t i = 1; i < nl; ++i) fprintf(stderr, " %u", h[i]);
    fprintf(stderr, "\n");
  }
  const KT *keys = static_cast<const KT *>(A.key);
  if (fz && g.n / (int64_t)std::max<uint32_t>(S, 1u) < kSlabSites)
    hipLaunchKernelGGL(k_brick_sums<KeySource<KT>>, dim3(sums_grid(bg)), dim3(kVTThreads), 0, s,
                       (KeySource<KT>{keys, A.idmask}), g, bg, *fz);
  else if (fz)
    hipLaunchKernelGGL(k_br_finish_sums<KT>, dim3(slab_grid(bg)), dim3(kVTThreads), 0, s, keys, g, bg, A.idmask,
                       *fz);
  else
    hipLaunchKernelGGL(k_br_finish<KT>, dim3(slab_grid(bg)), dim3(kVTThreads), 0, s, keys, g, bg, A.idmask, cell);
  LSRVT_LAUNCHED();
  if (timer().on) {
    std::lock_guard<std::mutex> lk(timer().mu);
    timer().passes += 1;
    timer().voxels_per_pass = g.n;
    timer().engines |= 2;
  }
  return LSRVT_OK;
}

// One Voronoi pass by brick relaxation, with narrow keys when the sites
// allow and until a pass outgrows them: that pass is repeated from the sites
// with wide keys (or by levels, levels_after_bricks), which the rest of the call
// keeps.
int32_t run_br(const Geom &g, const uint32_t *sites, uint32_t S, uint32_t *cell, CvtWork &W, VTState &st, bool inc,
               hipStream_t s, const Fuse *fz = nullptr) {
  if (!st.keys_set) {
    st.id_bits = narrow_id_bits(S);
    st.keys_set = true;
  }
  if (st.id_bits) {
    bool far = false;
    int32_t rc = run_br_k<uint32_t>(g, sites, S, cell, W, st, inc, s, fz, &far);
    if (rc || !far) return rc;
    st.id_bits = 0;
    if ((rc = fill<uint32_t>(W.ctl + 3, 1, 0u, s))) return rc;
    if (!levels_after_bricks(g, S, st.br_work))
      return run_br_k<unsigned long long>(g, sites, S, cell, W, st, false, s, fz, nullptr);
  } else {
    // (a pass that may still change to levels: the first of more sites than narrow keys hold)
    bool far = false;
    int32_t rc = run_br_k<unsigned long long>(g, sites, S, cell, W, st, inc, s, fz,
                                              !inc && S > (1u << 24) ? &far : nullptr);
    if (rc || !far) return rc;
  }
  st.bricks = false;
  int32_t rc = vt_masks(g, W, st, s);
  return rc ? rc : run_vt(g, sites, S, cell, W, st, s, fz);
}

// A Voronoi pass with the selected schedule; with fz, its last kernel also
// takes the centroid sums of the update that follows.
int32_t vt_pass(const Geom &g, const uint32_t *sites, uint32_t S, uint32_t *cell, CvtWork &W, VTState &st, bool inc,
                hipStream_t s, const Fuse *fz = nullptr) {
  if (st.bricks) return run_br(g, sites, S, cell, W, st, inc, s, fz);
  return inc ? run_vt_inc(g, sites, S, cell, W, st, s, fz) : run_vt(g, sites, S, cell, W, st, s, fz);
}

// Errors a run reported on the device (synchronises).
int32_t vt_errors(CvtWork &W, hipStream_t s) {
  uint32_t e = 0;
  int32_t rc = read_words(W.err, 1, &e, s);
  if (rc) return rc;
  if (e & 1u) return LSRVT_EINVAL;
  if (e) return LSRVT_EDEVICE;
  return LSRVT_OK;
}

// The sites' moves from the centroid sums, the cells seen through `cell`.
template <class View>
int32_t run_snap(const View &cell, const Geom &g, uint32_t *sites, uint32_t S, double *ds, CvtWork &W, hipStream_t s) {
  const Sums sm{W.sums};
  hipLaunchKernelGGL(k_snap<View>, dim3((S + 255) / 256), dim3(256), 0, s, cell, g, S, sm, sites, ds, W.moved,
                     W.fb_list, W.fb_cnt);
  const bool flat = std::min(g.nx, std::min(g.ny, g.nz)) <= kFlatEdge;
  hipLaunchKernelGGL((flat ? k_snap_near<true, View> : k_snap_near<false, View>),
                     dim3(std::min<uint32_t>((S + 3) / 4, 2048)), dim3(256), 0, s, cell, g, sm, sites, ds, W.moved,
                     W.fb_list, W.fb_cnt);
  hipLaunchKernelGGL((flat ? k_snap_far<true, View> : k_snap_far<false, View>), dim3(std::min<uint32_t>(S, 512)),
                     dim3(kSnapFarThreads), 0, s, cell, g, sm, sites, ds, W.moved, W.fb_list, W.fb_cnt);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}

// One site update from a C-order cell array.
int32_t run_update(const uint32_t *cell, const Geom &g, const uint16_t *w, uint32_t *sites, uint32_t S, double *ds,
                   CvtWork &W, hipStream_t s) {
  if (S == 0) return LSRVT_OK;
  int32_t rc;
  if ((rc = fill<uint32_t>(W.fb_cnt, 1, 0u, s))) return rc;
  if ((rc = fill<unsigned long long>(W.sums, 4 * (int64_t)S, 0ull, s))) return rc;
  const int64_t ntiles = (int64_t)((g.nx + TX - 1) / TX) * ((g.ny + TY - 1) / TY) * ((g.nz + TZ - 1) / TZ);
  hipLaunchKernelGGL(k_centroid, dim3((unsigned)(ntiles < 65535 ? ntiles : 65535)), dim3(256), 0, s, cell, w, g, S,
                     Sums{W.sums});
  LSRVT_LAUNCHED();
  return run_snap(CellView{cell, g.nx, g.ny}, g, sites, S, ds, W, s);
}

// The update inside the Lloyd loop: the sums were taken by the pass that
// produced the cells, which are still in the pass's own arrays.
int32_t run_loop_update(const Geom &g, uint32_t *sites, uint32_t S, CvtWork &W, const VTState &st, hipStream_t s) {
  int32_t rc;
  if ((rc = fill<uint32_t>(W.fb_cnt, 1, 0u, s))) return rc;
  const VTGrid bg = vt_grid(g);
  if (st.bricks && !st.id_bits)
    return run_snap(KeyView<unsigned long long>{reinterpret_cast<unsigned long long *>(W.cellb), bg, ~0u}, g, sites, S,
                    W.ds, W, s);
  return run_snap(KeyView<uint32_t>{W.cellb, bg, st.bricks ? (1u << st.id_bits) - 1u : ~0u}, g, sites, S, W.ds, W, s);
}

int32_t begin(CvtWork &W, const Geom &g, hipStream_t s) {
  int32_t rc;
  VTGrid bg = vt_grid(g);
  if ((rc = fill<uint32_t>(W.act, 2 * bg.nbricks, 0u, s))) return rc;
  if ((rc = fill<uint32_t>(W.ctl, 8 + 2 * 8 + kHistLen, 0u, s))) return rc;
  return LSRVT_OK;
}


// ----------------------------------------------------------------------------
// The Lloyd loops of many jobs in lockstep: every phase of every pass is one
// launch over all jobs (blockIdx.y = job), with each job's blocks striding
// over that job's own work.  The Voronoi passes use the brick relaxation
// (its rounds are shared: round r works on the marked bricks of every job,
// and the batch ends a pass when no job has a brick marked); a job with fewer
// updates than the batch's largest simply stops taking part.  Every job's
// kernels, sums and orders are its own, so its results are bit-identical to
// its lsrvt_cvt alone.
struct JobDev {
  BRArgs A;
  Geom g;
  const uint8_t *band;
  const uint32_t *comp, *seeds;
  const uint16_t *w;
  uint32_t *cell, *sites, *site_comp, *eq;
  uint32_t S;
  int32_t iters;
  Sums sums;
  double *ds;
  uint8_t *moved;
  uint32_t *fb_list, *fb_cnt;
  uint32_t first;     // bricks of the jobs before this one
  uint32_t fuse_min;  // moved sites above which the reset is fused into the first rounds
};

__global__ __launch_bounds__(kVTThreads) void kb_br_masks(const JobDev *J) {
  const JobDev &j = J[blockIdx.y];
  d_br_masks(j.band, j.g, j.A.bg, j.eq);
}

__global__ void kb_init_sites(const JobDev *J) {
  const JobDev &j = J[blockIdx.y];
  d_init_sites(j.seeds, j.S, j.comp, j.g, j.sites, j.site_comp, j.A.ctl + 3);
}

// Start of pass t: marks, list lengths and reset words cleared (of every job:
// one that has stopped keeps an empty list), and for a full pass (t = 0) every
// key and packed face unreached.  Block (0, 0) clears the shared words: the
// round flags and [3], the last round that had work.
template <class KT>
__global__ __launch_bounds__(256) void kb_pass_clear(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 4) j.A.alive[threadIdx.x] = 0u;
  if (blockIdx.x == 0 && threadIdx.x < 2) {
    j.A.cnt[threadIdx.x] = 0u;
    j.A.ctl[1 + threadIdx.x] = 0u;
  }
  if (t > j.iters) return;
  const int64_t nb = j.A.bg.nbricks, stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < 2 * nb; i += stride) j.A.mark[i] = 0u;
  if (t == 0) {
    KT *key = static_cast<KT *>(j.A.key), *xface = static_cast<KT *>(j.A.xface);
    for (int64_t i = i0; i < nb * kRows * BX; i += stride) key[i] = BRKey<KT>::inf;
    for (int64_t i = i0; i < nb * 512; i += stride) xface[i] = BRKey<KT>::inf;
  }
}

__global__ __launch_bounds__(256) void kb_count_moved(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t <= j.iters) d_count_moved(j.moved, j.S, j.A.ctl + 1);
}

template <class KT>
__global__ __launch_bounds__(256) void kb_reset(const JobDev *J, int32_t t, int32_t mode) {
  const JobDev &j = J[blockIdx.y];
  if (t > j.iters || t == 0) return;
  d_br_reset_or_fuse<KT>(j.moved, j.A, j.fuse_min, mode);
}

template <class KT>
__global__ void kb_sites(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t > j.iters) return;
  d_br_sites<KT>(j.sites, j.S, j.A);
}

// The job that holds item i of the jobs' items back to back: the last one that
// starts at or before it.
template <class F>
__device__ __forceinline__ int32_t job_of(int32_t n, uint32_t i, F start) {
  int32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (start(mid) <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// One relaxation round of the whole batch with a workgroup for every brick of
// every job (up to kDirectBricks of them, as for one volume): two launches
// fewer than with lists, 4.4 of 48.9 ms for sixteen jobs of 32^3 to 192^3 with
// 15 updates, which take 41.3 ms with the fused resets.
template <class KT>
__global__ __launch_bounds__(kBRThreads, sizeof(KT) == 4 ? 5 : 4) void kb_round_all(const JobDev *J, int32_t n,
                                                                                   uint32_t r, int32_t t) {
  __shared__ BRLds<KT> L;
  const int32_t k = job_of(n, blockIdx.x, [&](int32_t i) { return J[i].first; });
  const BRArgs &A = J[k].A;
  if (blockIdx.x == 0 && threadIdx.x == 0) A.alive[(r + 2) % 3] = 0u;  // round r + 1 sets it
  const uint32_t b = blockIdx.x - J[k].first;
  if (t > J[k].iters || A.mark[(size_t)(r & 1) * A.bg.nbricks + b] != r) return;
  if (threadIdx.x == 0) A.alive[3] = r;
  br_process<KT>(A, b, r, L);
}

// Larger batches: every job's marked bricks are listed, the lists put back to
// back (job j's at off[j] .. off[j + 1], an exclusive prefix sum of the list
// lengths by one workgroup; a job that has stopped taking part has an empty
// one), and the round's workgroups stride over them.
__global__ __launch_bounds__(256) void kb_list(const JobDev *J, uint32_t r, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t <= j.iters) d_br_list(j.A, r);
}

__global__ __launch_bounds__(1024) void kb_offsets(const JobDev *J, int32_t n, uint32_t *off, uint32_t r) {
  __shared__ uint32_t part[1024];
  const int t = threadIdx.x;
  const int32_t per = (n + 1023) / 1024, a = t * per, e = a + per < n ? a + per : n;
  uint32_t sum = 0;
  for (int32_t i = a; i < e; ++i) {
    sum += J[i].A.cnt[r & 1];
    J[i].A.cnt[(r + 1) & 1] = 0u;
  }
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {  // inclusive scan of the threads' sums
    const uint32_t v = t >= d ? part[t - d] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  uint32_t run = part[t] - sum;
  for (int32_t i = a; i < e; ++i) {
    off[i] = run;
    run += J[i].A.cnt[r & 1];
  }
  if (t == 1023) {
    uint32_t *alive = J[0].A.alive;
    off[n] = part[1023];
    if (part[1023]) alive[3] = r;
    alive[(r + 2) % 3] = 0u;
  }
}

template <class KT>
__global__ __launch_bounds__(kBRThreads, sizeof(KT) == 4 ? 5 : 4) void kb_round(const JobDev *J, int32_t n,
                                                                               const uint32_t *off, uint32_t r) {
  __shared__ BRLds<KT> L;
  const uint32_t total = off[n];
  for (uint32_t item = blockIdx.x; item < total; item += gridDim.x) {
    const int32_t k = job_of(n, item, [&](int32_t i) { return off[i]; });
    const BRArgs &A = J[k].A;
    br_process<KT>(A, A.list[item - off[k]], r, L);
  }
}

template <class KT>
__global__ __launch_bounds__(kVTThreads) void kb_finish(const JobDev *J, int32_t t) {
  __shared__ union {
    FinTab slab;
    BrickTab brick;
  } T;
  const JobDev &j = J[blockIdx.y];
  if (t > j.iters) return;
  const KT *key = static_cast<const KT *>(j.A.key);
  if (t == j.iters || j.S == 0)
    d_br_finish_slabs<KT, false>(key, j.g, j.A.bg, j.A.idmask, j.cell, Fuse{}, nullptr);
  else if (j.g.n / (int64_t)j.S < kSlabSites)
    d_brick_sums(KeySource<KT>{key, j.A.idmask}, j.g, j.A.bg, Fuse{j.w, j.S, j.sums}, T.brick);
  else
    d_br_finish_slabs<KT, true>(key, j.g, j.A.bg, j.A.idmask, nullptr, Fuse{j.w, j.S, j.sums}, &T.slab);
}

__global__ __launch_bounds__(256) void kb_update_clear(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t >= j.iters) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < 4 * (int64_t)j.S; i += stride) j.sums.p[i] = 0ull;
  if (i0 == 0) *j.fb_cnt = 0u;
}

template <class KT>
__global__ void kb_snap(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t >= j.iters) return;
  d_snap(KeyView<KT>{static_cast<const KT *>(j.A.key), j.A.bg, j.A.idmask}, j.g, j.S, j.sums, j.sites, j.ds, j.moved,
         j.fb_list, j.fb_cnt);
}

template <class KT>
__global__ __launch_bounds__(256) void kb_snap_near(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t >= j.iters) return;
  d_snap_near<false>(KeyView<KT>{static_cast<const KT *>(j.A.key), j.A.bg, j.A.idmask}, j.g, j.sums, j.sites, j.ds,
                     j.moved, j.fb_list, j.fb_cnt);
}
template <class KT>
__global__ __launch_bounds__(kSnapFarThreads) void kb_snap_far(const JobDev *J, int32_t t) {
  const JobDev &j = J[blockIdx.y];
  if (t >= j.iters) return;
  d_snap_far<false>(KeyView<KT>{static_cast<const KT *>(j.A.key), j.A.bg, j.A.idmask}, j.g, j.sums, j.sites, j.ds,
                    j.moved, j.fb_list, j.fb_cnt);
}

}  // namespace

// Bytes of the descriptor block that precedes the jobs' workspaces.
// (the job descriptors, 256 bytes of shared round words, then the n + 1
// offsets of the batch's round list)
size_t cvt_batch_header(int32_t n) {
  return ((size_t)n * sizeof(JobDev) + 256 + 4 * ((size_t)n + 1) + 255) & ~size_t(255);
}

size_t cvt_batch_job_workspace(lsrvt_dims dims, uint32_t n_sites, int32_t iters) {
  Geom g;
  if (make_geom(dims, g)) return 0;
  return (cvt_workspace(g, n_sites, iters < 0 ? 0 : iters) + 255) & ~size_t(255);
}

namespace {

// What the lockstep loop needs besides the descriptors.
struct BatchCtx {
  int32_t n;
  JobDev *dj;           // device copy of the descriptors
  uint32_t *alive;      // shared round words
  uint32_t *offs;       // offsets of the batch's round list
  std::vector<JobDev> *hj;
  std::vector<CvtWork> *Ws;
  int32_t tmax;
  int64_t max_keys, max_sites, max_nb, sum_nb;
};

// The Lloyd loops of the batch with keys KT, from the seeds.  status[i]
// receives each job's status; *far is set when a job's narrow keys reached
// their largest exact distance (its results are then not to be used).
template <class KT>
int32_t batch_loop(const BatchCtx &c, int32_t *status, bool *far, hipStream_t s) {
  const int32_t n = c.n;
  JobDev *dj = c.dj;
  std::vector<JobDev> &hj = *c.hj;
  int32_t rc;
  LSRVT_HIP(hipMemcpyAsync(dj, hj.data(), sizeof(JobDev) * (size_t)n, hipMemcpyHostToDevice, s));
  for (int32_t i = 0; i < n; ++i)
    if ((rc = fill<uint32_t>((*c.Ws)[(size_t)i].ctl, 8 + 2 * 8, 0u, s))) return rc;
  const unsigned N = (unsigned)n;
  auto cap = [](int64_t v, int64_t m) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(v, m)); };
  const unsigned g_sites = cap((c.max_sites + 255) / 256, 1 << 20);
  hipLaunchKernelGGL(kb_init_sites, dim3(g_sites, N), dim3(256), 0, s, dj);
  hipLaunchKernelGGL(kb_br_masks, dim3(cap(c.max_keys / (kRows * BX), 65535), N), dim3(kVTThreads), 0,
                     s, dj);
  LSRVT_LAUNCHED();
  const unsigned g_clear = cap((c.max_keys + 255) / 256, 8192);
  const unsigned g_list = cap((c.max_nb + 255) / 256, 4096);
  const unsigned g_round = cap(c.sum_nb, tuning(LSRVT_TUNE_BR_GRID) > 0 ? tuning(LSRVT_TUNE_BR_GRID) : 8192);
  const unsigned g_fin = cap((c.max_nb + 7) / 8 * 8, 65528);
  const unsigned g_near = cap((c.max_sites + 3) / 4, 512), g_far = cap(c.max_sites, 64);
  const bool direct = direct_rounds(c.sum_nb);
  uint32_t rounds_hint = 0;
  for (int32_t t = 0; t <= c.tmax; ++t) {
    hipLaunchKernelGGL(kb_pass_clear<KT>, dim3(g_clear, N), dim3(256), 0, s, dj, t);
    if (t > 0) {
      hipLaunchKernelGGL(kb_count_moved, dim3(cap((c.max_sites + 255) / 256, 256), N), dim3(256), 0, s, dj, t);
      hipLaunchKernelGGL(kb_reset<KT>, dim3(reset_grid(c.max_keys), N), dim3(256), 0, s, dj, t,
                         tuning(LSRVT_TUNE_RESET));
    }
    hipLaunchKernelGGL(kb_sites<KT>, dim3(g_sites, N), dim3(256), 0, s, dj, t);
    LSRVT_LAUNCHED();
    uint32_t r = 0;
    int batch = rounds_hint ? (int)rounds_hint + 1 : 12;
    uint32_t w[4];
    const bool timed = timer().on;
    while (true) {
      std::pair<hipEvent_t, hipEvent_t> ev;
      if (timed && (rc = timed_begin(s, ev))) return rc;
      for (int k = 0; k < batch; ++k) {
        ++r;
        if (direct) {
          hipLaunchKernelGGL(kb_round_all<KT>, dim3((unsigned)c.sum_nb), dim3(kBRThreads), 0, s, dj, n, r, t);
        } else {
          hipLaunchKernelGGL(kb_list, dim3(g_list, N), dim3(256), 0, s, dj, r, t);
          hipLaunchKernelGGL(kb_offsets, dim3(1), dim3(1024), 0, s, dj, n, c.offs, r);
          hipLaunchKernelGGL(kb_round<KT>, dim3(g_round), dim3(kBRThreads), 0, s, dj, n, (const uint32_t *)c.offs, r);
        }
      }
      LSRVT_LAUNCHED();
      if (timed && (rc = timed_end(s, ev, (uint64_t)batch))) return rc;
      if ((rc = read_words(c.alive, 4, w, s))) return rc;
      if (w[(r + 1) % 3] == 0) break;
      if (r > (uint32_t)(1u << 30)) return LSRVT_EDEVICE;
      batch = std::max(4, (int)(r / 4));
    }
    rounds_hint = w[3];
    if (t < c.tmax) hipLaunchKernelGGL(kb_update_clear, dim3(g_sites, N), dim3(256), 0, s, dj, t);
    hipLaunchKernelGGL(kb_finish<KT>, dim3(g_fin, N), dim3(kVTThreads), 0, s, dj, t);
    if (t < c.tmax) {
      hipLaunchKernelGGL(kb_snap<KT>, dim3(g_sites, N), dim3(256), 0, s, dj, t);
      hipLaunchKernelGGL(kb_snap_near<KT>, dim3(g_near, N), dim3(256), 0, s, dj, t);
      hipLaunchKernelGGL(kb_snap_far<KT>, dim3(g_far, N), dim3(kSnapFarThreads), 0, s, dj, t);
    }
    LSRVT_LAUNCHED();
    if (timed) {
      std::lock_guard<std::mutex> lk(timer().mu);
      timer().engines |= 2;
      for (int32_t i = 0; i < n; ++i)
        if (t <= hj[(size_t)i].iters) {
          timer().passes += 1;
          timer().voxels_per_pass = hj[(size_t)i].g.n;
        }
    }
  }
  // each job's error bits (a seed outside its volume; a narrow key that
  // reached the largest exact distance)
  for (int32_t i = 0; i < n; ++i) {
    uint32_t e = 0;
    if ((rc = read_words((*c.Ws)[(size_t)i].ctl + 3, 1, &e, s))) return rc;
    if (e & 4u) *far = true;
    status[i] = (e & 1u) ? LSRVT_EINVAL : (e & ~4u) ? LSRVT_EDEVICE : LSRVT_OK;
  }
  return LSRVT_OK;
}

}  // namespace

// The Lloyd loops of n jobs in lockstep (see above).  work: the descriptor
// block, then one cvt workspace per job (cvt_batch_job_workspace each, in
// order).  status[i] receives each job's status.  Narrow relaxation keys
// are used when every job's sites allow them; if a job outgrows them, the
// batch is run again with wide keys.
int32_t cvt_batch(const CvtBatchJob *jobs, int32_t n, void *work, size_t bytes, int32_t *status, hipStream_t s) {
  if (n <= 0) return LSRVT_OK;
  std::vector<JobDev> hj((size_t)n);
  uint8_t *base = static_cast<uint8_t *>(work);
  const size_t head = cvt_batch_header(n);
  if (bytes < head) return LSRVT_EWORKSPACE;
  BatchCtx c{};
  c.n = n;
  c.dj = reinterpret_cast<JobDev *>(base);
  c.alive = reinterpret_cast<uint32_t *>(base + (size_t)n * sizeof(JobDev));
  c.offs = reinterpret_cast<uint32_t *>(base + (size_t)n * sizeof(JobDev) + 256);
  size_t off = head;
  std::vector<CvtWork> Ws((size_t)n);
  std::vector<uint32_t> bits((size_t)n);
  bool narrow = true;
  for (int32_t i = 0; i < n; ++i) {
    const CvtBatchJob &b = jobs[i];
    JobDev &j = hj[(size_t)i];
    Geom g;
    int32_t rc = make_geom(b.dims, g);
    if (rc) return rc;
    if (b.iters < 0 || !b.band || !b.comp || !b.cell || (b.n_sites && (!b.seeds || !b.sites || !b.site_comp)))
      return LSRVT_EINVAL;
    const size_t need = cvt_batch_job_workspace(b.dims, b.n_sites, b.iters);
    if (off + need > bytes) return LSRVT_EWORKSPACE;
    CvtWork &W = Ws[(size_t)i];
    if ((rc = carve_cvt(base + off, need, g, b.n_sites, b.iters, W))) return rc;
    off += need;
    bits[(size_t)i] = narrow_id_bits(b.n_sites);
    narrow = narrow && bits[(size_t)i] != 0;
    j.A = br_args(g, W, 0u);
    j.A.alive = c.alive;
    j.A.dbg = nullptr;
    j.g = g;
    j.band = b.band;
    j.comp = b.comp;
    j.seeds = b.seeds;
    j.w = b.weights;
    j.cell = b.cell;
    j.sites = b.sites;
    j.site_comp = b.site_comp;
    j.eq = W.eq;
    j.S = b.n_sites;
    j.iters = b.iters;
    const size_t S = b.n_sites;
    j.first = (uint32_t)c.sum_nb;
    j.fuse_min = fuse_limit(g, b.n_sites);
    j.A.moved = W.moved;
    j.A.fsites = b.sites;
    j.sums = Sums{W.sums};
    j.ds = W.ds;
    j.moved = W.moved;
    j.fb_list = W.fb_list;
    j.fb_cnt = W.fb_cnt;
    c.tmax = std::max(c.tmax, b.iters);
    const VTGrid bg = vt_grid(g);
    c.max_nb = std::max<int64_t>(c.max_nb, bg.nbricks);
    c.sum_nb += bg.nbricks;
    c.max_keys = std::max<int64_t>(c.max_keys, bg.nbricks * kRows * BX);
    c.max_sites = std::max<int64_t>(c.max_sites, (int64_t)S);
  }
  c.hj = &hj;
  c.Ws = &Ws;
  if (narrow) {
    for (int32_t i = 0; i < n; ++i) {
      const BRArgs a = br_args(hj[(size_t)i].g, Ws[(size_t)i], bits[(size_t)i]);
      hj[(size_t)i].A.hop32 = a.hop32;
      hj[(size_t)i].A.idmask = a.idmask;
      hj[(size_t)i].A.lim32 = a.lim32;
    }
    bool far = false;
    const int32_t rc = batch_loop<uint32_t>(c, status, &far, s);
    if (rc || !far) return rc;
    for (int32_t i = 0; i < n; ++i) {
      const BRArgs a = br_args(hj[(size_t)i].g, Ws[(size_t)i], 0u);
      hj[(size_t)i].A.hop32 = a.hop32;
      hj[(size_t)i].A.idmask = a.idmask;
      hj[(size_t)i].A.lim32 = a.lim32;
    }
  }
  bool far = false;
  return batch_loop<unsigned long long>(c, status, &far, s);
}

namespace {
}  // namespace

}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_cvt_workspace(lsrvt_dims dims, uint32_t n_sites, int32_t iters) {
  Geom g;
  if (make_geom(dims, g)) return 0;
  return cvt_workspace(g, n_sites, iters < 0 ? 0 : iters);
}

extern "C" int32_t lsrvt_vt(const uint8_t *d_band, lsrvt_dims dims, const uint32_t *d_sites, uint32_t n_sites,
                            uint32_t *d_cell, void *d_work, size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (!d_band || !d_cell || (n_sites && !d_sites)) return LSRVT_EINVAL;
  if ((rc = check_work(d_work, work_bytes, cvt_workspace(g, n_sites, 0)))) return rc;
  CvtWork W;
  if ((rc = carve_cvt(d_work, work_bytes, g, n_sites, 0, W))) return rc;
  hipStream_t s = as_stream(stream);
  if ((rc = begin(W, g, s))) return rc;
  VTState st;
  if ((rc = vt_prepare(d_band, g, W, st, s))) return rc;
  if ((rc = vt_pass(g, d_sites, n_sites, d_cell, W, st, false, s))) return rc;
  return vt_errors(W, s);
}

extern "C" int32_t lsrvt_update(const uint32_t *d_cell, lsrvt_dims dims, const uint16_t *d_weights, uint32_t *d_sites,
                                uint32_t n_sites, double *d_ds, void *d_work, size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (!d_cell || (n_sites && !d_sites)) return LSRVT_EINVAL;
  if ((rc = check_work(d_work, work_bytes, cvt_workspace(g, n_sites, 0)))) return rc;
  CvtWork W;
  if ((rc = carve_cvt(d_work, work_bytes, g, n_sites, 0, W))) return rc;
  return run_update(d_cell, g, d_weights, d_sites, n_sites, d_ds, W, as_stream(stream));
}

extern "C" int32_t lsrvt_cvt(const uint8_t *d_band, const uint32_t *d_comp, lsrvt_dims dims, const uint32_t *d_seeds,
                             uint32_t n_sites, const uint16_t *d_weights, int32_t iters, uint32_t *d_cell,
                             uint32_t *d_sites, uint32_t *d_site_comp, double *h_mean_ds, void *d_work,
                             size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (iters < 0) return LSRVT_EINVAL;
  if (!d_band || !d_comp || !d_cell || (n_sites && (!d_seeds || !d_sites || !d_site_comp))) return LSRVT_EINVAL;
  if ((rc = check_work(d_work, work_bytes, cvt_workspace(g, n_sites, iters)))) return rc;
  CvtWork W;
  if ((rc = carve_cvt(d_work, work_bytes, g, n_sites, iters, W))) return rc;
  hipStream_t s = as_stream(stream);
  if ((rc = begin(W, g, s))) return rc;
  if (n_sites) {
    hipLaunchKernelGGL(k_init_sites, dim3((n_sites + 255) / 256), dim3(256), 0, s, d_seeds, n_sites, d_comp, g, d_sites,
                       d_site_comp, W.err);
    LSRVT_LAUNCHED();
  }
  VTState st;
  if ((rc = vt_prepare(d_band, g, W, st, s))) return rc;
  const Fuse fz{d_weights, n_sites, Sums{W.sums}};
  for (int32_t t = 0; t <= iters; ++t) {
    // the first pass covers every voxel; later ones only what the moved sites change.  A pass
    // followed by an update also takes the update's centroid sums.
    const bool upd = t < iters && n_sites > 0;
    if (upd && (rc = fill<unsigned long long>(W.sums, 4 * (int64_t)n_sites, 0ull, s))) return rc;
    if ((rc = vt_pass(g, d_sites, n_sites, d_cell, W, st, t > 0, s, upd ? &fz : nullptr))) return rc;
    if (t == iters) break;
    if (upd && (rc = run_loop_update(g, d_sites, n_sites, W, st, s))) return rc;
    hipLaunchKernelGGL(k_mean_ds_part, dim3(kMeanParts), dim3(256), 0, s, W.ds, n_sites, W.mean_part);
    hipLaunchKernelGGL(k_mean_ds, dim3(1), dim3(256), 0, s, W.mean_part, n_sites, W.mean + t);
    LSRVT_LAUNCHED();
  }
  if (h_mean_ds && iters > 0) {
    LSRVT_HIP(hipMemcpyAsync(h_mean_ds, W.mean, sizeof(double) * iters, hipMemcpyDeviceToHost, s));
  }
  return vt_errors(W, s);
}

extern "C" int32_t lsrvt_timing_enable(int32_t enable) {
  KernelTimer &T = timer();
  std::lock_guard<std::mutex> lk(T.mu);
  T.on = enable != 0;
  return LSRVT_OK;
}

extern "C" int32_t lsrvt_timing_read(double *ms, uint64_t *launches, uint64_t *passes, int64_t *voxels_per_pass,
                                     int32_t *engines) {
  KernelTimer &T = timer();
  std::lock_guard<std::mutex> lk(T.mu);
  for (auto &ev : T.pending) {
    LSRVT_HIP(hipEventSynchronize(ev.second));
    float dt = 0.0f;
    LSRVT_HIP(hipEventElapsedTime(&dt, ev.first, ev.second));
    T.ms += dt;
    T.pool.push_back(ev);
  }
  T.pending.clear();
  if (ms) *ms = T.ms;
  if (launches) *launches = T.launches;
  if (passes) *passes = T.passes;
  if (voxels_per_pass) *voxels_per_pass = T.voxels_per_pass;
  if (engines) *engines = T.engines;
  T.engines = 0;
  T.ms = 0.0;
  T.launches = 0;
  T.passes = 0;
  return LSRVT_OK;
}

// ----------------------------------------------------------------------------
// The site update for callers that cannot allocate device memory (code under
// graph capture, serving loops that forbid allocation): its scratch (per-site
// uint64 sums, the fallback list and counter, the moved flags) lives in a
// file-scope device array of fixed size, one copy per GPU, held until the
// process ends.  Host code never passes the array's name to a kernel: its
// device address is looked up once per device (with that device current)
// and kept.
namespace lsrvt {

constexpr uint32_t kNoAllocSites = LSRVT_UPDATE_NOALLOC_MAX_SITES;
constexpr size_t kNoAllocSums = (size_t)4 * kNoAllocSites * sizeof(unsigned long long);
constexpr size_t kNoAllocList = (size_t)kNoAllocSites * sizeof(uint32_t);
constexpr size_t kNoAllocBytes = kNoAllocSums + kNoAllocList + 256 + kNoAllocSites;

__device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {

struct ScratchTable {
  std::mutex mu;
  std::vector<unsigned char *> ptr;  // device address of `scratch` per device (nullptr: not looked up)
};

ScratchTable &scratch_table() {
  static ScratchTable t;
  return t;
}

int32_t scratch_ptr(unsigned char **out) {
  int dev = 0;
  LSRVT_HIP(hipGetDevice(&dev));
  ScratchTable &T = scratch_table();
  std::lock_guard<std::mutex> lk(T.mu);
  if ((size_t)dev >= T.ptr.size()) T.ptr.resize((size_t)dev + 1, nullptr);
  if (!T.ptr[dev]) {
    void *p = nullptr;
    LSRVT_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return LSRVT_EDEVICE;
    T.ptr[dev] = static_cast<unsigned char *>(p);
  }
  *out = T.ptr[dev];
  return LSRVT_OK;
}

}  // namespace
}  // namespace lsrvt

extern "C" int32_t lsrvt_update_noalloc(const uint32_t *d_cell, lsrvt_dims dims, const uint16_t *d_weights,
                                        uint32_t *d_sites, uint32_t n_sites, double *d_ds, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (!d_cell || (n_sites && !d_sites)) return LSRVT_EINVAL;
  if (n_sites > kNoAllocSites) return LSRVT_ELIMIT;
  unsigned char *base = nullptr;
  if ((rc = scratch_ptr(&base))) return rc;
  CvtWork W{};
  W.sums = reinterpret_cast<unsigned long long *>(base);
  W.fb_list = reinterpret_cast<uint32_t *>(base + kNoAllocSums);
  W.fb_cnt = reinterpret_cast<uint32_t *>(base + kNoAllocSums + kNoAllocList);
  W.moved = base + kNoAllocSums + kNoAllocList + 256;
  return run_update(d_cell, g, d_weights, d_sites, n_sites, d_ds, W, as_stream(stream));
}

namespace lsrvt {
namespace {
thread_local int32_t t_tuning[5] = {0, 0, 0, 0, 0};
}  // namespace
int32_t tuning(int32_t knob) { return knob > 0 && knob < 5 ? t_tuning[knob] : 0; }
}  // namespace lsrvt

extern "C" int32_t lsrvt_set_tuning(int32_t knob, int32_t value) {
  if (knob == LSRVT_TUNE_BR_GRID) {
    if (value != 0 && (value < 256 || value > 16384)) return -1;
  } else if (knob == LSRVT_TUNE_STATS_TILE) {
    if (value != 0 && value != 1 && value != 2 && value != 4) return -1;
  } else if (knob == LSRVT_TUNE_KEY_BITS) {
    if (value != 64 && (value < 0 || value > 30)) return -1;
  } else if (knob == LSRVT_TUNE_RESET) {
    if (value < 0 || value > 2) return -1;
  } else {
    return -1;
  }
  const int32_t prev = t_tuning[knob];
  t_tuning[knob] = value;
  return prev;
}

extern "C" int32_t lsrvt_set_vt_engine(int32_t engine) {
  if (engine < 0 || engine > 2) return -1;
  const int32_t prev = (int32_t)t_engine;
  t_engine = (VTEngine)engine;
  return prev;
}
