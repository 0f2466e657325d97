// Euclidean line-of-sight Voronoi tessellation and the geodesically weighted
// site update (Sec. 3.1 with Eq. 1 and Eq. 2; Sec. 3.2.2 and Sec. 3.2.3).
//
// State per voxel v: the path length d[v] (float64), its source src[v] (a
// voxel index, or LSRVT_LOS_SITE | s when v sees its site s directly) and,
// after the relaxation, phi[v] (the line-of-sight voxel of the path) and
// cell[v] (the site of phi[v]).  Sites are continuous points kept in fixed
// point with 8 fraction bits plus an anchor voxel.
//
// The relaxation is synchronous: a sweep reads the state the previous sweep
// left and writes proposals; an apply pass then installs the proposals.  A
// sweep re-evaluates a voxel only if something it reads changed in the
// previous sweep (itself, a face neighbour, its source, or the source of a
// face neighbour): every other voxel would recompute exactly what it computed
// before, so the sweep equals a full synchronous sweep.
//
// Rounding makes a path through a voxel on the straight line to the site as
// long as the straight line, or an ulp shorter, so a voxel takes a new path
// only when the shortest valid candidate is shorter by a relative 2^-40, and
// then takes the preferred candidate within 2^-40 of that shortest one (the
// site itself first, by id, else the lowest voxel index).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace lsrvt {
namespace {

constexpr uint32_t kSite = LSRVT_LOS_SITE;
constexpr int kLosThreads = 256;
constexpr int kSweepBatch = 16;  // sweeps launched before the host looks, when it has no better guess
constexpr int32_t kMaxSweeps = 100000;
constexpr int kPhiRounds = 40;
constexpr double kShorter = 1.0 - 0x1p-40;
constexpr double kNear = 1.0 + 0x1p-40;
constexpr int kPhiHops = 32;
constexpr int kRadius = 31;  // the largest cube radius (plus one) kept per voxel (5 bits)
constexpr int kSpec = 4;     // crossings of a ray looked at together

// A tile of a sweep: 32 x 4 x 4 voxels (along the axes of the bit planes,
// los_plane), one wave, one word of each bit plane per row.  Tiles of 512 voxels give a 3 Mvoxel volume about six waves for
// every SIMD, which its chains of dependent loads need.
constexpr int kTX = 32, kTY = 4, kTZ = 4;
constexpr int kTWords = kTY * kTZ;
constexpr int kLanes = kWave / kTWords;  // lanes that hold a word of the tile

// Division of u < 2^31 by a fixed d >= 1 as a multiplication: with
// 2^(l - 1) < d <= 2^l and m = ceil(2^(31 + l) / d), m d exceeds 2^(31 + l) by
// less than d <= 2^l, so u m / 2^(31 + l) is above u / d by less than 1 / d.
struct Div {
  uint32_t m, s;
};
Div make_div(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  return Div{(uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
__device__ __forceinline__ uint32_t quot(uint32_t u, Div d) { return (uint32_t)(((uint64_t)u * d.m) >> d.s); }

struct LosArgs {
  const uint32_t *comp;
  Geom g;
  const int32_t *site_q;  // [S][3] Q8
  const uint32_t *anchor; // [S]
  uint32_t n_sites;
  double *d;              // [N] path lengths (the caller's output)
  uint32_t *src;          // [N] sources (the caller's output)
  double *pd;             // [N] proposed lengths
  uint32_t *ps;           // [N] proposed sources
  uint32_t *nbh;          // [N] the neighbourhood word (k_los_nbh)
  uint8_t *blk;           // [N] bit i: the ray to the source of face neighbour i is blocked
  uint32_t *chg;          // bit plane: changed in this sweep
  uint32_t *flag;         // bit plane: v or its source changed in the sweep before
  uint32_t *last;         // the last sweep of the stage that changed a voxel (1-based)
  uint32_t *err;
  Div dx, dy;             // division by g.nx, g.ny
  int32_t axis;           // the axis along the words of the bit planes (0: x)
  int32_t pa, pb, pc;     // extents along it and the other two (in the order x, y, z)
  int32_t pw;             // words of a row of a bit plane
  int32_t ty;             // tiles along the second
  uint32_t ntiles;
};

// Plane coordinates of (x, y, z), and the coordinates of (a, b, c).
template <bool Turned>
__device__ __forceinline__ void to_plane(const LosArgs &A, int32_t x, int32_t y, int32_t z, int32_t &a, int32_t &b,
                                         int32_t &c) {
  a = !Turned || A.axis == 0 ? x : A.axis == 1 ? y : z;
  b = !Turned || A.axis == 0 ? y : x;
  c = !Turned || A.axis != 2 ? z : y;
}
template <bool Turned>
__device__ __forceinline__ void from_plane(const LosArgs &A, int32_t a, int32_t b, int32_t c, int32_t &x, int32_t &y,
                                           int32_t &z) {
  x = !Turned || A.axis == 0 ? a : b;
  y = !Turned || A.axis == 0 ? b : A.axis == 1 ? a : c;
  z = !Turned || A.axis != 2 ? c : a;
}
// The word of row (b, c) that holds place 32 i.
__device__ __forceinline__ int64_t plane_word(const LosArgs &A, int32_t i, int32_t b, int32_t c) {
  return i + (int64_t)A.pw * (b + (int64_t)A.pb * c);
}

__device__ __forceinline__ void xyz(uint32_t u, const LosArgs &A, int32_t &x, int32_t &y, int32_t &z) {
  const uint32_t row = quot(u, A.dx);
  const uint32_t zz = quot(row, A.dy);
  x = (int32_t)(u - row * (uint32_t)A.g.nx);
  y = (int32_t)(row - zz * (uint32_t)A.g.ny);
  z = (int32_t)zz;
}

// Coordinates of voxel v (v < 2^31, so 32-bit division is exact).
__device__ __forceinline__ void xyz(int64_t v, const Geom &g, int32_t &x, int32_t &y, int32_t &z) {
  const uint32_t u = (uint32_t)v, nx = (uint32_t)g.nx, ny = (uint32_t)g.ny;
  const uint32_t row = u / nx;
  const uint32_t zz = row / ny;
  x = (int32_t)(u - row * nx);
  y = (int32_t)(row - zz * ny);
  z = (int32_t)zz;
}

__device__ __forceinline__ double len_vox(int32_t ax, int32_t ay, int32_t az, int32_t bx, int32_t by, int32_t bz) {
  int64_t dx = ax - bx, dy = ay - by, dz = az - bz;
  return sqrt((double)(dx * dx + dy * dy + dz * dz));
}

__device__ __forceinline__ double len_site(int32_t x, int32_t y, int32_t z, const int32_t *q) {
  int64_t dx = 256 * (int64_t)x - q[0], dy = 256 * (int64_t)y - q[1], dz = 256 * (int64_t)z - q[2];
  return sqrt((double)(dx * dx + dy * dy + dz * dz)) / 256.0;
}

// The neighbourhood word of a voxel: bit b = (dx + 1) + 3 (dy + 1) + 9 (dz + 1),
// less one past the middle, says that the voxel at (dx, dy, dz) is in the same
// component (26 bits); the top bits hold r, one more than the radius of the
// largest cube around the voxel that lies in its component (the part of it in
// the volume).
constexpr int kNbhBits = 26;
__device__ __forceinline__ uint32_t nbh_bit(int32_t dx, int32_t dy, int32_t dz) {
  const int32_t b = 13 + dx + 3 * dy + 9 * dz;
  return (uint32_t)(b > 13 ? b - 1 : b);
}

// True when every voxel whose closed cube meets the segment between the
// centres of a and b belongs to a's component.  Plane crossings of axis i
// happen at t = (2k + 1) / (2 L_i); they are ordered by cross-multiplication
// ((2k + 1) L_j < 2^31 under the extent limit), and at a crossing shared by
// several axes every combination of their steps is touched.  The walk stays
// in the bounding box of a and b, so every read is in bounds.
//
// A ray is a chain of dependent loads, and nothing else bounds it, so the walk
// needs few: one word of a voxel tells all that a crossing from it touches; the
// words of the next kSpec voxels of the path are loaded together; and the
// walk leaps.  Every voxel within K = r - 1 of the current one is in the
// component, so a box that reaches no further needs no walk at all, and
// otherwise the next K crossings of the longest axis touch nothing else (the
// other axes cross at most as often in between, since their crossings lie no
// closer together).
__device__ __forceinline__ bool ray_clear(const LosArgs &A, int32_t ax, int32_t ay, int32_t az, int32_t bx, int32_t by,
                                          int32_t bz) {
  const uint32_t Lx = (uint32_t)abs(bx - ax), Ly = (uint32_t)abs(by - ay), Lz = (uint32_t)abs(bz - az);
  const int32_t nx = A.g.nx, nxy = A.g.nx * A.g.ny;
  const int32_t dx = bx > ax ? 1 : -1, dy = by > ay ? 1 : -1, dz = bz > az ? 1 : -1;
  const int32_t sx = dx, sy = dy * nx, sz = dz * nxy;
  const uint32_t LM = max(Lx, max(Ly, Lz));
  const int32_t start = ax + nx * ay + nxy * az;
  uint32_t mx = 0, my = 0, mz = 0;
  int32_t cur = start;
  for (;;) {
    // the next kSpec crossings: the voxel before each, and what it must hold
    uint32_t at[kSpec], must[kSpec];
#pragma unroll
    for (int k = 0; k < kSpec; ++k) {
      at[k] = (uint32_t)cur;
      // the smallest (2 m + 1) / L over the axes still to cross
      const bool wx = mx < Lx, wy = my < Ly, wz = mz < Lz;
      const uint32_t ox = 2 * mx + 1, oy = 2 * my + 1, oz = 2 * mz + 1;
      uint32_t bo = ox, bL = wx ? Lx : 0;
      if (wy && (!bL || oy * bL < bo * Ly)) { bo = oy; bL = Ly; }
      if (wz && (!bL || oz * bL < bo * Lz)) { bo = oz; bL = Lz; }
      const bool cx = wx && ox * bL == bo * Lx, cy = wy && oy * bL == bo * Ly, cz = wz && oz * bL == bo * Lz;
      uint32_t m = 0;
      if (cx) m |= 1u << nbh_bit(dx, 0, 0);
      if (cy) m |= 1u << nbh_bit(0, dy, 0);
      if (cz) m |= 1u << nbh_bit(0, 0, dz);
      if (cx && cy) m |= 1u << nbh_bit(dx, dy, 0);
      if (cx && cz) m |= 1u << nbh_bit(dx, 0, dz);
      if (cy && cz) m |= 1u << nbh_bit(0, dy, dz);
      if (cx && cy && cz) m |= 1u << nbh_bit(dx, dy, dz);
      must[k] = m;
      if (k + 1 < kSpec) {
        mx += cx;
        my += cy;
        mz += cz;
        cur += (cx ? sx : 0) + (cy ? sy : 0) + (cz ? sz : 0);
      }
    }
    uint32_t w[kSpec], r = 0;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < kSpec; ++k) w[k] = A.nbh[at[k]];
#pragma unroll
    for (int k = 0; k < kSpec; ++k) {
      r = w[k] >> kNbhBits;
      if (k + 1 < kSpec) ok = ok && (w[k] & must[k]) == must[k];
    }
    if ((w[0] >> kNbhBits) > LM) return true;  // (at the start: the whole box)
    if (!ok) return false;
    // now at the last of them
    const uint32_t rem = max(Lx - mx, max(Ly - my, Lz - mz));
    if (r > rem) return true;
    if (r > 1) {
      // the state right after the K-th next crossing of the longest axis
      const uint32_t M = (Lx == LM ? mx : Ly == LM ? my : mz) + r - 1;  // its crossings so far (M <= LM)
      const uint32_t t = 2 * M - 1;                                     // t / (2 LM)
      mx = Lx == LM ? M : (t * Lx + LM) / (2 * LM);
      my = Ly == LM ? M : (t * Ly + LM) / (2 * LM);
      mz = Lz == LM ? M : (t * Lz + LM) / (2 * LM);
      cur = start + sx * (int32_t)mx + sy * (int32_t)my + sz * (int32_t)mz;
    } else {
      const uint32_t m = must[kSpec - 1];
      if ((w[kSpec - 1] & m) != m) return false;
      const bool cx = m & (1u << nbh_bit(dx, 0, 0)), cy = m & (1u << nbh_bit(0, dy, 0)),
                 cz = m & (1u << nbh_bit(0, 0, dz));
      mx += cx;
      my += cy;
      mz += cz;
      cur += (cx ? sx : 0) + (cy ? sy : 0) + (cz ? sz : 0);
    }
  }
}

__device__ __forceinline__ uint32_t pref(uint32_t code) { return code ^ kSite; }

// ---------------------------------------------------------------- anchors
__global__ void k_los_check(const uint32_t *__restrict__ comp, Geom g, const int32_t *__restrict__ q,
                            const uint32_t *__restrict__ anchor, uint32_t S, uint32_t *err) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  uint32_t a = anchor[s];
  if ((int64_t)a >= g.n || comp[a] == kNone) { err[0] = 1u; return; }
  int32_t x, y, z;
  xyz(a, g, x, y, z);
  const int32_t *p = q + 3 * (size_t)s;
  if (abs(256 * x - p[0]) > 128 || abs(256 * y - p[1]) > 128 || abs(256 * z - p[2]) > 128) err[0] = 1u;
}

// Each anchor holds the site with the smallest (length, id): the smallest
// length by an atomic min on its bit pattern (non-negative doubles order as
// their bits), then the smallest id among the sites that reach it.
__global__ void k_anchor_reset(LosArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= A.n_sites) return;
  uint32_t a = A.anchor[s];
  reinterpret_cast<unsigned long long *>(A.pd)[a] = 0x7FF0000000000000ull;
  A.ps[a] = kNone;
}

__global__ void k_anchor_len(LosArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= A.n_sites) return;
  uint32_t a = A.anchor[s];
  int32_t x, y, z;
  xyz(a, A.g, x, y, z);
  double d = len_site(x, y, z, A.site_q + 3 * (size_t)s);
  atomicMin(reinterpret_cast<unsigned long long *>(A.pd) + a, (unsigned long long)__double_as_longlong(d));
}

__global__ void k_anchor_id(LosArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= A.n_sites) return;
  uint32_t a = A.anchor[s];
  int32_t x, y, z;
  xyz(a, A.g, x, y, z);
  double d = len_site(x, y, z, A.site_q + 3 * (size_t)s);
  if (d == A.pd[a]) atomicMin(A.ps + a, s);
}

__global__ void k_anchor_set(LosArgs A) {
  uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= A.n_sites) return;
  uint32_t a = A.anchor[s];
  if (A.ps[a] != s) return;
  A.d[a] = A.pd[a];
  A.src[a] = kSite | s;
  // the anchors' neighbourhoods are evaluated in the first sweep
  int32_t x, y, z;
  xyz(a, A, x, y, z);
  int32_t pa, pb, pc;
  to_plane<true>(A, x, y, z, pa, pb, pc);
  atomicOr(&A.flag[plane_word(A, pa / 32, pb, pc)], 1u << (pa & 31));
}

// ---------------------------------------------------------------- cube radii
// rad along one axis after the other: the largest r <= kRadius such that every
// voxel of the volume less than r away along the axes done so far is in v's
// component.  Along the next axis a voxel k away limits r to max(k, its own
// value) (to k if it is in another component).
template <int Axis>
__global__ __launch_bounds__(kLosThreads) void k_los_radius(const uint32_t *__restrict__ comp, Geom g, Div dx, Div dy,
                                                            const uint8_t *__restrict__ in, uint8_t *__restrict__ out) {
  const int64_t v = (int64_t)blockIdx.x * kLosThreads + threadIdx.x;
  if (v >= g.n) return;
  const uint32_t row = quot((uint32_t)v, dx), z = quot(row, dy);
  const uint32_t at = Axis == 0 ? (uint32_t)v - row * (uint32_t)g.nx : Axis == 1 ? row - z * (uint32_t)g.ny : z;
  const uint32_t len = (uint32_t)(Axis == 0 ? g.nx : Axis == 1 ? g.ny : g.nz);
  const int64_t step = Axis == 0 ? 1 : Axis == 1 ? g.nx : (int64_t)g.nx * g.ny;
  const uint32_t c = comp[v];
  uint32_t m = Axis == 0 ? kRadius : in[v];
  for (uint32_t k = 1; k < m; ++k) {
    const bool lo = at >= k, hi = at + k < len;
    const int64_t a = lo ? v - step * (int64_t)k : v, b = hi ? v + step * (int64_t)k : v;
    const uint32_t ca = comp[a], cb = comp[b];
    uint32_t q = m;
    if (Axis) q = min((uint32_t)(lo ? in[a] : m), (uint32_t)(hi ? in[b] : m));
    if (ca != c || cb != c) q = 0;
    m = min(m, max(k, q));
  }
  out[v] = (uint8_t)m;
}

// The neighbourhood words, from the radii along all three axes.
__global__ __launch_bounds__(kLosThreads) void k_los_nbh(const uint32_t *__restrict__ comp, Geom g, Div dx, Div dy,
                                                         const uint8_t *__restrict__ rad, uint32_t *__restrict__ nbh) {
  const int64_t v = (int64_t)blockIdx.x * kLosThreads + threadIdx.x;
  if (v >= g.n) return;
  const uint32_t row = quot((uint32_t)v, dx), zz = quot(row, dy);
  const int32_t x = (int32_t)((uint32_t)v - row * (uint32_t)g.nx), y = (int32_t)(row - zz * (uint32_t)g.ny), z = (int32_t)zz;
  const int64_t sy = g.nx, sz = (int64_t)g.nx * g.ny;
  const uint32_t c = comp[v];
  uint32_t w = (uint32_t)rad[v] << kNbhBits;
#pragma unroll
  for (int k = -1; k <= 1; ++k)
#pragma unroll
    for (int j = -1; j <= 1; ++j)
#pragma unroll
      for (int i = -1; i <= 1; ++i) {
        if (i == 0 && j == 0 && k == 0) continue;
        const bool in = x + i >= 0 && x + i < g.nx && y + j >= 0 && y + j < g.ny && z + k >= 0 && z + k < g.nz;
        const uint32_t o = comp[in ? v + i + sy * j + sz * k : v];
        w |= (in && o == c ? 1u : 0u) << nbh_bit(i, j, k);
      }
  nbh[v] = w;
}

// ---------------------------------------------------------------- sweeps
// A sweep is two launches.  eval: a wave takes a tile, spreads the flag plane
// to the face neighbours in registers (or takes every voxel, in the first
// sweep of stage 2), lists the voxels so marked in LDS, and each evaluates its
// candidates against the state of the previous sweep and writes a proposal if
// it changes.  apply: proposals are installed and flag is set for each voxel
// that changed or whose source changed.  A voxel left out reads nothing that
// changed since it was last evaluated, so it would compute the same result:
// the sweep equals a full synchronous sweep.

// The wave's tile: blocks b, b + 8, ... run on one XCD, so each gets a run of
// neighbouring tiles, which share their halos in its L2.
// (the grid's y counts runs of kTileRun tiles: a launch has fewer than 2^32
// threads along x)
constexpr uint32_t kTileRun = 1u << 22;
__device__ __forceinline__ uint32_t my_tile() {
  return blockIdx.y * kTileRun + (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

struct Tile {
  int32_t tx, y0, z0;  // word along the planes' rows, first row along the other two axes
};
__device__ __forceinline__ Tile tile_at(const LosArgs &A, uint32_t t) {
  const uint32_t q = t / (uint32_t)A.pw;
  return Tile{(int32_t)(t - q * (uint32_t)A.pw), (int32_t)(q % (uint32_t)A.ty) * kTY, (int32_t)(q / (uint32_t)A.ty) * kTZ};
}

// The set bits of the tile's words as a list of (word << 5 | bit), in order;
// lane l holds word l / kLanes and lists its part l % kLanes of it.  Returns
// their number.
__device__ __forceinline__ uint32_t tile_list(uint32_t word, uint16_t *list) {
  const int lane = lane_id();
  constexpr int kPart = 32 / kLanes;
  uint32_t bits = (word >> (kPart * (lane % kLanes))) & ((1u << kPart) - 1u);
  const uint32_t cnt = (uint32_t)__popc(bits);
  uint32_t inc = cnt;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t up = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += up;
  }
  uint32_t at = inc - cnt;
  while (bits) {
    const int b = __ffs(bits) - 1;
    list[at++] = (uint16_t)((lane / kLanes) << 5 | (lane % kLanes) * kPart | b);
    bits &= bits - 1;
  }
  return __shfl(inc, kWave - 1, kWave);
}

// Whether v takes a new path; its proposal is written if so.  The candidates
// of stage 1 are the sites of the face neighbours; those of stage 2 the
// sources of the neighbours, the neighbours themselves and the voxel's own
// path measured again.  A neighbour's source needs a clear ray; the other two
// are valid as they are.  Neighbours that share a source are one candidate, and
// one that has v's own source is none: its path is v's own measured again.
// What is left differs from lane to lane, so each lane walks its own few
// candidates, kept in LDS (in registers, under compile-time slots, every lane
// pays for all thirteen, and three waves fit a SIMD instead of five).
//
// Most marked voxels have no candidate that is short enough.  Probe says
// whether v has one; the wave then takes the voxels that have, packed, so that
// the rays, which cost most, do not run with a quarter of the lanes.
//
// Bit i of fresh: face neighbour i was flagged in the sweep before.  A ray
// that was found blocked is blocked for good, so it is remembered until the
// neighbour's flag is set (which has v evaluated): without this the same
// blocked rays are walked again in every sweep that a voxel takes part in.
template <int Stage, bool Probe>
__device__ __forceinline__ bool los_eval(const LosArgs &A, int32_t x, int32_t y, int32_t z, uint32_t fresh,
                                         double (*cds)[kWave], uint32_t (*code)[kWave],
                                         uint32_t (*aim)[kWave]) {
  const Geom g = A.g;
  const int lane = lane_id();
  const uint32_t sy = (uint32_t)g.nx, sz = (uint32_t)g.nx * (uint32_t)g.ny;
  const uint32_t v = (uint32_t)x + sy * (uint32_t)y + sz * (uint32_t)z;
  const uint32_t c = A.comp[v];
  const uint32_t sv = A.src[v];
  const double dh = A.d[v];
  const uint32_t blk0 = A.blk[v];
  const uint32_t nb[6] = {x > 0 ? v - 1 : v,  x < g.nx - 1 ? v + 1 : v,  y > 0 ? v - sy : v,
                          y < g.ny - 1 ? v + sy : v, z > 0 ? v - sz : v, z < g.nz - 1 ? v + sz : v};
  uint32_t nc[6], nu[6];
  double nd[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    nc[i] = A.comp[nb[i]];
    nu[i] = A.src[nb[i]];
    nd[i] = Stage == 2 ? A.d[nb[i]] : 0.0;
  }
  if (c == kNone) return false;
  const bool has_own = Stage == 2 && sv != kNone && !(sv & kSite);
  double own = __builtin_inf();
  if (has_own) {
    int32_t ux, uy, uz;
    xyz(sv, A, ux, uy, uz);
    own = len_vox(x, y, z, ux, uy, uz) + A.d[sv];
  }
  double base = own;  // the shortest candidate that needs no ray
  uint32_t ray = 0, valid = 0;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const uint32_t u = nu[i];
    const bool in = nb[i] != v && nc[i] == c && u != kNone;
    if (Stage == 2 && in) {
      nd[i] += 1.0;
      valid |= 1u << i;
      base = nd[i] < base ? nd[i] : base;
    }
    if (in && u != sv && u != v) {
      ray |= 1u << i;
      code[i][lane] = u;
    }
  }
  // one candidate for each source; blocked for one neighbour, blocked for all that share it
  auto sharing = [&](uint32_t u) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) m |= (nu[i] == u ? 1u : 0u) << i;
    return m & ray;
  };
  uint32_t blk = blk0 & ~fresh, cand = 0;
  double lim = base * kNear;
  for (uint32_t todo = ray; todo;) {
    const int i = __ffs(todo) - 1;
    const uint32_t u = code[i][lane], same = sharing(u);
    todo &= ~same;
    if (blk & same) {
      blk |= same;
      continue;
    }
    double cd;
    uint32_t t = u;
    if (u & kSite) {
      if (!Probe) t = A.anchor[u & ~kSite];
      cd = len_site(x, y, z, A.site_q + 3 * (size_t)(u & ~kSite));
    } else {
      int32_t ux, uy, uz;
      xyz(u, A, ux, uy, uz);
      cd = len_vox(x, y, z, ux, uy, uz) + A.d[u];
    }
    if (cd < dh && !(cd > lim)) {
      if (!Probe) {
        cds[i][lane] = cd;
        aim[i][lane] = t;
      }
      cand |= 1u << i;
    }
  }
  if (Probe) return cand != 0u || base < dh * kShorter;
  // First the shortest valid candidate, trying rays shortest first; then, of
  // the candidates near it, the preferred valid one, trying the rays of the
  // preferred first (the others' codes cannot win).
  bool found = false;
  double dmin = base, bestd = 0.0;
  uint32_t best = 0, bestc = 0;
  for (;;) {
    int bi = -1;
    double bd = 0.0;
    uint32_t bc = 0;
    for (uint32_t t = cand; t; t &= t - 1) {
      const int i = __ffs(t) - 1;
      const double d = cds[i][lane];
      const uint32_t u = code[i][lane];
      const bool take = !found ? bi < 0 || d < bd
                               : !(d > lim) && pref(u) < best && (bi < 0 || pref(u) < pref(bc));
      if (take) { bi = i; bd = d; bc = u; }
    }
    if (!found && (bi < 0 || !(bd < base) || !(bd < dh * kShorter))) {
      bi = -1;  // what needs no ray is as short, or nothing is short enough
      if (!(dmin < dh * kShorter)) break;
    }
    bool good = bi < 0;
    if (bi >= 0) {
      int32_t ux, uy, uz;
      xyz(aim[bi][lane], A, ux, uy, uz);
      good = ray_clear(A, x, y, z, ux, uy, uz);
      cand &= ~(1u << bi);
      if (!good) blk |= sharing(bc);
    }
    if (!good) continue;
    if (found) {
      if (bi >= 0) { bestc = bc; bestd = bd; }
      break;
    }
    found = true;
    best = ~0u;  // (no candidate's preference: kNone has no path)
    if (bi >= 0) { dmin = bd; best = pref(bc); bestc = bc; bestd = bd; }
    lim = dmin * kNear;
#pragma unroll
    for (int i = 0; i < 6; ++i)
      if (Stage == 2 && (valid >> i & 1u) && nd[i] < dh && !(nd[i] > lim) && pref(nb[i]) < best) {
        best = pref(nb[i]);
        bestc = nb[i];
        bestd = nd[i];
      }
    if (has_own && own < dh && !(own > lim) && pref(sv) < best) { best = pref(sv); bestc = sv; bestd = own; }
  }
  if (blk != blk0) A.blk[v] = (uint8_t)blk;
  if (found) {
    A.pd[v] = bestd;
    A.ps[v] = bestc;
  }
  return found;
}

// One synchronous sweep of stage 1 (paths only through sites) or stage 2
// over the marked voxels, the sweep-th of its stage.  A sweep past the one
// that changed nothing ends at once.
//
// Bound by the chains of dependent loads (the voxels, their sources, then one
// load a stretch of a ray) of the few voxels that each sweep works on, so it
// needs many waves and short chains.  At 160 x 144 x 128 voxels a sweep takes
// 15-100 us, where one launch for the marks, one for the evaluation and one for
// the proposals took 60-290 us, and a loop of 3 updates 17.4 ms instead of 43:
// 30.2 with the marks as bit planes and rays that leap, 28.2 with blocked rays
// remembered, 22.3 with each lane's own candidates, 19.0 with packed rays over
// neighbourhood words, 17.4 with fewer waits by the host.  (Tiles of 256 voxels
// instead of 512 cost 20.3 instead of 19.0, five waves a SIMD 19.5.)
template <int Stage, bool Turned>
__global__ __launch_bounds__(kWave, 4) void k_los_eval(LosArgs A, uint32_t sweep, int all_dirty) {
  __shared__ uint16_t list[kTWords * 32];
  __shared__ uint32_t chg[kTWords];
  __shared__ uint32_t nbf[6][kTWords];  // the flags of the face neighbours
  __shared__ double cds[6][kWave];      // each lane's candidates
  __shared__ uint32_t code[6][kWave], aim[6][kWave];
  const uint32_t t = my_tile();
  if (t >= A.ntiles || *A.last + 1 < sweep) return;
  const int lane = lane_id();
  const Tile T = tile_at(A, t);
  const int row = lane / kLanes, y = T.y0 + row % kTY, z = T.z0 + row / kTY;
  const bool in = y < A.pb && z < A.pc;
  const int64_t at = plane_word(A, T.tx, y, z);
  uint32_t w = 0;
  if (in) {
    const uint32_t *F = A.flag + at;
    const int64_t py = A.pw, pz = (int64_t)A.pw * A.pb;
    const int left = A.pa - T.tx * kTX;
    const uint32_t valid = left >= 32 ? ~0u : (1u << left) - 1u;
    const uint32_t m = F[0], xl = T.tx > 0 ? F[-1] : 0u, xr = T.tx < A.pw - 1 ? F[1] : 0u;
    const uint32_t f[6] = {m << 1 | xl >> 31,        m >> 1 | xr << 31,       y > 0 ? F[-py] : 0u,
                           y < A.pb - 1 ? F[py] : 0u, z > 0 ? F[-pz] : 0u, z < A.pc - 1 ? F[pz] : 0u};
    // the axes of the plane in the volume, whose face neighbours are numbered x-, x+, y-, y+, z-, z+
    const int ax[3] = {Turned ? A.axis : 0, Turned && A.axis ? 0 : 1, Turned && A.axis == 2 ? 1 : 2};
    w = m;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      w |= f[i];
      if (lane % kLanes == 0) nbf[2 * ax[i / 2] + i % 2][row] = f[i];
    }
    w = (all_dirty ? ~0u : w) & valid;
  }
  if (lane < kTWords) chg[lane] = 0u;
  const uint32_t n = tile_list(w, list);
  __syncthreads();
  auto fresh = [&](uint32_t e) {
    uint32_t f = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) f |= (nbf[k][e >> 5] >> (e & 31) & 1u) << k;
    return f;
  };
  auto eval = [&](uint32_t e, auto probe) {
    const uint32_t r = e >> 5;
    int32_t vx, vy, vz;
    from_plane<Turned>(A, T.tx * kTX + (int)(e & 31), T.y0 + (int)(r % kTY), T.z0 + (int)(r / kTY), vx, vy, vz);
    return los_eval<Stage, decltype(probe)::value>(A, vx, vy, vz, fresh(e), cds, code, aim);
  };
  uint32_t some = 0;  // listed voxels that have a candidate, moved to the front
  for (uint32_t i0 = 0; i0 < n; i0 += kWave) {
    const uint32_t e = i0 + lane < n ? list[i0 + lane] : 0u;
    const bool yes = i0 + lane < n && eval(e, std::true_type{});
    const uint64_t bal = __ballot(yes);
    if (yes) list[some + (uint32_t)__popcll(bal & lanemask_lt())] = (uint16_t)e;
    some += (uint32_t)__popcll(bal);
  }
  __syncthreads();
  for (uint32_t i = lane; i < some; i += kWave) {
    const uint32_t e = list[i];
    if (eval(e, std::false_type{})) atomicOr(&chg[e >> 5], 1u << (e & 31));
  }
  __syncthreads();
  const uint32_t out = chg[row];
  if (in && lane % kLanes == 0) A.chg[at] = out;
  if (__ballot(out != 0u) != 0ull && lane == 0) *A.last = sweep;
}

// Installs the proposals of a tile and writes its words of the flag plane.  In
// stage 1 no voxel has another voxel as its source, so only the changed ones
// are touched; stage 2 reads the source of every voxel and its change bit.
template <int Stage, bool Turned>
__global__ __launch_bounds__(kWave) void k_los_apply(LosArgs A, uint32_t sweep) {
  __shared__ uint16_t list[kTWords * 32];
  const uint32_t t = my_tile();
  if (t >= A.ntiles || *A.last + 1 < sweep) return;
  const int lane = lane_id();
  const Tile T = tile_at(A, t);
  const int row = lane / kLanes, yy = T.y0 + row % kTY, zz = T.z0 + row / kTY;
  const bool in = yy < A.pb && zz < A.pc;
  const int64_t at = plane_word(A, T.tx, yy, zz);
  const uint32_t w = in ? A.chg[at] : 0u;
  auto voxel = [&](int32_t a, int32_t b, int32_t c) {
    int32_t x, y, z;
    from_plane<Turned>(A, a, b, c, x, y, z);
    return x + (int64_t)A.g.nx * (y + (int64_t)A.g.ny * z);
  };
  if (Stage == 1) {
    if (in && lane % kLanes == 0) A.flag[at] = w;
    const uint32_t n = tile_list(w, list);
    __syncthreads();
    for (uint32_t i = lane; i < n; i += kWave) {
      const uint32_t e = list[i], r = e >> 5;
      const int64_t v = voxel(T.tx * kTX + (int)(e & 31), T.y0 + (int)(r % kTY), T.z0 + (int)(r / kTY));
      A.d[v] = A.pd[v];
      A.src[v] = A.ps[v];
    }
    return;
  }
  const int x = T.tx * kTX + (lane & 31), half = lane >> 5;
  uint32_t s[kTWords / 2];
#pragma unroll
  for (int k = 0; k < kTWords / 2; ++k) {
    const int r = 2 * k + half, y = T.y0 + r % kTY, z = T.z0 + r / kTY;
    const bool ok = x < A.pa && y < A.pb && z < A.pc;
    const int64_t v = voxel(x, y, z);
    const bool ch = (__shfl(w, kLanes * r, kWave) >> (lane & 31)) & 1u;
    s[k] = !ok ? kNone : ch ? A.ps[v] : A.src[v];
    if (ch) {
      A.d[v] = A.pd[v];
      A.src[v] = s[k];
    }
  }
  uint32_t sc[kTWords / 2];
#pragma unroll
  for (int k = 0; k < kTWords / 2; ++k) {
    sc[k] = 0u;
    if (s[k] != kNone && !(s[k] & kSite)) {
      int32_t ux, uy, uz, ua, ub, uc;
      xyz(s[k], A, ux, uy, uz);
      to_plane<Turned>(A, ux, uy, uz, ua, ub, uc);
      sc[k] = A.chg[plane_word(A, ua / 32, ub, uc)] >> (ua & 31);
    }
  }
#pragma unroll
  for (int k = 0; k < kTWords / 2; ++k) {
    const int r = 2 * k + half, y = T.y0 + r % kTY, z = T.z0 + r / kTY;
    const uint64_t bal = __ballot((sc[k] & 1u) != 0u);
    const uint32_t f = (uint32_t)(bal >> (32 * half)) | __shfl(w, kLanes * r, kWave);
    if ((lane & 31) == 0 && y < A.pb && z < A.pc) A.flag[plane_word(A, T.tx, y, z)] = f;
  }
}

// ---------------------------------------------------------------- phi, cells
// The line-of-sight voxel of each path (the last voxel before the site), and
// the site it sees.  Each thread follows its path for up to kPhiHops voxels;
// what is longer goes on in another launch, through the voxels that the
// launch before reached (any value read, old or new, lies on the same path, so
// in-place updates are safe).
template <bool First>
__global__ void k_phi(const uint32_t *__restrict__ src, int64_t n, uint32_t *phi, uint32_t *__restrict__ cell,
                      uint32_t *flag) {
  const int64_t v = (int64_t)blockIdx.x * kLosThreads + threadIdx.x;
  bool more = false;
  if (v < n) {
    uint32_t p = First ? (uint32_t)v : phi[v];
    uint32_t s = p == kNone ? kNone : src[p];
    if (s == kNone) p = kNone;
    for (int h = 0; h < kPhiHops && !(s & kSite); ++h) {
      p = First ? s : phi[p];
      s = src[p];
    }
    more = !(s & kSite);
    phi[v] = p;
    cell[v] = s == kNone ? kNone : s & ~kSite;
  }
  if (__ballot(more) != 0ull && lane_id() == 0) flag[0] = 1u;
}

// ---------------------------------------------------------------- update
// M and S = sum m x_phi per site.  One workgroup per 64 x 8 x 8 tile, one
// wave per row of 64 voxels along x: a segmented scan sums each run of equal
// cell, the last lane of a run adds it into an LDS table keyed by cell, and
// the table is flushed with one set of global atomics per distinct cell of
// the tile (a run that finds the table full adds straight to global memory).
// The sums are integers, so the order of the additions does not matter.
constexpr int kAccTX = 64, kAccTY = 8, kAccTZ = 8;
constexpr int kAccCap = 512;

__global__ void __launch_bounds__(256) k_los_accum(const uint32_t *__restrict__ cell,
                                                   const uint32_t *__restrict__ phi,
                                                   const uint16_t *__restrict__ w, Geom g, uint32_t S,
                                                   unsigned long long *acc, uint32_t *err) {
  __shared__ uint32_t tkey[kAccCap];
  __shared__ unsigned long long tM[kAccCap], tX[kAccCap], tY[kAccCap], tZ[kAccCap];
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  const int ntx = (g.nx + kAccTX - 1) / kAccTX, nty = (g.ny + kAccTY - 1) / kAccTY;
  const int ntz = (g.nz + kAccTZ - 1) / kAccTZ;
  const int64_t ntiles = (int64_t)ntx * nty * ntz;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    for (int i = t; i < kAccCap; i += 256) {
      tkey[i] = kNone;
      tM[i] = tX[i] = tY[i] = tZ[i] = 0ull;
    }
    __syncthreads();
    const int tx = (int)(tile % ntx), ty = (int)((tile / ntx) % nty), tz = (int)(tile / ((int64_t)ntx * nty));
    const int x = tx * kAccTX + lane;
    for (int r = wid; r < kAccTY * kAccTZ; r += 256 / kWave) {
      const int y = ty * kAccTY + (r % kAccTY), z = tz * kAccTZ + (r / kAccTY);
      if (y >= g.ny || z >= g.nz) continue;  // uniform across the wave
      const int64_t v = x + (int64_t)g.nx * (y + (int64_t)g.ny * z);
      uint32_t s = x < g.nx ? cell[v] : kNone;
      if (s != kNone && s >= S) {
        err[0] = 1u;
        s = kNone;
      }
      uint64_t m = 0, sx = 0, sy = 0, sz = 0;
      if (s != kNone) {
        m = w ? w[v] : 1u;
        int32_t px, py, pz;
        xyz(phi[v], g, px, py, pz);
        sx = m * (uint64_t)px;
        sy = m * (uint64_t)py;
        sz = m * (uint64_t)pz;
      }
      // segmented inclusive scan; a lane stops adding once its range holds
      // the start of its run
      const uint32_t sl_ = __shfl_up(s, 1, kWave), sr = __shfl_down(s, 1, kWave);
      uint32_t head = (lane == 0 || sl_ != s) ? 1u : 0u;
      const bool tail = lane == kWave - 1 || sr != s;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t ho = __shfl_up(head, d, kWave);
        const uint64_t mo = __shfl_up(m, d, kWave), xo = __shfl_up(sx, d, kWave);
        const uint64_t yo = __shfl_up(sy, d, kWave), zo = __shfl_up(sz, d, kWave);
        if (lane >= d && !head) { m += mo; sx += xo; sy += yo; sz += zo; head = ho; }
      }
      if (tail && s != kNone && m) {
        const int sl = lds_slot<kAccCap>(tkey, s);
        if (sl >= 0) {
          atomicAdd(&tM[sl], (unsigned long long)m);
          atomicAdd(&tX[sl], (unsigned long long)sx);
          atomicAdd(&tY[sl], (unsigned long long)sy);
          atomicAdd(&tZ[sl], (unsigned long long)sz);
        } else {
          unsigned long long *a = acc + 4 * (size_t)s;
          atomicAdd(a + 0, (unsigned long long)m);
          atomicAdd(a + 1, (unsigned long long)sx);
          atomicAdd(a + 2, (unsigned long long)sy);
          atomicAdd(a + 3, (unsigned long long)sz);
        }
      }
    }
    __syncthreads();
    for (int i = t; i < kAccCap; i += 256) {
      const uint32_t c = tkey[i];
      if (c != kNone && tM[i]) {
        unsigned long long *a = acc + 4 * (size_t)c;
        atomicAdd(a + 0, tM[i]);
        atomicAdd(a + 1, tX[i]);
        atomicAdd(a + 2, tY[i]);
        atomicAdd(a + 3, tZ[i]);
      }
    }
    __syncthreads();
  }
}

// Target X_c = round-half-up(256 S / M) per axis, then the walk from the
// anchor towards it, stopping where the segment first touches the closed
// cube of a voxel outside the component among the cubes it can move into.
__global__ void k_los_move(const uint32_t *__restrict__ comp, Geom g, uint32_t S,
                           const unsigned long long *__restrict__ acc, int32_t *q, uint32_t *anchor,
                           int32_t *target) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint64_t M = acc[4 * (size_t)s];
  int32_t *X = q + 3 * (size_t)s;
  if (M == 0) {
    if (target) target[3 * (size_t)s] = target[3 * (size_t)s + 1] = target[3 * (size_t)s + 2] = INT32_MIN;
    return;
  }
  int64_t T[3];
  for (int i = 0; i < 3; ++i) {
    const uint64_t Si = acc[4 * (size_t)s + 1 + i];
    const uint64_t qq = Si / M, r = Si % M;
    T[i] = (int64_t)(256 * qq + (512 * r + M) / (2 * M));
    if (target) target[3 * (size_t)s + i] = (int32_t)T[i];
  }
  const uint32_t a0 = anchor[s];
  const uint32_t c = comp[a0];
  int32_t cv[3];
  xyz(a0, g, cv[0], cv[1], cv[2]);
  const int32_t ext[3] = {g.nx, g.ny, g.nz};
  int64_t D[3], num[3], den[3];
  int32_t step[3];
  bool moving = false;
  for (int i = 0; i < 3; ++i) {
    D[i] = T[i] - X[i];
    step[i] = D[i] > 0 ? 1 : -1;
    den[i] = D[i] < 0 ? -D[i] : D[i];
    num[i] = (256 * (int64_t)cv[i] + 128 * step[i] - X[i]) * step[i];
    moving = moving || D[i] != 0;
  }
  if (!moving) return;
  for (;;) {
    int best = -1;
    for (int i = 0; i < 3; ++i) {
      if (den[i] == 0 || num[i] >= den[i]) continue;
      if (best < 0 || num[i] * den[best] < num[best] * den[i]) best = i;
    }
    if (best < 0) break;
    uint32_t tied = 0;
    for (int i = 0; i < 3; ++i)
      if (den[i] != 0 && num[i] < den[i] && num[i] * den[best] == num[best] * den[i]) tied |= 1u << i;
    bool blocked = false;
    for (uint32_t sub = tied; sub && !blocked; sub = (sub - 1) & tied) {
      int32_t p[3] = {cv[0], cv[1], cv[2]};
      for (int i = 0; i < 3; ++i)
        if (sub & (1u << i)) p[i] += step[i];
      if (p[0] < 0 || p[1] < 0 || p[2] < 0 || p[0] >= ext[0] || p[1] >= ext[1] || p[2] >= ext[2])
        blocked = true;
      else if (comp[p[0] + (int64_t)g.nx * (p[1] + (int64_t)g.ny * p[2])] != c)
        blocked = true;
    }
    if (blocked) {
      const int64_t tn = num[best], td = den[best];
      for (int i = 0; i < 3; ++i) X[i] = (int32_t)(X[i] + (tn * D[i]) / td);
      anchor[s] = (uint32_t)(cv[0] + (int64_t)g.nx * (cv[1] + (int64_t)g.ny * cv[2]));
      return;
    }
    for (int i = 0; i < 3; ++i)
      if (tied & (1u << i)) { cv[i] += step[i]; num[i] += 256; }
  }
  for (int i = 0; i < 3; ++i) X[i] = (int32_t)T[i];
  anchor[s] = (uint32_t)(cv[0] + (int64_t)g.nx * (cv[1] + (int64_t)g.ny * cv[2]));
}

__global__ void k_los_seed(const uint32_t *__restrict__ comp, Geom g, const uint32_t *__restrict__ seeds,
                           uint32_t S, int32_t *q, uint32_t *anchor, uint32_t *err) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint32_t v = seeds[s];
  if ((int64_t)v >= g.n || comp[v] == kNone) { err[0] = 1u; return; }
  int32_t x, y, z;
  xyz(v, g, x, y, z);
  q[3 * (size_t)s + 0] = 256 * x;
  q[3 * (size_t)s + 1] = 256 * y;
  q[3 * (size_t)s + 2] = 256 * z;
  anchor[s] = v;
}

// ---------------------------------------------------------------- host side
struct LosWork {
  double *pd;
  uint32_t *ps;
  uint32_t *nbh;
  uint8_t *blk;
  uint32_t *chg, *flag;
  uint32_t *ctl;  // [0] err, [1] phi flag, [2] last sweep
  unsigned long long *acc;
};

// The bit planes and their tiles: words along x, or, when x is too short to
// fill them and the volume is large, along the longer of the other two axes if
// that is longer.  A tile is a wave, so in a volume of one voxel along x words
// along x leave 16 voxels to each of 32 times as many waves; those run side by
// side until the card is full (4096 of these waves), and neighbours along the
// words lie nx apart in memory when turned, so a few waves of 16 voxels are
// better than fewer full ones.  One update with turned words over one without,
// e x e voxels across nx along x, 4 bands, 64 voxels a site: nx = 1 1.01 (e =
// 200), 0.94 (300), 0.86 (360), 0.70 (512), 0.55 (724); nx = 4 1.14, 1.05,
// 0.99, 0.81, 0.65; nx = 7 1.12, 1.06, 0.99, 0.86, 0.75.  The line is drawn
// between 300 and 360, at kTurnTiles tiles along x.  From 8 voxels on, x:
// 8 x 400 x 300 voxels 6.1 ms and 6.0 turned, 16 x 256 x 300 6.4 and 6.9.
struct LosPlane {
  int32_t axis, pa, pb, pc, pw, ty, tz;
};
constexpr int32_t kTurn = 8;
constexpr int64_t kTurnTiles = 6000;
LosPlane los_plane(const Geom &g) {
  LosPlane P{0, g.nx, g.ny, g.nz, 0, 0, 0};
  const int64_t tiles = (int64_t)((g.ny + kTY - 1) / kTY) * ((g.nz + kTZ - 1) / kTZ);  // of one word along x
  if (g.nx < kTurn && tiles > kTurnTiles && std::max(g.ny, g.nz) > g.nx)
    P = g.ny >= g.nz ? LosPlane{1, g.ny, g.nx, g.nz, 0, 0, 0} : LosPlane{2, g.nz, g.nx, g.ny, 0, 0, 0};
  P.pw = (P.pa + kTX - 1) / kTX;
  P.ty = (P.pb + kTY - 1) / kTY;
  P.tz = (P.pc + kTZ - 1) / kTZ;
  return P;
}

template <class C>
void los_layout(C &cv, const Geom &g, uint32_t S, LosWork *W) {
  double *pd = cv.template take<double>((size_t)g.n);
  uint32_t *ps = cv.template take<uint32_t>((size_t)g.n);
  uint32_t *nbh = cv.template take<uint32_t>((size_t)g.n);
  uint8_t *blk = cv.template take<uint8_t>((size_t)g.n);
  const LosPlane P = los_plane(g);
  const size_t words = (size_t)P.pw * P.pb * P.pc;
  uint32_t *chg = cv.template take<uint32_t>(words);
  uint32_t *flag = cv.template take<uint32_t>(words);
  uint32_t *ctl = cv.template take<uint32_t>(64);
  unsigned long long *acc = cv.template take<unsigned long long>(4 * (size_t)(S ? S : 1));
  if (W) *W = LosWork{pd, ps, nbh, blk, chg, flag, ctl, acc};
}

// The neighbourhood words of the component volume, which every pass over it
// reads (scratch: the proposals, which no sweep has written yet).
int32_t los_nbh(const uint32_t *d_comp, const Geom &g, const LosWork &W, hipStream_t s) {
  const dim3 gv((unsigned)((g.n + kLosThreads - 1) / kLosThreads)), b(kLosThreads);
  const Div dx = make_div((uint32_t)g.nx), dy = make_div((uint32_t)g.ny);
  uint8_t *p = reinterpret_cast<uint8_t *>(W.pd), *q = reinterpret_cast<uint8_t *>(W.ps);
  hipLaunchKernelGGL(k_los_radius<0>, gv, b, 0, s, d_comp, g, dx, dy, (const uint8_t *)nullptr, p);
  hipLaunchKernelGGL(k_los_radius<1>, gv, b, 0, s, d_comp, g, dx, dy, (const uint8_t *)p, q);
  hipLaunchKernelGGL(k_los_radius<2>, gv, b, 0, s, d_comp, g, dx, dy, (const uint8_t *)q, p);
  hipLaunchKernelGGL(k_los_nbh, gv, b, 0, s, d_comp, g, dx, dy, (const uint8_t *)p, W.nbh);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}

int32_t read_err(const uint32_t *d_err, hipStream_t s) {
  uint32_t e = 0;
  {
    const int32_t rc_ = read_words(d_err, 1, &e, s);
    if (rc_) return rc_;
  }
  return e ? LSRVT_EINVAL : LSRVT_OK;
}

// sweeps: in, what the stages took in the pass before (0: unknown); out, what
// they took.
int32_t los_vt(const uint32_t *d_comp, const Geom &g, const int32_t *d_q, const uint32_t *d_anchor, uint32_t S,
               double *d_dist, uint32_t *d_src, uint32_t *d_phi, uint32_t *d_cell, int32_t sweeps[2],
               const LosWork &W, hipStream_t s) {
  int32_t rc;
  const unsigned gs = grid_for(S, 256, 1 << 20);
  const unsigned gv = (unsigned)((g.n + kLosThreads - 1) / kLosThreads);
  const LosPlane P = los_plane(g);
  const uint32_t ntiles = (uint32_t)P.pw * (uint32_t)P.ty * (uint32_t)P.tz;
  LosArgs A{d_comp, g, d_q, d_anchor, S, d_dist, d_src, W.pd, W.ps, W.nbh, W.blk, W.chg, W.flag, W.ctl + 2,
            W.ctl,
            make_div((uint32_t)g.nx), make_div((uint32_t)g.ny), P.axis, P.pa, P.pb, P.pc, P.pw, P.ty, ntiles};
  const dim3 gt(std::min((ntiles + 7) / 8 * 8, kTileRun), (ntiles + kTileRun - 1) / kTileRun), bt(kWave);
  if ((rc = fill<uint32_t>(W.ctl, 2, 0u, s))) return rc;
  if (S) {
    hipLaunchKernelGGL(k_los_check, dim3(gs), dim3(256), 0, s, d_comp, g, d_q, d_anchor, S, W.ctl);
    LSRVT_LAUNCHED();
    if ((rc = read_err(W.ctl, s))) return rc;
  }
  if ((rc = fill<double>(d_dist, g.n, __builtin_inf(), s))) return rc;
  if ((rc = fill<uint32_t>(d_src, g.n, kNone, s))) return rc;
  if ((rc = fill<uint8_t>(W.blk, g.n, 0, s))) return rc;
  if ((rc = fill<uint32_t>(W.flag, (int64_t)P.pw * P.pb * P.pc, 0u, s))) return rc;
  if (S) {
    hipLaunchKernelGGL(k_anchor_reset, dim3(gs), dim3(256), 0, s, A);
    hipLaunchKernelGGL(k_anchor_len, dim3(gs), dim3(256), 0, s, A);
    hipLaunchKernelGGL(k_anchor_id, dim3(gs), dim3(256), 0, s, A);
    hipLaunchKernelGGL(k_anchor_set, dim3(gs), dim3(256), 0, s, A);
    LSRVT_LAUNCHED();
  }
  for (int stage = 1; stage <= 2; ++stage) {
    // as many sweeps as the stage took in the pass before, then a few at a time
    int32_t &took = sweeps[stage - 1];
    int32_t batch = took ? took + 2 : kSweepBatch;
    uint32_t launched = 0, last = 0;
    if ((rc = fill<uint32_t>(A.last, 1, 0u, s))) return rc;
    while (launched == last) {
      if (launched >= (uint32_t)kMaxSweeps) return LSRVT_ELIMIT;
      for (int32_t j = 0; j < batch && launched < (uint32_t)kMaxSweeps; ++j) {
        ++launched;
        // the first sweep of stage 2 re-evaluates everything: new candidates
        const int all = stage == 2 && launched == 1;
        hipLaunchKernelGGL((stage == 1 ? P.axis ? k_los_eval<1, true> : k_los_eval<1, false>
                                       : P.axis ? k_los_eval<2, true> : k_los_eval<2, false>),
                           gt, bt, 0, s, A, launched, all);
        hipLaunchKernelGGL((stage == 1 ? P.axis ? k_los_apply<1, true> : k_los_apply<1, false>
                                       : P.axis ? k_los_apply<2, true> : k_los_apply<2, false>),
                           gt, bt, 0, s, A, launched);
      }
      LSRVT_LAUNCHED();
      if ((rc = read_words(A.last, 1, &last, s))) return rc;
      batch = kSweepBatch;
    }
    took = (int32_t)last + 1;  // the sweep after the last change found none
  }
  for (int r = 0;; ++r) {
    if (r >= kPhiRounds) return LSRVT_ELIMIT;
    if (r && (rc = fill<uint32_t>(W.ctl + 1, 1, 0u, s))) return rc;
    if (r == 0)
      hipLaunchKernelGGL(k_phi<true>, dim3(gv), dim3(kLosThreads), 0, s, d_src, g.n, d_phi, d_cell, W.ctl + 1);
    else
      hipLaunchKernelGGL(k_phi<false>, dim3(gv), dim3(kLosThreads), 0, s, d_src, g.n, d_phi, d_cell, W.ctl + 1);
    LSRVT_LAUNCHED();
    uint32_t f = 0;
    if ((rc = read_words(W.ctl + 1, 1, &f, s))) return rc;
    if (!f) break;
  }
  return LSRVT_OK;
}

int32_t los_update(const uint32_t *d_comp, const Geom &g, const uint16_t *d_w, const uint32_t *d_cell,
                   const uint32_t *d_phi, uint32_t S, int32_t *d_q, uint32_t *d_anchor, int32_t *d_target,
                   const LosWork &W, hipStream_t s) {
  int32_t rc;
  if (S == 0) return LSRVT_OK;
  if ((rc = fill<uint32_t>(W.ctl, 1, 0u, s))) return rc;
  if ((rc = fill<unsigned long long>(W.acc, 4 * (int64_t)S, 0ull, s))) return rc;
  const int64_t ntiles = (int64_t)((g.nx + kAccTX - 1) / kAccTX) * ((g.ny + kAccTY - 1) / kAccTY) *
                         ((g.nz + kAccTZ - 1) / kAccTZ);
  hipLaunchKernelGGL(k_los_accum, dim3((unsigned)std::min<int64_t>(ntiles, 65535)), dim3(256), 0, s, d_cell, d_phi,
                     d_w, g, S, W.acc, W.ctl);
  hipLaunchKernelGGL(k_los_move, dim3(grid_for(S, 256, 1 << 20)), dim3(256), 0, s, d_comp, g, S, W.acc, d_q,
                     d_anchor, d_target);
  LSRVT_LAUNCHED();
  return read_err(W.ctl, s);
}

}  // namespace
}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_los_workspace(lsrvt_dims dims, uint32_t n_sites) {
  Geom g;
  if (make_geom(dims, g) != LSRVT_OK || n_sites >= kSite) return 0;
  Sizer sz;
  los_layout(sz, g, n_sites, nullptr);
  return sz.off;
}

static int32_t los_prepare(lsrvt_dims dims, uint32_t S, void *d_work, size_t work_bytes, Geom &g, LosWork &W) {
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (S >= kSite) return LSRVT_ELIMIT;
  if ((rc = check_work(d_work, work_bytes, lsrvt_los_workspace(dims, S)))) return rc;
  Carve cv(d_work, work_bytes);
  los_layout(cv, g, S, &W);
  return cv.ok ? LSRVT_OK : LSRVT_EWORKSPACE;
}

extern "C" int32_t lsrvt_los_vt(const uint32_t *d_comp, lsrvt_dims dims, const int32_t *d_site_q,
                                const uint32_t *d_anchor, uint32_t n_sites, double *d_dist, uint32_t *d_src,
                                uint32_t *d_phi, uint32_t *d_cell, int32_t *h_sweeps, void *d_work,
                                size_t work_bytes, void *stream) {
  if (!d_comp || !d_dist || !d_src || !d_phi || !d_cell || (n_sites && (!d_site_q || !d_anchor)))
    return LSRVT_EINVAL;
  Geom g;
  LosWork W;
  int32_t rc = los_prepare(dims, n_sites, d_work, work_bytes, g, W);
  if (rc || (rc = los_nbh(d_comp, g, W, as_stream(stream)))) return rc;
  int32_t sw[2] = {0, 0};
  rc = los_vt(d_comp, g, d_site_q, d_anchor, n_sites, d_dist, d_src, d_phi, d_cell, sw, W, as_stream(stream));
  for (int k = 0; k < 2; ++k)
    if (h_sweeps && sw[k]) h_sweeps[k] = sw[k];  // of every stage that ended
  return rc;
}

extern "C" int32_t lsrvt_los_update(const uint32_t *d_comp, lsrvt_dims dims, const uint16_t *d_weights,
                                    const uint32_t *d_cell, const uint32_t *d_phi, uint32_t n_sites,
                                    int32_t *d_site_q, uint32_t *d_anchor, int32_t *d_target_q, void *d_work,
                                    size_t work_bytes, void *stream) {
  if (!d_comp || !d_cell || !d_phi || (n_sites && (!d_site_q || !d_anchor))) return LSRVT_EINVAL;
  Geom g;
  LosWork W;
  int32_t rc = los_prepare(dims, n_sites, d_work, work_bytes, g, W);
  if (rc) return rc;
  return los_update(d_comp, g, d_weights, d_cell, d_phi, n_sites, d_site_q, d_anchor, d_target_q, W,
                    as_stream(stream));
}

extern "C" int32_t lsrvt_los_cvt(const uint32_t *d_comp, lsrvt_dims dims, const uint32_t *d_seeds,
                                 uint32_t n_sites, const uint16_t *d_weights, int32_t iters, int32_t *d_site_q,
                                 uint32_t *d_anchor, double *d_dist, uint32_t *d_src, uint32_t *d_phi,
                                 uint32_t *d_cell, int32_t *h_sweeps, void *d_work, size_t work_bytes,
                                 void *stream) {
  if (!d_comp || !d_dist || !d_src || !d_phi || !d_cell || iters < 0 ||
      (n_sites && (!d_seeds || !d_site_q || !d_anchor)))
    return LSRVT_EINVAL;
  Geom g;
  LosWork W;
  int32_t rc = los_prepare(dims, n_sites, d_work, work_bytes, g, W);
  if (rc) return rc;
  hipStream_t s = as_stream(stream);
  if (h_sweeps) *h_sweeps = 0;
  if (n_sites) {
    if ((rc = fill<uint32_t>(W.ctl, 1, 0u, s))) return rc;
    hipLaunchKernelGGL(k_los_seed, dim3(grid_for(n_sites, 256, 1 << 20)), dim3(256), 0, s, d_comp, g, d_seeds,
                       n_sites, d_site_q, d_anchor, W.ctl);
    LSRVT_LAUNCHED();
    if ((rc = read_err(W.ctl, s))) return rc;
  }
  if ((rc = los_nbh(d_comp, g, W, s))) return rc;
  int32_t sw[2] = {0, 0};
  for (int32_t t = 0; t <= iters; ++t) {
    rc = los_vt(d_comp, g, d_site_q, d_anchor, n_sites, d_dist, d_src, d_phi, d_cell, sw, W, s);
    if (rc) return rc;
    if (h_sweeps) *h_sweeps += sw[0] + sw[1];
    if (t == iters) break;
    rc = los_update(d_comp, g, d_weights, d_cell, d_phi, n_sites, d_site_q, d_anchor, nullptr, W, s);
    if (rc) return rc;
  }
  return LSRVT_OK;
}
