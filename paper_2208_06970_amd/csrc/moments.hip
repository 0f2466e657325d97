// Joint moments up to fourth order of every cell, component and band: the
// centred sums M2 (covariance), M3 (coskewness) and M4 (cokurtosis) that the
// joint plots compare between the raw data and the fitted distribution
// models (Sec. 4.4), merged up the hierarchy of Sec. 3.2.4 / Fig. 5.  Up to
// 18 variables: 7314 sums of orders 1 to 4 per unit.
//
// Cells: the voxels of a cell are one range of the structured layout, cut into
// items.  With d_0 = 1 and d_1 .. d_m the offsets x - x(site) in float64, every
// raw sum S1_i, S2_ij, S3_ijk, S4_ijkl about the site value is the sum over the
// voxels of a product (d_i d_j)(d_k d_l) with i <= j <= k <= l: a matrix
// product of pair rows, taken on the matrix cores (k_mom_cells).  The raw sums,
// written to the cell's output rows, then become centred sums in place with
// the mean offset a = S1 / n (k_mom_center).
// Components and bands: the members' centred sums shifted to the group's mean
// (k_mom_shift); the shifted sums only add, so members are taken in fixed
// chunks side by side and the chunk results added in order.  Everything is
// float64.
#include <algorithm>

#include "layout.h"

namespace lsrvt {
namespace {

constexpr int kMomMaxVars = 18;  // 7314 moments of orders 1..4 per unit at m = 18
constexpr int kMomThreads = 256;
constexpr int kMomRound = 64;    // voxels staged in LDS at a time
constexpr int kMergeChunk = 16;  // members of a group shifted and added by one workgroup
constexpr int kMaxPairs = (kMomMaxVars + 1) * (kMomMaxVars + 2) / 2;  // pairs i <= j of 0 .. m
constexpr int kMaxPairTiles = (kMaxPairs + 15) / 16;
constexpr int kMaxTiles = 44;  // 16 x 16 tiles of pair products (41 with 18 variables)

typedef double d4 __attribute__((ext_vector_type(4)));

struct MomShape {
  int m, P2, P3, P4, U;  // U = m + P2 + P3 + P4 raw units
};

MomShape mom_shape(int m) {
  MomShape s;
  s.m = m;
  s.P2 = m * (m + 1) / 2;
  s.P3 = m * (m + 1) * (m + 2) / 6;
  s.P4 = m * (m + 1) * (m + 2) * (m + 3) / 24;
  s.U = m + s.P2 + s.P3 + s.P4;
  return s;
}

// The pair products needed by the sums.  Rows of the product are the pairs
// (i, j), i <= j, of the indices 0 .. m ordered by j, columns the pairs (k, l)
// ordered by k; entry (ij, kl) is a sum of its own exactly when j <= k, so of the
// tiles of 16 x 16 only those with such an entry are taken: 41 of the 144 with
// 18 variables, whose 7315 entries would fill 29.
struct MomTiles {
  int n, pairs;
  uint8_t a[kMaxTiles], b[kMaxTiles];
};

MomTiles mom_tiles(int m) {
  MomTiles T{};
  const int M = m + 1;
  T.pairs = M * (M + 1) / 2;
  const int nt = (T.pairs + 15) / 16;
  int top[kMaxPairTiles];  // largest k of column tile b
  int q = 0;
  for (int k = 0; k < M; ++k)
    for (int l = k; l < M; ++l) top[q++ / 16] = k;
  for (int a = 0; a < nt; ++a) {
    int j = 0;  // smallest j of row tile a: that of its first pair
    while ((j + 1) * (j + 2) / 2 <= 16 * a) ++j;
    for (int b = 0; b < nt; ++b)
      if (j <= top[b]) {
        T.a[T.n] = (uint8_t)a;
        T.b[T.n] = (uint8_t)b;
        ++T.n;
      }
  }
  return T;
}

// Tables built on the device: code[u] = order | i << 4 | j << 9 | k << 14 |
// l << 19 of raw unit u (units of order 1, then 2, 3, 4, each in
// lexicographic order of i <= j <= k <= l), the packed position of every
// sorted pair and triple, and the unit of every entry of the product tiles in
// the lanes' order (kNoUnit where there is none).
struct MomTables {
  uint32_t *code;  // [U]
  uint16_t *idx2;  // [m][m]
  uint16_t *idx3;  // [m][m][m]
  uint16_t *unit;  // [tiles][64 lanes][4]
};
constexpr uint32_t kNoUnit = 0xFFFFu;

// Positions of sorted tuples among all of m variables, lexicographic.
__host__ __device__ inline int pos2(int m, int i, int j) { return i * m - i * (i - 1) / 2 + (j - i); }
__host__ __device__ inline int pos3(int m, int i, int j, int k) {
  const int r = m - i;
  return m * (m + 1) * (m + 2) / 6 - r * (r + 1) * (r + 2) / 6 + pos2(r, j - i, k - i);
}
__host__ __device__ inline int pos4(int m, int i, int j, int k, int l) {
  const int r = m - i;
  return m * (m + 1) * (m + 2) * (m + 3) / 24 - r * (r + 1) * (r + 2) * (r + 3) / 24 + pos3(r, j - i, k - i, l - i);
}

// Unit of the sorted tuple i <= j <= k <= l of 0 .. m (0: the constant 1).
__device__ inline uint32_t unit_of(const MomShape &S, int i, int j, int k, int l) {
  const int m = S.m;
  if (i > 0) return (uint32_t)(m + S.P2 + S.P3 + pos4(m, i - 1, j - 1, k - 1, l - 1));
  if (j > 0) return (uint32_t)(m + S.P2 + pos3(m, j - 1, k - 1, l - 1));
  if (k > 0) return (uint32_t)(m + pos2(m, k - 1, l - 1));
  return l > 0 ? (uint32_t)(l - 1) : kNoUnit;
}

// Pair p of the indices 0 .. M - 1 ordered by its larger (rows) or its
// smaller (columns) index.
__device__ inline void row_pair(int p, int &i, int &j) {
  j = 0;
  while ((j + 1) * (j + 2) / 2 <= p) ++j;
  i = p - j * (j + 1) / 2;
}
__device__ inline void col_pair(int M, int p, int &k, int &l) {
  k = 0;
  while (p >= M - k) p -= M - k++;
  l = k + p;
}

__global__ __launch_bounds__(256) void k_mom_tables(MomShape S, MomTables T, MomTiles P) {
  const int m = S.m, M = m + 1;
  const int at = blockIdx.x * 256 + threadIdx.x;
  if (at < M * M * M * M) {
    const int i = at / (M * M * M), j = at / (M * M) % M, k = at / M % M, l = at % M;
    if (i <= j && j <= k && k <= l && l > 0) {
      const uint32_t u = unit_of(S, i, j, k, l);
      T.code[u] = i > 0   ? 4u | (uint32_t)(i - 1) << 4 | (uint32_t)(j - 1) << 9 | (uint32_t)(k - 1) << 14 |
                              (uint32_t)(l - 1) << 19
                  : j > 0 ? 3u | (uint32_t)(j - 1) << 4 | (uint32_t)(k - 1) << 9 | (uint32_t)(l - 1) << 14
                  : k > 0 ? 2u | (uint32_t)(k - 1) << 4 | (uint32_t)(l - 1) << 9
                          : 1u | (uint32_t)(l - 1) << 4;
      if (i == 0 && j > 0) T.idx3[((j - 1) * m + k - 1) * m + l - 1] = (uint16_t)pos3(m, j - 1, k - 1, l - 1);
      if (i == 0 && j == 0 && k > 0) T.idx2[(k - 1) * m + l - 1] = (uint16_t)pos2(m, k - 1, l - 1);
    }
  }
  if (at < P.n * 256) {
    // lane `lane` of the tile's accumulator holds rows 4 r + lane / 16 of column lane % 16
    const int tile = at / 256, lane = at / 4 % 64, r = at % 4;
    const int pa = 16 * P.a[tile] + 4 * r + lane / 16, pb = 16 * P.b[tile] + lane % 16;
    uint32_t u = kNoUnit;
    if (pa < P.pairs && pb < P.pairs) {
      int i, j, k, l;
      row_pair(pa, i, j);
      col_pair(M, pb, k, l);
      if (j <= k) u = unit_of(S, i, j, k, l);
    }
    T.unit[at] = (uint16_t)u;
  }
}

struct MomOut {
  uint64_t *n;
  double *mean, *m2, *m3, *m4;
};

__device__ __forceinline__ int cidx(uint32_t code, int q) { return (int)((code >> (4 + 5 * q)) & 31u); }

// sorted-tuple lookups (a <= b <= c)
__device__ __forceinline__ int p2(const uint16_t *idx2, int m, int a, int b) { return idx2[a * m + b]; }
__device__ __forceinline__ int p3(const uint16_t *idx3, int m, int a, int b, int c) {
  return idx3[(a * m + b) * m + c];
}

// Entry u (order 1, then 2, 3, 4) of a unit's output rows.
__device__ __forceinline__ double *mom_row(const MomOut &o, const MomShape &sh, int64_t row, int u) {
  if (u < sh.m) return o.mean + row * sh.m + u;
  u -= sh.m;
  if (u < sh.P2) return o.m2 + row * sh.P2 + u;
  u -= sh.P2;
  if (u < sh.P3) return o.m3 + row * sh.P3 + u;
  return o.m4 + row * sh.P4 + (u - sh.P3);
}

// Items of at most `item` voxels; every cell has at least one, and the ones
// after its first are numbered by poff (by rank).
__global__ void k_mom_items(const uint32_t *__restrict__ cell_off, uint32_t S, uint32_t item, uint32_t *more) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= S) return;
  const uint32_t cnt = cell_off[r + 1] - cell_off[r];
  more[r] = cnt ? (cnt - 1) / item : 0u;
}
__global__ void k_mom_item_rank(const uint32_t *__restrict__ poff, uint32_t S, uint32_t *__restrict__ item_rank) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= S) return;
  const uint32_t hi = poff[r + 1];
  for (uint32_t p = poff[r]; p < hi; ++p) item_rank[r + 1 + p] = r;
  item_rank[r + poff[r]] = r;
}

// Raw sums about the site value of every item: the sum of unit (i, j, k, l)
// over the voxels is entry (ij, kl) of the product of the pair rows' values
// with the pair columns' values, taken in tiles of 16 x 16 with four voxels
// per matrix instruction.  The item's voxels are staged 64 at a time in LDS as
// float64 offsets (d_0 = 1; all zero past the item's end); a lane forms the
// one pair product of its operand from two of them, and keeps a row tile's
// operand over the column tiles that follow it.  Wave (tg, vg) of the
// workgroup owns the tiles of group tg (TG groups of up to TPW tiles each, the
// accumulators of all of them in registers) on every VG-th step of four
// voxels; the VG partial results are added in order at the end.  A cell's
// first item writes the cell's output rows, the others a row of `part` each.
//
// Bound by the float64 matrix rate: 41 tiles for 7314 sums, 30 TFLOP/s of the
// 59 that a large library product reaches.  256 x 128 x 128 voxels in 2036
// uneven cells with 18 variables take 2.9 ms; with one workgroup per cell and
// pass of 1024 units, each unit multiplied out from LDS by its own thread,
// they took 1199 ms (the largest cells ran alone at the end).
struct MomCellArgs {
  const uint32_t *perm, *cell_off, *order, *sites, *poff, *item_rank;
  uint32_t n_items, item;
  const float *vars;
  int64_t N;
  MomShape sh;
  MomTiles tiles;
  const uint16_t *unit;
  MomOut out;
  double *part;  // [items after the first][U]
};

template <int TPW, int TG>
__global__ __launch_bounds__(kMomThreads, TPW > 6 ? 2 : 3) void k_mom_cells(MomCellArgs A) {
  constexpr int VG = kMomThreads / kWave / TG;
  constexpr int kLd = kMomMaxVars + 1;  // row stride in doubles (odd)
  constexpr int kPerThread = (kMomRound * kMomMaxVars + kMomThreads - 1) / kMomThreads;
  __shared__ double d[2][kMomRound * kLd];
  __shared__ double K[kMomMaxVars];
  __shared__ d4 red[VG > 1 ? kMomThreads : 1];
  const int t = threadIdx.x, lane = lane_id();
  const int wid = __builtin_amdgcn_readfirstlane(t / kWave);
  const int tg = wid % TG, vg = wid / TG;
  const int m = A.sh.m, M = m + 1;
  // this wave's tiles, and each lane's offsets of the two factors of its operands
  const int per = (A.tiles.n + TG - 1) / TG;
  const int t0 = tg * per, nq = max(0, min(per, A.tiles.n - t0));
  uint32_t oa[TPW], ob[TPW], fresh = 0;
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    oa[q] = ob[q] = 0u;
    if (q >= nq) continue;
    const int a = A.tiles.a[t0 + q], b = A.tiles.b[t0 + q];
    if (q == 0 || a != A.tiles.a[t0 + q - 1]) fresh |= 1u << q;
    // a pair past the last gives entries that no unit takes
    int i, j;
    row_pair(min(16 * a + lane % 16, A.tiles.pairs - 1), i, j);
    oa[q] = (uint32_t)i | (uint32_t)j << 16;
    col_pair(M, min(16 * b + lane % 16, A.tiles.pairs - 1), i, j);
    ob[q] = (uint32_t)i | (uint32_t)j << 16;
  }
  fresh = __builtin_amdgcn_readfirstlane(fresh);

  for (uint32_t it = blockIdx.x; it < A.n_items; it += gridDim.x) {
    const uint32_t r = A.item_rank[it];
    const uint32_t k = it - (r + A.poff[r]);  // item k of its cell
    const uint32_t site = A.order[r];
    const uint32_t lo = A.cell_off[r] + k * A.item;
    const uint32_t hi = min(A.cell_off[r + 1], lo + A.item);
    __syncthreads();
    if (t < m) K[t] = hi > lo ? (double)A.vars[(int64_t)t * A.N + A.sites[site]] : 0.0;
    d4 acc[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) acc[q] = d4{0.0, 0.0, 0.0, 0.0};
    float x[kPerThread];
    auto fetch = [&](uint32_t base) {  // the thread's values of the round at base
      const int v = t % kMomRound;
      const bool in = base + v < hi;
      const uint32_t at = in ? A.perm[base + v] : 0u;
#pragma unroll
      for (int i = 0; i < kPerThread; ++i) {
        const int j = t / kMomRound + i * (kMomThreads / kMomRound);
        x[i] = in && j < m ? A.vars[(int64_t)j * A.N + at] : 0.0f;
      }
    };
    auto stage = [&](uint32_t base, double *dst) {
      const int v = t % kMomRound;
      const bool in = base + v < hi;
#pragma unroll
      for (int i = 0; i < kPerThread; ++i) {
        const int j = t / kMomRound + i * (kMomThreads / kMomRound);
        if (j < m) dst[v * kLd + 1 + j] = in ? (double)x[i] - K[j] : 0.0;
      }
      if (t < kMomRound) dst[v * kLd] = in ? 1.0 : 0.0;
    };
    if (lo < hi) fetch(lo);
    __syncthreads();  // K
    int buf = 0;
    for (uint32_t base = lo; base < hi; base += kMomRound, buf ^= 1) {
      // a buffer is written again only after the barrier of the round between
      stage(base, d[buf]);
      __syncthreads();
      if (base + kMomRound < hi) fetch(base + kMomRound);
      const int steps = (int)(min((uint32_t)kMomRound, hi - base) + 3) / 4;
      for (int s = vg; s < steps; s += VG) {
        const double *dv = d[buf] + (4 * s + lane / 16) * kLd;
        double av = 0.0;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
          if (q < nq) {
            if (fresh >> q & 1u) av = dv[oa[q] & 0xFFFFu] * dv[oa[q] >> 16];
            const double bv = dv[ob[q] & 0xFFFFu] * dv[ob[q] >> 16];
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[q], 0, 0, 0);
          }
        }
      }
    }
    // the voxel groups' partial results in order, then the units of this wave's tiles
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      d4 v = acc[q];
      if constexpr (VG > 1) {
        __syncthreads();
        red[t] = v;
        __syncthreads();
#pragma unroll
        for (int g = 1; g < VG; ++g) v += red[(t + g * TG * kWave) % kMomThreads];
      }
      if (q < nq && vg == 0) {
        const uint16_t *un = A.unit + ((t0 + q) * 64 + lane) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int u = un[i];
          if (u != (int)kNoUnit) {
            double *dst = k ? A.part + ((int64_t)A.poff[r] + k - 1) * A.sh.U + u : mom_row(A.out, A.sh, site, u);
            *dst = v[i];
          }
        }
      }
    }
  }
}

// The rows of a cell's later items added to its output rows, in order.
__global__ __launch_bounds__(kMomThreads) void k_mom_combine(const uint32_t *__restrict__ poff,
                                                             const uint32_t *__restrict__ order, uint32_t S,
                                                             const double *__restrict__ part, MomShape sh, MomOut out) {
  const int u = blockIdx.y * kMomThreads + threadIdx.x;
  if (u >= sh.U) return;
  for (uint32_t r = blockIdx.x; r < S; r += gridDim.x) {
    const uint32_t p0 = poff[r], p1 = poff[r + 1];
    if (p0 == p1) continue;
    double *dst = mom_row(out, sh, order[r], u);
    double v = *dst;
#pragma unroll 8
    for (uint32_t p = p0; p < p1; ++p) v += part[(int64_t)p * sh.U + u];
    *dst = v;
  }
}

// The raw sums of every cell about its site value become centred sums with
// the mean offset a = S1 / n, in place, highest order first (each order reads
// only lower orders' raw sums, which are rewritten later):
//   M4_ijkl = S4_ijkl - sum over the 4 indices of a_x S3_(other three)
//             + sum over the 6 index pairs of a_x a_y S2_(other two)
//             - 3 n a_i a_j a_k a_l
//   M3_ijk  = S3_ijk - (a_i S2_jk + a_j S2_ik + a_k S2_ij) + 2 n a_i a_j a_k
//   M2_ij   = S2_ij - n a_i a_j
//   mean_i  = x_i(site) + a_i
// One workgroup per cell.
__global__ __launch_bounds__(kMomThreads) void k_mom_center(const uint32_t *__restrict__ cell_off,
                                                            const uint32_t *__restrict__ order,
                                                            const uint32_t *__restrict__ sites, uint32_t S,
                                                            const float *__restrict__ vars, int64_t N, MomShape sh,
                                                            MomTables T, MomOut out) {
  __shared__ uint16_t i2[kMomMaxVars * kMomMaxVars], i3[kMomMaxVars * kMomMaxVars * kMomMaxVars];
  __shared__ double a_s[kMomMaxVars];
  const int t = threadIdx.x;
  const int m = sh.m;
  for (int i = t; i < m * m; i += kMomThreads) i2[i] = T.idx2[i];
  for (int i = t; i < m * m * m; i += kMomThreads) i3[i] = T.idx3[i];
  for (uint32_t r = blockIdx.x; r < S; r += gridDim.x) {
    const uint32_t lo = cell_off[r], hi = cell_off[r + 1];
    const uint32_t site = order[r];
    const double n = (double)(hi - lo);
    double *mean = out.mean + (int64_t)site * m, *m2 = out.m2 + (int64_t)site * sh.P2,
           *m3 = out.m3 + (int64_t)site * sh.P3, *m4 = out.m4 + (int64_t)site * sh.P4;
    __syncthreads();
    if (t < m) a_s[t] = hi > lo ? mean[t] / n : 0.0;
    __syncthreads();
    auto a = [&](int j) { return a_s[j]; };
    for (int q = t; q < sh.P4; q += kMomThreads) {
      const uint32_t code = T.code[m + sh.P2 + sh.P3 + q];
      const int i = cidx(code, 0), j = cidx(code, 1), k = cidx(code, 2), l = cidx(code, 3);
      double v = m4[q];
      v -= a(i) * m3[p3(i3, m, j, k, l)] + a(j) * m3[p3(i3, m, i, k, l)] + a(k) * m3[p3(i3, m, i, j, l)] +
           a(l) * m3[p3(i3, m, i, j, k)];
      v += a(i) * a(j) * m2[p2(i2, m, k, l)] + a(i) * a(k) * m2[p2(i2, m, j, l)] + a(i) * a(l) * m2[p2(i2, m, j, k)] +
           a(j) * a(k) * m2[p2(i2, m, i, l)] + a(j) * a(l) * m2[p2(i2, m, i, k)] + a(k) * a(l) * m2[p2(i2, m, i, j)];
      v -= 3.0 * n * a(i) * a(j) * a(k) * a(l);
      m4[q] = v;
    }
    __syncthreads();
    for (int q = t; q < sh.P3; q += kMomThreads) {
      const uint32_t code = T.code[m + sh.P2 + q];
      const int i = cidx(code, 0), j = cidx(code, 1), k = cidx(code, 2);
      m3[q] = m3[q] - (a(i) * m2[p2(i2, m, j, k)] + a(j) * m2[p2(i2, m, i, k)] + a(k) * m2[p2(i2, m, i, j)]) +
              2.0 * n * a(i) * a(j) * a(k);
    }
    __syncthreads();
    for (int q = t; q < sh.P2; q += kMomThreads) {
      const uint32_t code = T.code[m + q];
      const int i = cidx(code, 0), j = cidx(code, 1);
      m2[q] = m2[q] - n * a(i) * a(j);
    }
    if (t < m) mean[t] = hi > lo ? (double)vars[(int64_t)t * N + sites[site]] + a(t) : 0.0;
    if (t == 0) out.n[site] = (uint64_t)(hi - lo);
  }
}

// Group inputs: members of group g are member_id(lo + k) for k < hi - lo.
struct MergeIn {
  const uint64_t *n;  // member arrays in the MomOut layout
  const double *mean, *m2, *m3, *m4;
  const uint32_t *map;  // member index -> row (null: identity)
};

// Groups of members merge without an order of their own: with delta = the
// member's mean - the group's mean, the member's centred sums about the
// group's mean are
//   M2'_ab   = M2_ab + n d_a d_b
//   M3'_abc  = M3_abc + sum over the 3 indices x of d_x M2_(other two) + n d_a d_b d_c
//   M4'_abcd = M4_abcd + sum over the 4 indices x of d_x M3_(other three)
//              + sum over the 6 index pairs {x,y} of d_x d_y M2_(other two) + n d_a d_b d_c d_d
// (a member's first centred sums are zero), every term of the size of the
// result, and the group's sums are their sum over the members.  Groups longer
// than kMergeChunk are cut into chunks; a chunk's sums go to a row of `part`
// and the rows add in order.  2036 cells in 1231 components and 11 bands with 18
// variables take 0.37 ms, bound by the reads of M2 and M3 from LDS; one
// workgroup merging up to 128 members one after another by pairwise formulas
// took 7.8 ms (a serial chain of 128 rows).
struct MomGroups {
  uint32_t G;
  const uint32_t *off;     // members off[g] .. off[g + 1]
  const uint32_t *choff;   // chunks of the groups longer than kMergeChunk, by group
  const uint32_t *job_lo, *job_hi, *job_group;  // members and group of every chunk
  uint32_t J;
};

// Counts and first sums about the mean of the group's first member (about zero
// where that is not finite, so that what an infinite mean gives does not hang on
// which member has it): of every
// chunk (job = true: rows of `sum`, [m + 1] each) or of every group, whose
// mean is formed.
template <bool job>
__global__ __launch_bounds__(kWave) void k_mom_mean(MomGroups Q, MergeIn in, MomShape sh, double *sum, MomOut out) {
  const int m = sh.m, j = threadIdx.x;
  for (uint32_t b = blockIdx.x; b < (job ? Q.J : Q.G); b += gridDim.x) {
    const uint32_t g = job ? Q.job_group[b] : b;
    const uint32_t lo = job ? Q.job_lo[b] : Q.off[g], hi = job ? Q.job_hi[b] : Q.off[g + 1];
    if (j > m) continue;  // lane m: the counts
    const uint32_t f = Q.off[g];
    const double mean0 = j < m && hi > lo ? in.mean[(int64_t)(in.map ? in.map[f] : f) * m + j] : 0.0;
    const double first = __builtin_isfinite(mean0) ? mean0 : 0.0;
    const bool split = !job && hi - lo > (uint32_t)kMergeChunk;
    double s = 0.0;
    if (split) {
#pragma unroll 8
      for (uint32_t c = Q.choff[g]; c < Q.choff[g + 1]; ++c) s += sum[(int64_t)c * (m + 1) + j];
    } else {
#pragma unroll 4
      for (uint32_t k = lo; k < hi; ++k) {
        const uint32_t row = in.map ? in.map[k] : k;
        const double n = (double)in.n[row];
        s += j == m ? n : n > 0.0 ? n * (in.mean[(int64_t)row * m + j] - first) : 0.0;
      }
    }
    if (job) {
      sum[(int64_t)b * (m + 1) + j] = s;
    } else {
      const double n = __shfl(s, m, kWave);
      if (j == m)
        out.n[g] = (uint64_t)s;
      else
        out.mean[(int64_t)g * m + j] = n > 0.0 ? (hi - lo == 1 ? mean0 : first + s / n) : 0.0;
    }
  }
}

// The members' sums of orders 2 to 4 about the group's mean, units
// [blockIdx.y * kShiftUnits, + kShiftUnits) of the order-1-less rows: of every
// chunk into `part` (job = true), or of every group, a long one's from its
// chunks' rows.  The member's M2, M3 and offsets are staged in LDS.
constexpr int kShiftUnits = 2048;
template <bool job>
__global__ __launch_bounds__(kMomThreads) void k_mom_shift(MomGroups Q, MergeIn in, MomShape sh, MomTables T,
                                                           double *part, MomOut out) {
  constexpr int kPer = kShiftUnits / kMomThreads;
  __shared__ uint16_t i2[kMomMaxVars * kMomMaxVars], i3[kMomMaxVars * kMomMaxVars * kMomMaxVars];
  __shared__ double s2[kMomMaxVars * (kMomMaxVars + 1) / 2];
  __shared__ double s3[kMomMaxVars * (kMomMaxVars + 1) * (kMomMaxVars + 2) / 6];
  __shared__ double d[kMomMaxVars];
  const int t = threadIdx.x, m = sh.m, W = sh.U - m;
  const int u0 = blockIdx.y * kShiftUnits;
  for (int i = t; i < m * m; i += kMomThreads) i2[i] = T.idx2[i];
  for (int i = t; i < m * m * m; i += kMomThreads) i3[i] = T.idx3[i];
  for (uint32_t b = blockIdx.x; b < (job ? Q.J : Q.G); b += gridDim.x) {
    const uint32_t g = job ? Q.job_group[b] : b;
    const uint32_t lo = job ? Q.job_lo[b] : Q.off[g], hi = job ? Q.job_hi[b] : Q.off[g + 1];
    const bool split = !job && hi - lo > (uint32_t)kMergeChunk;
    const bool alone = !job && hi - lo == 1;  // its only member's sums as they are
    double acc[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) acc[i] = 0.0;
    if (split) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int u = u0 + i * kMomThreads + t;
        if (u >= W) continue;
#pragma unroll 8
        for (uint32_t c = Q.choff[g]; c < Q.choff[g + 1]; ++c) acc[i] += part[(int64_t)c * W + u];
      }
    } else {
      for (uint32_t k = lo; k < hi; ++k) {
        const uint32_t row = in.map ? in.map[k] : k;
        const double n = (double)in.n[row];
        if (n == 0.0) continue;  // uniform
        const double *m2 = in.m2 + (int64_t)row * sh.P2, *m3 = in.m3 + (int64_t)row * sh.P3,
                     *m4 = in.m4 + (int64_t)row * sh.P4;
        if (!alone) {
          __syncthreads();
          if (t < m) d[t] = in.mean[(int64_t)row * m + t] - out.mean[(int64_t)g * m + t];
          for (int i = t; i < sh.P2; i += kMomThreads) s2[i] = m2[i];
          for (int i = t; i < sh.P3; i += kMomThreads) s3[i] = m3[i];
          __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          const int u = u0 + i * kMomThreads + t;
          if (u >= W) continue;
          double v = u < sh.P2 ? m2[u] : u < sh.P2 + sh.P3 ? m3[u - sh.P2] : m4[u - sh.P2 - sh.P3];
          if (!alone) {
            const uint32_t cd = T.code[m + u];
            const int o = (int)(cd & 15u), a = cidx(cd, 0), e = cidx(cd, 1), f = cidx(cd, 2), h = cidx(cd, 3);
            auto v2 = [&](int x, int y) { return s2[p2(i2, m, x, y)]; };
            auto v3 = [&](int x, int y, int z) { return s3[p3(i3, m, x, y, z)]; };
            if (o == 4) {
              v += d[a] * v3(e, f, h) + d[e] * v3(a, f, h) + d[f] * v3(a, e, h) + d[h] * v3(a, e, f);
              v += d[a] * d[e] * v2(f, h) + d[a] * d[f] * v2(e, h) + d[a] * d[h] * v2(e, f) + d[e] * d[f] * v2(a, h) +
                   d[e] * d[h] * v2(a, f) + d[f] * d[h] * v2(a, e);
              v += n * d[a] * d[e] * d[f] * d[h];
            } else if (o == 3) {
              v += d[a] * v2(e, f) + d[e] * v2(a, f) + d[f] * v2(a, e) + n * d[a] * d[e] * d[f];
            } else {
              v += n * d[a] * d[e];
            }
          }
          acc[i] += v;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int u = u0 + i * kMomThreads + t;
      if (u >= W) continue;
      if (job)
        part[(int64_t)b * W + u] = acc[i];
      else
        *mom_row(out, sh, g, m + u) = acc[i];
    }
  }
}

// Chunks of the groups longer than kMergeChunk.
__global__ void k_mom_chunks(const uint32_t *goff, uint32_t G, uint32_t *nchunk) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  const uint32_t n = goff[g + 1] - goff[g];
  nchunk[g] = n > (uint32_t)kMergeChunk ? (n + kMergeChunk - 1) / kMergeChunk : 0u;
}

__global__ void k_mom_jobs(const uint32_t *goff, uint32_t G, const uint32_t *choff, uint32_t *job_lo, uint32_t *job_hi,
                           uint32_t *job_group) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  const uint32_t hi = goff[g + 1], j1 = choff[g + 1];
  uint32_t a = goff[g];
  for (uint32_t j = choff[g]; j < j1; ++j, a += kMergeChunk) {
    job_lo[j] = a;
    job_hi[j] = min(hi, a + kMergeChunk);
    job_group[j] = g;
  }
}

// Band ranges of components: comp_band is nondecreasing.
__global__ void k_mom_band_off(const uint8_t *comp_band, uint32_t C, int32_t nb, uint32_t *boff) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > nb) return;
  uint32_t lo = 0, hi = C;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((int)comp_band[mid] < b)
      lo = mid + 1;
    else
      hi = mid;
  }
  boff[b] = lo;
}

struct MomWork {
  LayoutWork lay;
  uint32_t *perm;
  MomTables tab;
  uint32_t *more, *poff, *item_rank;
  uint32_t *boff, *nchunk, *choff, *job_lo, *job_hi, *job_group;
  double *part;  // rows of the cells' later items, then of the groups' chunks
  double *sum;   // the chunks' counts and first sums
  void *scratch;
  size_t scratch_bytes;
};

// Voxels of an item: at most 2048, and at most 8192 items beyond the cells'
// first, so that a volume of a few cells still fills the card (a row of
// partial sums per item is 58 KB with 18 variables).
uint32_t mom_item(const Geom &g) {
  const int64_t v = (g.n + 8191) / 8192;
  return (uint32_t)(v > 2048 ? (v + 63) / 64 * 64 : 2048);
}

// Chunks of any grouping of `members`: a group of more than kMergeChunk has
// fewer than two chunks per kMergeChunk of its members.
int64_t chunk_cap(int64_t members) { return 2 * (members / kMergeChunk) + 1; }

template <class A>
void mom_layout(A &a, const Geom &g, uint32_t S, uint32_t C, int32_t nb, const MomShape &sh, MomWork *W) {
  const int64_t G = (int64_t)std::max<uint32_t>(C, (uint32_t)nb) + 1;
  const int64_t J = chunk_cap(std::max(S, C));
  const int64_t more = g.n / mom_item(g) + 1;
  layout_take(a, g, S, C, W ? &W->lay : nullptr);
  auto perm = a.template take<uint32_t>(g.n);
  auto code = a.template take<uint32_t>(sh.U);
  auto idx2 = a.template take<uint16_t>((size_t)sh.m * sh.m);
  auto idx3 = a.template take<uint16_t>((size_t)sh.m * sh.m * sh.m);
  auto unit = a.template take<uint16_t>((size_t)kMaxTiles * 256);
  auto mre = a.template take<uint32_t>((size_t)S + 1);
  auto pof = a.template take<uint32_t>((size_t)S + 1);
  auto irk = a.template take<uint32_t>((size_t)S + more);
  auto boff = a.template take<uint32_t>((size_t)nb + 1);
  auto nch = a.template take<uint32_t>(G + 1);
  auto cho = a.template take<uint32_t>(G + 1);
  auto jl = a.template take<uint32_t>(J);
  auto jh = a.template take<uint32_t>(J);
  auto jg = a.template take<uint32_t>(J);
  auto part = a.template take<double>(std::max(J, more) * sh.U);
  auto sum = a.template take<double>(J * (sh.m + 1));
  if (W) {
    W->perm = perm;
    W->tab.code = code;
    W->tab.idx2 = idx2;
    W->tab.idx3 = idx3;
    W->tab.unit = unit;
    W->more = mre;
    W->poff = pof;
    W->item_rank = irk;
    W->boff = boff;
    W->nchunk = nch;
    W->choff = cho;
    W->job_lo = jl;
    W->job_hi = jh;
    W->job_group = jg;
    W->part = part;
    W->sum = sum;
  }
}

size_t mom_scratch(const Geom &g, uint32_t S, uint32_t C, int32_t nb) {
  const int64_t G = (int64_t)std::max<uint32_t>(C, (uint32_t)nb) + 1;
  return std::max(layout_scratch(g, S, C), ScanU32::workspace(std::max<int64_t>(G, S))) + 256;
}

// Groups [goff[g], goff[g + 1]) of members (rows of `in`, through its map) to
// rows 0 .. G - 1 of `out`.
int32_t merge_groups(const uint32_t *goff, uint32_t G, const MergeIn &in, const MomOut &out, const MomShape &sh,
                     MomWork &W, hipStream_t s) {
  if (G == 0) return LSRVT_OK;
  int32_t rc;
  hipLaunchKernelGGL(k_mom_chunks, dim3((G + 255) / 256), dim3(256), 0, s, goff, G, W.nchunk);
  LSRVT_LAUNCHED();
  if ((rc = ScanU32::run(W.nchunk, G, W.choff, W.scratch, W.scratch_bytes, s))) return rc;
  uint32_t J = 0;
  {
    const int32_t rc_ = read_words(W.choff + G, 1, &J, s);
    if (rc_) return rc_;
  }
  const MomGroups Q{G, goff, W.choff, W.job_lo, W.job_hi, W.job_group, J};
  const unsigned slices = (unsigned)((sh.U - sh.m + kShiftUnits - 1) / kShiftUnits);
  const unsigned gj = std::min<uint32_t>(J, 65535), gg = std::min<uint32_t>(G, 65535);
  if (J) {
    hipLaunchKernelGGL(k_mom_jobs, dim3((G + 255) / 256), dim3(256), 0, s, goff, G, W.choff, W.job_lo, W.job_hi,
                       W.job_group);
    hipLaunchKernelGGL(k_mom_mean<true>, dim3(gj), dim3(kWave), 0, s, Q, in, sh, W.sum, out);
  }
  hipLaunchKernelGGL(k_mom_mean<false>, dim3(gg), dim3(kWave), 0, s, Q, in, sh, W.sum, out);
  if (J)
    hipLaunchKernelGGL(k_mom_shift<true>, dim3(gj, slices), dim3(kMomThreads), 0, s, Q, in, sh, W.tab, W.part, out);
  hipLaunchKernelGGL(k_mom_shift<false>, dim3(gg, slices), dim3(kMomThreads), 0, s, Q, in, sh, W.tab, W.part, out);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}

bool out_ok(const lsrvt_moments *o) { return o && o->n && o->mean && o->m2 && o->m3 && o->m4; }

}  // namespace
}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_comoments_workspace(lsrvt_dims dims, uint32_t n_sites, uint32_t n_comp, int32_t n_bands,
                                            int32_t n_vars) {
  Geom g;
  if (make_geom(dims, g) || n_vars < 1 || n_vars > kMomMaxVars || n_bands < 1 || n_bands > 255) return 0;
  const MomShape sh = mom_shape(n_vars);
  Sizer z;
  mom_layout(z, g, n_sites, n_comp, n_bands, sh, nullptr);
  return z.off + mom_scratch(g, n_sites, n_comp, n_bands);
}

extern "C" int32_t lsrvt_comoments(const uint32_t *d_cell, lsrvt_dims dims, const uint32_t *d_sites,
                                   const uint32_t *d_site_comp, uint32_t n_sites, const uint8_t *d_comp_band,
                                   uint32_t n_comp, int32_t n_bands, const float *d_vars, int32_t n_vars,
                                   const lsrvt_moments *cell, const lsrvt_moments *comp, const lsrvt_moments *band,
                                   void *d_work, size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (n_vars < 1 || n_vars > kMomMaxVars || n_bands < 1 || n_bands > 255) return LSRVT_EINVAL;
  if (!d_cell || !d_vars || !out_ok(cell) || !out_ok(comp) || !out_ok(band)) return LSRVT_EINVAL;
  if (n_sites && (!d_sites || !d_site_comp)) return LSRVT_EINVAL;
  if (n_comp && !d_comp_band) return LSRVT_EINVAL;
  const size_t need = lsrvt_comoments_workspace(dims, n_sites, n_comp, n_bands, n_vars);
  if ((rc = check_work(d_work, work_bytes, need))) return rc;
  const MomShape sh = mom_shape(n_vars);
  Carve cv(d_work, work_bytes);
  MomWork W;
  mom_layout(cv, g, n_sites, n_comp, n_bands, sh, &W);
  if (!cv.ok) return LSRVT_EWORKSPACE;
  W.scratch = cv.base + cv.off;
  W.scratch_bytes = cv.size - cv.off;
  W.lay.scratch = W.scratch;
  W.lay.scratch_bytes = W.scratch_bytes;
  hipStream_t s = as_stream(stream);
  const uint32_t S = n_sites, C = n_comp;
  const MomTiles tiles = mom_tiles(n_vars);
  {
    const int M = n_vars + 1;
    const int work = std::max(M * M * M * M, tiles.n * 256);
    hipLaunchKernelGGL(k_mom_tables, dim3((work + 255) / 256), dim3(256), 0, s, sh, W.tab, tiles);
    LSRVT_LAUNCHED();
  }
  // cells: the layout gives every cell one contiguous voxel range
  if ((rc = layout_sites(d_site_comp, S, C, W.lay, s))) return rc;
  if ((rc = layout_voxels(d_cell, g, S, W.lay, W.perm, s))) return rc;
  const MomOut co{cell->n, cell->mean, cell->m2, cell->m3, cell->m4};
  if (S) {
    const unsigned blocks = (S + 255) / 256;
    const uint32_t item = mom_item(g);
    hipLaunchKernelGGL(k_mom_items, dim3(blocks), dim3(256), 0, s, W.lay.cell_off, S, item, W.more);
    LSRVT_LAUNCHED();
    if ((rc = ScanU32::run(W.more, S, W.poff, W.scratch, W.scratch_bytes, s))) return rc;
    uint32_t more = 0;
    {
      const int32_t rc_ = read_words(W.poff + S, 1, &more, s);
      if (rc_) return rc_;
    }
    hipLaunchKernelGGL(k_mom_item_rank, dim3(blocks), dim3(256), 0, s, W.poff, S, W.item_rank);
    LSRVT_LAUNCHED();
    MomCellArgs A;
    A.perm = W.perm;
    A.cell_off = W.lay.cell_off;
    A.order = W.lay.order;
    A.sites = d_sites;
    A.poff = W.poff;
    A.item_rank = W.item_rank;
    A.n_items = S + more;
    A.item = item;
    A.vars = d_vars;
    A.N = g.n;
    A.sh = sh;
    A.tiles = tiles;
    A.unit = W.tab.unit;
    A.out = co;
    A.part = W.part;
    const unsigned grid = std::min<uint32_t>(A.n_items, 1u << 20);
    // tiles over the four waves: all of them in every wave, which then take
    // every fourth step (up to 6 tiles), in two groups (up to 22) or in four;
    // 11 accumulators of 8 registers are the most that leave two waves a SIMD
    auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(kMomThreads), 0, s, A); };
    if (tiles.n <= 1)
      launch(k_mom_cells<1, 1>);
    else if (tiles.n <= 6)
      launch(k_mom_cells<6, 1>);
    else if (tiles.n <= 12)
      launch(k_mom_cells<6, 2>);
    else if (tiles.n <= 22)
      launch(k_mom_cells<11, 2>);
    else
      launch(k_mom_cells<11, 4>);
    LSRVT_LAUNCHED();
    if (more) {
      hipLaunchKernelGGL(k_mom_combine, dim3(std::min<uint32_t>(S, 65535), (sh.U + kMomThreads - 1) / kMomThreads),
                         dim3(kMomThreads), 0, s, W.poff, W.lay.order, S, W.part, sh, co);
      LSRVT_LAUNCHED();
    }
    hipLaunchKernelGGL(k_mom_center, dim3((unsigned)std::min<uint32_t>(S, 65535)), dim3(kMomThreads), 0, s,
                       W.lay.cell_off, W.lay.order, d_sites, S, d_vars, g.n, sh, W.tab, co);
    LSRVT_LAUNCHED();
  }
  // components: their cells by site id (ranks coff[c] .. coff[c + 1])
  MergeIn cin{cell->n, cell->mean, cell->m2, cell->m3, cell->m4, W.lay.order};
  const MomOut go{comp->n, comp->mean, comp->m2, comp->m3, comp->m4};
  if ((rc = merge_groups(W.lay.coff, C, cin, go, sh, W, s))) return rc;
  // bands: their components by id
  hipLaunchKernelGGL(k_mom_band_off, dim3((n_bands + 1 + 255) / 256), dim3(256), 0, s, d_comp_band, C, n_bands,
                     W.boff);
  LSRVT_LAUNCHED();
  MergeIn bin{comp->n, comp->mean, comp->m2, comp->m3, comp->m4, nullptr};
  const MomOut bo{band->n, band->mean, band->m2, band->m3, band->m4};
  if ((rc = merge_groups(W.boff, (uint32_t)n_bands, bin, bo, sh, W, s))) return rc;
  return LSRVT_OK;
}
