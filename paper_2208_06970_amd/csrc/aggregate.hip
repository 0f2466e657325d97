// Statistics of every cell, merged cell -> component -> band (Sec. 3.3,
// "Aggregation"; the hierarchy of Sec. 3.2.4 / Fig. 5).
//
// Pipeline:
//  1. the structured layout (layout.hip) lists the voxels of every cell as
//     one contiguous range, cells in (component, site id) order and voxels
//     in index order;
//  2. every cell's range is cut into work items of at most kItemVoxels;
//  3. one workgroup per item (one wave for a small cell) gathers the item's
//     values and sums, per "unit", d_j and d_j d_k in float64, d being the
//     float32 difference from the value at the cell's site: exact products,
//     so the only rounding besides is that of the sums (2^-53 of their size).  With the
//     covariance the sums are a matrix product of the staged values with
//     themselves on the matrix cores; without, lanes own voxels.  The order
//     of every sum is fixed.  Histograms and extrema are integer / compare
//     operations and go through LDS and registers;
//  4. per cell, the item partials are combined in item order and the cell's
//     mean, M2 and co-moments formed in float64; the float32 cell outputs are
//     those values rounded once;
//  5. Chan et al.'s pairwise merge in float64: cells of a component in site
//     id order, then components of a band in component id order.  Counts,
//     extrema and histograms merge exactly with atomics.
#include <algorithm>

#include "layout.h"

namespace lsrvt {

namespace {

constexpr int kAggThreads = 256;
constexpr int kAggWaves = kAggThreads / kWave;
constexpr int kFold = 32;  // item partials of a large cell added together before the finalize
constexpr int kMaxVars = 32;
constexpr int kMaxPairs = kMaxVars * (kMaxVars + 1) / 2;
constexpr int64_t kItemVoxels = 4096;
constexpr int kSmallCell = 256;  // cells up to this size are summed by a single wave
constexpr int kMaxHist = 8192;  // n_vars * n_bins

struct Pairs {
  uint8_t j[kMaxPairs];
  uint8_t k[kMaxPairs];
};

struct BBox {
  uint32_t *x0, *x1, *y0, *y1, *z0, *z1;
};

typedef double d4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// 1-2. the voxels of every cell are a contiguous range of the structured
// layout (layout.hip); each cell's range is cut into items of at most
// kItemVoxels voxels, numbered in cell rank order.
__global__ void k_agg_items(const uint32_t *__restrict__ cnt_rank, uint32_t S, uint32_t *items) {
  uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < S) items[r] = (uint32_t)((cnt_rank[r] + kItemVoxels - 1) / kItemVoxels);
}

// item -> cell rank, and the split into cells small enough for one wave
// (their single item) and the items of larger cells
__global__ void k_item_cells(const uint32_t *__restrict__ item_off, const uint32_t *__restrict__ cnt_rank, uint32_t S,
                             int small_ok, uint32_t *item_rank, uint32_t *small_list, uint32_t *big_list,
                             uint32_t *counts) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = r < S;
  const uint32_t i0 = in ? item_off[r] : 0u, i1 = in ? item_off[r + 1] : 0u;
  const bool small = in && small_ok && cnt_rank[r] <= (uint32_t)kSmallCell;
  const uint32_t n = i1 - i0;
  // one counter atomic per wave and list: wave prefix sums of the item counts
  const int lane = lane_id();
  uint32_t ns = small ? n : 0u, nb = small ? 0u : n;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t a = __shfl_up(ns, o, kWave), b = __shfl_up(nb, o, kWave);
    if (lane >= o) {
      ns += a;
      nb += b;
    }
  }
  const uint32_t ts = __shfl(ns, kWave - 1, kWave), tb = __shfl(nb, kWave - 1, kWave);
  uint32_t bs = 0, bb = 0;
  if (lane == 0) {
    if (ts) bs = atomicAdd(&counts[0], ts);
    if (tb) bb = atomicAdd(&counts[1], tb);
  }
  bs = __shfl(bs, 0, kWave);
  bb = __shfl(bb, 0, kWave);
  const uint32_t p = small ? bs + ns - n : bb + nb - n;
  for (uint32_t i = i0; i < i1; ++i) {
    item_rank[i] = r;
    (small ? small_list : big_list)[p + (i - i0)] = i;
  }
}

// 3. per-item sums
struct CellArgs {
  const uint32_t *perm;       // layout order of the voxels
  const uint32_t *cell_off;   // [S + 1] by rank
  const uint32_t *order;      // rank -> site
  const uint32_t *sites;
  const float *vars;  // [m][N]
  const float *edges; // [m][B+1] or null
  int64_t n;
  int m, B, U, tile;          // tile: voxels staged in LDS per round, a multiple of 256
  uint32_t stage;             // bytes of the stage
  Pairs pairs;
  const uint32_t *item_off;   // [S + 1] by rank
  const uint32_t *item_rank;  // [n_items]
  const uint32_t *list;       // items of this launch
  const uint32_t *list_cnt;   // their number (device)
  double *part;               // [n_items][U]
  uint32_t *hist;            // cell histograms [S][m][B] (zeroed) or null
  uint32_t *kmin, *kmax;     // ordered keys [S][m]
};

// Wave-wide min / max by DPP lane moves (quad permutes, row mirrors, row
// broadcasts; every lane of the wave active): the result is read from the
// last lane and returned to all lanes.
#define LSRVT_DPP_STEP(OP, ID, CTRL, RMASK) \
  v = OP(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(ID), (int)v, CTRL, RMASK, 0xF, false))
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0xB1, 0xF);   // quad_perm [1,0,3,2]
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0x4E, 0xF);   // quad_perm [2,3,0,1]
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0x141, 0xF);  // row_half_mirror
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0x140, 0xF);  // row_mirror
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0x142, 0xA);  // row_bcast:15 into rows 1 and 3
  LSRVT_DPP_STEP(min, 0xFFFFFFFFu, 0x143, 0xC);  // row_bcast:31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  LSRVT_DPP_STEP(max, 0u, 0xB1, 0xF);
  LSRVT_DPP_STEP(max, 0u, 0x4E, 0xF);
  LSRVT_DPP_STEP(max, 0u, 0x141, 0xF);
  LSRVT_DPP_STEP(max, 0u, 0x140, 0xF);
  LSRVT_DPP_STEP(max, 0u, 0x142, 0xA);
  LSRVT_DPP_STEP(max, 0u, 0x143, 0xC);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}
#undef LSRVT_DPP_STEP
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Histogram bin of x: #{interior edges e_1..e_{B-1} <= x} for ascending
// edges e_0..e_B (sc = B / (e_B - e_0)).  A guess from the mean edge spacing
// is kept when the two edges around it confirm it (always, for evenly spaced
// edges); otherwise bisection.  NaN lands in bin 0, as every comparison with
// it is false.
__device__ __forceinline__ int hist_bin(float x, const float *e, int B, float e0, float sc) {
  const int g = (int)fminf(fmaxf((x - e0) * sc, 0.0f), (float)(B - 1));
  if ((g == 0 || e[g] <= x) && (g == B - 1 || x < e[g + 1])) return g;
  int a = 1, b = B;
  while (a < b) {
    const int mid = (a + b) >> 1;
    if (e[mid] <= x)
      a = mid + 1;
    else
      b = mid;
  }
  return a - 1;
}

// Count x of variable j in the histogram h (LDS) for the active lanes.  The
// values of a cell lie close together, so most lanes of a wave often meet in
// one bin, which the LDS would take one after another: the first lane's bin
// gets one addition for all of its lanes (2.97 ms for the statistics of
// 512 x 256 x 256 voxels with 18 variables; 3.11 ms without, 3.01 and 3.34 ms
// with two and four such bins).
__device__ __forceinline__ void hist_count(uint32_t *h, int bin, int lane) {
  const int lead = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t same = __ballot(bin == lead);
  if (bin != lead)
    atomicAdd(&h[bin], 1u);
  else if (lane == __ffsll((unsigned long long)same) - 1)
    atomicAdd(&h[bin], (uint32_t)__popcll(same));
}

// How the products are taken.  kDiag: squares only, lanes own voxels.  Else on
// the matrix cores, whose 16 x 16 x 4 instruction multiplies 16 values of four
// voxels with each other: k16 for up to 16 variables (with up to 8, or 4, the
// 16 rows hold the variables of two, or four, groups of voxels, and the
// diagonal blocks are added); k20 for 17 to 20, the last of them as the
// columns of 4 x 4 x 4 instructions; k32 for 21 to 32, three 16 x 16 tiles.
enum { kDiag = 0, k16 = 1, k20 = 2, k32 = 3 };

// Rows held by the variables of one voxel group (a power of two), and their groups.
__host__ __device__ inline int group_rows(int mode, int m) { return mode != k16 || m > 8 ? 16 : m > 4 ? 8 : 4; }

// The accumulators of one wave.  A lane's operand is variable `row` of voxel
// group g (k16) at one of four voxels; `extra` is its variable among the ones
// after the first 16.
template <int MODE>
struct CellSums {
  d4 t00, t01, t11;      // 16 x 16 tiles
  double e0, ee;         // 4 x 4 x 4 blocks: tile 0 with the extras, the extras with themselves
  double s0, s1;         // sums of the lane's operands
  __device__ __forceinline__ void zero() {
    t00 = t01 = t11 = d4{0.0, 0.0, 0.0, 0.0};
    e0 = ee = s0 = s1 = 0.0;
  }
  __device__ __forceinline__ void add(double x, double y) {
    t00 = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, t00, 0, 0, 0);
    s0 += x;
    if constexpr (MODE == k20) {
      e0 = __builtin_amdgcn_mfma_f64_4x4x4f64(x, y, e0, 0, 0, 0);
      ee = __builtin_amdgcn_mfma_f64_4x4x4f64(y, y, ee, 0, 0, 0);
      s1 += y;
    }
    if constexpr (MODE == k32) {
      t01 = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, t01, 0, 0, 0);
      t11 = __builtin_amdgcn_mfma_f64_16x16x4f64(y, y, t11, 0, 0, 0);
      s1 += y;
    }
  }
};

// The sums of `nw` waves to a row of unit sums: each accumulator in turn goes
// through `red` (256 doubles), wave by wave, and the units it holds are picked
// from there.  An accumulator register i of lane l is entry (4 i + l / 16,
// l % 16) of its 16 x 16 tile, or entry (l / 16, l % 4) of the 4 x 4 block of
// rows l / 4 % 4.  `sync` orders the LDS accesses of the cooperating threads.
template <int MODE, class Sync>
__device__ __forceinline__ void put_sums(const CellSums<MODE> &C, const CellArgs &A, double *red, int t, int nt, int w,
                                         int nw, double *row, Sync sync) {
  const int lane = lane_id(), m = A.m, P = A.U - m;
  const int gr = group_rows(MODE, m), G = 16 / gr;
  auto tile = [&](const d4 &v, int bj, int bk) {  // products of variables bj .. bj + 15 with bk .. bk + 15
    for (int i = 0; i < nw; ++i) {
      if (w == i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int at = (4 * q + lane / 16) * 16 + lane % 16;
          red[at] = i ? red[at] + v[q] : v[q];
        }
      sync();
    }
    for (int p = t; p < P; p += nt) {
      const int j = A.pairs.j[p] - bj, k = A.pairs.k[p] - bk;
      if (j < 0 || k < 0 || j > 15 || k > 15) continue;
      double x = red[j * 16 + k];
      for (int g = 1; g < G; ++g) x += red[(g * gr + j) * 16 + g * gr + k];
      row[m + p] = x;
    }
    sync();
  };
  // sums of the lanes' own operands: lane l holds variable b + l % gr
  auto lanes = [&](double v, int b, int gr, int G) {
    for (int i = 0; i < nw; ++i) {
      if (w == i) red[lane] = i ? red[lane] + v : v;
      sync();
    }
    for (int u = b + t; u < min(m, b + gr); u += nt) {
      double x = 0.0;
      for (int k = 0; k < 4; ++k)
        for (int g = 0; g < G; ++g) x += red[k * 16 + g * gr + u - b];
      row[u] = x;
    }
    sync();
  };
  tile(C.t00, 0, 0);
  lanes(C.s0, 0, gr, G);
  if constexpr (MODE == k32) {
    tile(C.t01, 0, 16);
    tile(C.t11, 16, 16);
    lanes(C.s1, 16, 16, 1);
  }
  if constexpr (MODE == k20) {
    auto block = [&](double v, bool first) {
      for (int i = 0; i < nw; ++i) {
        if (w == i) red[lane] = i ? red[lane] + v : v;
        sync();
      }
      for (int p = t; p < P; p += nt) {
        const int j = A.pairs.j[p], k = A.pairs.k[p] - 16;
        if (k < 0 || (j < 16) != first) continue;
        row[m + p] = first ? red[(j & 3) * 16 + (j >> 2) * 4 + k] : red[(j - 16) * 16 + k];
      }
      sync();
    };
    block(C.e0, true);
    block(C.ee, false);
    lanes(C.s1, 16, 4, 1);  // every block of four lanes holds the same extras: the first is taken
  }
}

// Items of large cells, one workgroup each.  A round's voxels are staged in
// LDS as [variable][voxel]: wave w gathers variables w, w + 4, ... (64 voxels
// of one variable per load, NS variables a wave), keeping their extrema in
// registers and counting their histograms on the way.  Each wave then takes
// every fourth chunk of 16 voxels (per voxel group): one 16-byte LDS read per
// lane feeds four matrix steps, and only the conversion to float64 and the
// subtraction of the site's value are left to the vector units.  Rows are
// tile + 4 floats apart, so the lanes' reads fall on all banks.
//
// Bound by the gathers and the histograms' LDS atomics, not by the products:
// 512 x 256 x 256 voxels, 18 variables, 32 bins and the covariance take 1.8 ms
// (1.0 TB/s of values), 0.8 ms of it the histograms and 0.15 ms the products
// (matrix cores 20 % busy, 69 % of the LDS cycles bank conflicts);
// float32 sums with error terms on the vector units, 11 operations per voxel
// and unit, took 4.1 ms.
template <int MODE, int NS>
__global__ __launch_bounds__(kAggThreads) void k_agg_cell(CellArgs A) {
  extern __shared__ uint8_t smem[];
  const int m = A.m, B = A.B, TL = A.tile, ld = A.tile + 4;
  double *red = reinterpret_cast<double *>(smem);                     // [256], after the rounds
  float *dv = reinterpret_cast<float *>(smem);                        // [m][tile + 4]
  uint32_t *hist_l = reinterpret_cast<uint32_t *>(smem + A.stage);    // [m*B]
  float *edg = reinterpret_cast<float *>(hist_l + m * B);             // [m][B+1]
  float *scl = edg + m * (B + 1);                                     // [m] B / (e_B - e_0)
  float *K = scl + m;                                                 // [m]
  const int t = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int gr = group_rows(MODE, m), G = 16 / gr;
  const int row0 = min(lane % gr, m - 1);
  const int row1 = min(16 + (MODE == k20 ? lane % 4 : lane % 16), m - 1);
  if (B > 0) {
    for (int i = t; i < m * (B + 1); i += kAggThreads) edg[i] = A.edges[i];
    for (int j = t; j < m; j += kAggThreads) scl[j] = (float)B / (A.edges[j * (B + 1) + B] - A.edges[j * (B + 1)]);
  }

  const uint32_t n_list = *A.list_cnt;
  for (uint32_t k = blockIdx.x; k < n_list; k += gridDim.x) {
    const uint32_t item = A.list[k];
    const uint32_t r = A.item_rank[item];
    const uint32_t s = A.order[r];
    const uint32_t part = item - A.item_off[r];
    const uint32_t start = A.cell_off[r] + part * (uint32_t)kItemVoxels;
    const uint32_t stop = min(A.cell_off[r + 1], start + (uint32_t)kItemVoxels);
    for (int i = t; i < m * B; i += kAggThreads) hist_l[i] = 0;
    if (t < m) K[t] = A.vars[(int64_t)t * A.n + A.sites[s]];
    uint32_t kmn[NS], kmx[NS];
    double d1[MODE == kDiag ? NS : 1], d2[MODE == kDiag ? NS : 1];
    CellSums<MODE> C;
    C.zero();
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      kmn[q] = 0xFFFFFFFFu;
      kmx[q] = 0u;
      if constexpr (MODE == kDiag) d1[q] = d2[q] = 0.0;
    }
    __syncthreads();
    const float K0 = K[row0], K1 = K[row1];

    for (uint32_t base = start; base < stop; base += (uint32_t)TL) {
      const int nt = (int)min((uint32_t)TL, stop - base);
      for (int sub = 0; sub < nt; sub += 4 * kWave) {
        uint32_t vv[4];
        bool ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ok[i] = sub + i * kWave + lane < nt;
          vv[i] = ok[i] ? A.perm[base + sub + i * kWave + lane] : 0u;
        }
        float xs[NS][4];  // all of the wave's gathers in flight at once
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          const int j = min(w + q * kAggWaves, m - 1);
          const float *col = A.vars + (int64_t)j * A.n;
#pragma unroll
          for (int i = 0; i < 4; ++i) xs[q][i] = col[vv[i]];
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          const int j = w + q * kAggWaves;
          if (j >= m) continue;  // uniform over the wave
          const float kj = K[j];
          float x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = ok[i] ? xs[q][i] : kj;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (MODE != kDiag) dv[j * ld + sub + i * kWave + lane] = x[i];
            if constexpr (MODE == kDiag) {  // a lane without a voxel adds zeros
              const double d = (double)(x[i] - kj);
              d1[q] += d;
              d2[q] = __builtin_fma(d, d, d2[q]);
            }
            if (ok[i]) {
              const uint32_t kk = f2key(x[i]);
              kmn[q] = min(kmn[q], kk);
              kmx[q] = max(kmx[q], kk);
            }
          }
          if (B > 0) {
            const float *e = edg + j * (B + 1);
            const float e0 = e[0], sc = scl[j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (ok[i]) hist_count(hist_l + j * B, hist_bin(x[i], e, B, e0, sc), lane);
          }
        }
      }
      if constexpr (MODE != kDiag) {
        __syncthreads();
        // the stage holds whole multiples of 256 voxels, the site's value past nt
        for (int c = w * 16 * G; c < nt; c += kAggWaves * 16 * G) {
          const int at = c + (lane % 16) / gr * 16 + lane / 16 * 4;
          const float4 a = *reinterpret_cast<const float4 *>(dv + row0 * ld + at);
          float4 b = a;
          if constexpr (MODE != k16) b = *reinterpret_cast<const float4 *>(dv + row1 * ld + at);
          C.add((double)(a.x - K0), (double)(b.x - K1));
          C.add((double)(a.y - K0), (double)(b.y - K1));
          C.add((double)(a.z - K0), (double)(b.z - K1));
          C.add((double)(a.w - K0), (double)(b.w - K1));
        }
        __syncthreads();
      }
    }
    double *out = A.part + (int64_t)item * A.U;
    if constexpr (MODE != kDiag)
      put_sums<MODE>(C, A, red, t, kAggThreads, w, kAggWaves, out, [] { __syncthreads(); });
    __syncthreads();
    // flush exact integer/compare statistics
    if (A.hist) {
      uint32_t *dst = A.hist + (int64_t)s * m * B;
      for (int i = t; i < m * B; i += kAggThreads)
        if (hist_l[i]) atomicAdd(&dst[i], hist_l[i]);
    }
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int j = w + q * kAggWaves;
      if (j >= m) continue;
      const uint32_t mn = wave_min_u32(kmn[q]), mx = wave_max_u32(kmx[q]);
      if constexpr (MODE == kDiag) {
        d1[q] = wave_sum(d1[q]);
        d2[q] = wave_sum(d2[q]);
      }
      if (lane == 0) {
        atomicMin(&A.kmin[(int64_t)s * m + j], mn);
        atomicMax(&A.kmax[(int64_t)s * m + j], mx);
        if constexpr (MODE == kDiag) {
          out[j] = d1[q];
          out[m + j] = d2[q];
        }
      }
    }
    __syncthreads();
  }
}

// The same sums for cells of at most kSmallCell voxels, one wave per cell:
// each wave has its own LDS region and synchronises only with itself.  A cell
// of at most 16 (32) voxels takes four (two) variables at a time, its voxels
// over 16 (32) lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

constexpr int kWaveLd = kWave + 4;  // floats between the rows of a wave's stage

// Bytes of a wave's stage ([m][kWaveLd] floats, then 256 doubles of put_sums; none for squares alone) and of its region.
__host__ __device__ inline size_t wave_stage_bytes(int mode, int m) {
  const size_t v = sizeof(float) * (size_t)m * kWaveLd;
  return mode == kDiag ? 0 : v > 2048 ? v : 2048;
}
__host__ __device__ inline size_t wave_region_bytes(int mode, int m, int B) {
  // stage, m sums and squares, histogram, extrema, site values
  return (wave_stage_bytes(mode, m) + sizeof(double) * 2 * m + sizeof(uint32_t) * ((size_t)m * B + 3 * (size_t)m) + 15) & ~size_t(15);
}

template <int MODE>
__global__ __launch_bounds__(kAggThreads) void k_agg_cell_wave(CellArgs A) {
  extern __shared__ uint8_t smem[];
  const int m = A.m, B = A.B;
  const int lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  float *edg = reinterpret_cast<float *>(smem);  // [m][B+1], shared by the waves
  const size_t head = (sizeof(float) * m * (B + 1) + 15) & ~size_t(15);
  uint8_t *own = smem + head + w * wave_region_bytes(MODE, m, B);
  float *dv = reinterpret_cast<float *>(own);
  double *red = reinterpret_cast<double *>(own);
  double *sum = reinterpret_cast<double *>(own + wave_stage_bytes(MODE, m));  // [2m] (kDiag)
  uint32_t *hist_l = reinterpret_cast<uint32_t *>(sum + 2 * m);               // [m*B]
  uint32_t *kmin_l = hist_l + m * B;
  uint32_t *kmax_l = kmin_l + m;
  float *K = reinterpret_cast<float *>(kmax_l + m);
  const int gr = group_rows(MODE, m), G = 16 / gr;
  const int row0 = min(lane % gr, m - 1);
  const int row1 = min(16 + (MODE == k20 ? lane % 4 : lane % 16), m - 1);
  if (B > 0)
    for (int i = threadIdx.x; i < m * (B + 1); i += kAggThreads) edg[i] = A.edges[i];
  __syncthreads();
  const uint32_t n_list = *A.list_cnt;
  for (uint32_t k = blockIdx.x * kAggWaves + w; k < n_list; k += gridDim.x * kAggWaves) {
    const uint32_t item = A.list[k];
    const uint32_t r = A.item_rank[item];
    const uint32_t s = A.order[r];
    const uint32_t start = A.cell_off[r];
    const int nt = (int)(A.cell_off[r + 1] - start);
    const int L = nt <= 16 ? 16 : nt <= 32 ? 32 : kWave;  // lanes of a variable
    for (int i = lane; i < m * B; i += kWave) hist_l[i] = 0;
    for (int j = lane; j < m; j += kWave) {
      K[j] = A.vars[(int64_t)j * A.n + A.sites[s]];
      kmin_l[j] = 0xFFFFFFFFu;
      kmax_l[j] = 0u;
      if constexpr (MODE == kDiag) sum[j] = sum[m + j] = 0.0;
    }
    wave_sync();
    const float K0 = K[row0], K1 = K[row1];
    CellSums<MODE> C;
    C.zero();
    for (int base = 0; base < nt; base += L) {
      const int v = lane & (L - 1);
      const bool in = base + v < nt;
      const uint32_t vv = in ? A.perm[start + base + v] : 0u;
      for (int j0 = 0; j0 < m; j0 += kWave / L) {
        const int j = j0 + lane / L;
        const bool ok = in && j < m;
        const float kj = K[min(j, m - 1)];
        const float x = ok ? A.vars[(int64_t)j * A.n + vv] : kj;
        const uint32_t kk = f2key(x);
        uint32_t mn = ok ? kk : 0xFFFFFFFFu, mx = ok ? kk : 0u;
        double a = 0.0, b = 0.0;
        if constexpr (MODE == kDiag) {
          a = (double)(x - kj);
          b = a * a;
        }
        for (int o = 1; o < L; o <<= 1) {
          mn = min(mn, (uint32_t)__shfl_xor(mn, o, kWave));
          mx = max(mx, (uint32_t)__shfl_xor(mx, o, kWave));
          if constexpr (MODE == kDiag) {
            a += __shfl_xor(a, o, kWave);
            b += __shfl_xor(b, o, kWave);
          }
        }
        if (v == 0 && j < m) {
          kmin_l[j] = min(kmin_l[j], mn);
          kmax_l[j] = max(kmax_l[j], mx);
          if constexpr (MODE == kDiag) {
            sum[j] += a;
            sum[m + j] += b;
          }
        }
        if constexpr (MODE != kDiag)
          if (j < m) dv[j * kWaveLd + v] = x;
        if (B > 0 && ok) {
          const float *e = edg + j * (B + 1);
          atomicAdd(&hist_l[j * B + hist_bin(x, e, B, e[0], (float)B / (e[B] - e[0]))], 1u);
        }
      }
      wave_sync();
      if constexpr (MODE != kDiag) {
        const int left = min(L, nt - base);
        for (int c = 0; c < left; c += 4 * G) {
          const int at = c + (lane % 16) / gr * 4 + lane / 16;
          const float a = dv[row0 * kWaveLd + at];
          float b = a;
          if constexpr (MODE != k16) b = dv[row1 * kWaveLd + at];
          C.add((double)(a - K0), (double)(b - K1));
        }
        wave_sync();
      }
    }
    double *out = A.part + (int64_t)item * A.U;
    if constexpr (MODE != kDiag)
      put_sums<MODE>(C, A, red, lane, kWave, 0, 1, out, [] { wave_sync(); });
    else
      for (int u = lane; u < 2 * m; u += kWave) out[u] = sum[u];
    // the cell's only item: plain stores
    if (A.hist) {
      uint32_t *dst = A.hist + (int64_t)s * m * B;
      for (int i = lane; i < m * B; i += kWave)
        if (hist_l[i]) dst[i] = hist_l[i];
    }
    for (int j = lane; j < m; j += kWave) {
      A.kmin[(int64_t)s * m + j] = kmin_l[j];
      A.kmax[(int64_t)s * m + j] = kmax_l[j];
    }
    wave_sync();
  }
}

// Runs of kFold item partials of a cell with more than kFold items, added into
// the run's first row: a cell of most of the volume has thousands.
__global__ __launch_bounds__(kAggThreads) void k_agg_fold(CellArgs A) {
  const uint32_t n_list = *A.list_cnt;
  for (uint32_t k = blockIdx.x; k < n_list; k += gridDim.x) {
    const uint32_t item = A.list[k];
    const uint32_t r = A.item_rank[item];
    const uint32_t i0 = A.item_off[r], i1 = A.item_off[r + 1];
    if (i1 - i0 <= (uint32_t)kFold || (item - i0) % kFold) continue;
    const uint32_t hi = min(i1, item + kFold);
    for (int u = threadIdx.x; u < A.U; u += kAggThreads) {
      double v = A.part[(int64_t)item * A.U + u];
#pragma unroll 8
      for (uint32_t i = item + 1; i < hi; ++i) v += A.part[(int64_t)i * A.U + u];
      A.part[(int64_t)item * A.U + u] = v;
    }
  }
}

// 4. per-cell finalize, one wave per cell: combine the item partials in item
// order, form the float32 statistics and the float64 merge inputs, and add
// the exact ones to the cell's component.
struct FinArgs {
  uint32_t S;
  int m, U, P;  // P = number of pair units (all pairs, or the diagonal only)
  Pairs pairs;
  const uint32_t *sites;
  const float *vars;
  int64_t n;
  const unsigned long long *cnt;
  const uint32_t *rank;      // site -> cell rank
  const uint32_t *item_off;  // by rank
  const double *part;
  const uint32_t *kmin, *kmax;
  // outputs
  uint64_t *out_n;
  float *mean32, *m2_32, *vmin, *vmax, *cov32;  // cov32 [S][m(m+1)/2] (only with cov)
  int with_cov;
  double *mean64;  // [S][m]
  double *c64;     // [S][P]
  // exact merges into the components
  int B;
  const uint32_t *hist;           // cell histograms [S][m][B] or null
  const uint32_t *site_comp;
  uint32_t n_comp;
  unsigned long long *cnt_c;
  uint32_t *kmin_c, *kmax_c, *hist_c;
};

constexpr int kHistAhead = 4;
__global__ __launch_bounds__(kAggThreads) void k_agg_finalize(FinArgs A) {
  extern __shared__ uint8_t smem[];
  const int m = A.m, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  double *th = reinterpret_cast<double *>(smem) + (size_t)w * A.U;  // [U] of this wave's cell
  for (uint32_t s = blockIdx.x * kAggWaves + w; s < A.S; s += gridDim.x * kAggWaves) {
    const uint64_t n = A.cnt[s];
    const uint32_t i0 = A.item_off[A.rank[s]], i1 = A.item_off[A.rank[s] + 1];
    const uint32_t c = A.site_comp[s];
    const uint32_t site = A.sites[s];
    // what does not hang on the items is loaded beside them: the first
    // variable and kHistAhead bins of every lane (123000 cells of 4 variables
    // with 32 bins: 100 us, 124 with one load after the other; several cells a
    // wave, their first loads a lane each, 155)
    const bool has = lane < m;
    const uint32_t lo0 = has ? A.kmin[(int64_t)s * m + lane] : 0u, hi0 = has ? A.kmax[(int64_t)s * m + lane] : 0u;
    const float at0 = has && n ? A.vars[(int64_t)lane * A.n + site] : 0.0f;
    uint32_t h0[kHistAhead];
#pragma unroll
    for (int k = 0; k < kHistAhead; ++k)
      h0[k] = A.hist && lane + kWave * k < m * A.B ? A.hist[(int64_t)s * m * A.B + lane + kWave * k] : 0u;
    const uint32_t step = i1 - i0 > (uint32_t)kFold ? kFold : 1;
    for (int u = lane; u < A.U; u += kWave) {
      double v = 0.0;
#pragma unroll 8
      for (uint32_t it = i0; it < i1; it += step) v += A.part[(int64_t)it * A.U + u];
      // an infinite value among the cell's leaves no mean
      th[u] = v + (v - v);
    }
    wave_sync();
    if (lane == 0) A.out_n[s] = n;
    if (n && c < A.n_comp) {
      if (lane == 0) atomicAdd(&A.cnt_c[c], (unsigned long long)n);
      for (int j = lane; j < m; j += kWave) {
        atomicMin(&A.kmin_c[(int64_t)c * m + j], j < kWave ? lo0 : A.kmin[(int64_t)s * m + j]);
        atomicMax(&A.kmax_c[(int64_t)c * m + j], j < kWave ? hi0 : A.kmax[(int64_t)s * m + j]);
      }
#pragma unroll
      for (int k = 0; k < kHistAhead; ++k)
        if (h0[k]) atomicAdd(&A.hist_c[(int64_t)c * m * A.B + lane + kWave * k], h0[k]);
      if (A.hist)
        for (int i = lane + kWave * kHistAhead; i < m * A.B; i += kWave) {
          uint32_t h = A.hist[(int64_t)s * m * A.B + i];
          if (h) atomicAdd(&A.hist_c[(int64_t)c * m * A.B + i], h);
        }
    }
    const double dn = (double)n;
    for (int j = lane; j < m; j += kWave) {
      float mean = 0.0f;
      double mean64 = 0.0;
      if (n) {
        mean64 = (double)(j < kWave ? at0 : A.vars[(int64_t)j * A.n + site]) + th[j] / dn;
        mean = (float)mean64;
      }
      A.mean32[(int64_t)s * m + j] = mean;
      A.mean64[(int64_t)s * m + j] = mean64;
      A.vmin[(int64_t)s * m + j] = n ? key2f(j < kWave ? lo0 : A.kmin[(int64_t)s * m + j]) : __builtin_inff();
      A.vmax[(int64_t)s * m + j] = n ? key2f(j < kWave ? hi0 : A.kmax[(int64_t)s * m + j]) : -__builtin_inff();
    }
    for (int p = lane; p < A.P; p += kWave) {
      const int j = A.pairs.j[p], k = A.pairs.k[p];
      float c32 = 0.0f;
      double c64 = 0.0;
      if (n) {
        // C = S_jk - S_j S_k / n cancels when the site's value is far from the
        // cell mean, so it is formed in float64 and rounded once
        c64 = th[m + p] - th[j] * th[k] / dn;
        if (j == k && c64 < 0.0) c64 = 0.0;
        c32 = (float)c64;
      }
      A.c64[(int64_t)s * A.P + p] = c64;
      if (j == k) A.m2_32[(int64_t)s * m + j] = c32;
      if (A.with_cov) A.cov32[(int64_t)s * A.P + p] = c32;
    }
    wave_sync();
  }
}

// 5a. exact band statistics from the components: one workgroup per run of at
// most kBandRun components in band order; each lane owns columns (count, minima,
// maxima, histogram bins) and flushes one atomic per column whenever the band
// changes.  What the time goes to is a lane's walk along its run, kAhead loads
// at a time, and the workgroups' atomics on one band's columns, 27 ns each, so
// there are about 1024 workgroups (123000 components, 4 variables of 32 bins:
// 41 us; 94 with 2048 workgroups whose loads waited for each other).
constexpr int kBandRun = 1024;
struct BandIntArgs {
  uint32_t n_comp, run;
  int m, B;
  const uint32_t *order;  // components sorted by band
  const uint8_t *comp_band;
  const unsigned long long *cnt_c;
  const uint32_t *kmin_c, *kmax_c, *hist_c;
  unsigned long long *cnt_b;
  uint32_t *kmin_b, *kmax_b, *hist_b;
};

__global__ __launch_bounds__(256) void k_band_int(BandIntArgs A) {
  const int m = A.m, B = A.B;
  const int64_t cols = 1 + 2 * (int64_t)m + (int64_t)m * B;
  const uint32_t q0 = blockIdx.x * A.run;
  const uint32_t q1 = q0 + A.run < A.n_comp ? q0 + A.run : A.n_comp;
  const int nq = (int)(q1 - q0);
  // the run's components and their bands, staged once (the order -> band
  // chain of loads would otherwise repeat for every column)
  __shared__ uint32_t cs[kBandRun];
  __shared__ uint8_t bs[kBandRun];
  for (int i = threadIdx.x; i < nq; i += 256) {
    const uint32_t c = A.order[q0 + i];
    cs[i] = c;
    bs[i] = A.comp_band[c];
  }
  __syncthreads();
  constexpr int kAhead = 16;  // loads issued together per column
  for (int64_t col = threadIdx.x; col < cols; col += 256) {
    const int kind = col == 0 ? 0 : col <= m ? 1 : col <= 2 * m ? 2 : 3;
    const int64_t sub = kind == 1 ? col - 1 : kind == 2 ? col - 1 - m : col - 1 - 2 * m;
    uint64_t acc = kind == 1 ? 0xFFFFFFFFull : 0ull;
    int band = -1;
    auto flush = [&]() {
      if (band < 0) return;
      if (kind == 0) {
        if (acc) atomicAdd(&A.cnt_b[band], (unsigned long long)acc);
      } else if (kind == 1) {
        if (acc != 0xFFFFFFFFull) atomicMin(&A.kmin_b[(int64_t)band * m + sub], (uint32_t)acc);
      } else if (kind == 2) {
        if (acc) atomicMax(&A.kmax_b[(int64_t)band * m + sub], (uint32_t)acc);
      } else {
        if (acc) atomicAdd(&A.hist_b[(int64_t)band * m * B + sub], (uint32_t)acc);
      }
    };
    // one address for all kinds: with a branch for each the loads of a step wait
    // for each other (a component has fewer than 2^31 voxels: the low word)
    const uint32_t *src = kind == 0   ? reinterpret_cast<const uint32_t *>(A.cnt_c)
                          : kind == 1 ? A.kmin_c + sub
                          : kind == 2 ? A.kmax_c + sub
                                      : A.hist_c + sub;
    const int64_t stride = kind == 0 ? 2 : kind < 3 ? m : (int64_t)m * B;
    for (int q = 0; q < nq; q += kAhead) {
      uint32_t v[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) v[k] = src[stride * cs[q + k < nq ? q + k : q]];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        if (q + k >= nq) break;
        const int bc = bs[q + k];
        if (bc != band) {
          flush();
          band = bc;
          acc = kind == 1 ? 0xFFFFFFFFull : 0ull;
        }
        if (kind == 0 || kind == 3)
          acc += v[k];
        else if (kind == 1)
          acc = v[k] < acc ? v[k] : acc;
        else
          acc = v[k] > acc ? v[k] : acc;
      }
    }
    flush();
  }
}

__global__ void k_decode_minmax(const uint32_t *kmin, const uint32_t *kmax, const unsigned long long *cnt, int64_t units,
                                int m, float *vmin, float *vmax, uint64_t *out_n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= units * m) return;
  int64_t u = i / m;
  bool any = cnt[u] != 0;
  vmin[i] = any ? key2f(kmin[i]) : __builtin_inff();
  vmax[i] = any ? key2f(kmax[i]) : -__builtin_inff();
  if (i % m == 0) out_n[u] = cnt[u];
}

// 5b. Chan pairwise merge in float64.  Members of group g are
// order[off[g] .. off[g+1]) in that order.  Groups of at most kSmallGroup
// members: one thread per (group, pair unit) merges them one after another.
// Larger groups: one workgroup per (group, pair unit); lane t merges members t,
// t + 256, ... in order, then the 256 lane states merge pairwise in a fixed tree
// (t with t + 128, ..., t with t + 1).  Neighbouring lanes take neighbouring
// members, because the members' values are a few doubles each and what bounds
// the merge is the lines they lie in: with a contiguous share for each lane the
// bands of 123000 components and 4 variables take 125 us, now 71.
constexpr uint32_t kSmallGroup = 32;
constexpr int kChanAhead = 8;  // members of a lane whose values are loaded together

struct MergeArgs {
  uint32_t n_groups;
  int m, P;
  Pairs pairs;
  const uint32_t *order;
  const uint32_t *off;
  const unsigned long long *in_cnt;
  const double *in_mean;           // [members][m]
  const double *in_c;              // [members][P]
  double *out_mean;                // [groups][m]
  double *out_m2;                  // [groups][m]
  double *out_c;                   // [groups][P] (internal, always)
  double *out_cov;                 // [groups][P] user output, or null
  int with_cov;
  const uint32_t *big;             // groups larger than kSmallGroup
  const uint32_t *big_cnt;
};

struct ChanState {
  double n, mj, mk, c;
};

__device__ __forceinline__ void chan_add(ChanState &a, double ni, double aj, double ak, double ci) {
  if (ni == 0.0) return;
  if (a.n == 0.0) {
    a = ChanState{ni, aj, ak, ci};
    return;
  }
  const double nn = a.n + ni;
  const double dj = aj - a.mj, dk = ak - a.mk;
  a.c = a.c + ci + dj * dk * (a.n * ni / nn);
  a.mj = a.mj + dj * (ni / nn);
  a.mk = a.mk + dk * (ni / nn);
  a.n = nn;
}

__device__ __forceinline__ void chan_write(const MergeArgs &A, uint32_t gidx, int p, const ChanState &st) {
  const int j = A.pairs.j[p], k = A.pairs.k[p];
  A.out_c[(int64_t)gidx * A.P + p] = st.c;
  if (j == k) {
    A.out_mean[(int64_t)gidx * A.m + j] = st.mj;
    A.out_m2[(int64_t)gidx * A.m + j] = st.c;
  }
  if (A.with_cov) A.out_cov[(int64_t)gidx * A.P + p] = st.c;
}

__global__ void k_chan_small(MergeArgs A) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)A.n_groups * A.P) return;
  const uint32_t gidx = (uint32_t)(i / A.P);
  const int p = (int)(i % A.P);
  const uint32_t q0 = A.off[gidx], q1 = A.off[gidx + 1];
  if (q1 - q0 > kSmallGroup) return;
  const int j = A.pairs.j[p], k = A.pairs.k[p];
  ChanState st{0.0, 0.0, 0.0, 0.0};
  for (uint32_t q = q0; q < q1; ++q) {
    const uint32_t mem = A.order[q];
    chan_add(st, (double)A.in_cnt[mem], A.in_mean[(int64_t)mem * A.m + j], A.in_mean[(int64_t)mem * A.m + k],
             A.in_c[(int64_t)mem * A.P + p]);
  }
  chan_write(A, gidx, p, st);
}

__global__ void k_chan_list_big(const uint32_t *off, uint32_t n_groups, uint32_t *big, uint32_t *big_cnt) {
  uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n_groups && off[g + 1] - off[g] > kSmallGroup) big[atomicAdd(big_cnt, 1u)] = g;
}

__global__ __launch_bounds__(256) void k_chan_big(MergeArgs A) {
  __shared__ double sn[256], sj[256], sk[256], sc[256];
  const int t = threadIdx.x;
  const int64_t work = (int64_t)(*A.big_cnt) * A.P;
  for (int64_t w = blockIdx.x; w < work; w += gridDim.x) {
    const uint32_t gidx = A.big[w / A.P];
    const int p = (int)(w % A.P);
    const int j = A.pairs.j[p], k = A.pairs.k[p];
    const uint32_t q0 = A.off[gidx], q1 = A.off[gidx + 1];
    ChanState st{0.0, 0.0, 0.0, 0.0};
    for (uint32_t q = q0 + t; q < q1; q += 256 * kChanAhead) {
      double n[kChanAhead], vj[kChanAhead], vk[kChanAhead], vc[kChanAhead];
      uint32_t mem[kChanAhead];
#pragma unroll
      for (int i = 0; i < kChanAhead; ++i) mem[i] = A.order[q + 256 * i < q1 ? q + 256 * i : q];
#pragma unroll
      for (int i = 0; i < kChanAhead; ++i) {
        n[i] = q + 256 * i < q1 ? (double)A.in_cnt[mem[i]] : 0.0;  // (an empty member adds nothing)
        vj[i] = A.in_mean[(int64_t)mem[i] * A.m + j];
        vk[i] = A.in_mean[(int64_t)mem[i] * A.m + k];
        vc[i] = A.in_c[(int64_t)mem[i] * A.P + p];
      }
#pragma unroll
      for (int i = 0; i < kChanAhead; ++i) chan_add(st, n[i], vj[i], vk[i], vc[i]);
    }
    sn[t] = st.n;
    sj[t] = st.mj;
    sk[t] = st.mk;
    sc[t] = st.c;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (t < o) {
        ChanState a{sn[t], sj[t], sk[t], sc[t]};
        chan_add(a, sn[t + o], sj[t + o], sk[t + o], sc[t + o]);
        sn[t] = a.n;
        sj[t] = a.mj;
        sk[t] = a.mk;
        sc[t] = a.c;
      }
      __syncthreads();
    }
    if (t == 0) chan_write(A, gidx, p, ChanState{sn[0], sj[0], sk[0], sc[0]});
    __syncthreads();
  }
}

// helpers for ordering components by band
__global__ void k_permute(const uint32_t *key, const uint32_t *val, const uint32_t *pos, uint32_t n, uint32_t *key_out,
                          uint32_t *val_out) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    key_out[pos[i]] = key[i];
    val_out[pos[i]] = val[i];
  }
}
__global__ void k_iota(uint32_t *p, uint32_t n) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i;
}

struct AggWork {
  LayoutWork lay;
  uint32_t *perm;  // [N]
  unsigned long long *cnt_c, *cnt_b;
  uint32_t *items, *item_off;
  double *part;
  uint32_t *kmin, *kmax, *kmin_c, *kmax_c, *kmin_b, *kmax_b;
  double *mean64, *c64, *mean64_c, *c64_c, *m2tmp_c, *mean64_b, *c64_b, *m2tmp_b;
  uint32_t *key_b, *val_b, *pos, *corder, *bucket;
  uint32_t *item_rank, *small_list, *big_list, *big, *big_cnt;
  void *scratch;
  size_t scratch_bytes;
  int64_t item_cap;
};

// Items: one per started kItemVoxels of every cell.
int64_t item_capacity(const Geom &g, uint32_t S) { return (int64_t)S + g.n / kItemVoxels + 1; }

template <class A>
void agg_layout(A &a, const Geom &g, uint32_t S, uint32_t n_comp, int32_t n_bands, int m, int U, int P, AggWork *W) {
  size_t s1 = S ? S : 1, c1 = n_comp + 2, b1 = (size_t)n_bands + 1;
  int64_t ic = item_capacity(g, S);
  layout_take(a, g, S, n_comp, W ? &W->lay : nullptr);
  auto perm = a.template take<uint32_t>(g.n);
  auto cnt_c = a.template take<unsigned long long>(c1);
  auto cnt_b = a.template take<unsigned long long>(b1);
  auto items = a.template take<uint32_t>(s1);
  auto ioff = a.template take<uint32_t>(s1 + 1);
  auto part = a.template take<double>(ic * U);
  auto kmin = a.template take<uint32_t>(s1 * m);
  auto kmax = a.template take<uint32_t>(s1 * m);
  auto kminc = a.template take<uint32_t>(c1 * m);
  auto kmaxc = a.template take<uint32_t>(c1 * m);
  auto kminb = a.template take<uint32_t>(b1 * m);
  auto kmaxb = a.template take<uint32_t>(b1 * m);
  auto mean64 = a.template take<double>(s1 * m);
  auto c64 = a.template take<double>(s1 * P);
  auto mean64c = a.template take<double>(c1 * m);
  auto c64c = a.template take<double>(c1 * P);
  auto m2c = a.template take<double>(c1 * m);
  auto mean64b = a.template take<double>(b1 * m);
  auto c64b = a.template take<double>(b1 * P);
  auto m2b = a.template take<double>(b1 * m);
  auto kb = a.template take<uint32_t>(c1);
  auto vb = a.template take<uint32_t>(c1);
  auto pos = a.template take<uint32_t>(c1);
  auto corder = a.template take<uint32_t>(c1);
  auto bucket = a.template take<uint32_t>(257);
  auto irank = a.template take<uint32_t>(ic);
  auto slist = a.template take<uint32_t>(ic);
  auto blist = a.template take<uint32_t>(ic);
  auto big = a.template take<uint32_t>(c1 > b1 ? c1 : b1);
  auto bigc = a.template take<uint32_t>(4);
  if (W) {
    W->perm = perm;
    W->cnt_c = cnt_c;
    W->cnt_b = cnt_b;
    W->items = items;
    W->item_off = ioff;
    W->part = part;
    W->kmin = kmin;
    W->kmax = kmax;
    W->kmin_c = kminc;
    W->kmax_c = kmaxc;
    W->kmin_b = kminb;
    W->kmax_b = kmaxb;
    W->mean64 = mean64;
    W->c64 = c64;
    W->mean64_c = mean64c;
    W->c64_c = c64c;
    W->m2tmp_c = m2c;
    W->mean64_b = mean64b;
    W->c64_b = c64b;
    W->m2tmp_b = m2b;
    W->key_b = kb;
    W->val_b = vb;
    W->pos = pos;
    W->corder = corder;
    W->bucket = bucket;
    W->item_rank = irank;
    W->small_list = slist;
    W->big_list = blist;
    W->big = big;
    W->big_cnt = bigc;
    W->item_cap = ic;
  }
}

struct SizerT : Sizer {
  template <class T>
  T *take(size_t c) {
    Sizer::take<T>(c);
    return nullptr;
  }
};

// Variables and bins that the call takes.  The limit is the one that an earlier
// form of the cell kernel set (histograms, edges and a stage of one value per
// group of units in 64 KiB); the present kernels need less LDS for whatever it
// lets through, and what the call refuses has stayed the same.
bool hist_fits(int m, int B, int U) {
  int G = 1, NT = kAggThreads;
  if (U <= kAggThreads) {
    G = 2 * U <= kAggThreads ? kAggThreads / U : 2;
    NT = std::max(kAggThreads, (G * U + kWave - 1) / kWave * kWave);
  }
  return sizeof(float) * (2 * (size_t)m * B + 5 * (size_t)m + 2 * (size_t)G * U + (size_t)(m + 1) * (NT + 4)) <= 65536;
}

void units_for(int m, bool cov, int &P, int &U, Pairs &pairs) {
  P = 0;
  for (int j = 0; j < m; ++j)
    for (int k = j; k < m; ++k)
      if (cov || j == k) {
        pairs.j[P] = (uint8_t)j;
        pairs.k[P] = (uint8_t)k;
        ++P;
      }
  U = m + P;
}

size_t scratch_need(const Geom &g, uint32_t S, uint32_t n_comp) {
  size_t a = ScanU32::workspace((int64_t)S + 1);
  size_t b = StableSort8::workspace((int64_t)n_comp + 2);
  size_t c = ScanU32::workspace((int64_t)n_comp + 2);
  size_t d = layout_scratch(g, S, n_comp);
  size_t r = a > b ? a : b;
  r = r > c ? r : c;
  return (r > d ? r : d) + 256;
}

}  // namespace

}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_aggregate_workspace(lsrvt_dims dims, uint32_t n_sites, uint32_t n_comp, int32_t n_bands,
                                            int32_t n_vars, int32_t n_bins, uint32_t flags) {
  (void)n_bins;
  Geom g;
  if (make_geom(dims, g)) return 0;
  if (n_vars < 1 || n_vars > kMaxVars || n_bands < 1 || n_bands > 255) return 0;
  int P, U;
  Pairs pairs;
  units_for(n_vars, (flags & LSRVT_STATS_COV) != 0, P, U, pairs);
  SizerT z;
  agg_layout(z, g, n_sites, n_comp, n_bands, n_vars, U, P, nullptr);
  return z.off + scratch_need(g, n_sites, n_comp);
}

extern "C" int32_t lsrvt_aggregate(const uint32_t *d_cell, lsrvt_dims dims, const uint32_t *d_sites,
                                   const uint32_t *d_site_comp, uint32_t n_sites, const uint8_t *d_comp_band,
                                   uint32_t n_comp, int32_t n_bands, const float *d_vars, int32_t n_vars,
                                   const float *d_edges, int32_t n_bins, uint32_t flags, const lsrvt_cell_stats *cell,
                                   const lsrvt_group_stats *comp, const lsrvt_group_stats *band, void *d_work,
                                   size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (n_vars < 1 || n_vars > kMaxVars || n_bands < 1 || n_bands > 255) return LSRVT_EINVAL;
  if (!d_cell || !d_vars || !cell || !comp || !band) return LSRVT_EINVAL;
  if (n_sites && (!d_sites || !d_site_comp)) return LSRVT_EINVAL;
  if (n_comp && !d_comp_band) return LSRVT_EINVAL;
  const bool want_hist = (flags & LSRVT_STATS_HIST) != 0;
  const bool want_cov = (flags & LSRVT_STATS_COV) != 0;
  const int B = want_hist ? n_bins : 0;
  if (want_hist && (n_bins < 1 || !d_edges || (int64_t)n_vars * n_bins > kMaxHist)) return LSRVT_EINVAL;
  const lsrvt_cell_stats &cs = *cell;
  const lsrvt_group_stats *lv[2] = {comp, band};
  if (!cs.n || !cs.mean || !cs.m2 || !cs.vmin || !cs.vmax || (want_hist && !cs.hist) || (want_cov && !cs.cov))
    return LSRVT_EINVAL;
  for (const lsrvt_group_stats *q : lv)
    if (!q->n || !q->mean || !q->m2 || !q->vmin || !q->vmax || (want_hist && !q->hist) || (want_cov && !q->cov))
      return LSRVT_EINVAL;
  const size_t need = lsrvt_aggregate_workspace(dims, n_sites, n_comp, n_bands, n_vars, n_bins, flags);
  if ((rc = check_work(d_work, work_bytes, need))) return rc;
  int P, U;
  Pairs pairs;
  units_for(n_vars, want_cov, P, U, pairs);
  const int m = n_vars;
  Carve cv(d_work, work_bytes);
  AggWork W;
  agg_layout(cv, g, n_sites, n_comp, n_bands, m, U, P, &W);
  if (!cv.ok) return LSRVT_EWORKSPACE;
  W.scratch = cv.base + cv.off;
  W.scratch_bytes = cv.size - cv.off;
  hipStream_t s = as_stream(stream);
  const uint32_t S = n_sites;
  const uint32_t C = n_comp;
  const int64_t Pfull = (int64_t)m * (m + 1) / 2;

  // zero / identity initialisation
  if ((rc = fill<unsigned long long>(W.cnt_c, C + 2, 0ull, s))) return rc;
  if ((rc = fill<unsigned long long>(W.cnt_b, n_bands + 1, 0ull, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmin, (int64_t)(S ? S : 1) * m, 0xFFFFFFFFu, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmax, (int64_t)(S ? S : 1) * m, 0u, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmin_c, (int64_t)(C + 2) * m, 0xFFFFFFFFu, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmax_c, (int64_t)(C + 2) * m, 0u, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmin_b, (int64_t)(n_bands + 1) * m, 0xFFFFFFFFu, s))) return rc;
  if ((rc = fill<uint32_t>(W.kmax_b, (int64_t)(n_bands + 1) * m, 0u, s))) return rc;
  if (want_hist) {
    if ((rc = fill<uint32_t>(cs.hist, (int64_t)S * m * B, 0u, s))) return rc;
    if ((rc = fill<uint32_t>(comp->hist, (int64_t)C * m * B, 0u, s))) return rc;
    if ((rc = fill<uint32_t>(band->hist, (int64_t)n_bands * m * B, 0u, s))) return rc;
  }

  // 1. sites in (component, id) order and the voxels of every cell as one range
  W.lay.scratch = W.scratch;
  W.lay.scratch_bytes = W.scratch_bytes;
  if ((rc = layout_sites(d_site_comp, S, C, W.lay, s))) return rc;
  if ((rc = layout_voxels(d_cell, g, S, W.lay, W.perm, s))) return rc;

  // 2. items
  uint32_t n_items = 0;
  if (S) {
    hipLaunchKernelGGL(k_agg_items, dim3((S + 255) / 256), dim3(256), 0, s, W.lay.cnt_rank, S, W.items);
    LSRVT_LAUNCHED();
    if ((rc = ScanU32::run(W.items, S, W.item_off, W.scratch, W.scratch_bytes, s))) return rc;
    {
      const int32_t rc_ = read_words(W.item_off + S, 1, &n_items, s);
      if (rc_) return rc_;
    }
    if ((int64_t)n_items > W.item_cap) return LSRVT_EDEVICE;  // cannot happen: the capacity is an upper bound
  }

  // 3. per-item sums: cells of at most kSmallCell voxels one wave each, larger cells one workgroup per item
  if (n_items) {
    if (!hist_fits(m, B, U)) return LSRVT_EINVAL;
    CellArgs A;
    A.perm = W.perm;
    A.cell_off = W.lay.cell_off;
    A.order = W.lay.order;
    A.sites = d_sites;
    A.vars = d_vars;
    A.edges = d_edges;
    A.n = g.n;
    A.m = m;
    A.B = B;
    A.U = U;
    A.pairs = pairs;
    A.item_off = W.item_off;
    A.item_rank = W.item_rank;
    A.part = W.part;
    A.hist = want_hist ? cs.hist : nullptr;
    A.kmin = W.kmin;
    A.kmax = W.kmax;
    A.stage = 0;
    A.tile = 0;
    const int mode = !want_cov ? kDiag : m <= 16 ? k16 : m <= 20 ? k20 : k32;
    // wave path, while four waves' regions fit in LDS
    const size_t lds_w = ((sizeof(float) * m * (B + 1) + 15) & ~size_t(15)) + kAggWaves * wave_region_bytes(mode, m, B);
    const bool small_ok = lds_w <= 65536;
    if ((rc = fill<uint32_t>(W.big_cnt + 1, 2, 0u, s))) return rc;
    uint32_t *counts = W.big_cnt + 1;
    hipLaunchKernelGGL(k_item_cells, dim3((S + 255) / 256), dim3(256), 0, s, W.item_off, W.lay.cnt_rank, S,
                       small_ok ? 1 : 0, W.item_rank, W.small_list, W.big_list, counts);
    LSRVT_LAUNCHED();
    if (small_ok) {
      A.list = W.small_list;
      A.list_cnt = counts;
      const unsigned grid = (unsigned)std::min<uint64_t>(65535, (n_items + 3) / 4);
      auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(kAggThreads), lds_w, s, A); };
      mode == kDiag ? launch(k_agg_cell_wave<kDiag>)
      : mode == k16 ? launch(k_agg_cell_wave<k16>)
      : mode == k20 ? launch(k_agg_cell_wave<k20>)
                    : launch(k_agg_cell_wave<k32>);
      LSRVT_LAUNCHED();
    }
    A.list = W.big_list;
    A.list_cnt = counts + 1;
    // a staging round of 256 voxels, or the asked multiple of it if that fits in 64 KiB (not the next
    // smaller one that does: larger rounds leave fewer workgroups a CU, 18 variables with 32 bins and the
    // covariance of 1024 x 512 x 512 voxels take 18.3 ms with 256 voxels and 21.8 with 512)
    const size_t fixed = sizeof(float) * ((size_t)m * B + (size_t)m * (B + 1) + 2 * m);
    auto stage = [&](int tile) {
      return mode == kDiag ? (size_t)0 : std::max<size_t>(2048, sizeof(float) * (size_t)m * (tile + 4));
    };
    A.tile = kAggThreads;
    const int32_t tv = tuning(LSRVT_TUNE_STATS_TILE);
    if (tv && fixed + stage(tv * kAggThreads) <= 65536) A.tile = tv * kAggThreads;
    A.stage = (uint32_t)stage(A.tile);
    const size_t lds = fixed + A.stage;  // within 64 KiB: less than hist_fits asks for
    const unsigned grid = n_items < 16384 ? n_items : 16384;
    auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(kAggThreads), lds, s, A); };
    const int ns = (m + kAggWaves - 1) / kAggWaves;  // variables of a wave
    if (mode == kDiag)
      ns == 1 ? launch(k_agg_cell<kDiag, 1>) : ns == 2 ? launch(k_agg_cell<kDiag, 2>)
      : ns <= 5 ? launch(k_agg_cell<kDiag, 5>) : launch(k_agg_cell<kDiag, 8>);
    else if (mode == k16)
      ns == 1 ? launch(k_agg_cell<k16, 1>) : ns == 2 ? launch(k_agg_cell<k16, 2>) : launch(k_agg_cell<k16, 4>);
    else if (mode == k20)
      launch(k_agg_cell<k20, 5>);
    else
      launch(k_agg_cell<k32, 8>);
    LSRVT_LAUNCHED();
    if (n_items > (uint32_t)kFold) {
      hipLaunchKernelGGL(k_agg_fold, dim3(std::min<uint32_t>(grid, 4096)), dim3(kAggThreads), 0, s, A);
      LSRVT_LAUNCHED();
    }
  }

  // 4. per-cell finalize, plus exact merges of counts, extrema and histograms into components
  if (S) {
    FinArgs F;
    F.S = S;
    F.m = m;
    F.U = U;
    F.P = P;
    F.pairs = pairs;
    F.sites = d_sites;
    F.vars = d_vars;
    F.n = g.n;
    F.cnt = W.lay.cnt;
    F.rank = W.lay.rank;
    F.item_off = W.item_off;
    F.part = W.part;
    F.kmin = W.kmin;
    F.kmax = W.kmax;
    F.out_n = cs.n;
    F.mean32 = cs.mean;
    F.m2_32 = cs.m2;
    F.vmin = cs.vmin;
    F.vmax = cs.vmax;
    F.cov32 = cs.cov;
    F.with_cov = want_cov;
    F.mean64 = W.mean64;
    F.c64 = W.c64;
    F.B = B;
    F.hist = want_hist ? cs.hist : nullptr;
    F.site_comp = d_site_comp;
    F.n_comp = C;
    F.cnt_c = W.cnt_c;
    F.kmin_c = W.kmin_c;
    F.kmax_c = W.kmax_c;
    F.hist_c = want_hist ? comp->hist : nullptr;
    const size_t lds = sizeof(double) * (size_t)U * kAggWaves;
    const unsigned grid = std::min<uint32_t>((S + kAggWaves - 1) / kAggWaves, 16384);
    hipLaunchKernelGGL(k_agg_finalize, dim3(grid), dim3(kAggThreads), lds, s, F);
    LSRVT_LAUNCHED();
  }

  // 5a. components sorted by band (stable in id); exact band statistics
  if (C) {
    hipLaunchKernelGGL(k_iota, dim3((C + 255) / 256), dim3(256), 0, s, W.corder, C);
    LSRVT_LAUNCHED();
    if ((rc = StableSort8::run(d_comp_band, C, W.pos, W.bucket, W.scratch, W.scratch_bytes, s))) return rc;
    hipLaunchKernelGGL(k_permute, dim3((C + 255) / 256), dim3(256), 0, s, W.corder, W.corder, W.pos, C, W.key_b,
                       W.val_b);
    LSRVT_LAUNCHED();
    BandIntArgs BI;
    BI.n_comp = C;
    BI.run = std::min<uint32_t>(kBandRun, std::max<uint32_t>(8, C / 1024));
    BI.m = m;
    BI.B = B;
    BI.order = W.val_b;
    BI.comp_band = d_comp_band;
    BI.cnt_c = W.cnt_c;
    BI.kmin_c = W.kmin_c;
    BI.kmax_c = W.kmax_c;
    BI.hist_c = want_hist ? comp->hist : nullptr;
    BI.cnt_b = W.cnt_b;
    BI.kmin_b = W.kmin_b;
    BI.kmax_b = W.kmax_b;
    BI.hist_b = want_hist ? band->hist : nullptr;
    hipLaunchKernelGGL(k_band_int, dim3((C + BI.run - 1) / BI.run), dim3(256), 0, s, BI);
    LSRVT_LAUNCHED();
    hipLaunchKernelGGL(k_decode_minmax, dim3(grid_for((int64_t)C * m, 256, 1 << 30)), dim3(256), 0, s, W.kmin_c,
                       W.kmax_c, W.cnt_c, (int64_t)C, m, comp->vmin, comp->vmax, comp->n);
    LSRVT_LAUNCHED();
  } else {
    if ((rc = fill<uint32_t>(W.bucket, 257, 0u, s))) return rc;
  }
  hipLaunchKernelGGL(k_decode_minmax, dim3(grid_for((int64_t)n_bands * m, 256, 1 << 30)), dim3(256), 0, s, W.kmin_b,
                     W.kmax_b, W.cnt_b, (int64_t)n_bands, m, band->vmin, band->vmax, band->n);
  LSRVT_LAUNCHED();

  auto run_merge = [&](MergeArgs &M) -> int32_t {
    int32_t r;
    if ((r = fill<uint32_t>(W.big_cnt, 1, 0u, s))) return r;
    M.big = W.big;
    M.big_cnt = W.big_cnt;
    hipLaunchKernelGGL(k_chan_small, dim3(grid_for((int64_t)M.n_groups * M.P, 256, 1 << 30)), dim3(256), 0, s, M);
    hipLaunchKernelGGL(k_chan_list_big, dim3((M.n_groups + 255) / 256), dim3(256), 0, s, M.off, M.n_groups, W.big,
                       W.big_cnt);
    hipLaunchKernelGGL(k_chan_big, dim3(1024), dim3(256), 0, s, M);
    LSRVT_LAUNCHED();
    return LSRVT_OK;
  };

  // 5b. the cell -> component merge, cells of a component in site id order
  if (C) {
    if (S) {
      MergeArgs M;
      M.n_groups = C;
      M.m = m;
      M.P = P;
      M.pairs = pairs;
      M.order = W.lay.order;
      M.off = W.lay.coff;
      M.in_cnt = W.lay.cnt;
      M.in_mean = W.mean64;
      M.in_c = W.c64;
      M.out_mean = comp->mean;
      M.out_m2 = comp->m2;
      M.out_c = W.c64_c;
      M.out_cov = comp->cov;
      M.with_cov = want_cov;
      if ((rc = run_merge(M))) return rc;
      // keep float64 component means for the band merge
      LSRVT_HIP(hipMemcpyAsync(W.mean64_c, comp->mean, sizeof(double) * (size_t)C * m, hipMemcpyDeviceToDevice, s));
    } else {
      if ((rc = fill<double>(comp->mean, (int64_t)C * m, 0.0, s))) return rc;
      if ((rc = fill<double>(comp->m2, (int64_t)C * m, 0.0, s))) return rc;
      if (want_cov && (rc = fill<double>(comp->cov, (int64_t)C * Pfull, 0.0, s))) return rc;
      if ((rc = fill<double>(W.mean64_c, (int64_t)C * m, 0.0, s))) return rc;
      if ((rc = fill<double>(W.c64_c, (int64_t)C * P, 0.0, s))) return rc;
    }
  }

  // 5c. component -> band merge, components of a band in id order
  {
    MergeArgs M;
    M.n_groups = (uint32_t)n_bands;
    M.m = m;
    M.P = P;
    M.pairs = pairs;
    M.order = W.val_b;
    M.off = W.bucket;
    M.in_cnt = W.cnt_c;
    M.in_mean = W.mean64_c;
    M.in_c = W.c64_c;
    M.out_mean = band->mean;
    M.out_m2 = band->m2;
    M.out_c = W.c64_b;
    M.out_cov = band->cov;
    M.with_cov = want_cov;
    if ((rc = run_merge(M))) return rc;
  }
  return LSRVT_OK;
}
