// Structured hierarchical layout (Sec. 3.2.4 "Data Reduction and Structured
// Data Layout", Fig. 5): the voxels that lie in a cell, ordered by band, then
// component, then cell, then linear index, with offsets per cell, component
// and band, so that every feature of the hierarchy is one contiguous range.
//
// Cells are ordered by (component, site id): the sites are sorted stably by
// component with an LSD radix sort, and rank[s] is the position of site s.
// Components are numbered band-major, so this order is also band-major.
//
// Voxels are placed by a deterministic counting sort.  The volume is cut
// into tiles of 4096 consecutive linear indices.  One workgroup per tile sorts
// its voxels stably by cell in LDS (k_lay_sort) and keeps the order as one
// 16-bit word per voxel.  Every (tile, cell) pair becomes one segment of the
// output.  The pairs are sorted stably by cell rank, so the segments of a cell
// follow each other in tile order, and an exclusive scan of their sizes gives
// every segment's start.  A last pass over the tiles' orders writes each voxel
// to its segment (k_lay_runs).
#include "layout.h"

namespace lsrvt {

namespace {

constexpr int kLayThreads = 256;
constexpr int kLayWaves = kLayThreads / kWave;
constexpr int kLayGroups = kLayTile / kLayThreads;  // 64-voxel groups of a wave, consecutive
// Hash tables of a tile's distinct cells: a small one for almost all tiles, so
// that eight workgroups fit a CU, and one that holds a whole tile (a tile
// that overflows the small table is listed for it).  A thread adds one cell
// between two looks at the count, so at most kLayThreads more than MaxD are
// added and the tables keep free slots.
constexpr int kSmallCap = 1024, kSmallMax = 640;
constexpr int kBigCap = 2 * kLayTile, kBigMax = kLayTile;
static_assert(kSmallMax + kLayThreads < kSmallCap, "free slots in the small table");
constexpr uint32_t kLayHead = 0x8000u;  // first voxel of its cell in the tile's order

struct LayArgs {
  const uint32_t *cell;
  int64_t n;
  uint32_t S;
  int64_t n_tiles;
  unsigned long long *cnt;
  uint32_t *tile_nd;    // distinct cells of every tile
  uint32_t *tile_nv;    // placed voxels of every tile
  uint16_t *order;      // [tiles][4096] the placed voxels' places in the tile, by cell, kLayHead at each cell's first
  uint32_t *big_list;   // tiles deferred by the small table
  uint32_t *big_cnt;    // their number
  const uint32_t *pair_off;
  uint32_t *pair_cell, *pair_cnt;
  const uint32_t *seg_off;
  uint32_t *perm;
};

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v) {
  const int lane = lane_id();
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// A tile's voxels sorted stably by cell.  Wave w holds the tile's groups
// [16 w, 16 w + 16) of 64 voxels, one voxel a lane.  The first voxel of every
// run of equal cells in a group looks its cell up in a hash table of the tile
// (LDS, atomicCAS), the occupied slots are numbered in slot order (the order
// of the cells inside a tile is of no consequence, as the pairs are sorted by
// cell rank), and the voxels are sorted by that number, six bits a pass and
// so one pass for up to 63 cells: ballots rank a lane among the equal digits
// of its group, counters in LDS carry the ranks over a wave's groups, and one
// scan of the counters gives the places.  Unplaced voxels (no cell) take the
// last number and are left out.
//
// Bound by the ballots and the LDS round trips of a pass; four waves a tile
// and no serial walk over runs of equal cells, so the time depends little on
// how fragmented the cells are.  The three walks of a wave per tile that this
// and k_lay_runs replace took 1.8 ms on 512 x 256 x 256 voxels in 9155 cells
// (now 0.35 + 0.08 + 0.05 ms), 2.5 ms on 333 x 255 x 201 in 322209 (now 0.37)
// and 5.0 ms on 131 x 121 x 77 in 123464 (now 0.1): there a tile's ~1000 runs
// were taken one after another.  Four waves a SIMD: five and six spill more
// and are 3 % and 5 % slower on the whole call.
template <int Cap, int MaxD, bool small>
__global__ __launch_bounds__(kLayThreads, small ? 4 : 3) void k_lay_sort(LayArgs A) {
  __shared__ uint32_t key[Cap];         // cell id (kNone: free), then its number
  __shared__ uint32_t item[kLayTile];   // number << 12 | place in the tile
  __shared__ uint32_t cnt[kLayWaves][kWave];
  __shared__ uint32_t part[kLayWaves];
  __shared__ uint32_t found, placed;
  const int t = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const uint32_t n_list = small ? (uint32_t)A.n_tiles : *A.big_cnt;
  for (uint32_t b = blockIdx.x; b < n_list; b += gridDim.x) {
    const uint32_t tile = small ? b : A.big_list[b];
    const int64_t v0 = (int64_t)tile * kLayTile;
    uint32_t c[kLayGroups];
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      const int64_t v = v0 + (w * kLayGroups + g) * kWave + lane;
      c[g] = v < A.n ? A.cell[v] : kNone;
      if (c[g] >= A.S) c[g] = kNone;
    }
    for (int i = t; i < Cap; i += kLayThreads) key[i] = kNone;
    if (t == 0) found = placed = 0u;
    __syncthreads();
    // slots of the table
    bool over = false;
    uint32_t n_placed = 0;
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      const uint32_t cl = c[g], left = __shfl_up(cl, 1, kWave);
      const bool first = lane == 0 || cl != left;
      const uint64_t firsts = __ballot(first);
      n_placed += (uint32_t)__popcll(__ballot(cl != kNone));
      uint32_t h = 0;
      if (first && cl != kNone && !over) {
        h = (cl * 2654435761u) & (Cap - 1);
        for (int probe = 0; probe < Cap; ++probe) {
          const uint32_t k = __hip_atomic_load(&key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (k == cl) break;
          if (k == kNone) {
            const uint32_t old = atomicCAS(&key[h], kNone, cl);
            if (old == kNone) {
              over = atomicAdd(&found, 1u) >= (uint32_t)MaxD;
              break;
            }
            if (old == cl) break;
          }
          h = (h + 1) & (Cap - 1);
        }
        if (small)
          over = over || __hip_atomic_load(&found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > (uint32_t)MaxD;
      }
      // the run's slot from its first voxel
      const int leader = kWave - 1 - __clzll((long long)(firsts & (lanemask_lt() | (1ull << lane))));
      h = __shfl(h, leader, kWave);
      c[g] = cl == kNone ? kNone : h;
    }
    if (lane == 0) atomicAdd(&placed, n_placed);
    __syncthreads();
    const uint32_t nd = found;
    if (small && nd > (uint32_t)MaxD) {
      if (t == 0) A.big_list[atomicAdd(A.big_cnt, 1u)] = tile;
      __syncthreads();
      continue;
    }
    if (nd == 1 && placed == (uint32_t)kLayTile) {  // a tile inside one cell is in order
#pragma unroll
      for (int g = 0; g < kLayGroups; ++g) {
        const uint32_t q = (uint32_t)((w * kLayGroups + g) * kWave + lane);
        A.order[v0 + q] = (uint16_t)(q | (q == 0 ? kLayHead : 0u));
      }
      if (t == 0) {
        A.tile_nd[tile] = 1;
        A.tile_nv[tile] = kLayTile;
      }
      __syncthreads();
      continue;
    }
    // numbers of the occupied slots, in slot order
    constexpr int kOwn = Cap / kLayThreads;
    uint32_t own = 0;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) own += key[t * kOwn + i] != kNone ? 1u : 0u;
    const uint32_t inc = wave_scan_add(own);
    if (lane == kWave - 1) part[w] = inc;
    __syncthreads();
    uint32_t num = inc - own;
    for (int i = 0; i < w; ++i) num += part[i];
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
      if (key[t * kOwn + i] != kNone) key[t * kOwn + i] = num++;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g)
      c[g] = (c[g] == kNone ? nd : key[c[g]]) << 12 | (uint32_t)((w * kLayGroups + g) * kWave + lane);
    // stable passes of six bits
    for (uint32_t bits = 0; nd >> bits; bits += 6) {
      const int shift = 12 + (int)bits;
      uint32_t r[kLayGroups];
      cnt[w][lane] = 0u;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int g = 0; g < kLayGroups; ++g) {
        const uint32_t dg = c[g] >> shift & 63u;
        uint64_t same = ~0ull;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          const uint64_t bal = __ballot(dg >> k & 1u);
          same &= dg >> k & 1u ? bal : ~bal;
        }
        // LDS operations of a wave complete in order
        const uint32_t base = __hip_atomic_load(&cnt[w][dg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        r[g] = base + (uint32_t)__popcll(same & lanemask_lt());
        __builtin_amdgcn_wave_barrier();
        if (same >> lane == 1ull)
          __hip_atomic_store(&cnt[w][dg], base + (uint32_t)__popcll(same), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_wave_barrier();
      }
      __syncthreads();
      if (w == 0) {
        uint32_t of[kLayWaves], all = 0;
#pragma unroll
        for (int i = 0; i < kLayWaves; ++i) {
          of[i] = all;
          all += cnt[i][lane];
        }
        const uint32_t start = wave_scan_add(all) - all;
#pragma unroll
        for (int i = 0; i < kLayWaves; ++i) cnt[i][lane] = start + of[i];
      }
      __syncthreads();
#pragma unroll
      for (int g = 0; g < kLayGroups; ++g) item[cnt[w][c[g] >> shift & 63u] + r[g]] = c[g];
      __syncthreads();
#pragma unroll
      for (int g = 0; g < kLayGroups; ++g) c[g] = item[(w * kLayGroups + g) * kWave + lane];
      __syncthreads();
    }
    // (with nd = 0 nothing is placed)
    const uint32_t nv = placed;
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      const uint32_t q = (uint32_t)((w * kLayGroups + g) * kWave + lane);
      if (q < nv) {
        const bool head = q == 0 || item[q - 1] >> 12 != c[g] >> 12;
        A.order[v0 + q] = (uint16_t)((c[g] & 0xFFFu) | (head ? kLayHead : 0u));
      }
    }
    if (t == 0) {
      A.tile_nd[tile] = nd;
      A.tile_nv[tile] = nv;
    }
    __syncthreads();
  }
}

// The runs of equal cells in every tile's order.  place = false: the (tile,
// cell) pairs with their voxel counts, also added to the cells' totals; place
// = true: every voxel to its pair's segment start plus its place in the run.
// One streaming read of the order (2 B per voxel); the runs are numbered by
// ballots, a wave's total carried to the next waves through LDS.
template <bool place>
__global__ __launch_bounds__(kLayThreads) void k_lay_runs(LayArgs A) {
  __shared__ uint32_t at[kLayTile + 1];  // per run: its first place in the order, or its segment start less that
  __shared__ uint32_t part[kLayWaves];
  const int t = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  for (uint32_t tile = blockIdx.x; tile < (uint32_t)A.n_tiles; tile += gridDim.x) {
    const uint32_t nv = A.tile_nv[tile];
    if (nv == 0) continue;  // uniform
    const uint32_t p0 = A.pair_off[tile];
    const int64_t v0 = (int64_t)tile * kLayTile;
    uint32_t e[kLayGroups];
    uint64_t heads[kLayGroups];
    uint32_t total = 0;
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      const uint32_t q = (uint32_t)((w * kLayGroups + g) * kWave + lane);
      e[g] = q < nv ? A.order[v0 + q] : 0u;
    }
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      heads[g] = __ballot(e[g] & kLayHead);
      total += (uint32_t)__popcll(heads[g]);
    }
    if (lane == 0) part[w] = total;
    __syncthreads();
    uint32_t before = 0, nd = 0;
    for (int i = 0; i < kLayWaves; ++i) {
      if (i < w) before += part[i];
      nd += part[i];
    }
    uint32_t run = before;
#pragma unroll
    for (int g = 0; g < kLayGroups; ++g) {
      const uint32_t q = (uint32_t)((w * kLayGroups + g) * kWave + lane);
      if (e[g] & kLayHead) {
        const uint32_t k = run + (uint32_t)__popcll(heads[g] & lanemask_lt());
        at[k] = place ? A.seg_off[p0 + k] - q : q;
        if (!place) A.pair_cell[p0 + k] = A.cell[v0 + (e[g] & 0xFFFu)];
      }
      run += (uint32_t)__popcll(heads[g]);
    }
    if (!place && t == 0) at[nd] = nv;
    __syncthreads();
    if (place) {
      run = before;
#pragma unroll
      for (int g = 0; g < kLayGroups; ++g) {
        const uint32_t q = (uint32_t)((w * kLayGroups + g) * kWave + lane);
        const uint32_t k = run + (uint32_t)__popcll(heads[g] & (lanemask_lt() | (1ull << lane)));  // runs begun up to q
        if (q < nv) A.perm[at[k - 1] + q] = (uint32_t)(v0 + (e[g] & 0xFFFu));
        run += (uint32_t)__popcll(heads[g]);
      }
    } else {
      for (uint32_t k = t; k < nd; k += kLayThreads) {
        const uint32_t len = at[k + 1] - at[k];
        A.pair_cnt[p0 + k] = len;
        atomicAdd(&A.cnt[A.pair_cell[p0 + k]], (unsigned long long)len);
      }
    }
    __syncthreads();
  }
}

// ---- small helpers ---------------------------------------------------------
__global__ void k_iota32(uint32_t *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (uint32_t)i;
}
// dst[pos[i]] = src[i]
__global__ void k_scatter32(const uint32_t *src, const uint32_t *pos, int64_t n, uint32_t *dst) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[pos[i]] = src[i];
}
// dst[i] = src[idx[i]]
__global__ void k_gather32(const uint32_t *src, const uint32_t *idx, int64_t n, uint32_t *dst) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[idx[i]];
}

// site sort: key = min(site_comp, C) (out-of-range components last)
__global__ void k_site_count(const uint32_t *site_comp, uint32_t S, uint32_t C, uint32_t *ccount) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < S) atomicAdd(&ccount[min(site_comp[i], C)], 1u);
}
__global__ void k_site_digit(const uint32_t *val, uint32_t S, const uint32_t *site_comp, uint32_t C, int shift,
                             uint8_t *digit) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < S) digit[i] = (uint8_t)(min(site_comp[val[i]], C) >> shift);
}
__global__ void k_site_rank(const uint32_t *order, uint32_t S, uint32_t *rank) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < S) rank[order[i]] = i;
}
__global__ void k_pair_digit(const uint32_t *val, int64_t P, const uint32_t *pair_cell, const uint32_t *rank,
                             int shift, uint8_t *digit) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P) digit[i] = (uint8_t)(rank[pair_cell[val[i]]] >> shift);
}
__global__ void k_cnt_rank(const unsigned long long *cnt, const uint32_t *order, uint32_t S, uint32_t *cnt_rank) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < S) cnt_rank[i] = (uint32_t)cnt[order[i]];
}

int bits_for(uint64_t maxval) {
  int b = 0;
  while (b < 64 && (maxval >> b) != 0) ++b;
  return b;
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

}  // namespace

size_t layout_scratch(const Geom &g, uint32_t S, uint32_t C) {
  const int64_t P = layout_pair_cap(g, S);
  const int64_t T = layout_tiles(g);
  int64_t m = P > (int64_t)S ? P : (int64_t)S;
  if (m < (int64_t)C + 3) m = (int64_t)C + 3;
  if (m < T + 1) m = T + 1;
  size_t a = StableSort8::workspace(m);
  size_t b = ScanU32::workspace(m + 1);
  return (a > b ? a : b) + 256;
}

int32_t layout_sites(const uint32_t *site_comp, uint32_t S, uint32_t C, LayoutWork &W, hipStream_t s) {
  int32_t rc;
  if ((rc = fill<uint32_t>(W.ccount, (int64_t)C + 2, 0u, s))) return rc;
  if (S) {
    hipLaunchKernelGGL(k_site_count, dim3(blocks_for(S)), dim3(256), 0, s, site_comp, S, C, W.ccount);
    hipLaunchKernelGGL(k_iota32, dim3(blocks_for(S)), dim3(256), 0, s, W.order, (int64_t)S);
    LSRVT_LAUNCHED();
    const int passes = (bits_for(C) + 7) / 8;
    uint32_t *cur = W.order, *other = W.sval;
    for (int p = 0; p < passes; ++p) {
      hipLaunchKernelGGL(k_site_digit, dim3(blocks_for(S)), dim3(256), 0, s, cur, S, site_comp, C, 8 * p, W.sdigit);
      LSRVT_LAUNCHED();
      if ((rc = StableSort8::run(W.sdigit, S, W.spos, nullptr, W.scratch, W.scratch_bytes, s))) return rc;
      hipLaunchKernelGGL(k_scatter32, dim3(blocks_for(S)), dim3(256), 0, s, cur, W.spos, (int64_t)S, other);
      LSRVT_LAUNCHED();
      uint32_t *t = cur;
      cur = other;
      other = t;
    }
    if (cur != W.order) {
      LSRVT_HIP(hipMemcpyAsync(W.order, cur, sizeof(uint32_t) * S, hipMemcpyDeviceToDevice, s));
    }
    hipLaunchKernelGGL(k_site_rank, dim3(blocks_for(S)), dim3(256), 0, s, W.order, S, W.rank);
    LSRVT_LAUNCHED();
  }
  return ScanU32::run(W.ccount, (int64_t)C + 2, W.coff, W.scratch, W.scratch_bytes, s);
}

int32_t layout_voxels(const uint32_t *cell, const Geom &g, uint32_t S, LayoutWork &W, uint32_t *perm, hipStream_t s) {
  int32_t rc;
  if ((rc = fill<unsigned long long>(W.cnt, S ? S : 1, 0ull, s))) return rc;
  if ((rc = fill<uint32_t>(W.big_cnt, 1, 0u, s))) return rc;
  if (S == 0) return fill<uint32_t>(W.cell_off, 1, 0u, s);
  const int64_t T = W.n_tiles;
  LayArgs A;
  A.cell = cell;
  A.n = g.n;
  A.S = S;
  A.n_tiles = T;
  A.cnt = W.cnt;
  A.tile_nd = W.tile_nd;
  A.tile_nv = W.tile_nv;
  A.order = W.tile_order;
  A.big_list = W.big_list;
  A.big_cnt = W.big_cnt;
  A.pair_off = W.pair_off;
  A.pair_cell = W.pair_cell;
  A.pair_cnt = W.pair_cnt;
  A.seg_off = W.pair_cnt;  // segment starts replace the counts before the place pass
  A.perm = perm;
  const unsigned grid = (unsigned)(T < 65535 ? T : 65535);
  // 1. every tile's order and distinct cells
  hipLaunchKernelGGL((k_lay_sort<kSmallCap, kSmallMax, true>), dim3(grid), dim3(kLayThreads), 0, s, A);
  hipLaunchKernelGGL((k_lay_sort<kBigCap, kBigMax, false>), dim3((unsigned)(T < 768 ? T : 768)), dim3(kLayThreads), 0,
                     s, A);
  LSRVT_LAUNCHED();
  if ((rc = ScanU32::run(W.tile_nd, T, W.pair_off, W.scratch, W.scratch_bytes, s))) return rc;
  uint32_t P = 0;
  {
    const int32_t rc_ = read_words(W.pair_off + T, 1, &P, s);
    if (rc_) return rc_;
  }
  if ((int64_t)P > W.pair_cap) return LSRVT_EDEVICE;  // cannot happen: the capacity is an upper bound
  // 2. the pairs, in tile order, and the voxels per site
  hipLaunchKernelGGL(k_lay_runs<false>, dim3(grid), dim3(kLayThreads), 0, s, A);
  LSRVT_LAUNCHED();
  // 3. stable sort of the pairs by cell rank
  if (P) {
    hipLaunchKernelGGL(k_iota32, dim3(blocks_for(P)), dim3(256), 0, s, W.val_a, (int64_t)P);
    LSRVT_LAUNCHED();
    const int passes = (bits_for(S - 1) + 7) / 8;
    uint32_t *cur = W.val_a, *other = W.val_b;
    for (int p = 0; p < passes; ++p) {
      hipLaunchKernelGGL(k_pair_digit, dim3(blocks_for(P)), dim3(256), 0, s, cur, (int64_t)P, W.pair_cell, W.rank,
                         8 * p, W.digit);
      LSRVT_LAUNCHED();
      if ((rc = StableSort8::run(W.digit, P, W.pos, nullptr, W.scratch, W.scratch_bytes, s))) return rc;
      hipLaunchKernelGGL(k_scatter32, dim3(blocks_for(P)), dim3(256), 0, s, cur, W.pos, (int64_t)P, other);
      LSRVT_LAUNCHED();
      uint32_t *t = cur;
      cur = other;
      other = t;
    }
    // 4. segment starts: scan the sizes in sorted order, scatter back to pair order
    hipLaunchKernelGGL(k_gather32, dim3(blocks_for(P)), dim3(256), 0, s, W.pair_cnt, cur, (int64_t)P, W.pos);
    LSRVT_LAUNCHED();
    if ((rc = ScanU32::run(W.pos, P, other, W.scratch, W.scratch_bytes, s))) return rc;
    hipLaunchKernelGGL(k_scatter32, dim3(blocks_for(P)), dim3(256), 0, s, other, cur, (int64_t)P, W.pair_cnt);
    LSRVT_LAUNCHED();
    // 5. place every voxel
    hipLaunchKernelGGL(k_lay_runs<true>, dim3(grid), dim3(kLayThreads), 0, s, A);
    LSRVT_LAUNCHED();
  }
  // cell offsets by rank
  hipLaunchKernelGGL(k_cnt_rank, dim3(blocks_for(S)), dim3(256), 0, s, W.cnt, W.order, S, W.cnt_rank);
  LSRVT_LAUNCHED();
  return ScanU32::run(W.cnt_rank, S, W.cell_off, W.scratch, W.scratch_bytes, s);
}

namespace {

// comp_off[c] = cell_off[coff[c]] for c <= C
__global__ void k_comp_off(const uint32_t *cell_off, const uint32_t *coff, uint32_t C, uint32_t *comp_off) {
  uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c <= C) comp_off[c] = cell_off[coff[c]];
}
// band_off[b] = comp_off[first component whose band is >= b] (bands nondecreasing in component id)
__global__ void k_band_off(const uint8_t *comp_band, uint32_t C, int32_t n_bands, const uint32_t *comp_off,
                           uint32_t *band_off) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > n_bands) return;
  uint32_t lo = 0, hi = C;
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if ((int)comp_band[mid] < b)
      lo = mid + 1;
    else
      hi = mid;
  }
  band_off[b] = comp_off[lo];
}

// out[j][k] = vars[j][perm[k]]
__global__ void k_extract(const float *__restrict__ vars, int64_t n, int m, const uint32_t *__restrict__ perm,
                          int64_t count, float *__restrict__ out) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  const int64_t v = perm[k];
  for (int j = 0; j < m; ++j) out[(int64_t)j * count + k] = v < n ? vars[(int64_t)j * n + v] : __builtin_nanf("");
}

struct LaySizer : Sizer {
  template <class T>
  T *take(size_t c) {
    Sizer::take<T>(c);
    return nullptr;
  }
};

}  // namespace

}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_layout_workspace(lsrvt_dims dims, uint32_t n_sites, uint32_t n_comp) {
  Geom g;
  if (make_geom(dims, g)) return 0;
  LaySizer z;
  layout_take(z, g, n_sites, n_comp, nullptr);
  return z.off + layout_scratch(g, n_sites, n_comp);
}

extern "C" int32_t lsrvt_layout(const uint32_t *d_cell, lsrvt_dims dims, const uint32_t *d_site_comp, uint32_t n_sites,
                                const uint8_t *d_comp_band, uint32_t n_comp, int32_t n_bands, uint32_t *d_perm,
                                uint32_t *d_site_order, uint32_t *d_cell_off, uint32_t *d_comp_off,
                                uint32_t *d_band_off, uint32_t *h_n_placed, void *d_work, size_t work_bytes,
                                void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (n_bands < 1 || n_bands > 255) return LSRVT_EINVAL;
  if (!d_cell || !d_perm || !d_cell_off || !d_comp_off || !d_band_off) return LSRVT_EINVAL;
  if (n_sites && (!d_site_comp || !d_site_order)) return LSRVT_EINVAL;
  if (n_comp && !d_comp_band) return LSRVT_EINVAL;
  if ((rc = check_work(d_work, work_bytes, lsrvt_layout_workspace(dims, n_sites, n_comp)))) return rc;
  Carve cv(d_work, work_bytes);
  LayoutWork W;
  layout_take(cv, g, n_sites, n_comp, &W);
  if (!cv.ok) return LSRVT_EWORKSPACE;
  W.scratch = cv.base + cv.off;
  W.scratch_bytes = cv.size - cv.off;
  hipStream_t s = as_stream(stream);
  if ((rc = layout_sites(d_site_comp, n_sites, n_comp, W, s))) return rc;
  if ((rc = layout_voxels(d_cell, g, n_sites, W, d_perm, s))) return rc;
  if (n_sites) {
    LSRVT_HIP(hipMemcpyAsync(d_site_order, W.order, sizeof(uint32_t) * n_sites, hipMemcpyDeviceToDevice, s));
  }
  LSRVT_HIP(hipMemcpyAsync(d_cell_off, W.cell_off, sizeof(uint32_t) * ((size_t)n_sites + 1), hipMemcpyDeviceToDevice,
                           s));
  hipLaunchKernelGGL(k_comp_off, dim3(blocks_for((int64_t)n_comp + 1)), dim3(256), 0, s, W.cell_off, W.coff, n_comp,
                     d_comp_off);
  hipLaunchKernelGGL(k_band_off, dim3(blocks_for(n_bands + 1)), dim3(256), 0, s, d_comp_band, n_comp, n_bands,
                     d_comp_off, d_band_off);
  LSRVT_LAUNCHED();
  uint32_t placed = 0;
  {
    const int32_t rc_ = read_words(W.cell_off + n_sites, 1, &placed, s);
    if (rc_) return rc_;
  }
  if (h_n_placed) *h_n_placed = placed;
  return LSRVT_OK;
}

extern "C" int32_t lsrvt_extract(const float *d_vars, int32_t n_vars, lsrvt_dims dims, const uint32_t *d_perm,
                                 uint32_t n_placed, float *d_out, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (n_vars < 1 || (int64_t)n_placed > g.n) return LSRVT_EINVAL;
  if (n_placed == 0) return LSRVT_OK;
  if (!d_vars || !d_perm || !d_out) return LSRVT_EINVAL;
  hipLaunchKernelGGL(k_extract, dim3(blocks_for(n_placed)), dim3(256), 0, as_stream(stream), d_vars, g.n, n_vars,
                     d_perm, (int64_t)n_placed, d_out);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}
