// Stratified initial sites (Sec. 3.2.1, Eq. 3 and Eq. 4).
//
// Voxel mass m(v) = lut[w(v)] (m = w without a table, 1 without weights).
// A component C gets n_c = max(ceil(m(C) N / (rho M)), 1) sites, M the total
// mass and rho the voxels per site (Eq. 3 with the density as one site per
// rho voxels of average mass).  The volume is cut into cubes of edge B; the
// (component, block) pairs of C share its n_c sites by floor shares
// floor(n_c m(b) / m(C)) plus one each for the largest remainders
// n_c m(b) mod m(C), ties to the lower block index (Eq. 4, "most
// under-represented blocks").  Inside a pair, the n_b sites are placed by
// systematic sampling proportional to mass over the pair's voxels in
// linear-index order: with o in [0, m(b)) the j-th point is
// p_j = floor((o + j m(b)) / n_b) and the site is the voxel whose cumulative
// mass interval holds p_j.  o comes from Philox4x32-10 (Salmon et al., SC
// 2011) keyed by the seed, counter (block, component, 0, 0).  A component
// of zero mass gets one site, its first voxel (smallest linear index).  Sites are numbered by
// (component, block, j).  Every decision is taken in exact integer
// arithmetic, so the result does not depend on scheduling.
//
// Steps: per block, the distinct components and their masses (LDS hash);
// a scan gives the pairs block-major; a stable radix sort by component puts
// them in (component, block) order; a wave (a workgroup for the components of
// many pairs) apportions a component's sites: the r-th largest remainder is
// found by bisection (by digits) on its value; a scan numbers the sites; per block, each pair with sites runs a prefix
// sum of its mass over the block's voxels and places its points.
#include <algorithm>

#include "common.h"

namespace lsrvt {
namespace {

constexpr int kSeedThreads = 256;
constexpr int kMaxBlockEdge = 16;
constexpr int kBlockCap = kMaxBlockEdge * kMaxBlockEdge * kMaxBlockEdge;  // voxels (and components) per block

struct SeedGeom {
  Geom g;
  int32_t B;
  int32_t nbx, nby, nbz;
  int64_t nblocks;
};

SeedGeom seed_geom(const Geom &g, int32_t B) {
  SeedGeom G;
  G.g = g;
  G.B = B;
  G.nbx = (g.nx + B - 1) / B;
  G.nby = (g.ny + B - 1) / B;
  G.nbz = (g.nz + B - 1) / B;
  G.nblocks = (int64_t)G.nbx * G.nby * G.nbz;
  return G;
}

struct MassIn {
  const uint16_t *w;    // weights or null (mass 1)
  const uint32_t *lut;  // mass of every weight value or null (mass = weight)
};

__device__ __forceinline__ uint32_t voxel_mass(const MassIn &mi, int64_t v) {
  if (!mi.w) return 1u;
  const uint32_t x = mi.w[v];
  return mi.lut ? mi.lut[x] : x;
}

// Voxel k (x fastest) of block b as a linear index; -1 outside the volume.
// Within a block k increases with the linear index.
__device__ __forceinline__ int64_t block_voxel(const SeedGeom &G, int64_t b, int k) {
  const int bx = (int)(b % G.nbx), by = (int)((b / G.nbx) % G.nby), bz = (int)(b / ((int64_t)G.nbx * G.nby));
  const int x = bx * G.B + k % G.B, y = by * G.B + (k / G.B) % G.B, z = bz * G.B + k / (G.B * G.B);
  if (x >= G.g.nx || y >= G.g.ny || z >= G.g.nz) return -1;
  return x + (int64_t)G.g.nx * (y + (int64_t)G.g.ny * z);
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (published multipliers and key increments)
struct U4 {
  uint32_t v[4];
};

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t lo0 = 0xD2511F53u * c.v[0], hi0 = __umulhi(0xD2511F53u, c.v[0]);
    const uint32_t lo1 = 0xCD9E8D57u * c.v[2], hi1 = __umulhi(0xCD9E8D57u, c.v[2]);
    U4 o;
    o.v[0] = hi1 ^ c.v[1] ^ k0;
    o.v[1] = lo1;
    o.v[2] = hi0 ^ c.v[3] ^ k1;
    o.v[3] = lo0;
    c = o;
  }
  return c;
}

// ---------------------------------------------------------------------------
// exact 128-bit helpers
typedef unsigned __int128 u128;

__device__ __forceinline__ double u128_to_double(u128 a) {
  return (double)(uint64_t)(a >> 64) * 18446744073709551616.0 + (double)(uint64_t)a;
}

// floor(num / den) for a quotient below 2^32 (the estimate in double is then
// within one of it; the loops correct it exactly).  *err is set if the
// quotient is out of range.
__device__ __forceinline__ uint64_t div_small(u128 num, u128 den, uint32_t *err) {
  if (den == 0) {
    atomicOr(err, 2u);
    return 0;
  }
  double e = u128_to_double(num) / u128_to_double(den);
  if (!(e < 4294967296.0 * 2.0)) {
    atomicOr(err, 2u);
    return 0;
  }
  uint64_t q = (uint64_t)e;
  for (int i = 0; i < 4 && (u128)q * den > num; ++i) --q;
  for (int i = 0; i < 4 && (u128)(q + 1) * den <= num; ++i) ++q;
  if ((u128)q * den > num || (u128)(q + 1) * den <= num) atomicOr(err, 2u);
  return q;
}

// ---------------------------------------------------------------------------
// Components and masses of row t of the block (its voxels B t .. B t + B - 1);
// returns the mask of those inside the volume.  Sixteen voxels are read in four
// (two for the weights) wide loads, whatever the edge: what lies past the row is
// not used, and only where it would lie past the volume's last voxel are they
// read one by one.  (The call on 501 x 333 x 187 voxels in 6 isobands with weights and
// edge 15 takes 0.58 ms so, 2.16 reading a row voxel by voxel, 1.55 with
// sixteen voxels a thread across the rows and 1.50 with neighbouring lanes on
// neighbouring voxels.)
constexpr int kPer = kBlockCap / kSeedThreads;
__device__ __forceinline__ uint32_t load_row(const uint32_t *__restrict__ comp, const SeedGeom &G, const MassIn &mi,
                                             int64_t b, int t, uint32_t vc[kPer], uint32_t vm[kPer]) {
  static_assert(kPer == kMaxBlockEdge, "a thread's voxels are a row of the largest block");
  if (t >= G.B * G.B) return 0u;
  const int64_t v = block_voxel(G, b, t * G.B);
  if (v < 0) return 0u;
  const int left = min(G.B, G.g.nx - (int)(b % G.nbx) * G.B);
  if (v + kPer <= G.g.n) {
    uint16_t w[kPer];
    __builtin_memcpy(vc, comp + v, sizeof(uint32_t) * kPer);
    if (mi.w) __builtin_memcpy(w, mi.w + v, sizeof(w));
#pragma unroll
    for (int j = 0; j < kPer; ++j) vm[j] = !mi.w ? 1u : mi.lut ? mi.lut[w[j]] : (uint32_t)w[j];
  } else {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (j < left) {
        vc[j] = comp[v + j];
        vm[j] = voxel_mass(mi, v + j);
      }
  }
  return (1u << left) - 1u;
}

// per block: distinct components (pass 0 counts them and sums the block's
// mass; pass 1 writes the pairs: component, block, mass, in any order).  A
// block of one component needs no table; in the others each thread adds the
// runs of its row (501 x 333 x 187 voxels with 5 isobands and a table of
// masses: the two passes took 0.34 ms with an atomic for each voxel, now 0.28).
// Edge: the block edge where it is known to the compiler (the usual 16: 2 to 4 % of the
// call on labels of many small components), else 0.
template <int Pass, int Edge>
__global__ __launch_bounds__(kSeedThreads) void k_seed_blocks(const uint32_t *__restrict__ comp, SeedGeom G,
                                                              uint32_t n_comp, MassIn mi, uint32_t *pcnt,
                                                              unsigned long long *bmass, const uint32_t *poff,
                                                              uint32_t *pair_comp, uint32_t *pair_block,
                                                              unsigned long long *pair_mass, uint32_t *err) {
  __shared__ uint32_t key[kBlockCap];
  __shared__ unsigned long long msum[Pass ? kBlockCap : 1];
  __shared__ uint32_t wsum[kSeedThreads / kWave];
  __shared__ unsigned long long red[kSeedThreads / kWave];
  if (Edge) G.B = Edge;
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  for (int64_t b = blockIdx.x; b < G.nblocks; b += gridDim.x) {
    const uint32_t c0 = comp[block_voxel(G, b, 0)];  // a block's first voxel is inside the volume
    uint32_t vc[kPer], vm[kPer];
    uint32_t in = load_row(comp, G, mi, b, t, vc, vm);
    bool one = true;
    unsigned long long mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (in >> j & 1u) {
        if (vc[j] >= n_comp) {
          atomicOr(err, 1u);
          in &= ~(1u << j);
          one = false;
        } else {
          one = one && vc[j] == c0;
          mine += vm[j];
        }
      }
    const unsigned long long wm = wave_sum_u64(mine);
    if (lane == 0) red[wid] = wm;
    one = __syncthreads_and(one);
    unsigned long long mass = 0;
    for (int q = 0; q < kSeedThreads / kWave; ++q) mass += red[q];
    if (one) {
      if (t == 0) {
        if (Pass == 0) {
          pcnt[b] = 1u;
          bmass[b] = mass;
        } else {
          pair_comp[poff[b]] = c0;
          pair_block[poff[b]] = (uint32_t)b;
          pair_mass[poff[b]] = mass;
        }
      }
      __syncthreads();
      continue;
    }
    for (int i = t; i < kBlockCap; i += kSeedThreads) {
      key[i] = kNone;
      if (Pass) msum[i] = 0ull;
    }
    __syncthreads();
    uint32_t run_c = kNone;
    unsigned long long run_m = 0;
    auto flush = [&]() {
      if (run_c == kNone) return;
      const int sl = lds_slot<kBlockCap>(key, run_c);  // a block holds at most kBlockCap components
      if (Pass && sl >= 0) atomicAdd(&msum[sl], run_m);
    };
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (in >> j & 1u) {
        if (vc[j] != run_c) {
          flush();
          run_c = vc[j];
          run_m = 0;
        }
        run_m += vm[j];
      }
    flush();
    __syncthreads();
    // slots in use: count (pass 0) or compact (pass 1)
    uint32_t cnt = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) cnt += key[t + j * kSeedThreads] != kNone;
    uint32_t inc = cnt;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t x = __shfl_up(inc, o, kWave);
      if (lane >= o) inc += x;
    }
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int q = 0; q < kSeedThreads / kWave; ++q) {
      if (q < wid) before += wsum[q];
      total += wsum[q];
    }
    if (Pass == 0) {
      if (t == 0) {
        pcnt[b] = total;
        bmass[b] = mass;
      }
    } else {
      uint32_t pos = poff[b] + before + inc - cnt;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int sl = t + j * kSeedThreads;
        if (key[sl] != kNone) {
          pair_comp[pos] = key[sl];
          pair_block[pos] = (uint32_t)b;
          pair_mass[pos] = msum[sl];
          ++pos;
        }
      }
    }
    __syncthreads();
  }
}

// Total mass: one workgroup over the per-block sums (fixed order).
__global__ __launch_bounds__(kSeedThreads) void k_seed_total(const unsigned long long *bmass, int64_t nb,
                                                             unsigned long long *total) {
  __shared__ unsigned long long red[kSeedThreads];
  unsigned long long s = 0;
  for (int64_t i = threadIdx.x; i < nb; i += kSeedThreads) s += bmass[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = kSeedThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = red[0];
}

__global__ void k_seed_iota(uint32_t *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (uint32_t)i;
}

__global__ void k_seed_digit(const uint32_t *val, int64_t n, const uint32_t *pair_comp, int shift, uint8_t *digit) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) digit[i] = (uint8_t)(pair_comp[val[i]] >> shift);
}

__global__ void k_seed_scatter(const uint32_t *src, const uint32_t *pos, int64_t n, uint32_t *dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[pos[i]] = src[i];
}

// sorted views of the pairs and the segment of every component
__global__ void k_seed_sorted(const uint32_t *idx, int64_t P, const uint32_t *pair_comp,
                              const unsigned long long *pair_mass, uint32_t *scomp, unsigned long long *smass,
                              uint32_t *cbeg, uint32_t *cend) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const uint32_t c = pair_comp[idx[i]];
  scomp[i] = c;
  smass[i] = pair_mass[idx[i]];
  if (i == 0 || pair_comp[idx[i - 1]] != c) cbeg[c] = (uint32_t)i;
  if (i == P - 1 || pair_comp[idx[i + 1]] != c) cend[c] = (uint32_t)(i + 1);
}

// n_c and the share of each pair of a component (sorted order, blocks
// ascending), written to snb: one wave for a component of up to kNarrow pairs,
// whose remainders stay in registers, a workgroup for the others (wide: their
// list and number).  The walk over the pairs is a chain of loads for every
// step of the search: with a wave for each component the largest one's 30000
// pairs took 0.92 ms of a 501 x 333 x 187 volume (0.05 now) and
// 3.1 ms at 1024 x 512 x 512 (0.19 now).
constexpr int kNarrowPer = 4;
constexpr uint32_t kNarrow = kNarrowPer * kWave;
constexpr int kWideThreads = 1024;

// Eq. 3: n_c = max(ceil(m(C) N / (rho M)), 1), den = rho M
__device__ __forceinline__ uint64_t site_count(unsigned long long mc, int64_t N, u128 den, uint32_t *err) {
  const u128 num = (u128)mc * (u128)(uint64_t)N;
  uint64_t nc = div_small(num, den, err);
  if ((u128)nc * den < num) ++nc;
  return nc ? nc : 1;
}

__global__ __launch_bounds__(kSeedThreads) void k_seed_apportion(uint32_t n_comp, const uint32_t *cbeg,
                                                                 const uint32_t *cend,
                                                                 const unsigned long long *smass,
                                                                 const unsigned long long *total, int64_t N,
                                                                 uint32_t rho, uint32_t *snb, uint32_t *wide,
                                                                 uint32_t *n_wide, uint32_t *err) {
  const int lane = lane_id();
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  const u128 den = (u128)rho * (u128)(*total);
  for (int64_t c = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; c < n_comp; c += waves) {
    const uint32_t b0 = cbeg[c], b1 = cend[c];
    if (b1 <= b0) continue;
    if (b1 - b0 > kNarrow) {
      if (lane == 0) wide[atomicAdd(n_wide, 1u)] = (uint32_t)c;
      continue;
    }
    unsigned long long m[kNarrowPer], mc = 0;
#pragma unroll
    for (int k = 0; k < kNarrowPer; ++k) {
      const uint32_t i = b0 + k * kWave + lane;
      m[k] = i < b1 ? smass[i] : 0ull;
      mc += m[k];
    }
    mc = wave_sum_u64(mc);
    if (mc == 0) {
      // zero mass: one site (the component's first voxel), numbered with its first pair
      for (uint32_t i = b0 + lane; i < b1; i += kWave) snb[i] = i == b0 ? 1u : 0u;
      continue;
    }
    const uint64_t nc = site_count(mc, N, den, err);
    // floor shares and remainders
    unsigned long long rem[kNarrowPer];
    uint32_t share[kNarrowPer];
    uint64_t given = 0;
#pragma unroll
    for (int k = 0; k < kNarrowPer; ++k) {
      rem[k] = 0;
      share[k] = 0;
      if (b0 + k * kWave < b1) {  // uniform
        const u128 q = (u128)nc * (u128)m[k];
        const uint64_t base = div_small(q, (u128)mc, err);
        rem[k] = (unsigned long long)(q - (u128)base * mc);
        share[k] = (uint32_t)base;
        given += base;
      }
    }
    given = wave_sum_u64(given);
    const uint64_t r = nc - given;
    if (r) {
      auto count = [&](unsigned long long v) {  // pairs with a remainder of at least v (v > 0)
        uint64_t n = 0;
#pragma unroll
        for (int k = 0; k < kNarrowPer; ++k) n += (uint64_t)__popcll(__ballot(rem[k] >= v));
        return n;
      };
      // the r-th largest remainder v: the largest v with #(rem >= v) >= r
      unsigned long long lo = 0, hi = mc;
      while (hi - lo > 1) {
        const unsigned long long mid = lo + (hi - lo) / 2;
        if (count(mid) >= r)
          lo = mid;
        else
          hi = mid;
      }
      // remainders above v all get one more; those equal to v in block order
      uint64_t ties = r - count(lo + 1);
#pragma unroll
      for (int k = 0; k < kNarrowPer; ++k) {
        const bool eq = b0 + k * kWave + lane < b1 && rem[k] == lo;
        const uint64_t em = __ballot(eq);
        const uint64_t rank = (uint64_t)__popcll(em & lanemask_lt());
        if (rem[k] > lo || (eq && rank < ties)) share[k] += 1u;
        const uint64_t used = (uint64_t)__popcll(em);
        ties = ties > used ? ties - used : 0;
      }
    }
#pragma unroll
    for (int k = 0; k < kNarrowPer; ++k) {
      const uint32_t i = b0 + k * kWave + lane;
      if (i < b1) snb[i] = share[k];
    }
  }
}

__device__ __forceinline__ uint64_t wide_sum(uint64_t v, unsigned long long *part) {
  v = wave_sum_u64(v);
  __syncthreads();
  if (lane_id() == 0) part[threadIdx.x / kWave] = v;
  __syncthreads();
  uint64_t s = 0;
  for (int q = 0; q < kWideThreads / kWave; ++q) s += part[q];
  return s;
}

// The same by a workgroup.  The r-th largest remainder comes from its digits of
// eight bits, the highest first: a histogram of the remainders that agree with
// the digits found so far.
__global__ __launch_bounds__(kWideThreads) void k_seed_apportion_wide(
    const uint32_t *cbeg, const uint32_t *cend, const unsigned long long *smass, const unsigned long long *total,
    int64_t N, uint32_t rho, unsigned long long *srem, uint32_t *snb, const uint32_t *wide, const uint32_t *n_wide,
    uint32_t *err) {
  __shared__ unsigned long long part[kWideThreads / kWave];
  __shared__ uint32_t hist[256];
  __shared__ uint32_t digit_s, above_s;
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  const u128 den = (u128)rho * (u128)(*total);
  const uint32_t n = *n_wide;
  for (uint32_t e = blockIdx.x; e < n; e += gridDim.x) {
    const uint32_t c = wide[e], b0 = cbeg[c], b1 = cend[c];
    uint64_t mc = 0;
    for (uint32_t i = b0 + t; i < b1; i += kWideThreads) mc += smass[i];
    mc = wide_sum(mc, part);
    if (mc == 0) {
      for (uint32_t i = b0 + t; i < b1; i += kWideThreads) snb[i] = i == b0 ? 1u : 0u;
      continue;
    }
    const uint64_t nc = site_count(mc, N, den, err);
    uint64_t given = 0;
    for (uint32_t i = b0 + t; i < b1; i += kWideThreads) {
      const u128 q = (u128)nc * (u128)smass[i];
      const uint64_t base = div_small(q, (u128)mc, err);
      srem[i] = (unsigned long long)(q - (u128)base * mc);
      snb[i] = (uint32_t)base;
      given += base;
    }
    given = wide_sum(given, part);
    uint64_t r = nc - given;
    if (r == 0) continue;
    uint64_t v = 0;  // the digits found, then r: the rank among the remainders that agree with them
    for (int shift = (63 - __clzll((long long)mc)) / 8 * 8; shift >= 0; shift -= 8) {
      __syncthreads();
      if (t < 256) hist[t] = 0u;
      __syncthreads();
      for (uint32_t i = b0 + t; i < b1; i += kWideThreads) {
        const uint64_t x = srem[i] >> shift;
        if (x >> 8 == v) atomicAdd(&hist[x & 255u], 1u);
      }
      __syncthreads();
      if (wid == 0) {  // lane l holds digits 255 - 4 l down to 252 - 4 l
        uint32_t h[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          h[k] = hist[255 - 4 * lane - k];
          sum += h[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
          const uint32_t up = __shfl_up(inc, o, kWave);
          if (lane >= o) inc += up;
        }
        uint32_t before = inc - sum;
        if (before < r && r <= inc)
          for (int k = 0; k < 4; ++k) {
            if (before < r && r <= before + h[k]) {
              digit_s = (uint32_t)(255 - 4 * lane - k);
              above_s = before;
            }
            before += h[k];
          }
      }
      __syncthreads();
      v = v << 8 | digit_s;
      r -= above_s;
    }
    // remainders above v all get one more; those equal to v in block order
    for (uint32_t i0 = b0; i0 < b1; i0 += kWideThreads) {
      const uint32_t i = i0 + t;
      const bool eq = i < b1 && srem[i] == v;
      const uint64_t em = __ballot(eq);
      __syncthreads();
      if (lane == 0) hist[wid] = (uint32_t)__popcll(em);
      __syncthreads();
      uint64_t rank = (uint64_t)__popcll(em & lanemask_lt()), all = 0;
      for (int q = 0; q < kWideThreads / kWave; ++q) {
        if (q < wid) rank += hist[q];
        all += hist[q];
      }
      if (i < b1 && (srem[i] > v || (eq && rank < r))) snb[i] += 1u;
      r = r > all ? r - all : 0;
    }
  }
}

// back to block-major pair order
__global__ void k_seed_unsort(const uint32_t *idx, int64_t P, const uint32_t *snb, const uint32_t *ssoff,
                              uint32_t *nb_pair, uint32_t *soff_pair) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  nb_pair[idx[i]] = snb[i];
  soff_pair[idx[i]] = ssoff[i];
}

// Per block, each pair with sites: prefix sums of the pair's mass over the
// block's voxels in linear order, then the systematic points.  The block's
// components and masses are read once into registers (thread t holds row t);
// per pair the prefix sums are a wave scan of the
// per-thread sums plus the four wave totals.  They lie in LDS with one place
// unused after every 16, so that the threads' stores meet different banks
// (501 x 333 x 187 voxels: 0.45 ms before, 0.22 now).
template <int Edge>
__global__ __launch_bounds__(kSeedThreads) void k_seed_place(const uint32_t *__restrict__ comp, SeedGeom G,
                                                             MassIn mi, const uint32_t *poff,
                                                             const uint32_t *pair_comp,
                                                             const unsigned long long *pair_mass,
                                                             const uint32_t *comp_first, const uint32_t *nb_pair,
                                                             const uint32_t *soff_pair, uint32_t key_lo,
                                                             uint32_t key_hi, uint32_t *sites, uint32_t cap) {
  __shared__ unsigned long long cum[kBlockCap + kBlockCap / kPer];
  __shared__ unsigned long long wtot[kSeedThreads / kWave];
  if (Edge) G.B = Edge;
  const int t = threadIdx.x, lane = lane_id(), wid = t / kWave;
  for (int64_t b = blockIdx.x; b < G.nblocks; b += gridDim.x) {
    const uint32_t k0 = poff[b], k1 = poff[b + 1];
    uint32_t any = 0;
    for (uint32_t k = k0 + t; k < k1; k += kSeedThreads) any |= nb_pair[k];
    if (!__syncthreads_or(any != 0u)) continue;  // no site in this block
    uint32_t vc[kPer], vm[kPer];
    const uint32_t in = load_row(comp, G, mi, b, t, vc, vm);
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (!(in >> j & 1u)) {
        vc[j] = kNone;
        vm[j] = 0u;
      }
    for (uint32_t k = k0; k < k1; ++k) {
      const uint32_t nb = nb_pair[k];
      if (nb == 0) continue;  // uniform across the workgroup
      const uint32_t c = pair_comp[k];
      const unsigned long long mb = pair_mass[k];
      const uint32_t so = soff_pair[k];
      if (mb == 0) {
        if (t == 0 && so < cap) sites[so] = comp_first[c];
        continue;
      }
      unsigned long long run = 0, loc[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        run += vc[j] == c ? vm[j] : 0u;
        loc[j] = run;
      }
      unsigned long long inc = run;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const unsigned long long x = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += x;
      }
      if (lane == kWave - 1) wtot[wid] = inc;
      __syncthreads();
      unsigned long long before = inc - run;
      for (int q = 0; q < wid; ++q) before += wtot[q];
#pragma unroll
      for (int j = 0; j < kPer; ++j) cum[t * (kPer + 1) + j] = before + loc[j];
      __syncthreads();
      U4 ctr;
      ctr.v[0] = (uint32_t)b;
      ctr.v[1] = c;
      ctr.v[2] = 0u;
      ctr.v[3] = 0u;
      const U4 rnd = philox4x32_10(ctr, key_lo, key_hi);
      const unsigned long long o = ((unsigned long long)rnd.v[0] | ((unsigned long long)rnd.v[1] << 32)) % mb;
      const unsigned long long qm = mb / nb, rm = mb % nb;
      for (uint32_t j = t; j < nb; j += kSeedThreads) {
        // p_j = floor((o + j mb) / nb) without 128-bit products
        const unsigned long long p = (unsigned long long)j * qm + (o + (unsigned long long)j * rm) / nb;
        // first voxel whose cumulative mass exceeds p
        int lo = 0, hi = kBlockCap - 1;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (cum[mid + mid / kPer] > p)
            hi = mid;
          else
            lo = mid + 1;
        }
        const int64_t v = block_voxel(G, b, lo / kPer * G.B) + lo % kPer;  // place lo: voxel lo % 16 of row lo / 16
        if (so + j < cap) sites[so + j] = (uint32_t)v;
      }
      __syncthreads();
    }
  }
}

struct SeedWork {
  uint32_t *pcnt, *poff, *err;
  unsigned long long *bmass, *total;
  uint32_t *pair_comp, *pair_block;
  unsigned long long *pair_mass;
  uint32_t *val_a, *val_b, *pos;
  uint8_t *digit;
  void *scratch;
  size_t scratch_bytes;
  uint32_t *scomp, *snb, *ssoff, *cbeg, *cend, *nb_pair, *soff_pair;
  unsigned long long *smass, *srem;
};

template <class A>
void seed_layout(A &a, const SeedGeom &G, uint32_t n_comp, uint32_t cap_pairs, SeedWork *W) {
  const size_t nb = (size_t)G.nblocks;
  const size_t P = cap_pairs ? cap_pairs : 1;
  auto pcnt = a.template take<uint32_t>(nb + 1);
  auto poff = a.template take<uint32_t>(nb + 1);
  auto err = a.template take<uint32_t>(2);  // [0] errors, [1] components with many pairs
  auto bmass = a.template take<unsigned long long>(nb);
  auto total = a.template take<unsigned long long>(1);
  auto pc = a.template take<uint32_t>(P);
  auto pb = a.template take<uint32_t>(P);
  auto pm = a.template take<unsigned long long>(P);
  auto va = a.template take<uint32_t>(P);
  auto vb = a.template take<uint32_t>(P);
  auto pos = a.template take<uint32_t>(P);
  auto dig = a.template take<uint8_t>(P);
  const size_t sb = std::max(StableSort8::workspace((int64_t)P), ScanU32::workspace((int64_t)std::max(P, nb)));
  auto scr = a.template take<uint8_t>(sb);
  auto sc = a.template take<uint32_t>(P);
  auto snb = a.template take<uint32_t>(P + 1);
  auto sso = a.template take<uint32_t>(P + 1);
  auto cb = a.template take<uint32_t>(n_comp ? n_comp : 1);
  auto ce = a.template take<uint32_t>(n_comp ? n_comp : 1);
  auto nbp = a.template take<uint32_t>(P);
  auto sop = a.template take<uint32_t>(P);
  auto sm = a.template take<unsigned long long>(P);
  auto sr = a.template take<unsigned long long>(P);
  if (W) {
    W->pcnt = pcnt;
    W->poff = poff;
    W->err = err;
    W->bmass = bmass;
    W->total = total;
    W->pair_comp = pc;
    W->pair_block = pb;
    W->pair_mass = pm;
    W->val_a = va;
    W->val_b = vb;
    W->pos = pos;
    W->digit = dig;
    W->scratch = scr;
    W->scratch_bytes = sb;
    W->scomp = sc;
    W->snb = snb;
    W->ssoff = sso;
    W->cbeg = cb;
    W->cend = ce;
    W->nb_pair = nbp;
    W->soff_pair = sop;
    W->smass = sm;
    W->srem = sr;
  }
}

unsigned blocks_for_n(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + 255) / 256); }

}  // namespace
}  // namespace lsrvt

using namespace lsrvt;

extern "C" size_t lsrvt_seed_workspace(lsrvt_dims dims, uint32_t n_comp, int32_t block, uint32_t cap_pairs) {
  Geom g;
  if (make_geom(dims, g) != LSRVT_OK || block < 1 || block > kMaxBlockEdge || cap_pairs == 0) return 0;
  SeedGeom G = seed_geom(g, block);
  Sizer sz;
  seed_layout(sz, G, n_comp, cap_pairs, nullptr);
  return sz.off;
}

extern "C" int32_t lsrvt_seed(const uint32_t *d_comp, const uint32_t *d_comp_first, lsrvt_dims dims, uint32_t n_comp,
                              const uint16_t *d_weights,
                              const uint32_t *d_mass_lut, uint32_t rho, int32_t block, uint64_t seed,
                              uint32_t cap_pairs, uint32_t *d_sites, uint32_t cap_sites, uint32_t *h_n_sites,
                              uint32_t *h_n_pairs, void *d_work, size_t work_bytes, void *stream) {
  Geom g;
  int32_t rc = make_geom(dims, g);
  if (rc) return rc;
  if (!d_comp || !d_comp_first || rho == 0 || block < 1 || block > kMaxBlockEdge || cap_pairs == 0 || n_comp == 0 ||
      (cap_sites > 0 && !d_sites) || (d_mass_lut && !d_weights))
    return LSRVT_EINVAL;
  if (h_n_sites) *h_n_sites = 0;
  if (h_n_pairs) *h_n_pairs = 0;
  const SeedGeom G = seed_geom(g, block);
  const size_t need = lsrvt_seed_workspace(dims, n_comp, block, cap_pairs);
  if ((rc = check_work(d_work, work_bytes, need))) return rc;
  Carve cv(d_work, work_bytes);
  SeedWork W;
  seed_layout(cv, G, n_comp, cap_pairs, &W);
  if (!cv.ok) return LSRVT_EWORKSPACE;
  hipStream_t s = as_stream(stream);
  const MassIn mi{d_weights, d_mass_lut};
  const unsigned gb = (unsigned)std::min<int64_t>(G.nblocks, 65535);
  if ((rc = fill<uint32_t>(W.err, 2, 0u, s))) return rc;
  // pairs per block, block masses, total mass
  const bool usual = block == kMaxBlockEdge;
  hipLaunchKernelGGL((usual ? k_seed_blocks<0, kMaxBlockEdge> : k_seed_blocks<0, 0>), dim3(gb), dim3(kSeedThreads), 0, s,
                     d_comp, G, n_comp, mi, W.pcnt, W.bmass, nullptr, nullptr, nullptr, nullptr, W.err);
  hipLaunchKernelGGL(k_seed_total, dim3(1), dim3(kSeedThreads), 0, s, W.bmass, G.nblocks, W.total);
  LSRVT_LAUNCHED();
  if ((rc = ScanU32::run(W.pcnt, G.nblocks, W.poff, W.scratch, W.scratch_bytes, s))) return rc;
  uint32_t hdr[2] = {0, 0};
  LSRVT_HIP(hipMemcpyAsync(&hdr[0], W.poff + G.nblocks, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  LSRVT_HIP(hipMemcpyAsync(&hdr[1], W.err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  LSRVT_HIP(hipStreamSynchronize(s));
  if (hdr[1] & 1u) return LSRVT_EINVAL;
  const uint32_t P = hdr[0];
  if (h_n_pairs) *h_n_pairs = P;
  if (P > cap_pairs) return LSRVT_ECAPACITY;
  hipLaunchKernelGGL((usual ? k_seed_blocks<1, kMaxBlockEdge> : k_seed_blocks<1, 0>), dim3(gb), dim3(kSeedThreads), 0, s,
                     d_comp, G, n_comp, mi, W.pcnt, W.bmass, W.poff, W.pair_comp, W.pair_block, W.pair_mass, W.err);
  // stable radix sort of the pairs by component (block order is kept)
  hipLaunchKernelGGL(k_seed_iota, dim3(blocks_for_n(P)), dim3(256), 0, s, W.val_a, (int64_t)P);
  LSRVT_LAUNCHED();
  uint32_t *cur = W.val_a, *other = W.val_b;
  for (int p = 0; p < 4 && (p == 0 || (n_comp - 1) >> (8 * p)); ++p) {
    hipLaunchKernelGGL(k_seed_digit, dim3(blocks_for_n(P)), dim3(256), 0, s, cur, (int64_t)P, W.pair_comp, 8 * p,
                       W.digit);
    LSRVT_LAUNCHED();
    if ((rc = StableSort8::run(W.digit, P, W.pos, nullptr, W.scratch, W.scratch_bytes, s))) return rc;
    hipLaunchKernelGGL(k_seed_scatter, dim3(blocks_for_n(P)), dim3(256), 0, s, cur, W.pos, (int64_t)P, other);
    LSRVT_LAUNCHED();
    std::swap(cur, other);
  }
  if ((rc = fill<uint32_t>(W.cbeg, n_comp, 0u, s))) return rc;
  if ((rc = fill<uint32_t>(W.cend, n_comp, 0u, s))) return rc;
  hipLaunchKernelGGL(k_seed_sorted, dim3(blocks_for_n(P)), dim3(256), 0, s, cur, (int64_t)P, W.pair_comp,
                     W.pair_mass, W.scomp, W.smass, W.cbeg, W.cend);
  hipLaunchKernelGGL(k_seed_apportion, dim3(grid_for(n_comp, kSeedThreads / kWave, 65535)), dim3(kSeedThreads), 0,
                     s, n_comp, W.cbeg, W.cend, W.smass, W.total, g.n, rho, W.snb, W.pos, W.err + 1, W.err);
  // (the positions of the sort are not needed any more: their place takes the
  // list of at most P / kNarrow components)
  if (P > kNarrow)
    hipLaunchKernelGGL(k_seed_apportion_wide, dim3(std::min<uint32_t>(P / kNarrow, 256)), dim3(kWideThreads), 0, s,
                       W.cbeg, W.cend, W.smass, W.total, g.n, rho, W.srem, W.snb, W.pos, W.err + 1, W.err);
  LSRVT_LAUNCHED();
  if ((rc = ScanU32::run(W.snb, P, W.ssoff, W.scratch, W.scratch_bytes, s))) return rc;
  uint32_t S = 0;
  LSRVT_HIP(hipMemcpyAsync(&S, W.ssoff + P, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  LSRVT_HIP(hipMemcpyAsync(&hdr[1], W.err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  LSRVT_HIP(hipStreamSynchronize(s));
  if (hdr[1] & 1u) return LSRVT_EINVAL;
  if (hdr[1]) return LSRVT_ELIMIT;
  if (h_n_sites) *h_n_sites = S;
  if (S > cap_sites) return LSRVT_ECAPACITY;
  hipLaunchKernelGGL(k_seed_unsort, dim3(blocks_for_n(P)), dim3(256), 0, s, cur, (int64_t)P, W.snb, W.ssoff,
                     W.nb_pair, W.soff_pair);
  hipLaunchKernelGGL((usual ? k_seed_place<kMaxBlockEdge> : k_seed_place<0>), dim3(gb), dim3(kSeedThreads), 0, s, d_comp,
                     G, mi, W.poff, W.pair_comp, W.pair_mass, d_comp_first, W.nb_pair, W.soff_pair, (uint32_t)seed, (uint32_t)(seed >> 32),
                     d_sites, cap_sites);
  LSRVT_LAUNCHED();
  return LSRVT_OK;
}
