// Grouped scan order for X against X.
//
// The rows are partitioned by their nearest of G seed rows (the rows at
// positions floor(c n / G), squared distance in fp32, ties to the lower
// seed; G from order_groups) and laid out group by group, each group in input
// order (a stable counting sort).  The quantised copy, its norms and radii
// are written in that order; a tile workgroup starts its scan at the first
// row of the group holding its first query, so near references come first
// and the filter's thresholds tighten early.  The exact kNN set of every row
// does not depend on the order: the recheck maps positions back to input rows
// before it ranks and writes anything.
//
// Pruned scan.  On clustered rows most of the references cannot be among a
// query's nearest: the boxes of sub-tiles and stages bound the distance between a
// wave's queries and a stage from below, and the tile (mtile.h) skips what lies
// beyond the wave's worst list entry.  At 10^6 rows of 64 in ten clusters the tile's
// 16 launches take 50 ms instead of 165, at 10^5 of 32 in five 1.2 instead of 2.2.
// The order then makes the boxes small: rows of more than 16 elements by the nearest
// of kPivots pivots and the distance from it, shorter ones by a k-d tree.  Where the
// boxes rule too little out, the plain scan runs (kFlatShare, kPruneWorth).
#include "tod_internal.h"

namespace tod {

namespace {

constexpr int kAssignThreads = 256;
constexpr int kSmallD = 16;       // rows this short keep the row in registers
constexpr int kWideGroups = 16;   // seed groups for longer rows

// The G seed rows of short rows, zero-padded to DT columns, gathered once.
__global__ void __launch_bounds__(256)
seeds_kernel(const float* __restrict__ x, int64_t n, int d, int G, int DT,
             float* __restrict__ seeds) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G * DT) return;
  const int c = i / DT, t = i - c * DT;
  const int64_t srow = (int64_t)c * n / G;
  seeds[i] = t < d ? x[srow * d + t] : 0.0f;
}

// Rows of at most kSmallD elements: lab[row] = nearest of G seeds (the row in
// registers, zero-padded to DT = d rounded up to 4 columns; every lane reads
// the same seed, so the seeds come through the scalar cache as wave-uniform
// loads).
template <int DT>
__global__ void __launch_bounds__(kAssignThreads)
assign_small_kernel(const float* __restrict__ x, int64_t n, int d, int G,
                    const float4* __restrict__ gseeds, int32_t* __restrict__ lab) {
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n) return;
  float v[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) v[t] = t < d ? x[row * d + t] : 0.0f;
  float best_d = INFINITY;
  int best = 0;
  // (Unrolled so that the scalar loads of several seeds are in flight at once.)
#pragma unroll 8
  for (int c = 0; c < G; ++c) {
    float acc = 0.0f;
#pragma unroll
    for (int q = 0; q < DT / 4; ++q) {
      const float4 s4 = gseeds[c * (DT / 4) + q];
      const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float df = v[4 * q + t] - sv[t];
        acc = fmaf(df, df, acc);
      }
    }
    if (acc < best_d) {
      best_d = acc;
      best = c;
    }
  }
  lab[row] = best;
}

// Longer rows, kWideGroups seeds: lab[row] = nearest seed (one thread per
// row; the seeds sit in LDS).
__global__ void __launch_bounds__(kAssignThreads)
assign_kernel(const float* __restrict__ x, int64_t n, int d, int32_t* __restrict__ lab) {
  extern __shared__ float seeds[];  // [kWideGroups][d]
  for (int i = threadIdx.x; i < kWideGroups * d; i += blockDim.x) {
    const int c = i / d, t = i - c * d;
    const int64_t srow = (int64_t)c * n / kWideGroups;
    seeds[i] = x[srow * d + t];
  }
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n) return;
  float acc[kWideGroups];
#pragma unroll
  for (int c = 0; c < kWideGroups; ++c) acc[c] = 0.0f;
  const float* in = x + row * d;
  for (int t = 0; t < d; ++t) {
    const float v = in[t];
#pragma unroll
    for (int c = 0; c < kWideGroups; ++c) {
      const float df = v - seeds[c * d + t];
      acc[c] = fmaf(df, df, acc[c]);
    }
  }
  int best = 0;
#pragma unroll
  for (int c = 1; c < kWideGroups; ++c) best = acc[c] < acc[best] ? c : best;
  lab[row] = best;
}

// An input element as the quantisation sees it: centred and scaled in fp64, |w| <
// 2^E, then rounded to fp32 (by at most 2^(E-25)).  Differences of such values
// neither overflow nor turn into NaN, whatever the magnitude of finite rows (the
// scale alone can exceed fp32's range, and so can a difference of two rows).
__device__ __forceinline__ float scaled_elem(float x, float mu, double s) {
  return (float)(s * ((double)x - (double)mu));
}

// The pivots: kPivots of up to kSeedSamples evenly spaced rows (as many as fit
// in LDS), the first one given, each next one drawn with probability
// proportional to its squared distance from the nearest pivot so far
// (k-means++ seeding, with a fixed low-discrepancy sequence in place of random
// numbers).  Rows at random would leave some of ten clusters without a pivot in
// four runs of five, and stages of two such clusters can hardly be told apart:
// at 10^6 rows of 64 the tile took 65 to 85 ms from seed to seed, against 47.
// One workgroup, bound by its kPivots dependent rounds over the samples in LDS
// (16-byte reads: 59 us at 75,000 rows of 128, 84 with 4-byte ones; 37 at rows
// of 32).
//
// Rows that the pivots cannot tell apart are recognised here, before the rest of
// the preparation is paid: of the pairs of up to kFlatQueries samples (no pivots
// themselves) with all samples, the share that no pivot's distances separate by
// more than twice the first one's distance to its nearest pivot, the plan's
// estimate of a neighbour's distance.  Boxes hold whole stages, so they rule out
// no more than that: on Gaussian and uniform rows of 17 to 256 elements the share
// was 0.85 and more (boxes: 0.998 and more), on ten or five clusters 0.09 to 0.22
// (0.14 to 0.38), on a curved sheet 0.16 to 0.22 (0.45 to 0.54).  From kFlatShare
// on the call keeps to the plain scan over evenly spaced seeds, input order within
// their groups: pivots and distance bins made that 3 to 15 % slower there (their
// order puts the outliers into tiles of their own, and a group's rows in the order
// of their distance, not at random, fill the lists more often).  In several splits
// it scans the rows in input order, whose splits are all alike (100,000 normal rows
// of 32 in blocks of 8,192 took 1.2 times as long in eight pieces of the groups).
constexpr int kFlatQueries = 32;
constexpr float kFlatShare = 0.75f;
constexpr int kSeedSamples = 512;
constexpr int kSeedThreads = 1024;
constexpr int kSeedFloats = 36 * 1024;  // LDS for the samples

// Floats from one sample to the next: whole 16-byte chunks, zero-padded, and one
// more to spread the samples over the banks.
__host__ __device__ constexpr int seed_stride(int d) { return (d + 3) / 4 * 4 + 4; }

int seed_samples(int64_t n, int d) {
  int64_t m = kSeedFloats / seed_stride(d);
  m = m < kSeedSamples ? m : kSeedSamples;
  return (int)(m < n ? m : n);
}

__global__ void __launch_bounds__(kSeedThreads)
pivot_seed_kernel(const float* __restrict__ x, int64_t n, int d, int m, int tps,
                  const float* __restrict__ mu32, Ctrl* __restrict__ ctrl, int scale_exp,
                  int flat_as, float* __restrict__ dist, int32_t* __restrict__ srow) {
  extern __shared__ __align__(16) float smp[];  // [m][stride], centred and scaled
  __shared__ float wsum[kSeedThreads / 64];
  __shared__ int32_t rows[kSeedSamples], piv[kPivots];
  __shared__ int pick, cnt[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double sc = scale_from_maxabs(ctrl->maxabs_bits, scale_exp);
  // (One 64-bit division per sample, and eight elements' loads at once.)
  if (tid < m) rows[tid] = (int32_t)((int64_t)tid * n / m);
  __syncthreads();
  const int stride = seed_stride(d), dp = stride - 4;
  constexpr int kLoads = 8;
  for (int e0 = tid; e0 < m * dp; e0 += kLoads * kSeedThreads) {
    float v[kLoads], mu[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = e0 + u * kSeedThreads < m * dp ? e0 + u * kSeedThreads : e0;
      const int i = e / dp, t = e - i * dp < d ? e - i * dp : d - 1;
      v[u] = x[(int64_t)rows[i] * d + t];
      mu[u] = mu32[t];
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = e0 + u * kSeedThreads;
      const int i = e / dp, t = e - i * dp;
      if (i < m) smp[i * stride + t] = t < d ? scaled_elem(v[u], mu[u], sc) : 0.0f;
    }
  }
  if (tid == 0) {
    pick = m - 1;
    cnt[0] = cnt[1] = 0;
  }
  __syncthreads();
  const int i = tid / tps, sub = tid & (tps - 1);  // sample, one of its tps threads
  const float4* const smp4 = reinterpret_cast<const float4*>(smp);
  const float4* in = smp4 + (i < m ? i : 0) * (stride / 4);
  float near = INFINITY;
  int p = 0;
  for (int c = 0; c < kPivots; ++c) {
    if (tid == 0) piv[c] = rows[p];
    const float4* pv = smp4 + p * (stride / 4);
    float acc = 0.0f;
#pragma unroll 4
    for (int t = sub; t < dp / 4; t += tps) {
      const float4 a = in[t], b = pv[t];
      const float d0 = a.x - b.x, d1 = a.y - b.y, d2 = a.z - b.z, d3 = a.w - b.w;
      acc = fmaf(d0, d0, fmaf(d1, d1, fmaf(d2, d2, fmaf(d3, d3, acc))));
    }
    for (int off = 1; off < tps; off <<= 1) acc += __shfl_xor(acc, off, 64);
    near = fminf(near, acc);
    if (flat_as && i < m && sub == 0) dist[(int64_t)i * kPivots + c] = sqrtf(acc);
    // Inclusive sums of the weights in sample order.
    float incl = i < m && sub == 0 ? near : 0.0f;
    for (int off = 1; off < 64; off <<= 1) {
      const float o = __shfl_up(incl, off, 64);
      if (lane >= off) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    float before = 0.0f, total = 0.0f;
#pragma unroll
    for (int w = 0; w < kSeedThreads / 64; ++w) {
      before += w < wave ? wsum[w] : 0.0f;
      total += wsum[w];
    }
    const float u = (float)(c + 1) * 0.61803399f;
    // (One atomic a wave: its first sample at or past the mark.)
    const uint64_t at = __ballot(i < m && before + incl >= (u - floorf(u)) * total);
    if (at && lane == __builtin_ctzll(at)) atomicMin(&pick, i);
    __syncthreads();
    p = pick;
    __syncthreads();  // every thread has read pick before it is reset
    if (tid == 0) pick = m - 1;
  }
  if (!flat_as) {  // uniform
    if (tid < kPivots) srow[tid] = piv[tid];
    return;
  }
  // The samples' distances (each thread reads what it wrote) take the samples'
  // place in LDS: [m][kPivots], then each sample's distance to its nearest pivot.
  float* const near_of = smp + m * kPivots;
  if (i < m && sub == 0) {
    for (int c = 0; c < kPivots; ++c) smp[i * kPivots + c] = dist[(int64_t)i * kPivots + c];
    near_of[i] = sqrtf(near);
  }
  __syncthreads();
  const int j = tid % m, nq = m < kFlatQueries ? m : kFlatQueries;
  float dj[kPivots];
#pragma unroll
  for (int c = 0; c < kPivots; ++c) dj[c] = smp[j * kPivots + c];
  int seen = 0, live = 0;
  for (int q = tid / m; tid < kSeedThreads / m * m && q < nq; q += kSeedThreads / m) {
    const int s = q * m / nq;
    float lb = 0.0f;
#pragma unroll
    for (int c = 0; c < kPivots; c += 4) {
      const float4 dq = smp4[(s * kPivots + c) / 4];
      lb = fmaxf(fmaxf(lb, fabsf(dq.x - dj[c])), fabsf(dq.y - dj[c + 1]));
      lb = fmaxf(fmaxf(lb, fabsf(dq.z - dj[c + 2])), fabsf(dq.w - dj[c + 3]));
    }
    if (near_of[s] > 0.0f) {
      ++seen;
      live += lb > 2.0f * near_of[s] ? 0 : 1;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    seen += __shfl_xor(seen, off, 64);
    live += __shfl_xor(live, off, 64);
  }
  if (lane == 0) {
    atomicAdd(&cnt[0], seen);
    atomicAdd(&cnt[1], live);
  }
  __syncthreads();
  const bool flat = cnt[0] > 0 && (float)cnt[1] >= kFlatShare * (float)cnt[0];
  if (tid < kPivots) srow[tid] = flat ? (int32_t)((int64_t)tid * n / kPivots) : piv[tid];
  if (tid == 0) ctrl->flat = flat ? (uint32_t)flat_as : 0u;
}

// Longer rows with the pruned scan: groups by the nearest pivot.  Per row the
// distances to the pivots, in the quantisation's units (scaled_elem), go to
// pdist, and lab = 64 c + bin of the nearest pivot c, bin by half octaves of the
// squared distance: the rows of a group are laid out by their distance from its
// pivot, so that rows far from every pivot (outliers, clusters without one) do
// not widen the boxes of the group's bulk.  Rows the pivots cannot tell apart
// (ctrl->flat): srow holds evenly spaced rows, and a group is one bin.
__global__ void __launch_bounds__(kAssignThreads)
assign_pivot_kernel(const float* __restrict__ x, int64_t n, int d,
                    const float* __restrict__ mu32, const Ctrl* __restrict__ ctrl, int scale_exp,
                    const int32_t* __restrict__ srow, float* __restrict__ pdist,
                    int32_t* __restrict__ lab) {
  extern __shared__ float seeds[];  // [kPivots][d], centred and scaled
  const double sc = scale_from_maxabs(ctrl->maxabs_bits, scale_exp);
  for (int i = threadIdx.x; i < kPivots * d; i += blockDim.x) {
    const int c = i / d, t = i - c * d;
    seeds[i] = scaled_elem(x[(int64_t)srow[c] * d + t], mu32[t], sc);
  }
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n) return;
  if (ctrl->flat == 2) {  // input order
    lab[row] = 0;
    return;
  }
  float acc[kPivots];
#pragma unroll
  for (int c = 0; c < kPivots; ++c) acc[c] = 0.0f;
  const float* in = x + row * d;
  for (int t = 0; t < d; ++t) {
    const float v = scaled_elem(in[t], mu32[t], sc);
#pragma unroll
    for (int c = 0; c < kPivots; ++c) {
      const float df = v - seeds[c * d + t];
      acc[c] = fmaf(df, df, acc[c]);
    }
  }
  int best = 0;
  float bd = acc[0];
#pragma unroll
  for (int c = 1; c < kPivots; ++c) {
    best = acc[c] < bd ? c : best;
    bd = acc[c] < bd ? acc[c] : bd;
  }
  // The difference is below 2^(E+1) in every column: D^2 < 4 d 4^E.
  const int top = (int)(__float_as_uint(ldexpf((float)d, 2 * scale_exp + 2)) >> 22);
  int bin = (int)(__float_as_uint(bd) >> 22) - top + (kRadBins - 1);
  bin = bin < 0 ? 0 : (bin > kRadBins - 1 ? kRadBins - 1 : bin);
  const bool flat = ctrl->flat != 0;
  lab[row] = best * kRadBins + (flat ? 0 : bin);
  if (flat) return;
  float4* out = reinterpret_cast<float4*>(pdist + row * kPivots);
#pragma unroll
  for (int c = 0; c < kPivots / 4; ++c)
    out[c] = make_float4(sqrtf(acc[4 * c]), sqrtf(acc[4 * c + 1]), sqrtf(acc[4 * c + 2]),
                         sqrtf(acc[4 * c + 3]));
}

// ---------------------------------------------------------------------------
// k-d order (rows of at most 16 elements with the pruned scan).  A tree of
// medians over a sample gives up to 1024 leaves, which the counting sort lays
// out in tree order; then every chunk of 1024 or 4096 positions is split on its own
// rows' medians down to 32, so that sub-tiles, stages and chunks of stages are
// compact boxes.  Each split takes the dimension of the largest variance.
// ---------------------------------------------------------------------------
constexpr int kKdThreads = 1024;
constexpr int kKdSamples = 4;      // sample rows per leaf
constexpr int kKdChunkMost = 4096;  // rows of the local splits (fewer: 1024, see kd_chunk)
constexpr int kKdLook = 64;        // rows of a node its variances are taken from

// Order-preserving bits of a float.
__device__ __forceinline__ uint32_t ord_bits(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Lanes t + 16 g: variance of dimension t over the values of the lanes' rows,
// given as each lane's count, sum and sum of squares; returns the dimension of
// the largest one (ties to the lower one), the same in every lane.
__device__ __forceinline__ int widest(float c, float s, float q, int d, int lane) {
  for (int off = 16; off < 64; off <<= 1) {
    c += __shfl_xor(c, off, 64);
    s += __shfl_xor(s, off, 64);
    q += __shfl_xor(q, off, 64);
  }
  int best = lane & 15;
  float v = best < d && c > 0.0f ? q - s * s / c : -1.0f;
  for (int off = 1; off < 16; off <<= 1) {
    const float o = __shfl_xor(v, off, 64);
    const int b = __shfl_xor(best, off, 64);
    if (o > v || (o == v && b < best)) {
      v = o;
      best = b;
    }
  }
  return __shfl(best < d ? best : 0, 0, 64);
}

// Bitonic sort of segments of 2^lseg entries.  (A pass whose pairs lie within
// the 128 entries one wave handles needs no workgroup barrier.)
template <typename K>
__device__ __forceinline__ void bitonic_segments(K* key, int n, int lseg) {
  for (int lsize = 1; lsize <= lseg; ++lsize)
    for (int ls = lsize - 1; ls >= 0; --ls) {
      for (int e = threadIdx.x; e < n / 2; e += kKdThreads) {
        const int lo = ((e >> ls) << (ls + 1)) | (e & ((1 << ls) - 1)), hi = lo + (1 << ls);
        const bool asc = lsize == lseg || ((lo >> lsize) & 1) == 0;
        const K a = key[lo], b = key[hi];
        if ((b < a) == asc && a != b) {
          key[lo] = b;
          key[hi] = a;
        }
      }
      // Strides up to 64 stay within a wave's 128 consecutive entries; the next
      // pass's stride is smaller, or (at ls = 0) as large as the segments grow.
      const int next = ls > 0 ? ls - 1 : lsize;
      if (ls > 6 || next > 6) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      }
    }
  __syncthreads();
}

// The tree over m = kKdSamples 2^levels evenly spaced rows: node h (1 = root)
// splits at tree[h] = (dimension, value); rows with a value >= it go right.
// One workgroup; the keys (value, sample) of a node's samples are a segment.
__global__ void __launch_bounds__(kKdThreads)
kd_build_kernel(const float* __restrict__ x, int64_t n, int d, int m, int levels,
                int2* __restrict__ tree) {
  extern __shared__ uint64_t skey[];  // [m]
  __shared__ int sdim[kOrdMaxC / 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto row_of = [&](uint64_t k) { return (int64_t)(uint32_t)k * n / m; };
  for (int i = tid; i < m; i += kKdThreads) skey[i] = (uint64_t)i;
  __syncthreads();
  for (int l = 0; l < levels; ++l) {
    const int seg = m >> l, nodes = 1 << l;
    const int look = seg < kKdLook ? seg : kKdLook, step = seg / look;
    for (int nd = wave; nd < nodes; nd += kKdThreads / 64) {
      const int t = lane & 15;
      float c = 0.0f, s = 0.0f, q = 0.0f;
      if (t < d) {
        const float r0 = x[row_of(skey[nd * seg]) * d + t];
        for (int i = lane >> 4; i < look; i += 4) {
          const float v = x[row_of(skey[nd * seg + i * step]) * d + t] - r0;
          c += 1.0f;
          s += v;
          q = fmaf(v, v, q);
        }
      }
      const int w = widest(c, s, q, d, lane);
      if (lane == 0) sdim[nd] = w;
    }
    __syncthreads();
    for (int i = tid; i < m; i += kKdThreads) {
      const uint64_t k = skey[i];
      skey[i] = ((uint64_t)ord_bits(x[row_of(k) * d + sdim[i >> __builtin_ctz(seg)]]) << 32) |
                (uint32_t)k;
    }
    __syncthreads();
    bitonic_segments(skey, m, __builtin_ctz(seg));
    for (int nd = tid; nd < nodes; nd += kKdThreads)
      tree[nodes + nd] = make_int2(
          sdim[nd],
          __float_as_int(x[row_of(skey[nd * seg + seg / 2]) * d + sdim[nd]]));
    __syncthreads();
  }
}

// lab[row] = leaf of the row.
__global__ void __launch_bounds__(kAssignThreads)
assign_kd_kernel(const float* __restrict__ x, int64_t n, int d, int levels,
                 const int2* __restrict__ tree, int32_t* __restrict__ lab) {
  __shared__ int2 st[kOrdMaxC];
  for (int i = threadIdx.x + 1; i < (1 << levels); i += kAssignThreads) st[i] = tree[i];
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n) return;
  const float* in = x + row * d;
  int h = 1;
  for (int l = 0; l < levels; ++l) {
    const int2 nd = st[h];
    h = 2 * h + (in[nd.x] >= __int_as_float(nd.y) ? 1 : 0);
  }
  lab[row] = h - (1 << levels);
}

// Local splits: one workgroup per chunk of kKdChunk positions, down to 32 rows.
// The rows' values sit in LDS as fp16 (centred and scaled as for the quantisation;
// only the order matters), a key is (far flag, value, local row).  Rows more than
// kKdFar times the chunk's mean squared distance from its mean are flagged and end
// up last in the chunk, so that a few far rows widen the boxes of the last sub-tiles
// only.
constexpr float kKdFar = 5.0f;

template <int kKdChunk>
__global__ void __launch_bounds__(kKdThreads)
kd_local_kernel(const float* __restrict__ x, int64_t n, int d, const float* __restrict__ mu32,
                const Ctrl* __restrict__ ctrl, int scale_exp, int32_t* __restrict__ perm) {
  extern __shared__ uint32_t lkey[];  // [kKdChunk], then the values [d][kKdChunk]
  _Float16* const val = reinterpret_cast<_Float16*>(lkey + kKdChunk);
  __shared__ int sdim[kKdChunk / 64];
  __shared__ float smean[16], red[kKdThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kKdChunk;
  const int rows = n - base < kKdChunk ? (int)(n - base) : kKdChunk;
  const double sc = scale_from_maxabs(ctrl->maxabs_bits, scale_exp);
  constexpr int kPer = kKdChunk / kKdThreads;
  int32_t mine[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid + e * kKdThreads;
    mine[e] = i < rows ? perm[base + i] : 0;
    for (int t = 0; t < d; ++t)
      val[t * kKdChunk + i] =
          i < rows ? (_Float16)scaled_elem(x[(int64_t)mine[e] * d + t], mu32[t], sc)
                   : (_Float16)0.0f;
  }
  __syncthreads();
  if (wave < d) {
    float s = 0.0f;
    for (int i = lane; i < rows; i += 64) s += (float)val[wave * kKdChunk + i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) smean[wave] = s / (float)rows;
  }
  __syncthreads();
  float dist[kPer], tot = 0.0f;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid + e * kKdThreads;
    dist[e] = 0.0f;
    for (int t = 0; t < d; ++t) {
      const float df = (float)val[t * kKdChunk + i] - smean[t];
      dist[e] = fmaf(df, df, dist[e]);
    }
    tot += i < rows ? dist[e] : 0.0f;
  }
  for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
  if (lane == 0) red[wave] = tot;
  __syncthreads();
  tot = 0.0f;
  for (int w = 0; w < kKdThreads / 64; ++w) tot += red[w];
  constexpr uint32_t kFar = 1u << 28, kNone = 1u << 29;  // flags above value << 12 | row
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid + e * kKdThreads;
    lkey[i] = (uint32_t)i | (i >= rows ? kNone : dist[e] * (float)rows > kKdFar * tot ? kFar : 0u);
  }
  __syncthreads();
  for (int seg = kKdChunk; seg > 32; seg >>= 1) {
    const int lseg = __builtin_ctz(seg), nodes = kKdChunk >> lseg;
    constexpr int look = kKdLook;
    const int step = seg >> 6;  // seg / look
    for (int nd = wave; nd < nodes; nd += kKdThreads / 64) {
      const int t = lane & 15;
      float c = 0.0f, s = 0.0f, q = 0.0f;
      if (t < d)
        for (int i = lane >> 4; i < look; i += 4) {
          const uint32_t k = lkey[nd * seg + i * step];
          if (k >= kFar) continue;
          const float v = ((float)val[t * kKdChunk + (k & (kKdChunk - 1))] - smean[t]) * 0x1p-14f;
          c += 1.0f;
          s += v;
          q = fmaf(v, v, q);
        }
      const int w = widest(c, s, q, d, lane);
      if (lane == 0) sdim[nd] = w;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int i = tid + e * kKdThreads;
      const uint32_t k = lkey[i], r = k & (kKdChunk - 1);
      const uint16_t hb = __builtin_bit_cast(uint16_t, val[sdim[i >> lseg] * kKdChunk + r]);
      const uint32_t code = (uint16_t)((hb & 0x8000u) ? ~hb : (hb | 0x8000u));
      lkey[i] = (k & (kFar | kNone)) | (code << 12) | r;
    }
    __syncthreads();
    bitonic_segments(lkey, kKdChunk, lseg);
  }
  // (Every row of the chunk is in a register: they change places through LDS.)
  int32_t* const out = reinterpret_cast<int32_t*>(val);
#pragma unroll
  for (int e = 0; e < kPer; ++e) out[tid + e * kKdThreads] = mine[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid + e * kKdThreads;
    if (i < rows) perm[base + i] = out[lkey[i] & (kKdChunk - 1)];
  }
}

// Rows per group in each block of kOrdRows rows.
__global__ void __launch_bounds__(256)
count_kernel(const int32_t* __restrict__ lab, int64_t n, int G, int32_t* __restrict__ bcnt) {
  __shared__ int32_t cnt[kOrdMaxC];
  for (int c = threadIdx.x; c < G; c += blockDim.x) cnt[c] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * kOrdRows;
  const int64_t r1 = r0 + kOrdRows < n ? r0 + kOrdRows : n;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += blockDim.x) atomicAdd(&cnt[lab[r]], 1);
  __syncthreads();
  for (int c = threadIdx.x; c < G; c += blockDim.x) bcnt[(int64_t)blockIdx.x * G + c] = cnt[c];
}

// Inclusive prefix sum over the wave.
__device__ __forceinline__ int32_t wave_incl_sum(int32_t v, int lane) {
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}

// Each block's first position within its group: one wave per group walks
// the blocks' counts 64 at a time (exclusive prefix sums), and leaves the
// group's total in cstart[c + 1].
__global__ void __launch_bounds__(256)
block_offsets_kernel(const int32_t* __restrict__ bcnt, int nb, int G,
                     int32_t* __restrict__ boff, int32_t* __restrict__ cstart) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= G) return;  // uniform per wave
  int32_t at = 0;
  for (int b0 = 0; b0 < nb; b0 += 64) {
    const int b = b0 + lane;
    const int32_t v = b < nb ? bcnt[(int64_t)b * G + c] : 0;
    const int32_t incl = wave_incl_sum(v, lane);
    if (b < nb) boff[(int64_t)b * G + c] = at + incl - v;
    at += __shfl(incl, 63, 64);
  }
  if (lane == 0) cstart[c + 1] = at;
}

// Group starts: cstart[0..G] becomes the exclusive prefix sums of the group
// totals (one workgroup, 64 groups per step).
__global__ void __launch_bounds__(64)
group_starts_kernel(int G, int32_t* __restrict__ cstart) {
  const int lane = threadIdx.x;
  int32_t at = 0;
  for (int c0 = 0; c0 < G; c0 += 64) {
    const int c = c0 + lane;
    const int32_t v = c < G ? cstart[c + 1] : 0;
    const int32_t incl = wave_incl_sum(v, lane);
    if (c < G) cstart[c + 1] = at + incl;
    at += __shfl(incl, 63, 64);
  }
  if (lane == 0) cstart[0] = 0;
}

// Key starts of the pivot order: one wave per seed group, lane = distance bin.
// Bins more than four half octaves above the group's median bin (rows more
// than twice as far from the seed as the median row) form the group's far
// class.  Layout: the near classes group by group, then the far classes; within
// a class by bin.  start[key] replaces the key's total; kstart[key] is the
// start of the key's class.
__global__ void __launch_bounds__(kPivots * kRadBins)
pivot_starts_kernel(int32_t* __restrict__ start, int32_t* __restrict__ kstart) {
  __shared__ int32_t tot[2][kPivots];
  const int g = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int32_t v = start[threadIdx.x + 1];
  __syncthreads();  // every total is read before a start overwrites it
  const int32_t incl = wave_incl_sum(v, lane);
  const int32_t all = __shfl(incl, 63, 64);
  const uint64_t past = __ballot(2 * (int64_t)incl >= all);
  const int cut = __builtin_ctzll(past) + 4;  // lane 63's sum is `all`: past is never 0
  const int32_t near = __shfl(incl, cut < 63 ? cut : 63, 64);
  if (lane == 0) {
    tot[0][g] = near;
    tot[1][g] = all - near;
  }
  __syncthreads();
  int32_t at = 0;
  const bool far = lane > cut;
  for (int i = 0; i < kPivots; ++i) at += (far || i < g) ? tot[0][i] : 0;
  if (far)
    for (int i = 0; i < g; ++i) at += tot[1][i];
  kstart[threadIdx.x] = at;
  start[threadIdx.x] = at + incl - v - (far ? near : 0);
}

// perm[position] = row, stable within each group: one wave per block walks
// its rows 64 at a time; each lane counts the lanes of the same group below
// it (its rank) and in all (the group's count in these 64 rows), writes its
// row at the group's next position plus its rank, and the group's first lane
// advances the group's next position.  (A group's next position starts at
// the group's start plus the block's offset within the group.)
__global__ void __launch_bounds__(64)
scatter_kernel(const int32_t* __restrict__ lab, int64_t n, int G, int bits,
               const int32_t* __restrict__ boff, const int32_t* __restrict__ cstart,
               int32_t* __restrict__ perm) {
  __shared__ int32_t next[kOrdMaxC];
  const int lane = threadIdx.x;
  for (int c = lane; c < G; c += 64) next[c] = cstart[c] + boff[(int64_t)blockIdx.x * G + c];
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * kOrdRows;
  const int64_t r1 = r0 + kOrdRows < n ? r0 + kOrdRows : n;
  for (int64_t r = r0; r < r1; r += 64) {
    const int64_t row = r + lane;
    const int l = row < r1 ? lab[row] : -1;
    // Lanes of the same group: one ballot per bit of the group number.
    uint64_t same = __ballot(l >= 0);
    for (int b = 0; b < bits; ++b) {
      const uint64_t m = __ballot((l >> b) & 1);
      same &= ((l >> b) & 1) ? m : ~m;
    }
    const int cnt = __popcll(same);
    const int rank = __popcll(same & ((1ull << lane) - 1));
    if (l >= 0) perm[next[l] + rank] = (int32_t)row;
    __syncthreads();  // every lane has read next[] before it moves
    if (l >= 0 && rank == 0) next[l] += cnt;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Boxes and the work plan of the pruned scan.
// ---------------------------------------------------------------------------
constexpr int kSubsPerBlock = 16;

// Pivot boxes of the 32-row sub-tiles: one thread per (sub-tile, pivot).  The
// quantised rows' distances differ from the rows' own by at most the two
// radii (<= 2 P): every box is widened by P.  eps covers the fp32 rounding of
// the distances' arithmetic, `wide` that of the elements (scaled_elem: each row
// of a pair is off by at most sqrt(d) 2^(E-25)) and differences below the
// smallest normal number.  A box with a value that is not finite bounds nothing
// (finite rows have none).
__global__ void __launch_bounds__(kSubsPerBlock * kBoxDim)
pivot_box_kernel(const float* __restrict__ pdist, const int32_t* __restrict__ perm,
                 const int32_t* __restrict__ lab, const int32_t* __restrict__ kstart, int64_t n,
                 int64_t subs, float eps, float wide, const Ctrl* __restrict__ ctrl,
                 float* __restrict__ box32, int32_t* __restrict__ substart) {
  const int t = threadIdx.x & (kBoxDim - 1);
  const int64_t sub = (int64_t)blockIdx.x * kSubsPerBlock + (threadIdx.x / kBoxDim);
  if (sub >= subs) return;
  const int64_t r0 = 32 * sub;
  if (t == 0) substart[sub] = kstart[lab[perm[r0]]];
  if (ctrl->flat) return;  // (no distances; no box is read)
  const int rows = n - r0 < 32 ? (int)(n - r0) : 32;
  float lo = INFINITY, hi = 0.0f;
  bool bounded = true;
#pragma unroll 8
  for (int i = 0; i < rows; ++i) {
    const float v = pdist[(int64_t)perm[r0 + i] * kPivots + t];
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
    bounded = bounded && v < INFINITY;
  }
  const double pmax = __longlong_as_double((long long)ctrl->pmax_bits);
  const float w = (float)(pmax * (1.0 + 0x1p-20)) + wide;
  box32[sub * (2 * kBoxDim) + t] = bounded ? lo * (1.0f - eps) - w : -INFINITY;
  box32[sub * (2 * kBoxDim) + kBoxDim + t] = bounded ? hi * (1.0f + eps) + w : INFINITY;
}

// Boxes of the quantised columns of the 32-row sub-tiles (exact values).
template <typename T>
__global__ void __launch_bounds__(kSubsPerBlock * kBoxDim)
column_box_kernel(const T* __restrict__ xq, int64_t n, int64_t subs, int d, int dpad,
                  float* __restrict__ box32, int32_t* __restrict__ substart) {
  const int t = threadIdx.x & (kBoxDim - 1);
  const int64_t sub = (int64_t)blockIdx.x * kSubsPerBlock + (threadIdx.x / kBoxDim);
  if (sub >= subs) return;
  const int64_t r0 = 32 * sub;
  const int rows = n - r0 < 32 ? (int)(n - r0) : 32;
  float lo = 0.0f, hi = 0.0f;
  if (t < d) {
    lo = hi = (float)xq[r0 * dpad + t];
#pragma unroll 8
    for (int i = 1; i < rows; ++i) {
      const float v = (float)xq[(r0 + i) * dpad + t];
      lo = fminf(lo, v);
      hi = fmaxf(hi, v);
    }
  }
  box32[sub * (2 * kBoxDim) + t] = lo;
  box32[sub * (2 * kBoxDim) + kBoxDim + t] = hi;
  if (t == 0) substart[sub] = (int32_t)r0;
}

// Boxes of the stages (nsub sub-tiles each) from those of their sub-tiles, and
// of chunks of stages from those of the stages.
__global__ void __launch_bounds__(256)
stage_box_kernel(const float* __restrict__ box32, int64_t subs, int64_t stages, int nsub,
                 const Ctrl* __restrict__ ctrl, float* __restrict__ sbox) {
  if (ctrl->flat) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t st = i / (2 * kBoxDim);
  const int t = (int)(i % (2 * kBoxDim));
  if (st >= stages) return;
  const int64_t s0 = st * nsub, s1 = s0 + nsub < subs ? s0 + nsub : subs;
  float v = box32[s0 * (2 * kBoxDim) + t];
#pragma unroll 8
  for (int64_t s = s0 + 1; s < s1; ++s) {
    const float o = box32[s * (2 * kBoxDim) + t];
    v = t < kBoxDim ? fminf(v, o) : fmaxf(v, o);
  }
  sbox[i] = v;
}

// Work estimate of every query tile: the stages its box cannot rule out at an
// estimated distance of the K'-th neighbour.  Pivots: the rows of a sub-tile
// lie within twice its smallest pivot distance of each other; a sub-tile far
// above both its neighbours (one that holds rows of two clusters) counts as the
// larger of them, then the largest of the tile counts.  One wave per tile; at most
// kPlanSamples stages are tested, evenly spaced.  The estimate only balances the
// pieces (at 10^5 rows of 32 and 10^6 of 64 it is within 1% of the stages scanned).
constexpr int kPlanSamples = 2048;

__global__ void __launch_bounds__(256)
plan_estimate_kernel(const float* __restrict__ box32, const float* __restrict__ sbox,
                     int64_t stages, int64_t sub0, int64_t nsubs, int subs_per_tile,
                     int64_t tiles, int prune, const Ctrl* __restrict__ ctrl,
                     int32_t* __restrict__ rec) {
  if (ctrl->flat) return;
  const int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (t >= tiles) return;  // uniform per wave
  const int64_t s0 = t * subs_per_tile;
  const int64_t s1 = s0 + subs_per_tile < nsubs ? s0 + subs_per_tile : nsubs;
  // Lane t < 32 holds entry t of the tile's box (lo, then hi).
  const int e = lane & (2 * kBoxDim - 1);
  float v = e < kBoxDim ? INFINITY : -INFINITY;
  // (near: the sub-tile's smallest upper end; two sub-tiles trail.)
  float near = 0.0f, n1 = INFINITY, n2 = INFINITY;
  for (int64_t s = s0 - 2; s <= s1; ++s) {
    float o = INFINITY;
    if (s >= 0 && s < nsubs) {
      o = box32[(sub0 + s) * (2 * kBoxDim) + e];
      if (s >= s0 && s < s1) v = e < kBoxDim ? fminf(v, o) : fmaxf(v, o);
    }
    if (prune != kPrunePivot) continue;
    o = e < kBoxDim ? INFINITY : o;
    for (int off = 32; off > 0; off >>= 1) o = fminf(o, __shfl_xor(o, off, 64));
    // (Off the ends of the rows the neighbour's place is empty: it counts as 0.)
    const float a = n2 < INFINITY ? n2 : 0.0f, b = o < INFINITY ? o : 0.0f;
    if (s > s0) near = fmaxf(near, fminf(n1, fmaxf(a, b)));
    n2 = n1;
    n1 = o;
  }
  float lo[kBoxDim], hi[kBoxDim];
#pragma unroll
  for (int i = 0; i < kBoxDim; ++i) {
    lo[i] = __shfl(v, i, 64);
    hi[i] = __shfl(v, kBoxDim + i, 64);
  }
  float lim;  // squared
  if (prune == kPrunePivot) {
    lim = 2.0f * near;
    lim *= lim;
  } else {
    lim = 0.0f;
#pragma unroll
    for (int i = 0; i < kBoxDim; ++i) lim += (hi[i] - lo[i]) * (hi[i] - lo[i]);
    lim *= 0.0625f;  // a quarter of the tile's diagonal
  }
  const int64_t step = (stages + kPlanSamples - 1) / kPlanSamples;
  int32_t cnt = 0, seen = 0;
  for (int64_t s = (int64_t)lane * step; s < stages; s += 64 * step) {
    const float4* b = reinterpret_cast<const float4*>(sbox + s * (2 * kBoxDim));
    float lb = 0.0f;
#pragma unroll
    for (int i = 0; i < kBoxDim / 4; ++i) {
      const float4 l4 = b[i], h4 = b[kBoxDim / 4 + i];
      const float g[4] = {fmaxf(l4.x - hi[4 * i], lo[4 * i] - h4.x),
                          fmaxf(l4.y - hi[4 * i + 1], lo[4 * i + 1] - h4.y),
                          fmaxf(l4.z - hi[4 * i + 2], lo[4 * i + 2] - h4.z),
                          fmaxf(l4.w - hi[4 * i + 3], lo[4 * i + 3] - h4.w)};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float gc = fmaxf(g[c], 0.0f);
        lb = prune == kPrunePivot ? fmaxf(lb, gc * gc) : lb + gc * gc;
      }
    }
    ++seen;
    cnt += lb > lim ? 0 : 1;
  }
  for (int off = 32; off > 0; off >>= 1) {
    cnt += __shfl_xor(cnt, off, 64);
    seen += __shfl_xor(seen, off, 64);
  }
  if (lane == 0) rec[3 * t + 2] = (int32_t)((int64_t)cnt * stages / (seen > 0 ? seen : 1)) + 1;
}

// Pieces per tile (one workgroup).  Tiles longer than a target length are cut
// into equal pieces.  The target is picked from a geometric series by the time
// it should take: the work over the slots (and half a mean piece idle at the
// end), and no less than the longest piece, plus a charge for the number of
// pieces.  A scan of L stages
// costs L for the distances and kSelCost L for the selection while nearly every
// sub-tile holds a survivor, i.e. up to l0 stages (1024 K' rows: 32 x 32 pairs
// a sub-tile, each in the first K' of t rows with probability K'/t); beyond,
// the selection grows with the logarithm only, so cutting such a scan repeats
// it.  Each piece costs `fixed` on top (its first rows fill the lists: 60 us at
// K' = 32).  At 10^5 rows of 32 (Gaussian mixture, 2% outliers, K' = 32) the outliers'
// tiles scan everything: cut, the tile kernel takes 1.2 ms instead of 1.64.  At
// 10^6 rows of 64 cutting tiles of 800 stages (l0 = 256) in two took 59 ms
// instead of 47.  Where the last round would leave compute units idle, its
// tiles (those taken last: the first ones) are cut too, as tail_pieces does.
constexpr int kPlanThreads = 1024;
constexpr int kMaxPieces = 32;
constexpr float kPruneWorth = 0.8f;
constexpr float kSelCost = 1.7f;
constexpr float kPieceCharge = 0.25f;

__global__ void __launch_bounds__(kPlanThreads)
plan_pieces_kernel(int64_t tiles, int64_t stages, int slots, int cus, int cap, float l0,
                   float fixed, const Ctrl* __restrict__ ctrl, int32_t* __restrict__ plan,
                   int64_t rec_at, int32_t* __restrict__ ran) {
  if (ctrl->flat) {
    if (threadIdx.x == 0) {
      plan[0] = -1;
      *ran = 0;
    }
    return;  // uniform
  }
  __shared__ float red[3][kPlanThreads / 64];
  __shared__ int32_t wsum[kPlanThreads / 64];
  int32_t* rec = plan + rec_at;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Sums of v and w and maximum of m over the workgroup.
  auto block_red = [&](float& v, float& w, float& m) {
    for (int off = 32; off > 0; off >>= 1) {
      v += __shfl_xor(v, off, 64);
      w += __shfl_xor(w, off, 64);
      m = fmaxf(m, __shfl_xor(m, off, 64));
    }
    __syncthreads();
    if (lane == 0) {
      red[0][wave] = v;
      red[1][wave] = w;
      red[2][wave] = m;
    }
    __syncthreads();
    v = w = m = 0.0f;
    for (int i = 0; i < kPlanThreads / 64; ++i) {
      v += red[0][i];
      w += red[1][i];
      m = fmaxf(m, red[2][i]);
    }
  };
  float total = 0.0f, top = 0.0f, unused = 0.0f;
  for (int64_t t = tid; t < tiles; t += kPlanThreads) {
    const float e = (float)rec[3 * t + 2];
    total += e;
    top = fmaxf(top, e);
  }
  block_red(total, unused, top);
  // Where the boxes rule out less than a fifth of the pairs the plain scan is
  // the faster one (its sequence of stages is known): 6.1 ms against 6.6 at
  // 97,549 uniform rows of 26 (K' = 64), 27.1 against 29.4 at 269,454 of 65.
  if (total > kPruneWorth * (float)tiles * (float)stages) {
    if (tid == 0) {
      plan[0] = -1;
      *ran = 0;
    }
    return;  // uniform over the workgroup
  }
  auto pieces_of = [&](float est, float target) -> float {
    const float p = ceilf(est / target - 1e-4f);
    return p < 1.0f ? 1.0f : p < kMaxPieces ? p : (float)kMaxPieces;
  };
  auto cost = [&](float l) -> float {
    return fixed + l + kSelCost * (l < l0 ? l : l0 * (1.0f + __logf(l / l0)));
  };
  // (All of this is uniform over the workgroup.)
  float best = INFINITY, target = top, count = (float)tiles;
  const float low = fmaxf(4.0f, total / slots * 0.25f);
  for (float c = top; c >= low || c == top; c *= 0.62f) {
    float n = 0.0f, work = 0.0f, len = 0.0f;
    for (int64_t t = tid; t < tiles; t += kPlanThreads) {
      const float est = (float)rec[3 * t + 2], p = pieces_of(est, c), one = cost(est / p);
      n += p;
      work += p * one;
      len = fmaxf(len, one);
    }
    block_red(n, work, len);
    if (n - (float)tiles > (float)cap) break;  // shorter targets need more
    // (More pieces than slots: half a piece of idle time at the end.)
    const float span = fmaxf(n > slots ? work / slots + 0.5f * work / n : 0.0f, len) *
                       (1.0f + kPieceCharge * (1.0f - (float)tiles / n));
    if (span < best) {
      best = span;
      target = c;
      count = n;
    }
  }
  // The last round's tiles.
  const int64_t tw = (int64_t)count % slots;
  int tailp = 1;
  if (tw > 0 && tw < cus && tw < tiles) {
    float tbest = 1.0f;
    for (int p = 2; p <= 8; ++p) {
      if (count - (float)tiles + (float)(tw * (p - 1)) > (float)cap) break;
      const float c = (float)((tw * p + slots - 1) / slots) / p + 0.02f * (p - 1);
      if (c < tbest - 1e-6f) {
        tbest = c;
        tailp = p;
      }
    }
  }
  auto pieces = [&](int64_t t) -> int32_t {
    const int32_t p = (int32_t)pieces_of((float)rec[3 * t + 2], target);
    return t < tw && p < tailp && rec[3 * t + 2] >= 4 * tailp ? tailp : p;
  };
  int32_t base = 0;
  for (int64_t t0 = 0; t0 < tiles; t0 += kPlanThreads) {
    const int64_t t = t0 + tid;
    const int32_t ex = t < tiles ? pieces(t) - 1 : 0;
    const int32_t incl = wave_incl_sum(ex, lane);
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int32_t at = base + incl - ex;
    int32_t all = 0;
    for (int w = 0; w < kPlanThreads / 64; ++w) {
      at += w < wave ? wsum[w] : 0;
      all += wsum[w];
    }
    if (t < tiles) {
      rec[3 * t] = at;
      rec[3 * t + 1] = ex;
      for (int32_t i = 0; i < ex; ++i) {
        plan[1 + 2 * (int64_t)(at + i)] = (int32_t)t;
        plan[2 + 2 * (int64_t)(at + i)] = i + 1;
      }
    }
    base += all;
  }
  if (tid == 0) {
    plan[0] = base;
    *ran = 1;
  }
}

}  // namespace

// Seed groups: kWideGroups for rows of more than kSmallD elements; for
// shorter rows the most powers of two up to kOrdMaxC that leave each group
// at least kOrdRowsPerGroup rows.  Fine groups pay where neighbours are near
// in few dimensions: at 4 10^6 uniform rows of 8 elements, 256 groups against
// 16 cut the tile's time by 8% (577 -> 530 ms; 512 and 1024 groups measured
// the same within the spread and cost more in the assignment); rows of 32 and
// 64 elements (Gaussian mixtures, 10^5 and 10^6 rows) were slower with 64 or
// 256 groups, whose workgroups share fewer reference streams.
constexpr int64_t kOrdRowsPerGroup = 8192;

int32_t order_groups(int64_t nr, int64_t d) {
  if (d > kSmallD) return kWideGroups;
  int64_t g = kWideGroups;
  while (g * 2 <= kOrdMaxC && g * 2 * kOrdRowsPerGroup <= nr) g *= 2;
  return (int32_t)g;
}

int32_t order_blocks(int64_t nr) { return (int32_t)((nr + kOrdRows - 1) / kOrdRows); }

hipError_t launch_order(const Plan& p, const Args& a, hipStream_t st) {
  const int64_t n = p.nr;
  const int nb = order_blocks(n);
  const int G = p.groups;
  const unsigned ga = (unsigned)((n + kAssignThreads - 1) / kAssignThreads);
  if (p.prune == kPruneBox) {
    int levels = 0;
    while ((1 << levels) < G) ++levels;
    const int m = kKdSamples << levels;
    const size_t lds = sizeof(uint64_t) * (size_t)m;
    static_assert(sizeof(uint64_t) * kKdSamples * kOrdMaxC <= 65536, "no opt-in needed");
    hipLaunchKernelGGL(kd_build_kernel, dim3(1), dim3(kKdThreads), lds, st, a.xr, n, (int)p.d, m,
                       levels, reinterpret_cast<int2*>(a.oseed));
    hipLaunchKernelGGL(assign_kd_kernel, dim3(ga), dim3(kAssignThreads), 0, st, a.xr, n, (int)p.d,
                       levels, reinterpret_cast<const int2*>(a.oseed), a.lab);
  } else if (p.d <= kSmallD) {
    const int DT = (int)((p.d + 3) & ~3);
    hipLaunchKernelGGL(seeds_kernel, dim3((unsigned)((G * DT + 255) / 256)), dim3(256), 0, st,
                       a.xr, n, (int)p.d, G, DT, a.oseed);
    const auto kern = DT == 4   ? assign_small_kernel<4>
                      : DT == 8 ? assign_small_kernel<8>
                      : DT == 12 ? assign_small_kernel<12>
                                 : assign_small_kernel<16>;
    hipLaunchKernelGGL(kern, dim3(ga), dim3(kAssignThreads), 0, st, a.xr, n, (int)p.d, G,
                       reinterpret_cast<const float4*>(a.oseed), a.lab);
  } else if (p.prune == kPrunePivot) {
    if (G != kPivots * kRadBins) return hipErrorInvalidValue;
    int32_t* const srow = reinterpret_cast<int32_t*>(a.oseed);
    const int m = seed_samples(n, (int)p.d);
    int tps = 2;  // threads per sample
    while (m * tps * 2 <= kSeedThreads && tps < 64) tps *= 2;
    const size_t lds = sizeof(float) * (size_t)m * (size_t)seed_stride((int)p.d);
    // (The attribute is the function's, not the call's: its bound, whatever this
    // call needs, so that calls of other threads stay within it.)
    hipError_t e = hipFuncSetAttribute((const void*)pivot_seed_kernel,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(sizeof(float) * kSeedFloats));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pivot_seed_kernel, dim3(1), dim3(kSeedThreads), lds, st, a.xr, n, (int)p.d,
                       m, tps, a.mu32, a.ctrl, p.scale_exp, !a.plan ? 0 : p.splits > 1 ? 2 : 1,
                       a.pdist, srow);
    hipLaunchKernelGGL(assign_pivot_kernel, dim3(ga), dim3(kAssignThreads),
                       sizeof(float) * kPivots * (size_t)p.d, st, a.xr, n, (int)p.d, a.mu32,
                       a.ctrl, p.scale_exp, srow, a.pdist, a.lab);
  } else {
    if (G != kWideGroups) return hipErrorInvalidValue;
    hipLaunchKernelGGL(assign_kernel, dim3(ga), dim3(kAssignThreads),
                       sizeof(float) * kWideGroups * (size_t)p.d, st, a.xr, n, (int)p.d, a.lab);
  }
  hipLaunchKernelGGL(count_kernel, dim3((unsigned)nb), dim3(256), 0, st, a.lab, n, G, a.bcnt);
  hipLaunchKernelGGL(block_offsets_kernel, dim3((unsigned)((G + 3) / 4)), dim3(256), 0, st,
                     a.bcnt, nb, G, a.boff, a.cstart);
  if (p.prune == kPrunePivot)
    hipLaunchKernelGGL(pivot_starts_kernel, dim3(1), dim3(kPivots * kRadBins), 0, st, a.cstart,
                       a.kstart);
  else
    hipLaunchKernelGGL(group_starts_kernel, dim3(1), dim3(64), 0, st, G, a.cstart);
  int bits = 0;
  while ((1 << bits) < G) ++bits;
  hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)nb), dim3(64), 0, st, a.lab, n, G, bits,
                     a.boff, a.cstart, a.perm);
  if (p.prune == kPruneBox) {
    const int chunk = kd_chunk(n);
    const size_t lds = (size_t)chunk * (sizeof(uint32_t) + sizeof(_Float16) * (p.d < 2 ? 2 : p.d));
    const auto kern = chunk == kKdChunkMost ? kd_local_kernel<kKdChunkMost> : kd_local_kernel<1024>;
    // (The most any row length takes, as above.)
    const size_t most = (size_t)chunk * (sizeof(uint32_t) + sizeof(_Float16) * kBoxDim);
    hipError_t e = hipFuncSetAttribute((const void*)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + chunk - 1) / chunk)),
                       dim3(kKdThreads), lds, st, a.xr, n, (int)p.d, a.mu32, a.ctrl, p.scale_exp,
                       a.perm);
  }
  return hipGetLastError();
}

// Rows of the local splits: as few as the tree's 1024 leaves allow.
int kd_chunk(int64_t nr) { return nr <= (int64_t)1024 * kOrdMaxC ? 1024 : kKdChunkMost; }

// Leaves of the k-d order's tree: one per chunk of the local splits.
int32_t kd_leaves(int64_t nr) {
  int32_t g = 2;
  while (g < kOrdMaxC && (int64_t)g * kd_chunk(nr) < nr) g *= 2;
  return g;
}

hipError_t launch_boxes(const Plan& p, const Args& a, hipStream_t st) {
  const int64_t subs = p.nr_pad / 32;
  const int64_t stages = (p.nr + p.stage_rows - 1) / p.stage_rows;
  const unsigned gsub = (unsigned)((subs + kSubsPerBlock - 1) / kSubsPerBlock);
  const dim3 bsub(kSubsPerBlock * kBoxDim);
  if (p.prune == kPrunePivot) {
    const float eps = (float)(p.d + 16) * 0x1p-24f;
    const float wide = 0x1p-6f + ldexpf(sqrtf((float)p.d), p.scale_exp - 24);
    hipLaunchKernelGGL(pivot_box_kernel, dim3(gsub), bsub, 0, st, a.pdist, a.perm, a.lab, a.kstart,
                       p.nr, subs, eps, wide, a.ctrl, a.box32, a.substart);
  } else if (p.precision == TOD_PREC_FP16) {
    hipLaunchKernelGGL(column_box_kernel<_Float16>, dim3(gsub), bsub, 0, st,
                       (const _Float16*)a.xq_r, p.nr, subs, (int)p.d, p.dpad, a.box32, a.substart);
  } else {
    hipLaunchKernelGGL(column_box_kernel<__bf16>, dim3(gsub), bsub, 0, st, (const __bf16*)a.xq_r,
                       p.nr, subs, (int)p.d, p.dpad, a.box32, a.substart);
  }
  const auto grid = [](int64_t boxes) {
    return dim3((unsigned)((boxes * 2 * kBoxDim + 255) / 256));
  };
  const int64_t chunks = (stages + 63) / 64;
  hipLaunchKernelGGL(stage_box_kernel, grid(stages), dim3(256), 0, st, a.box32, subs, stages,
                     p.stage_rows / 32, a.ctrl, a.sbox);
  hipLaunchKernelGGL(stage_box_kernel, grid(chunks), dim3(256), 0, st, a.sbox, stages, chunks, 64,
                     a.ctrl, a.xbox);
  return hipGetLastError();
}

hipError_t launch_plan(const Plan& p, const Args& a, int64_t q_begin, int64_t q_rows, int slots,
                       int cus, hipStream_t st) {
  const int64_t tiles = (q_rows + p.tile_rows - 1) / p.tile_rows;
  const int64_t stages = (p.nr + p.stage_rows - 1) / p.stage_rows;
  hipLaunchKernelGGL(plan_estimate_kernel, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st,
                     a.box32, a.sbox, stages, q_begin / 32, (q_rows + 31) / 32, p.tile_rows / 32,
                     tiles, p.prune, a.ctrl, a.plan + a.plan_tiles);
  hipLaunchKernelGGL(plan_pieces_kernel, dim3(1), dim3(kPlanThreads), 0, st, tiles, stages, slots,
                     cus, (int)a.plan_cap, 1024.0f * p.kprime / p.stage_rows,
                     200.0f * p.kprime / p.stage_rows, a.ctrl, a.plan, a.plan_tiles,
                     a.ran + q_begin / p.query_block);
  return hipGetLastError();
}

}  // namespace tod
