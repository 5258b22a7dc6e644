// Scalar quantization: codebook training, encoding, and query folding.
// Paper Appendix G (SQ-b: uniform levels over the value range of a dimension)
// and Section 5.2 (stored squared norm; query terms precomputed before search).
#include <math.h>

#include "ann_internal.hpp"
#include "device_utils.hpp"

namespace ann {

// ------------------------------------------------------------- codebook
// Column-wise min/max.  Bound: one read of x.  The threads of a workgroup lie
// side by side over the row's VEC-wide pieces and, where the row has fewer pieces
// than the workgroup threads, over several rows at a time, with eight loads in
// flight per thread.  The partial results of the workgroups (about a thousand) are
// reduced by a workgroup per 16 columns whose 64 threads per column walk them in
// parallel.  1M x 128: 244 + 491 us (half of the threads idle; one thread per
// column over all partial results) -> 97 + 5 us (5.3 TB/s).
//
// The workgroups go through the rows together, from the first to the last, and
// sq_encode_kernel from the last to the first: what the encoder reads first is then
// still in the 256 MB of the Infinity Cache, and what it reads last is there for the
// copy into an index.  Codebook and codes of 1M x 128, 8 bits: 243.6 -> 235 us; 130,000 x 960,
// 4 bits 242.4 -> 230.6; a whole index of 200,000 x 960 993 -> 973.
constexpr int kMinmaxThreads = 256, kMinmaxUnroll = 8;

template <int VEC>
__global__ __launch_bounds__(kMinmaxThreads) void sq_minmax_partial_kernel(const float *__restrict__ x, uint64_t n, uint32_t d,
                                                                           float *__restrict__ pmin, float *__restrict__ pmax) {
  __shared__ float red[2][kMinmaxThreads * VEC];
  const uint32_t pieces = d / VEC, p0 = blockIdx.y * kMinmaxThreads;
  const uint32_t width = pieces - p0 < (uint32_t)kMinmaxThreads ? pieces - p0 : (uint32_t)kMinmaxThreads;
  const uint32_t side = kMinmaxThreads / width;   // rows side by side
  const uint32_t r = threadIdx.x / width, c = threadIdx.x % width;
  float mn[VEC], mx[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    mn[e] = INFINITY;
    mx[e] = -INFINITY;
  }
  auto take = [&](const float *p, float (&v)[VEC]) {
    if constexpr (VEC == 4) {
      const float4 t = *reinterpret_cast<const float4 *>(p);
      v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
    } else {
      v[0] = p[0];
    }
  };
  auto fold = [&](const float (&v)[VEC]) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      mn[e] = fminf(mn[e], v[e]);
      mx[e] = fmaxf(mx[e], v[e]);
    }
  };
  if (r < side) {
    const float *col = x + (uint64_t)(p0 + c) * VEC;
    // (rows past the last are the last again)
    for (uint64_t i = (uint64_t)blockIdx.x * kMinmaxUnroll * side + r; i < n; i += (uint64_t)gridDim.x * kMinmaxUnroll * side) {
      float v[kMinmaxUnroll][VEC];
#pragma unroll
      for (int u = 0; u < kMinmaxUnroll; ++u) {
        const uint64_t row = i + (uint64_t)u * side;
        take(col + (row < n ? row : n - 1) * d, v[u]);
      }
#pragma unroll
      for (int u = 0; u < kMinmaxUnroll; ++u) fold(v[u]);
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    red[0][threadIdx.x * VEC + e] = mn[e];
    red[1][threadIdx.x * VEC + e] = mx[e];
  }
  __syncthreads();
  if (threadIdx.x < width) {
    for (uint32_t k = 1; k < side; ++k)
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        mn[e] = fminf(mn[e], red[0][(k * width + threadIdx.x) * VEC + e]);
        mx[e] = fmaxf(mx[e], red[1][(k * width + threadIdx.x) * VEC + e]);
      }
    const uint64_t at = (uint64_t)blockIdx.x * d + (uint64_t)(p0 + threadIdx.x) * VEC;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      pmin[at + e] = mn[e];
      pmax[at + e] = mx[e];
    }
  }
}

constexpr int kFinalCols = 16, kFinalRows = 64;

__global__ __launch_bounds__(kFinalCols *kFinalRows) void sq_minmax_final_kernel(const float *__restrict__ pmin,
                                                                                 const float *__restrict__ pmax, uint32_t nblocks,
                                                                                 uint32_t d, float levels, float *__restrict__ lo,
                                                                                 float *__restrict__ delta) {
  __shared__ float smn[kFinalRows][kFinalCols], smx[kFinalRows][kFinalCols];
  const uint32_t c = threadIdx.x % kFinalCols, r = threadIdx.x / kFinalCols, j = blockIdx.x * kFinalCols + c;
  float mn = INFINITY, mx = -INFINITY;
  if (j < d)
#pragma unroll 8
    for (uint32_t b = r; b < nblocks; b += kFinalRows) {
      mn = fminf(mn, pmin[(uint64_t)b * d + j]);
      mx = fmaxf(mx, pmax[(uint64_t)b * d + j]);
    }
  smn[r][c] = mn;
  smx[r][c] = mx;
  for (uint32_t h = kFinalRows / 2; h > 0; h >>= 1) {
    __syncthreads();
    if (r < h) {
      smn[r][c] = fminf(smn[r][c], smn[r + h][c]);
      smx[r][c] = fmaxf(smx[r][c], smx[r + h][c]);
    }
  }
  if (r == 0 && j < d) {
    mn = smn[0][c];
    mx = smx[0][c];
    lo[j] = mn;
    delta[j] = (mx > mn) ? __fdiv_rn(__fsub_rn(mx, mn), levels) : 1.0f;
  }
}

// ------------------------------------------------------------- truncated range
// Exact order statistics of every column by radix selection on the ordered
// bit pattern of the floats: four passes of 8 bits; each pass histograms the
// next digit of the elements that still match the prefix found so far.  Two
// selections per column run side by side (lower and upper end of the range).
// Bound: four reads of x.  The counters of a digit lie side by side over the
// columns, so that the lanes of a wavefront (32 columns of two rows) count in
// different LDS banks; with the digits of a column side by side one exponent's
// values all met in one bank.  200,000 x 960: 814 -> 186 us a pass.
constexpr int kSelCols = 32;  // columns per workgroup
constexpr int kSelBlock = 512, kSelUnroll = 8;

__global__ __launch_bounds__(kSelBlock) void radix_hist_kernel(const float *__restrict__ x, uint64_t n, uint32_t d,
                                                               uint32_t rows_per_block, int shift,
                                                               const uint32_t *__restrict__ prefix /*[2][d]*/,
                                                               uint32_t *__restrict__ hist /*[2][d][256]*/) {
  __shared__ uint32_t lh[2][256][kSelCols];
  for (int e = threadIdx.x; e < 2 * kSelCols * 256; e += kSelBlock) (&lh[0][0][0])[e] = 0;
  __syncthreads();
  const uint32_t c = threadIdx.x % kSelCols, col = blockIdx.y * kSelCols + c;
  const uint64_t r0 = (uint64_t)blockIdx.x * rows_per_block;
  const uint64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  constexpr uint32_t side = kSelBlock / kSelCols;
  if (col < d) {
    const uint32_t p0 = prefix[col], p1 = prefix[d + col];
    auto take = [&](float v) {
      const uint32_t key = order_u32(v);
      const uint32_t digit = (key >> shift) & 255u;
      if (shift == 24) {   // (nothing tells the two selections apart yet: they share the first table)
        atomicAdd(&lh[0][digit][c], 1u);
        return;
      }
      const uint32_t high = key >> (shift + 8);
      if (high == p0) atomicAdd(&lh[0][digit][c], 1u);
      if (high == p1) atomicAdd(&lh[1][digit][c], 1u);
    };
    const float *at = x + col;
    uint64_t i = r0 + threadIdx.x / kSelCols;
    for (; i + (uint64_t)(kSelUnroll - 1) * side < r1; i += kSelUnroll * side) {
      float v[kSelUnroll];
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) v[u] = at[(i + (uint64_t)u * side) * d];
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) take(v[u]);
    }
    for (; i < r1; i += side) take(at[i * d]);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * kSelCols * 256; e += kSelBlock) {
    const int sel = e / (kSelCols * 256), cc = (e / 256) % kSelCols, b = e % 256;
    const uint32_t v = lh[shift == 24 ? 0 : sel][b][cc], gc = blockIdx.y * kSelCols + cc;
    if (v != 0 && gc < d) atomicAdd(&hist[((size_t)sel * d + gc) * 256 + b], v);
  }
}

// One wavefront per (selection, column): the digit whose bucket holds the
// wanted rank, four buckets per lane; the table is left cleared for the next pass.
__global__ __launch_bounds__(64) void radix_pick_kernel(uint32_t *__restrict__ hist, uint32_t *__restrict__ prefix,
                                                        uint32_t *__restrict__ rank) {
  const uint32_t t = blockIdx.x, lane = threadIdx.x;
  uint4 *h4 = reinterpret_cast<uint4 *>(hist + (size_t)t * 256) + lane;
  const uint4 h = *h4;
  *h4 = make_uint4(0, 0, 0, 0);
  const uint32_t sum = h.x + h.y + h.z + h.w;
  const uint32_t before = (uint32_t)wave_inclusive_scan_i32((int)sum) - sum, want = rank[t];
  // (the last bucket takes what no other does)
  const bool mine = (want >= before && want < before + sum) || (lane == kWave - 1 && want >= before + sum);
  if (mine) {
    uint32_t cum = before, b = 0;
    if (want >= cum + h.x) {
      cum += h.x, b = 1;
      if (want >= cum + h.y) {
        cum += h.y, b = 2;
        if (want >= cum + h.z) cum += h.z, b = 3;
      }
    }
    rank[t] = want - cum;
    prefix[t] = (prefix[t] << 8) | (lane * 4 + b);
  }
}

// prefix[2][d], rank[2][d], hist[2][d][256] before the first pass
__global__ void radix_init_kernel(uint32_t d, uint32_t low, uint32_t high, uint32_t *__restrict__ prefix, uint32_t *__restrict__ rank,
                                  uint32_t *__restrict__ hist) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 2ull * d) {
    prefix[t] = 0;
    rank[t] = t < d ? low : high;
  }
  if (t < 512ull * d) hist[t] = 0;
}

__global__ void truncated_range_kernel(const uint32_t *__restrict__ prefix, uint32_t d, float levels,
                                       float *__restrict__ lo, float *__restrict__ delta) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  const float mn = unorder_f32(prefix[j]), mx = unorder_f32(prefix[d + j]);
  lo[j] = mn;
  delta[j] = (mx > mn) ? __fdiv_rn(__fsub_rn(mx, mn), levels) : 1.0f;
}

// The same in one read of x where a sample says between which two values an order
// statistic must lie.  Per column and end of the range, from a stratified random sample of
// m rows: `a` and `b`, kBracketWidth standard deviations of the sample's order statistic (and a
// little) to either side of it.  One pass over x then counts what lies outside of
// the two brackets and what equals an end of one, and lists what lies strictly inside (1 % of
// the values); the wanted one is picked from the list by its rank.  Any order of the
// rows and any distribution: a bracket that does not hold the wanted rank or has more values
// inside than there is room for (many equal ones) is noticed, and the call takes
// the four radix passes.  Bound: the pass' read of x (4 TB/s of it: the rest of its time is
// the walk over the values inside).  200,000 x 960, coverage 0.99: four passes and
// picks 738 us; sample 19, brackets 33, pass 190, picks 24: 270 with the host's wait.
// 1M x 128 521 / 252, 33,000 x 100 145 / 75.
constexpr double kBracketWidth = 5.5;
constexpr uint32_t kBracketMost = 1u << 18;   // values of a list at most
constexpr int kBracketKeys = 32;              // keys of the sample per thread

// What the pass finds out about an end (0: low, 1: high) of column j, at [end * d + j].
struct BracketArgs {
  const float *x;
  uint64_t n;
  uint32_t d, k;          // rank of the low end; of the high one, from above
  uint32_t m, room;       // rows of the sample; values a list has room for
  double below, beyond, slack;   // ranks in the sample between which the bracket reaches, and how much further it may
  uint32_t *sample;       // [d][m] ordered keys
  uint32_t *a, *b;        // brackets
  uint32_t *outside;      // values below a (low end), above b (high end)
  uint32_t *at_a, *at_b, *inside;
  uint32_t *list;         // [2 * d][room]
  uint32_t *failed;
};

// Rows of the sample, column by column: a workgroup turns 64 rows x 64 columns in LDS.
__global__ __launch_bounds__(256) void bracket_sample_kernel(BracketArgs g) {
  __shared__ uint32_t tile[64][65];
  const uint32_t lane = threadIdx.x % 64, w = threadIdx.x / 64, j = blockIdx.y * 64 + lane;
  const double stretch = (double)g.n / g.m;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint64_t r = sample_row(blockIdx.x * 64 + w * 16 + i, stretch);
    tile[w * 16 + i][lane] = j < g.d ? order_u32(g.x[r * g.d + j]) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t c = blockIdx.y * 64 + w * 16 + i;
    if (c < g.d) g.sample[(uint64_t)c * g.m + blockIdx.x * 64 + lane] = tile[lane][w * 16 + i];
  }
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *g.failed = 0;
}

// Keys in registers, EPT per thread of THREADS; a step of a bisection counts those up to the middle.
template <int EPT, int THREADS>
struct KeyCounter {
  static constexpr int kWaves = THREADS / kWave;
  uint32_t key[EPT];
  uint32_t *red;   // LDS [2][kWaves]
  int parity = 0;
  __device__ __forceinline__ uint32_t up_to(uint32_t v) {
    uint32_t c = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) c += (uint32_t)__popcll(__ballot(key[e] <= v));
    return total(c);
  }
  __device__ __forceinline__ uint32_t total(uint32_t c) {   // of the wavefronts' counts
    if (threadIdx.x % kWave == 0) red[parity * kWaves + threadIdx.x / kWave] = c;
    __syncthreads();
    c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += red[parity * kWaves + w];
    parity ^= 1;
    return c;
  }
};

// One workgroup per column: the brackets of both ends.  A few steps over the whole
// sample find a value that the keys of interest do not reach and at most four keys per thread do;
// the bracket's ends are then searched among those (a step over 32 keys per thread is bound by
// vector instructions; 960 columns: 50 us with all steps over all keys -> 33).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void bracket_bounds_kernel(BracketArgs g) {
  constexpr int EPT = kBracketKeys, kWaves = THREADS / kWave, kFew = 4;
  __shared__ uint32_t red[2 * kWaves], ends[kWaves], few_s[kFew * THREADS], n_few;
  const uint32_t j = blockIdx.x, tid = threadIdx.x;
  KeyCounter<EPT, THREADS> s;
  s.red = red;
  uint32_t mn = 0xFFFFFFFFu, mx = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    s.key[e] = g.sample[(uint64_t)j * g.m + e * THREADS + tid];
    mn = s.key[e] < mn ? s.key[e] : mn;
    mx = s.key[e] > mx ? s.key[e] : mx;
  }
  auto least = [&](uint32_t v) {   // of all threads' values
#pragma unroll
    for (int x = 1; x < kWave; x <<= 1) {
      const uint32_t o = (uint32_t)xor_lane_i32((int)v, x);
      v = o < v ? o : v;
    }
    __syncthreads();
    if (tid % kWave == 0) ends[tid / kWave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v = ends[w] < v ? ends[w] : v;
    return v;
  };
  mn = least(mn);
  mx = ~least(~mx);
  for (int end = 0; end < 2; ++end) {
    // the high end is the low end of the complements
    if (end == 1) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) s.key[e] = ~s.key[e];
      const uint32_t t = ~mx;
      mx = ~mn;
      mn = t;
    }
    uint32_t a = 0, b = 0xFFFFFFFFu, between = 0;
    const uint32_t under = mn > 0 ? mn - 1 : 0;
    auto bracket = [&](auto &s, uint32_t most) {
      constexpr int kEach = sizeof(s.key) / sizeof(s.key[0]);
      // a: the smallest key above a value that few enough keys reach (no bound if the wanted rank is among the first)
      if (g.below >= 1.0) {
        uint32_t lo = under, hi = most;   // count(lo) <= below < count(hi)
        while (hi - lo > 1) {
          const uint32_t mid = lo + (hi - lo) / 2;
          const double n = s.up_to(mid);
          if (n <= g.below) {
            lo = mid;
            if (n >= g.below - g.slack) break;
          } else {
            hi = mid;
          }
        }
        uint32_t next = 0xFFFFFFFFu;
#pragma unroll
        for (int e = 0; e < kEach; ++e) next = s.key[e] > lo && s.key[e] < next ? s.key[e] : next;
        a = least(next);
      }
      // b: the first value that enough keys reach, or one not far above it
      if (g.beyond <= (double)g.m) {
        uint32_t lo = under, hi = most;   // count(lo) < beyond <= count(hi)
        while (hi - lo > 1) {
          const uint32_t mid = lo + (hi - lo) / 2;
          const double n = s.up_to(mid);
          if (n >= g.beyond) {
            hi = mid;
            if (n <= g.beyond + g.slack) break;
          } else {
            lo = mid;
          }
        }
        b = hi;
      }
      between = a < b ? s.up_to(b - 1) - s.up_to(a) : 0u;
    };
    // the few: keys up to `most`, which at least `beyond` and at most kFew * THREADS keys reach
    uint32_t most = mx;
    bool some = false;
    if (g.beyond <= (double)(kFew * THREADS)) {
      uint32_t lo = under, hi = mx;   // count(lo) < beyond <= count(hi)
      while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        const double n = s.up_to(mid);
        if (n >= g.beyond) {
          hi = mid;
          if (n <= (double)(kFew * THREADS)) break;
        } else {
          lo = mid;
        }
      }
      most = hi;
      some = s.up_to(most) <= (uint32_t)(kFew * THREADS);
    }
    if (some) {
      if (tid == 0) n_few = 0;
      __syncthreads();
      uint32_t mine = 0, to = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) mine += (uint32_t)__popcll(__ballot(s.key[e] <= most));
      if (tid % kWave == 0) to = atomicAdd(&n_few, mine);
      to = (uint32_t)__builtin_amdgcn_readfirstlane((int)to);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint64_t m = __ballot(s.key[e] <= most);
        if (s.key[e] <= most) few_s[to + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = s.key[e];
        to += (uint32_t)__popcll(m);
      }
      __syncthreads();
      KeyCounter<kFew, THREADS> few;
      few.red = red;
      few.parity = s.parity;
#pragma unroll
      for (int e = 0; e < kFew; ++e) few.key[e] = e * THREADS + tid < n_few ? few_s[e * THREADS + tid] : 0xFFFFFFFFu;
      bracket(few, most);
      s.parity = few.parity;
    } else {
      bracket(s, mx);
    }
    if (tid == 0) {
      const uint64_t at = (uint64_t)end * g.d + j;
      g.a[at] = end ? ~b : a;
      g.b[at] = end ? ~a : b;
      g.outside[at] = g.at_a[at] = g.at_b[at] = g.inside[at] = 0;
      if ((double)between * ((double)g.n / g.m) > 0.75 * g.room) atomicOr(g.failed, 1u);
    }
  }
}

// The pass over x.  A thread stays in its column (32 columns x 16 rows at a time),
// carries kSelUnroll values and then walks those of them that lie in a bracket; these
// collect in LDS and go to their lists when the workgroup's rows are done.  A workgroup
// takes every gridDim.x-th group of 16 rows: rows in an order that puts a bracket's
// values side by side spread over the workgroups.
constexpr int kBracketLocal = 128;   // values of a column and end collected in LDS
__global__ __launch_bounds__(kSelBlock) void bracket_collect_kernel(BracketArgs g) {
  __shared__ uint32_t local[2 * kSelCols][kBracketLocal], n_local[2 * kSelCols], tally[6][kSelCols], base_s[2 * kSelCols];
  if (*(volatile uint32_t *)g.failed) return;   // (set by an earlier kernel only)
  const uint32_t tid = threadIdx.x, c = tid % kSelCols, col = blockIdx.y * kSelCols + c;
  if (tid < 2 * kSelCols) n_local[tid] = 0;
  for (uint32_t e = tid; e < 6 * kSelCols; e += kSelBlock) (&tally[0][0])[e] = 0;
  __syncthreads();
  constexpr uint32_t side = kSelBlock / kSelCols;
  if (col < g.d) {
    const uint32_t a0 = g.a[col], b0 = g.b[col], a1 = g.a[g.d + col], b1 = g.b[g.d + col];
    uint32_t below = 0, above = 0, eq[4] = {0, 0, 0, 0};
    auto put = [&](uint32_t key, uint32_t end) {
      const uint32_t at = end * kSelCols + c, pos = atomicAdd(&n_local[at], 1u);
      if (pos < kBracketLocal) {
        local[at][pos] = key;
      } else {
        const uint64_t l = (uint64_t)end * g.d + col;
        const uint32_t to = atomicAdd(&g.inside[l], 1u);
        if (to < g.room) g.list[l * g.room + to] = key;
      }
    };
    // nearly all values lie between the brackets: for those a subtraction and a comparison
    const uint32_t after = b0 + 1u, gap = a1 > b0 ? a1 - after : 0u;
    auto take = [&](const float (&v)[kSelUnroll], uint32_t valid) {
      uint32_t key[kSelUnroll], mine = 0;
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) {
        key[u] = order_u32(v[u]);
        mine |= key[u] - after < gap ? 0u : 1u << u;
      }
      mine &= valid;
      while (mine) {
        const int u = __builtin_ctz(mine);
        mine &= mine - 1;
        static_assert(kSelUnroll == 8, "three selects");
        const uint32_t s0 = u & 1 ? key[1] : key[0], s1 = u & 1 ? key[3] : key[2], s2 = u & 1 ? key[5] : key[4], s3 = u & 1 ? key[7] : key[6];
        const uint32_t t0 = u & 2 ? s1 : s0, t1 = u & 2 ? s3 : s2, v_ = u & 4 ? t1 : t0;
        below += v_ < a0 ? 1u : 0u;
        above += v_ > b1 ? 1u : 0u;
        eq[0] += v_ == a0 ? 1u : 0u;
        eq[1] += v_ == b0 ? 1u : 0u;
        eq[2] += v_ == a1 ? 1u : 0u;
        eq[3] += v_ == b1 ? 1u : 0u;
        if (v_ > a0 && v_ < b0) put(v_, 0u);
        if (v_ > a1 && v_ < b1) put(v_, 1u);
      }
    };
    const float *at = g.x + col;
    const uint64_t step = (uint64_t)gridDim.x * side;
    for (uint64_t i = (uint64_t)blockIdx.x * side + tid / kSelCols; i < g.n; i += kSelUnroll * step) {
      float v[kSelUnroll];
      uint32_t valid = 0;
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) {
        const uint64_t r = i + (uint64_t)u * step;
        v[u] = at[(r < g.n ? r : g.n - 1) * g.d];
        valid |= r < g.n ? 1u << u : 0u;
      }
      take(v, valid);
    }
    if (below) atomicAdd(&tally[0][c], below);
    if (above) atomicAdd(&tally[1][c], above);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (eq[e]) atomicAdd(&tally[2 + e][c], eq[e]);
  }
  __syncthreads();
  if (tid < 2 * kSelCols) {
    const uint32_t end = tid / kSelCols, gc = blockIdx.y * kSelCols + tid % kSelCols;
    if (gc < g.d) {
      const uint64_t l = (uint64_t)end * g.d + gc;
      const uint32_t out = tally[end][tid % kSelCols], ea = tally[2 + 2 * end][tid % kSelCols], eb = tally[3 + 2 * end][tid % kSelCols];
      const uint32_t n_l = n_local[tid] < kBracketLocal ? n_local[tid] : kBracketLocal;
      if (out) atomicAdd(&g.outside[l], out);
      if (ea) atomicAdd(&g.at_a[l], ea);
      if (eb) atomicAdd(&g.at_b[l], eb);
      base_s[tid] = n_l ? atomicAdd(&g.inside[l], n_l) : 0u;
      n_local[tid] = n_l;
    } else {
      n_local[tid] = 0;
    }
  }
  __syncthreads();
  for (uint32_t e = tid; e < 2 * kSelCols * kBracketLocal; e += kSelBlock) {
    const uint32_t at = e / kBracketLocal, i = e % kBracketLocal;
    if (i >= n_local[at]) continue;
    const uint64_t l = (uint64_t)(at / kSelCols) * g.d + blockIdx.y * kSelCols + at % kSelCols;
    const uint32_t to = base_s[at] + i;
    if (to < g.room) g.list[l * g.room + to] = local[at][i];
  }
}

// One workgroup per column and end: the wanted value, as radix_pick_kernel leaves it.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void bracket_pick_kernel(BracketArgs g, uint32_t *__restrict__ prefix) {
  __shared__ uint32_t red[2 * THREADS / kWave];
  if (*(volatile uint32_t *)g.failed & 1u) return;   // (by bracket_bounds_kernel; the other bit may be set meanwhile)
  const uint32_t end = blockIdx.x / g.d, tid = threadIdx.x;
  const uint64_t l = blockIdx.x;
  // from the end inwards: outside, equal to the outer end, inside, equal to the inner end
  const uint32_t out = g.outside[l], ea = g.at_a[l], eb = g.at_b[l], n_l = g.inside[l], a = g.a[l], b = g.b[l];
  const uint32_t outer = end ? eb : ea, inner = end ? ea : eb, want = g.k - out;   // (wraps below)
  if (g.k < out || n_l > g.room || (uint64_t)want >= (uint64_t)outer + n_l + (a < b ? inner : 0u)) {
    if (tid == 0) atomicOr(g.failed, 2u);
    return;
  }
  if (want < outer || want - outer >= n_l) {
    if (tid == 0) prefix[l] = (want < outer) == (end == 0) ? a : b;
    return;
  }
  const uint32_t from_low = end ? n_l - 1 - (want - outer) : want - outer;
  const uint32_t *list = g.list + l * g.room;
  auto bisect = [&](auto &&count) {
    uint32_t lo = a, hi = b;   // count(lo) <= from_low < count(hi)
    while (hi - lo > 1) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (count(mid) > from_low)
        hi = mid;
      else
        lo = mid;
    }
    if (tid == 0) prefix[l] = hi;
  };
  auto in_registers = [&](auto &s) {
    s.red = red;
    constexpr int kEach = sizeof(s.key) / sizeof(s.key[0]);
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
      const uint32_t i = (uint32_t)e * THREADS + tid;
      s.key[e] = i < n_l ? list[i] : 0xFFFFFFFFu;   // (none inside a bracket is that large)
    }
    bisect([&](uint32_t mid) { return s.up_to(mid); });
  };
  if (n_l <= 16u * THREADS) {
    KeyCounter<16, THREADS> s;
    in_registers(s);
  } else if (n_l <= 64u * THREADS) {
    KeyCounter<64, THREADS> s;
    in_registers(s);
  } else {   // (millions of rows: the list is read again for every step)
    KeyCounter<1, THREADS> s;
    s.red = red;
    bisect([&](uint32_t mid) {
      uint32_t c = 0;
      for (uint32_t i = tid; i < n_l; i += THREADS) c += list[i] <= mid ? 1u : 0u;
      return s.total((uint32_t)group_sum_i32<kWave>((int)c));
    });
  }
}

// ------------------------------------------------------------- encoder
// Bound: one read of x, one write of the codes (vector instructions are close
// behind).  A group of LPR lanes takes a row, VEC dimensions per lane and piece
// (a row of more than LPR * VEC dimensions has several pieces), and every lane
// carries kEncRows rows at a time, so that many loads are in flight and what
// depends on the column alone is read once for all of them.
//
// The quotient of two floats is taken as a product in fp64 with the reciprocal
// of the step (one division per column and workgroup instead of one per
// element) and rounded to fp32: the product is within 2^-51 of the quotient,
// relatively, and a quotient of two floats is never closer than 2^-49 to the
// middle between two floats, so the rounding is that of the division.
//
// The squared norm is defined as the fp64 sum in dimension order, rounded once
// to fp32.  It is formed as a tree instead (certain_f32 says when both round to
// the same float) and again by one lane in dimension order where the two may
// differ: about one row in 2^28 / d.
// 1M x 128, 8 bits: 782 us (one row per wavefront, the sum by one lane) -> 114 us (5.7 TB/s read and written);
// 200,000 x 960, 4 bits: 1,179 us -> 189 us (4.6 TB/s).
constexpr int kEncRows = 8;

// Code of value v in a column with the given range and reciprocal step, and the value it decodes to.
template <int BITS>
__device__ __forceinline__ uint32_t sq_code(float v, float lo, float delta, double inv, float &decoded) {
  constexpr uint32_t top = (1u << BITS) - 1u;
  const float quot = (float)((double)__fsub_rn(v, lo) * inv);
  const float u = __fadd_rn(quot, 0.5f);
  // (a NaN counts as 0)
  const uint32_t c = !(u > 0.0f) ? 0u : (u >= (float)(top + 1) ? top : (uint32_t)u);
  decoded = __fadd_rn(lo, __fmul_rn(delta, (float)c));
  return c;
}

// Squared norm of a decoded row in dimension order, by a whole wavefront (rarely needed, see above).
template <int BITS>
__device__ __forceinline__ float sq_norm_in_order(const float *xr, uint32_t d, const float *lo, const float *delta, const double *inv,
                                                  double *room) {
  double acc = 0.0;
  for (uint32_t base = 0; base < d; base += kWave) {
    const uint32_t j = base + (uint32_t)lane_id();
    float v = 0.0f;
    if (j < d) (void)sq_code<BITS>(xr[j], lo[j], delta[j], inv[j], v);
    acc = add_in_order(acc, j < d ? (double)v * (double)v : 0.0, room);
  }
  return (float)acc;
}

// SINGLE: one piece per row, the columns' ranges stay in registers.
template <int BITS, int VEC, int LPR, bool SINGLE>
__global__ __launch_bounds__(256) void sq_encode_kernel(const float *__restrict__ x, uint64_t n, uint32_t d,
                                                        const float *__restrict__ lo, const float *__restrict__ delta,
                                                        uint8_t *__restrict__ codes, float *__restrict__ norm_term) {
  extern __shared__ double inv_s[];                        // [d]
  __shared__ double order_room[4][kWave];
  float *lo_s = reinterpret_cast<float *>(inv_s + d);      // [d]
  float *delta_s = lo_s + d;                               // [d]
  for (uint32_t j = threadIdx.x; j < d; j += blockDim.x) {
    const float dl = delta[j];
    lo_s[j] = lo[j];
    delta_s[j] = dl;
    inv_s[j] = 1.0 / (double)dl;
  }
  __syncthreads();
  constexpr int RPG = kWave / LPR;   // rows side by side in a wavefront
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, sub = lane % LPR, grp = lane / LPR;
  const uint32_t row_bytes = BITS == 8 ? d : d / 2, nv = d / VEC;
  const uint32_t pieces = SINGLE ? 1u : (nv + LPR - 1) / LPR;
  const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / kWave);
  float lo_r[VEC], delta_r[VEC];
  double inv_r[VEC];
  auto columns = [&](uint32_t j0) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      lo_r[e] = lo_s[j0 + e];
      delta_r[e] = delta_s[j0 + e];
      inv_r[e] = inv_s[j0 + e];
    }
  };
  if (SINGLE) columns((uint32_t)sub < nv ? (uint32_t)sub * VEC : 0u);
  const uint64_t groups = (n + kEncRows * RPG - 1) / (kEncRows * RPG);
  for (uint64_t t = (uint64_t)blockIdx.x * (blockDim.x / kWave) + wave; t < groups; t += waves) {
    const uint64_t base = (groups - 1 - t) * (kEncRows * RPG);
    double acc[kEncRows];
#pragma unroll
    for (int r = 0; r < kEncRows; ++r) acc[r] = 0.0;
    for (uint32_t p = 0; p < pieces; ++p) {
      const uint32_t v = p * LPR + (uint32_t)sub;
      const bool in = v < nv;
      const uint32_t j0 = in ? v * VEC : 0u;
      if (!SINGLE) columns(j0);
      // (loads past the last row or the row's end are clamped into the array, so that none is conditional)
      float xv[kEncRows][VEC];
#pragma unroll
      for (int r = 0; r < kEncRows; ++r) {
        const uint64_t i = base + (uint32_t)(r * RPG + grp);
        const float *at = x + (i < n ? i : n - 1) * d + j0;
        if constexpr (VEC == 4) {
          const float4 t = *reinterpret_cast<const float4 *>(at);
          xv[r][0] = t.x, xv[r][1] = t.y, xv[r][2] = t.z, xv[r][3] = t.w;
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) xv[r][e] = at[e];
        }
      }
#pragma unroll
      for (int r = 0; r < kEncRows; ++r) {
        const uint64_t i = base + (uint32_t)(r * RPG + grp);
        uint32_t word = 0;
        double sum = acc[r];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          float dec;
          word |= sq_code<BITS>(xv[r][e], lo_r[e], delta_r[e], inv_r[e], dec) << (BITS * e);
          sum = fma((double)dec, (double)dec, sum);
        }
        acc[r] = in ? sum : acc[r];
        if (in && i < n) {
          uint8_t *to = codes + i * row_bytes + (BITS == 8 ? j0 : j0 / 2);
          if constexpr (BITS * VEC == 32)
            *reinterpret_cast<uint32_t *>(to) = word;
          else if constexpr (BITS * VEC == 16)
            *reinterpret_cast<uint16_t *>(to) = (uint16_t)word;
          else
            *to = (uint8_t)word;
        }
      }
    }
    if (!norm_term) continue;
    // Sums over the row's lanes, all rows of the lane together: an exchange
    // with the lane next door halves the rows a lane still carries, so that
    // after three of them lane `sub` holds a part of row sub % 8 alone.
    static_assert(kEncRows == 8, "three halvings");
    double part;
    {
      double h4[4], h2[2];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double keep = (sub & 1) ? acc[2 * k + 1] : acc[2 * k], give = (sub & 1) ? acc[2 * k] : acc[2 * k + 1];
        h4[k] = keep + xor_lane_f64(give, 1);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double keep = (sub & 2) ? h4[2 * k + 1] : h4[2 * k], give = (sub & 2) ? h4[2 * k] : h4[2 * k + 1];
        h2[k] = keep + xor_lane_f64(give, 2);
      }
      const double keep = (sub & 4) ? h2[1] : h2[0], give = (sub & 4) ? h2[0] : h2[1];
      part = keep + xor_lane_f64(give, 4);
#pragma unroll
      for (int m = 8; m < LPR; m <<= 1) part += xor_lane_f64(part, m);
    }
    const uint64_t i = base + (uint32_t)((sub & 7) * RPG + grp);
    const bool mine = sub < 8 && i < n;
    float norm;
    const bool sure = certain_f32(part, part, d, norm);
    if (mine && sure) norm_term[i] = norm;
    for (uint64_t todo = __ballot(mine && !sure); todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const uint64_t row = base + (uint32_t)(((l % LPR) & 7) * RPG + l / LPR);
      const float in_order = sq_norm_in_order<BITS>(x + row * d, d, lo_s, delta_s, inv_s, order_room[wave]);
      if (lane == 0) norm_term[row] = in_order;
    }
  }
}

// ------------------------------------------------------------- query folding
// One wavefront per query.  a_j = delta_j q_j; s = max|a|/127; t_j =
// rint(a_j * (127/max|a|)) in [-127,127]; qlo = sum_j q_j lo_j, the fp64 sum in
// dimension order rounded once to fp32.  Writes the folded query in the layout the
// search kernels load (see chunk_dot) and optionally as plain [nq][d] int8.
// Bound: latency.  The three arrays are read once, four loads each in flight, the
// products kept in LDS and the bytes written four at a time; the sum is formed by
// all lanes (certain_f32 tells whether dimension order could round to another
// float; then it is formed that way).  1,000 x 960: 28 us (a load, a byte and one
// lane's addition after the other) -> 13.
template <int BITS>
__global__ __launch_bounds__(64) void query_prep_kernel(const float *__restrict__ q, uint32_t nq, uint32_t d,
                                                        const float *__restrict__ lo, const float *__restrict__ delta,
                                                        uint8_t *__restrict__ tq, uint32_t tq_stride,
                                                        uint32_t tq_plane, uint32_t nq_cap,
                                                        float *__restrict__ s_ws, float *__restrict__ qlo_ws,
                                                        int32_t *__restrict__ sum_t_ws, int8_t *__restrict__ t_plain,
                                                        float *__restrict__ s_out, float *__restrict__ qlo_out) {
  // One plane: the int8 query.  Two planes (tq_stride == 2 * tq_plane): the
  // 15-bit query t = 128 * hi + lo with lo in [-64, 63], high bytes first.
  const bool q15 = tq_stride != tq_plane;
  const float top = q15 ? 16256.0f : 127.0f;
  const uint32_t qi = blockIdx.x;
  if (qi >= nq) return;
  const int lane = threadIdx.x;
  const float *qr = q + (uint64_t)qi * d;
  extern __shared__ float a_s[];   // [d] the products delta_j q_j
  __shared__ double order_room[kWave];
  float amax = 0.0f;
  double part = 0.0, mag = 0.0;    // sum of q_j lo_j (every product is exact in fp64) and of its terms' magnitudes
  constexpr int kBatch = 4;        // loads in flight per lane and array
  for (uint32_t base = 0; base < d; base += kBatch * kWave) {
    float qv[kBatch], dv[kBatch], lv[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const uint32_t j = base + u * kWave + lane, jc = j < d ? j : d - 1;
      qv[u] = qr[jc];
      dv[u] = delta[jc];
      lv[u] = lo[jc];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const uint32_t j = base + u * kWave + lane;
      if (j >= d) continue;
      const float a = __fmul_rn(dv[u], qv[u]);
      a_s[j] = a;
      amax = fmaxf(amax, fabsf(a));
      const double p = (double)qv[u] * (double)lv[u];
      part += p;
      mag += fabs(p);
    }
  }
  amax = wave_max_f32(amax);
  float s = 1.0f, r = 0.0f;
  if (amax > 0.0f) {
    s = __fdiv_rn(amax, top);
    r = __fdiv_rn(top, amax);
  }
  __syncthreads();
  uint32_t *tq_row = reinterpret_cast<uint32_t *>(tq + (uint64_t)qi * tq_stride);
  int sum = 0, sum_lo = 0;
  const int limit = q15 ? 16256 : 127;
  // four bytes of the kernel layout per lane and step
  for (uint32_t w = lane; w < tq_plane / 4; w += kWave) {
    uint32_t word = 0, word_lo = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t dim = folded_dim<BITS>(w, (uint32_t)e);
      int ti = 0;
      if (dim < d) {
        ti = __float2int_rn(__fmul_rn(a_s[dim], r));  // round half to even
        ti = ti > limit ? limit : (ti < -limit ? -limit : ti);
        if (t_plain) {
          if (q15)
            reinterpret_cast<int16_t *>(t_plain)[(uint64_t)qi * d + dim] = (int16_t)ti;
          else
            t_plain[(uint64_t)qi * d + dim] = (int8_t)ti;
        }
      }
      if (q15) {
        const int low = ((ti + 64) & 127) - 64, high = (ti - low) >> 7;
        word |= (uint32_t)(uint8_t)(int8_t)high << (8 * e);
        word_lo |= (uint32_t)(uint8_t)(int8_t)low << (8 * e);
        sum += high;
        sum_lo += low;
      } else {
        word |= (uint32_t)(uint8_t)(int8_t)ti << (8 * e);
        sum += ti;
      }
    }
    tq_row[w] = word;
    if (q15) tq_row[tq_plane / 4 + w] = word_lo;
  }
  sum = group_sum_i32<64>(sum);
  sum_lo = group_sum_i32<64>(sum_lo);
  part = group_sum_f64<64>(part);
  mag = group_sum_f64<64>(mag);
  float qlo;
  if (!certain_f32(part, mag, d, qlo)) qlo = dot_in_order(qr, lo, d, order_room);   // (the same in all lanes)
  if (lane == 0) {
    s_ws[qi] = s;
    qlo_ws[qi] = qlo;
    sum_t_ws[qi] = sum;
    sum_t_ws[nq_cap + qi] = sum_lo;
    if (s_out) s_out[qi] = s;
    if (qlo_out) qlo_out[qi] = qlo;
  }
}

ann_status launch_query_prep_into(const ann_index *ix, uint32_t level, const float *q, uint32_t nq, const Workspace &w,
                                  int8_t *t_plain, float *s_out, float *qlo_out, hipStream_t st) {
  const LevelDev &L = ix->level[level];
  const size_t smem = (size_t)ix->d * sizeof(float);
  if (L.bits == 8)
    query_prep_kernel<8><<<nq, 64, smem, st>>>(q, nq, ix->d, L.lo, L.delta, w.tq, w.tq_stride, w.tq_plane, w.nq_cap, w.s, w.qlo, w.sum_t,
                                               t_plain, s_out, qlo_out);
  else
    query_prep_kernel<4><<<nq, 64, smem, st>>>(q, nq, ix->d, L.lo, L.delta, w.tq, w.tq_stride, w.tq_plane, w.nq_cap, w.s, w.qlo, w.sum_t,
                                               t_plain, s_out, qlo_out);
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

ann_status launch_query_prep(ann_index *ix, uint32_t level, const float *q, uint32_t nq, int8_t *t_plain, float *s_out,
                             float *qlo_out, hipStream_t st, WorkspaceLease &lease) {
  ann_status rc = workspace_for(ix, level, nq, st, lease);
  if (rc != ANN_OK) return rc;
  rc = launch_query_prep_into(ix, level, q, nq, *lease.ws, t_plain, s_out, qlo_out, st);
  if (rc != ANN_OK) return rc;
  lease.ws->folded_q = q;
  lease.ws->folded_nq = nq;
  return ANN_OK;
}

// Workgroups of 256 to 4,096 rows, about a thousand (two and more fit a compute unit).
static dim3 select_grid(uint64_t n, uint32_t d, uint64_t &rows_per_block) {
  const uint32_t groups = (d + kSelCols - 1) / kSelCols;
  rows_per_block = n * groups / 1024;
  rows_per_block = rows_per_block < 256 ? 256 : (rows_per_block > 4096 ? 4096 : rows_per_block);
  return dim3((uint32_t)((n + rows_per_block - 1) / rows_per_block), groups);
}

// For bracket_collect_kernel: whole turns of workgroups (four to a compute unit) of at most
// 6,144 rows, of which about 1.4 % lie in a bracket and find room in LDS.  200,000 x 960: 1,470 workgroups
// of 4,096 rows, a second turn less than half full, 207 us; 1,020 of 5,883 190.
static dim3 collect_grid(uint64_t n, uint32_t d) {
  const uint32_t turn = 4 * compute_units(), groups = (d + kSelCols - 1) / kSelCols, side = groups < turn ? turn / groups : 1;
  uint64_t blocks = (n + 6144ull * side - 1) / (6144ull * side) * side;
  if (blocks > (n + 255) / 256) blocks = (n + 255) / 256;
  return dim3((uint32_t)blocks, groups);
}

// The truncated range by brackets from a sample, if that is to be expected to work (`done`: it did).
static ann_status train_bracketed(const float *x, uint64_t n, uint32_t d, uint32_t k, float levels, float *lo, float *delta,
                                  hipStream_t st, bool &done) {
  // the smallest sample whose brackets hold few values
  const double p = ((double)k + 0.5) / (double)n;
  BracketArgs g{};
  double expected = 0.0, deviation = 0.0;
  for (uint32_t m = 8192; m <= 32768 && n >= 4ull * m && (g.m == 0 || expected > 6000.0); m *= 2) {
    g.m = m;
    deviation = sqrt((double)m * p * (1.0 - p)) + 1.0;
    expected = (2.0 * (kBracketWidth + 0.5) * deviation + 4.0) / m * (double)n;
  }
  // (with more values in the brackets the lists cost more than three passes: 1M x 128, coverage 0.9, 2 %: 524 us / 290, 0.6, 3.3 %: 527 / 900)
  if (g.m == 0 || expected > 0.3 * kBracketMost || expected > 0.022 * (double)n) return ANN_OK;
  g.x = x;
  g.n = n;
  g.d = d;
  g.k = k;
  g.below = p * g.m - kBracketWidth * deviation - 1.0;
  g.beyond = p * g.m + kBracketWidth * deviation + 2.0;
  g.slack = deviation;
  g.room = 3.0 * expected + 256.0 < kBracketMost ? (uint32_t)(3.0 * expected) + 256 : kBracketMost;
  const uint64_t ends = 2ull * d, words = (uint64_t)d * g.m + ends * g.room + 7 * ends + 1;
  uint32_t *base = nullptr;
  if (device_alloc((void **)&base, words * sizeof(uint32_t)) != hipSuccess) {
    (void)hipGetLastError();
    return ANN_OK;   // (the radix passes need less)
  }
  g.sample = base;
  g.list = g.sample + (uint64_t)d * g.m;
  g.a = g.list + ends * g.room;
  g.b = g.a + ends;
  g.outside = g.b + ends;
  g.at_a = g.outside + ends;
  g.at_b = g.at_a + ends;
  g.inside = g.at_b + ends;
  uint32_t *prefix = g.inside + ends;
  g.failed = prefix + ends;
  bracket_sample_kernel<<<dim3(g.m / 64, (d + 63) / 64), 256, 0, st>>>(g);
  static_assert(kBracketKeys * 1024 == 32768, "keys per thread");
  if (g.m == 8192)
    bracket_bounds_kernel<256><<<d, 256, 0, st>>>(g);
  else if (g.m == 16384)
    bracket_bounds_kernel<512><<<d, 512, 0, st>>>(g);
  else
    bracket_bounds_kernel<1024><<<d, 1024, 0, st>>>(g);
  bracket_collect_kernel<<<collect_grid(n, d), kSelBlock, 0, st>>>(g);
  if (expected <= 8192.0)
    bracket_pick_kernel<256><<<(uint32_t)ends, 256, 0, st>>>(g, prefix);
  else
    bracket_pick_kernel<1024><<<(uint32_t)ends, 1024, 0, st>>>(g, prefix);
  truncated_range_kernel<<<(d + 255) / 256, 256, 0, st>>>(prefix, d, levels, lo, delta);
  uint32_t failed = 1;
  const hipError_t e = hipGetLastError();
  const hipError_t e2 = e == hipSuccess ? read_words(g.failed, &failed, 1, st) : hipStreamSynchronize(st);
  device_free(base, e2 == hipSuccess);
  if (e != hipSuccess) return hip_fail(e, "ann_sq_train_truncated");
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  done = failed == 0;
  return ANN_OK;
}

}  // namespace ann

using namespace ann;

extern "C" {

ann_status ann_sq_train(const float *x, uint64_t n, uint32_t d, uint32_t bits, float *lo, float *delta, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!x || !lo || !delta) return fail(ANN_EINVAL, "ann_sq_train: NULL argument");
  if (n == 0 || d == 0) return fail(ANN_EINVAL, "ann_sq_train: empty input");
  if (bits != 8 && bits != 4) return fail(ANN_EINVAL, "ann_sq_train: bits must be 4 or 8");
  // about a thousand workgroups (four per compute unit), none with so few rows that a thread has fewer than eight
  const bool vec4 = d % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
  const uint32_t pieces = vec4 ? d / 4 : d;
  const uint32_t side = pieces < (uint32_t)kMinmaxThreads ? kMinmaxThreads / pieces : 1u;
  uint64_t rows_per_block = (n + 1023) / 1024;
  if (rows_per_block < (uint64_t)kMinmaxUnroll * side) rows_per_block = (uint64_t)kMinmaxUnroll * side;
  const uint32_t nblocks = (uint32_t)((n + rows_per_block - 1) / rows_per_block);
  float *pmin = nullptr;
  ANN_HIP(device_alloc((void **)&pmin, (size_t)nblocks * d * 2 * sizeof(float)));
  float *pmax = pmin + (size_t)nblocks * d;
  const dim3 grid(nblocks, (pieces + kMinmaxThreads - 1) / kMinmaxThreads);
  if (vec4)
    sq_minmax_partial_kernel<4><<<grid, kMinmaxThreads, 0, st>>>(x, n, d, pmin, pmax);
  else
    sq_minmax_partial_kernel<1><<<grid, kMinmaxThreads, 0, st>>>(x, n, d, pmin, pmax);
  sq_minmax_final_kernel<<<(d + kFinalCols - 1) / kFinalCols, kFinalCols * kFinalRows, 0, st>>>(
      pmin, pmax, nblocks, d, (float)((1u << bits) - 1u), lo, delta);
  hipError_t e = hipGetLastError();
  hipError_t e2 = hipStreamSynchronize(st);
  device_free(pmin, e2 == hipSuccess);
  if (e != hipSuccess) return hip_fail(e, "sq_minmax launch");
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  return ANN_OK;
}

ann_status ann_sq_train_truncated(const float *x, uint64_t n, uint32_t d, uint32_t bits, double coverage, float *lo,
                                  float *delta, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!x || !lo || !delta) return fail(ANN_EINVAL, "ann_sq_train_truncated: NULL argument");
  if (n == 0 || n >= (1ull << 31) || d == 0) return fail(ANN_EINVAL, "ann_sq_train_truncated: empty input or n >= 2^31");
  if (bits != 8 && bits != 4) return fail(ANN_EINVAL, "ann_sq_train_truncated: bits must be 4 or 8");
  if (!(coverage > 0.5 && coverage <= 1.0)) return fail(ANN_EINVAL, "ann_sq_train_truncated: coverage must be in (0.5, 1]");
  const uint64_t k = (uint64_t)floor((1.0 - coverage) * (double)(n - 1));
  bool done = false;
  ann_status rc = train_bracketed(x, n, d, (uint32_t)k, (float)((1u << bits) - 1u), lo, delta, st, done);
  if (rc != ANN_OK || done) return rc;
  uint32_t *hist = nullptr;  // [2][d][256], then prefix[2][d] and rank[2][d]
  const size_t n_hist = (size_t)512 * d;
  ANN_HIP(device_alloc((void **)&hist, (n_hist + (size_t)4 * d) * sizeof(uint32_t)));
  uint32_t *prefix = hist + n_hist, *rank = prefix + (size_t)2 * d;
  uint64_t rows_per_block;
  const dim3 grid = select_grid(n, d, rows_per_block);
  radix_init_kernel<<<(uint32_t)((n_hist + 255) / 256), 256, 0, st>>>(d, (uint32_t)k, (uint32_t)(n - 1 - k), prefix, rank, hist);
  for (int shift = 24; shift >= 0; shift -= 8) {
    radix_hist_kernel<<<grid, kSelBlock, 0, st>>>(x, n, d, (uint32_t)rows_per_block, shift, prefix, hist);
    radix_pick_kernel<<<2 * d, 64, 0, st>>>(hist, prefix, rank);
  }
  truncated_range_kernel<<<(d + 255) / 256, 256, 0, st>>>(prefix, d, (float)((1u << bits) - 1u), lo, delta);
  hipError_t e = hipGetLastError();
  const hipError_t e2 = hipStreamSynchronize(st);
  device_free(hist, e2 == hipSuccess);
  if (e != hipSuccess) return hip_fail(e, "ann_sq_train_truncated");
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  return ANN_OK;
}

ann_status ann_sq_encode(const float *x, uint64_t n, uint32_t d, uint32_t bits, const float *lo, const float *delta,
                         uint8_t *codes, float *norm_term, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!x || !lo || !delta || !codes) return fail(ANN_EINVAL, "ann_sq_encode: NULL argument");
  if (n == 0 || d == 0) return fail(ANN_EINVAL, "ann_sq_encode: empty input");
  if (bits != 8 && bits != 4) return fail(ANN_EINVAL, "ann_sq_encode: bits must be 4 or 8");
  if (bits == 4 && (d & 1)) return fail(ANN_EINVAL, "ann_sq_encode: 4-bit codes need an even d");
  if (d > 2048) return fail(ANN_ECAPACITY, "ann_sq_encode: d = %u exceeds 2048", d);
  // pieces of four dimensions need 16-byte rows of x and codes that can be
  // stored four (8 bits) or two (4 bits) bytes at a time
  const bool vec4 = d % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(codes) % 4 == 0;
  const uint32_t vec = vec4 ? 4u : (bits == 8 ? 1u : 2u), pieces = d / vec;
  uint32_t lpr = 8;
  while (lpr < pieces && lpr < (uint32_t)kWave) lpr <<= 1;
  const uint64_t rows_per_block = (uint64_t)(256 / kWave) * kEncRows * (kWave / lpr);
  const uint64_t want = (n + rows_per_block - 1) / rows_per_block;
  const int grid = (int)(want > 2048 ? 2048 : want);   // eight workgroups per compute unit
  const size_t smem = (size_t)d * (sizeof(double) + 2 * sizeof(float));
#define ANN_ENC(B, V, L, S) sq_encode_kernel<B, V, L, S><<<grid, 256, smem, st>>>(x, n, d, lo, delta, codes, norm_term)
#define ANN_ENC_LPR(B, V)                                    \
  do {                                                       \
    switch (lpr) {                                           \
      case 8: ANN_ENC(B, V, 8, true); break;                 \
      case 16: ANN_ENC(B, V, 16, true); break;               \
      case 32: ANN_ENC(B, V, 32, true); break;               \
      default:                                               \
        if (pieces <= (uint32_t)kWave)                       \
          ANN_ENC(B, V, 64, true);                           \
        else                                                 \
          ANN_ENC(B, V, 64, false);                          \
    }                                                        \
  } while (0)
  if (bits == 8) {
    if (vec4)
      ANN_ENC_LPR(8, 4);
    else
      ANN_ENC_LPR(8, 1);
  } else {
    if (vec4)
      ANN_ENC_LPR(4, 4);
    else
      ANN_ENC_LPR(4, 2);
  }
#undef ANN_ENC_LPR
#undef ANN_ENC
  ANN_HIP(hipGetLastError());
  ANN_HIP(hipStreamSynchronize(st));
  return ANN_OK;
}

ann_status ann_query_prep(ann_index *index, uint32_t level, const float *q, uint32_t nq, int8_t *t, float *s, float *qlo,
                          void *stream) {
  if (!index || !q) return fail(ANN_EINVAL, "ann_query_prep: NULL argument");
  if (level >= index->n_levels) return fail(ANN_EINVAL, "ann_query_prep: level %u not in the index", level);
  if (nq == 0) return fail(ANN_EINVAL, "ann_query_prep: nq == 0");
  WorkspaceLease lease;
  return launch_query_prep(index, level, q, nq, t, s, qlo, (hipStream_t)stream, lease);
}

}  // extern "C"
