// Exact k nearest neighbours by exhaustive search: the ground truth NN_k of
// the paper's recall measure (Section 6.1).
//
// Scores that only select candidates: -2 q.x + |x|^2 (or -q.x) from a dense
// contraction on the matrix cores, every fp32 value split into three bf16
// parts and six of the nine partial products accumulated in fp32, or into two
// half-precision parts and three of the four products; for vectors of like
// sizes neither loses more than fp32 products do (see bf_score_kernel).  With many queries only the product of the first
// half-precision parts is taken, and every row that this product, less the most it can err, leaves among the best is
// re-evaluated in fp64 before it is selected (see screen_room).  Between `want` = k + 8 and
// `most`, half as many again, of a query's best rows are re-evaluated in fp64 by
// the rerank kernel and sorted by (distance, id).
//
// Selection without a top-k structure in the contraction kernel:
//   few rows   all scores are written out and a selection kernel takes the best
//              of every stretch of 4,096, another the best of those;
//   otherwise  a stratified random sample of 4,096 or 8,192 rows gives every
//              query a (score, id) bound that k + 8 rows of the sample reach; a
//              sample `growth` times larger (at most 32 times), of which only
//              what reaches the bound is written, gives a tighter one, and so on
//              until the sample would be the whole set; the last pass takes all
//              rows in order and writes what reaches the last bound: about
//              `growth` times k + 8 .. `most_bound` entries per query (room for
//              `cap`) whatever the distribution of the data, since the rank of a
//              random sample's order statistic does not depend on it.
// A result is certain if its k-th distance is smaller than the score of the first
// row left out allows, less the error that score may have.  Ordinary data leave
// many times that error between the k-th row and the first left out (no query of
// the calls below was uncertain); those that are not certain (vectors far from
// the origin, many equal distances, entries beyond their room) are taken up
// again, see settle().
//
// Whole calls, before (fp32 products, top-k lists in LDS kept by the contraction
// kernel, every slab's list re-evaluated) and now: 10,000 queries x 1M x 128,
// k = 10: 25.8 -> 3.51 to 3.75 ms, by the card (15.5 with three parts, 7.4 to 8.3 with two); 2,000 x 200,000
// x 768, k = 100: 13.9 -> 1.38 to 1.43 (3.8, 2.27 to 2.41); 100 x 10,000 x 128, k = 10: 2.56 -> 0.056.
#include <math.h>

#include <type_traits>

#include "ann_internal.hpp"
#include "device_utils.hpp"
#include "kept_blocks.hpp"

namespace ann {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kQT = 32;    // queries per workgroup
constexpr int kBT = 128;   // base vectors per tile (4 wavefronts x 32)
constexpr int kKC = 32;    // K chunk staged in LDS
constexpr int kLd = kKC + 1;  // padded row length (floats): conflict-free column reads

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, uint32_t n, uint32_t v) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void row_norm_kernel(const float *__restrict__ x, uint64_t n, uint32_t d, float *__restrict__ out) {
  const int lane = threadIdx.x % kWave;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const uint64_t n_waves = (uint64_t)gridDim.x * blockDim.x / kWave;
  for (uint64_t i = wave; i < n; i += n_waves) {
    float acc = 0.f;
    for (uint32_t j = lane; j < d; j += kWave) {
      float v = x[i * d + j];
      acc = fmaf(v, v, acc);
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) acc += __int_as_float(xor_lane_i32(__float_as_int(acc), m));
    if (lane == 0) out[i] = acc;
  }
}

// One workgroup: kQT queries against base rows [slab*rows_per_slab, ...).
// The K dimension is walked in chunks of kKC; the next chunk of Q and X is
// fetched into registers while the matrix cores work on the current one, then
// written to the other half of a double-buffered LDS tile (one barrier per
// chunk).  LDS: Qs[2][kQT][kLd], Xs[2][kBT][kLd], thr[kQT], cnt[kQT],
// buf[kQT][cb] (u64).
// VEC4: rows are read as float4 (needs d % 4 == 0).
template <bool VEC4>
__global__ __launch_bounds__(256) void bf_tile_kernel(const float *__restrict__ X, const float *__restrict__ xnorm,
                                                      uint64_t n, uint32_t d, const float *__restrict__ Q, uint32_t nq,
                                                      uint32_t metric, uint64_t rows_per_slab, uint32_t kp, uint32_t cb,
                                                      uint32_t *__restrict__ cand_out /*[nq][slabs][kp]*/) {
  extern __shared__ float smem_f[];
  float *Qs = smem_f;                    // [2][kQT][kLd]
  float *Xs = Qs + 2 * kQT * kLd;        // [2][kBT][kLd]
  float *thr = Xs + 2 * kBT * kLd;
  uint32_t *cnt = reinterpret_cast<uint32_t *>(thr + kQT);
  uint64_t *buf = reinterpret_cast<uint64_t *>(cnt + kQT);  // offset is a multiple of 8 bytes

  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const uint32_t q0 = blockIdx.x * kQT;
  const uint32_t slab = blockIdx.y, n_slabs = gridDim.y;
  const uint64_t b_begin = (uint64_t)slab * rows_per_slab;
  const uint64_t b_end = b_begin + rows_per_slab < n ? b_begin + rows_per_slab : n;

  if (tid < kQT) {
    thr[tid] = INFINITY;
    cnt[tid] = 0;
  }

  // staging registers: one float4 of Q and four of X per thread and chunk
  // (kQT*kKC = 1024 and kBT*kKC = 4096 floats over 256 threads)
  const int sc = (tid % 8) * 4;  // column inside the chunk
  const int sr = tid / 8;        // row 0..31 (+32 i for X)
  float4 rq, rx[4];
  auto fetch = [&](uint64_t t0, uint32_t k0) {
    const uint32_t kk = k0 + sc;
    const uint32_t qi = q0 + sr;
    rq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (qi < nq) {
      const float *p = Q + (uint64_t)qi * d + kk;
      if (VEC4) {
        if (kk < d) rq = *reinterpret_cast<const float4 *>(p);
      } else {
        if (kk + 0 < d) rq.x = p[0];
        if (kk + 1 < d) rq.y = p[1];
        if (kk + 2 < d) rq.z = p[2];
        if (kk + 3 < d) rq.w = p[3];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t bi = t0 + sr + 32 * i;
      rx[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (bi < b_end) {
        const float *p = X + bi * d + kk;
        if (VEC4) {
          if (kk < d) rx[i] = *reinterpret_cast<const float4 *>(p);
        } else {
          if (kk + 0 < d) rx[i].x = p[0];
          if (kk + 1 < d) rx[i].y = p[1];
          if (kk + 2 < d) rx[i].z = p[2];
          if (kk + 3 < d) rx[i].w = p[3];
        }
      }
    }
  };
  auto stage = [&](int b) {
    float *qd = Qs + (b * kQT + sr) * kLd + sc;
    qd[0] = rq.x;
    qd[1] = rq.y;
    qd[2] = rq.z;
    qd[3] = rq.w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float *xd = Xs + (b * kBT + sr + 32 * i) * kLd + sc;
      xd[0] = rx[i].x;
      xd[1] = rx[i].y;
      xd[2] = rx[i].z;
      xd[3] = rx[i].w;
    }
  };

  const uint32_t n_chunks = (d + kKC - 1) / kKC;
  int cur = 0;
  if (b_begin < b_end) {
    fetch(b_begin, 0);
    stage(0);
  }
  __syncthreads();

  for (uint64_t t0 = b_begin; t0 < b_end; t0 += kBT) {
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    for (uint32_t c = 0; c < n_chunks; ++c) {
      // next chunk (of this tile, or the first of the next tile) on its way
      const bool last_chunk = c + 1 == n_chunks;
      const uint64_t nt0 = last_chunk ? t0 + kBT : t0;
      const bool more = nt0 < b_end;
      if (more) fetch(nt0, last_chunk ? 0 : (c + 1) * kKC);
      const float *ap = Qs + (cur * kQT + lane % 32) * kLd + lane / 32;
      const float *bp = Xs + (cur * kBT + wave * 32 + lane % 32) * kLd + lane / 32;
#pragma unroll
      for (int kk = 0; kk < kKC; kk += 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ap[kk], bp[kk], acc, 0, 0, 0);
      if (more) stage(cur ^ 1);
      __syncthreads();
      cur ^= 1;
    }
    // scores and threshold filter.  acc[i] belongs to query row
    // 8*(i/4) + 4*(lane/32) + i%4 and base column lane%32 of this wave.
    const uint64_t bi = t0 + wave * 32 + lane % 32;
    const bool live = bi < b_end;
    const float xn = (live && metric == ANN_L2) ? xnorm[bi] : 0.f;
    bool pushed = false;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = 8 * (i / 4) + 4 * (lane / 32) + (i % 4);
      const float score = metric == ANN_L2 ? fmaf(-2.0f, acc[i], xn) : -acc[i];
      if (live && q0 + row < nq && score < thr[row]) {
        uint32_t pos = atomicAdd(&cnt[row], 1u);
        buf[(size_t)row * cb + pos] = ((uint64_t)order_u32(score) << 32) | (uint32_t)bi;
        pushed = true;
      }
    }
    // tiles that pushed nothing (the common case once the thresholds have
    // settled) skip the compaction pass
    if (__syncthreads_or(pushed ? 1 : 0) == 0) continue;
    // keep the kp best of every row that grew beyond kp (each wave owns 8 rows)
    for (int row = wave; row < kQT; row += 4) {
      const uint32_t c = cnt[row];
      if (c <= kp) continue;
      uint64_t *list = buf + (size_t)row * cb;
      uint64_t mine[8];
      uint32_t rank[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t i = lane + u * kWave;
        mine[u] = i < c ? list[i] : ~0ull;
        rank[u] = 0;
      }
      for (uint32_t j = 0; j < c; ++j) {
        const uint64_t o = list[j];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank[u] += o < mine[u] ? 1u : 0u;   // ids differ, so no ties
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t i = lane + u * kWave;
        if (i < c && rank[u] < kp) {
          list[rank[u]] = mine[u];
          if (rank[u] == kp - 1) thr[row] = unorder_f32((uint32_t)(mine[u] >> 32));
        }
      }
      if (lane == 0) cnt[row] = kp;
    }
    __syncthreads();
  }
  // hand the survivors of this slab to the exact stage
  for (int e = tid; e < kQT * (int)kp; e += 256) {
    const int row = e / kp, j = e % kp;
    const uint32_t qi = q0 + row;
    if (qi < nq)
      cand_out[((uint64_t)qi * n_slabs + slab) * kp + j] = (uint32_t)j < cnt[row] ? (uint32_t)buf[(size_t)row * cb + j] : ANN_PAD_ID;
  }
}

// ---------------------------------------------------------------------------
// Scores on the 16-bit matrix cores.
//
// PARTS = 3: a float is the sum of three bf16 values (8 + 8 + 8 bits; rounding to nearest
// each time, the remainders are exact).  Of the nine products of two such sums
// the three smallest (below 2^-25 of the product) are left out.  The fp32 matrix
// rate is 157 TFLOP/s; six bf16 products at 2.5 PFLOP/s leave 417 of the same.
// Root mean square error of a score against 64 bits, relative to that of the
// scores (128 queries x 4,096 rows; in brackets: fp32 products and norms):
//   inner products of mixtures   d = 24 5.5e-8 (7.5e-8), 128 1.4e-7 (1.7e-7),
//                                960 3.1e-7 (4.2e-7), 2,048 4.0e-7 (6.1e-7)
//   L2, centred normal vectors   128 5.7e-8 (6.0e-8), 960 5.2e-8 (5.5e-8),
//                                2,048 6.2e-8 (6.3e-8)
//   L2, offset of 1,000 spreads  128 2.2e-7 (3.0e-7), 960 8.7e-7 (8.6e-7),
//                                2,048 1.3e-6 (1.2e-6)
// (likewise for uniform, unit-norm and stretched vectors).  Only the last two are
// larger than with fp32 products; such results are settled with centred rows.
//
// PARTS = 2: half precision carries 11 bits, so two parts hold a float but for one
// bit (a remainder below 2^-23 of it), if its size allows: rows times one power of
// two, each query times its own, have norms of about 2^12, of 2^16 that the format ends at;
// what falls below its smallest value, 2^-24, is 2^-36 of the norm.  Rows 8 times larger than
// the largest of a sample are left out (L2: a result they might belong to is uncertain; inner product:
// they are listed, and the call is repeated with three parts if they are many).  The product of the
// two second parts, below 2^-22 of the product, is left out.  That is half the products, and
// half the roundings of the accumulators, which are the larger error from 65 columns on.
// Error as above, three parts / two (norms in fp64):
//   L2 of mixtures   d = 72 7.3e-8 / 6.8e-8, 128 1.04e-7 / 8.5e-8, 960 2.1e-7 / 1.8e-7,
//                    2,048 3.0e-7 / 2.7e-7
//   inner products   128 1.4e-7 / 1.0e-7, 960 3.1e-7 / 2.6e-7; centred normal 128 1.6e-7 /
//                    1.4e-7, 48 9.1e-8 / 1.04e-7, 24 6.0e-8 / 9.2e-8 (there three are taken)
//   offset of 1,000 spreads, L2   128 2.2e-7 / 1.8e-7, 960 8.7e-7 / 5.3e-7
// The format holds 22 to 23 bits of a float's 24, so two parts are not the more exact ones everywhere: of
// mixtures with 8 to 100 centres and 65 to 128 columns the scores of a query's 50 nearest rows err 15 to 28 %
// less than with three, all scores together between 25 % less and (65 columns, inner product) 4 % more; inner
// products of centred normal vectors 10 % more at 65 columns, 5 % at 96 and less from 128 on; of norms spread
// over four orders of magnitude 6 to 28 % more up to 256 columns, rows below 2^-14 of the largest far more
// (the arithmetic in numpy, a rounding per instruction).  Scores only select; what an error could
// change is found out from half_room() and settled.
//
// A workgroup of four wavefronts takes QT queries x 128 base rows per tile.
// The queries come split, in the order the matrix instruction wants them
// (bf_split_queries_kernel), straight from global memory (they stay in the L2),
// one step ahead of their use.  The base rows are fetched a K chunk (32
// columns) ahead, split on the way into LDS (three planes of 64 bytes per row,
// the 16-byte slots of a row permuted with the row number so that eight rows
// read side by side hit all banks); their squared norms are summed on the way.
// One barrier per chunk.  128 queries: a wavefront has 128 rows x 32 queries,
// four accumulators (64 x 64 scores fetch twice the query parts per product: 3 to
// 5 % slower); up to 64 queries: 32 rows x 64; up to 32: 32 x 32 (then the kernel
// is bound by reading the base rows: 1M x 128 in 0.113 ms).
//
// Workgroup b runs on die b mod 8; slabs of rows belong to dies, and a die takes
// 16 query tiles (1.6 MB of parts at 128 dimensions) through all its slabs before
// the next 16, so that both stay in its 4 MB of L2 (all tiles at once: 66 GB fetched
// per pass instead of 10, 6 % slower).  From about 340 dimensions on 16 tiles'
// parts are more than that; other group sizes have not been measured there.
//
// Three parts, 10,112 queries x 1M x 128, a pass without entries: 13.4 ms = 193 TFLOP/s of fp32
// work = 1,160 on the matrix cores, at the 1.96 GHz the card runs such work (peak
// 2,050 there; a large bf16 matrix product reaches 1,420).  Without the query
// loads it takes 12.1, without the splitting 12.8.  Two parts: 10.2, bound by the
// splitting and the end of a tile.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

constexpr int kSK = 32;           // columns per chunk
constexpr int kSB = 128;          // base rows per tile
constexpr int kPlane = kSB * kSK * 2;   // bytes of one plane of a chunk
constexpr uint64_t kScreenBytes = 128ull << 20;   // of rows' first parts at a time
constexpr uint32_t kCallCounters = 12;   // of CallState
// One query in kVoters votes (additions to one counter, one after the other: by all of 10,000 queries 110 us; an odd number, so that
// workgroups that do are on all dies: 9,000 queries x 20,000 rows, one in sixteen 15 us, in seventeen 3).
constexpr uint32_t kVoters = 17;
constexpr int kHitList = 96;      // entries a wavefront collects before they go to global memory
constexpr float kFarNorm2 = 0x1.fp31f;   // two parts: rows of this squared norm and more, scaled, are left out (half precision ends at 2^16)
constexpr uint32_t kSampleRows = 4096;   // scores one selection workgroup takes; first sample (or twice that, see ann_bruteforce_topk)

// a, b -> their three bf16 parts, a's in the low halves
__device__ __forceinline__ void split3(float a, float b, uint32_t (&w)[3]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const floatx2 v = {a, b};
    w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    if (p < 2) {
      a = __fsub_rn(a, __uint_as_float(w[p] << 16));
      b = __fsub_rn(b, __uint_as_float(w[p] & 0xFFFF0000u));
    }
  }
}

// a and b times the power of two `scale` -> their two half-precision parts, a's in the low halves
__device__ __forceinline__ void split2(float a, float b, float scale, uint32_t (&w)[2]) {
  const halfx2 hi = {(_Float16)__builtin_fmaf(a, scale, 0.0f), (_Float16)__builtin_fmaf(b, scale, 0.0f)};
  const halfx2 lo = {(_Float16)__builtin_fmaf(a, scale, -(float)hi.x), (_Float16)__builtin_fmaf(b, scale, -(float)hi.y)};
  w[0] = __builtin_bit_cast(uint32_t, hi);
  w[1] = __builtin_bit_cast(uint32_t, lo);
}

// The power of two that brings a vector of squared norm sq to a norm of 2^12 to 2^13
// (2^-60 to 2^60; 1 for zero).
__device__ __forceinline__ int half_exponent(float sq) {
  if (!(sq > 0.0f && sq < INFINITY)) return 0;
  const int e = 12 - (ilogbf(sq) >> 1);
  return e < -60 ? -60 : (e > 60 ? 60 : e);
}

// Queries split and laid out as the second operand of the 32x32x16 matrix
// instruction: 16-byte unit (((q / 32) * KB + kb) * 3 + plane) * 64 + lane holds
// columns kb * 16 + 8 * (lane / 32) .. + 7 of query lane % 32.  Zero past the
// batch and past d.  centre (NULL: none) is subtracted.  Also the start of every
// query's selection (bound NULL: not wanted): no bound, no entries; and of a
// call (zero: its counters, or NULL).
__global__ __launch_bounds__(256) void bf_split_queries_kernel(const float *__restrict__ Q, uint32_t nq, uint32_t d, uint32_t kb_n,
                                                               uint32_t q32_n, const float *__restrict__ centre, uint4 *__restrict__ out,
                                                               uint64_t *__restrict__ bound, uint32_t *__restrict__ count,
                                                               uint32_t *__restrict__ zero) {
  if (zero && blockIdx.x == 0 && threadIdx.x < kCallCounters) zero[threadIdx.x] = 0u;
  const uint64_t total = (uint64_t)q32_n * kb_n * 64;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t lane = (uint32_t)(e % 64), kb = (uint32_t)(e / 64 % kb_n), q32 = (uint32_t)(e / 64 / kb_n);
    const uint32_t qi = q32 * 32 + lane % 32, k0 = kb * 16 + 8 * (lane / 32);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bool in = qi < nq && k0 + j < d;
      v[j] = in ? Q[(uint64_t)qi * d + k0 + j] : 0.0f;
      if (centre && in) v[j] = __fsub_rn(v[j], centre[k0 + j]);
    }
    if (bound && kb == 0 && lane < 32 && qi < nq) {
      bound[qi] = ~0ull;
      count[qi] = 0;
    }
    uint32_t w[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j) split3(v[2 * j], v[2 * j + 1], w[j]);
    uint4 *to = out + ((uint64_t)q32 * kb_n + kb) * 192 + lane;
#pragma unroll
    for (int p = 0; p < 3; ++p) to[p * 64] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
  }
}

// Largest squared norm (of those that are floats) of each 64th of a sample of
// kNormSample rows: out[64].  A wavefront per row.  Also the start of a call's counters.
constexpr uint32_t kNormSample = 1024;
__global__ __launch_bounds__(1024) void bf_sample_norms_kernel(const float *__restrict__ x, uint32_t d, double stretch, float *__restrict__ out,
                                                               uint32_t *__restrict__ zero) {
  __shared__ float sq_s[16];
  if (blockIdx.x == 0 && threadIdx.x < kCallCounters) zero[threadIdx.x] = 0u;
  const uint32_t wave = threadIdx.x / kWave;
  const float *row = x + sample_row(blockIdx.x * 16 + wave, stretch) * d;
  float sq = 0.0f;
  for (uint32_t j0 = 0; j0 < d; j0 += 4 * kWave) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t j = j0 + i * kWave + lane_id();
      v[i] = row[j < d ? j : 0];
      v[i] = j < d ? v[i] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sq = fmaf(v[i], v[i], sq);
  }
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) sq += __int_as_float(xor_lane_i32(__float_as_int(sq), m));
  if (lane_id() == 0) sq_s[wave] = sq < INFINITY ? sq : 0.0f;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) sq_s[0] = fmaxf(sq_s[0], sq_s[w]);
    out[blockIdx.x] = sq_s[0];
  }
}
__device__ __forceinline__ float rows_sq(const float *sample_sq) { return wave_max_f32(sample_sq[lane_id()]); }

// The same in two half-precision parts, each query times a power of two (2^-60 to
// 2^60) that brings its norm to 2^12 .. 2^13.  One workgroup per 32 queries and 16 blocks
// of columns: the norms first.  unscale[q]: what takes a product of parts back, the rows' scale included; norm[q]: at
// least |q|; rest[q]: at least the norm of what the first part leaves of it.
__global__ __launch_bounds__(1024) void bf_halve_queries_kernel(const float *__restrict__ Q, uint32_t nq, uint32_t d, uint32_t kb_n,
                                                                const float *__restrict__ sample_sq, uint4 *__restrict__ out,
                                                                float *__restrict__ unscale, float *__restrict__ norm, float *__restrict__ rest,
                                                                uint64_t *__restrict__ bound, uint32_t *__restrict__ count) {
  __shared__ float scale_s[32];
  const uint32_t q32 = blockIdx.x, tid = threadIdx.x;
  {
    const uint32_t qi = q32 * 32 + tid / 32;
    float sq = 0.0f;
    if (qi < nq)
      for (uint32_t j = tid % 32; j < d; j += 32) {
        const float v = Q[(uint64_t)qi * d + j];
        sq = fmaf(v, v, sq);
      }
#pragma unroll
    for (int m = 1; m < 32; m <<= 1) sq += __int_as_float(xor_lane_i32(__float_as_int(sq), m));
    const int e = half_exponent(sq), ex = half_exponent(rows_sq(sample_sq));
    const float scale = ldexpf(1.0f, e);
    float left = 0.0f;
    if (qi < nq && blockIdx.y == 0)
      for (uint32_t j = tid % 32; j < d; j += 32) {
        const float v = Q[(uint64_t)qi * d + j] * scale, lo = v - (float)(_Float16)v;
        left = fmaf(lo, lo, left);
      }
#pragma unroll
    for (int m = 1; m < 32; m <<= 1) left += __int_as_float(xor_lane_i32(__float_as_int(left), m));
    if (tid % 32 == 0) {
      scale_s[tid / 32] = scale;
      if (qi < nq && blockIdx.y == 0) {
        rest[qi] = __fsqrt_rn(left) * (1.0f + 0x1p-10f) * ldexpf(1.0f, -e);
        unscale[qi] = ldexpf(1.0f, -e - ex);
        norm[qi] = __fsqrt_rn(sq) * (1.0f + 0x1p-10f);   // (rounded up; infinite where the square is no float)
        bound[qi] = ~0ull;
        count[qi] = 0;
      }
    }
  }
  __syncthreads();
  const uint32_t lane = tid % 64, kb = blockIdx.y * 16 + tid / 64;
  if (kb < kb_n) {
    const uint32_t qi = q32 * 32 + lane % 32, k0 = kb * 16 + 8 * (lane / 32);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = qi < nq && k0 + j < d ? Q[(uint64_t)qi * d + k0 + j] : 0.0f;
    uint32_t w[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) split2(v[2 * j], v[2 * j + 1], scale_s[lane % 32], w[j]);
    uint4 *to = out + ((uint64_t)q32 * kb_n + kb) * 128 + lane;
#pragma unroll
    for (int p = 0; p < 2; ++p) to[p * 64] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
  }
}

// What a call learns on the device and the host reads at its end (or between steps).
constexpr uint32_t kFewFarRows = 64;   // two parts: with more of them the call is repeated with three
constexpr uint32_t kFarRows = 3840;   // (with 256 results they fit the 4,096 candidates of a rerank)
// (the kCallCounters words in front of the list of rows start at zero)
struct CallState {
  uint32_t n_uncertain;   // queries whose k-th distance is not certain (listed by the rerank kernel)
  uint32_t far_rows;      // inner product: rows whose squared norm is no float; the first kFarRows are listed
  uint32_t n_wide;        // two parts: queries whose scores would be nearer to their value with three
  uint32_t n_lost;        // first parts: queries for whose entries there was no room
  uint32_t abandoned;     // first parts: not 0: the passes were given up, all queries of the round and of those after it are lost
  uint32_t left_out;      // two parts, L2: not 0: rows were left out for their size
  uint32_t max_norm;      // inner product, or first parts: bits of the largest squared norm of the others
  uint32_t most_entries;  // of a query in the last pass over uncertain queries
  uint32_t n_next, n_fp32;   // uncertain queries for another pass; for the fp32 kernel
  uint32_t max_rest;      // first parts: bits of the largest squared norm of what they leave of a scaled row
  uint32_t n_hopeless;    // first parts: queries of which the pass before this one tells that they will be lost, see vote()
  uint32_t far_row[kFarRows];
};

// A pass of scores: its rows and queries, and where the scores go.
struct ScoreArgs {
  const float *x;
  const uint4 *qfrag;
  uint64_t first, rows;    // rows first .. first + rows - 1 of x, or of a sample of it
  double stretch;    // sample: rows of x per row of the sample; 0: none
  uint32_t d, kb_n, nq, metric;
  uint32_t q_tiles, q_group, slabs, tiles_per_slab;
  float *scores;     // not NULL: every score goes here, [nq][ld]
  uint32_t ld;
  const uint64_t *bound;   // [nq] otherwise: (score, id) pairs up to the bound go to buf
  uint64_t *buf;     // [nq][cap]
  uint32_t *count;   // [nq]
  uint32_t cap;
  const float *centre;     // [d] subtracted from every row (kernels with CENTRE)
  const float *sample_sq;  // [64] two parts: squared norms that settle the rows' scale
  const float *unscale;    // [nq] two parts: takes a product back
  const uint4 *xfrag;      // rows' parts (bf_pair_kernel; bf_screen_kernel: first parts) and their squared norms
  const float *norm;
  CallState *state;        // inner product: norms are noted here (NULL: not in this pass)
  bool list_far;           // and the rows without one listed
};
static_assert(sizeof(ScoreArgs) == 176, "every launch of a score kernel pays for what is added here, see ScreenArgs");

// A pass of first parts.  (Arguments of its own: with these in ScoreArgs the smallest calls took 0.3 us longer, of 56.)
struct ScreenArgs : ScoreArgs {
  uint64_t n;        // part_w != 0: rows of x; the pass takes part_w of every 2^part_log2 rows, see part_row()
  uint32_t part_log2, part_from, part_w;
  const float *q_norm, *q_rest;   // [nq] at least |q|, and the norm of what its first part leaves
};

// Row of x that row v of a pass over a part of the rows is: of each stretch of 2^part_log2 rows the pass takes
// places part_from .. part_from + part_w - 1 of a random order (places exchanged by a random mask), so
// that passes over disjoint places share out all rows and each is a stratified random sample.  n or more: no row.
__device__ __forceinline__ uint64_t part_row(const ScreenArgs &a, uint64_t v) {
  const uint32_t stretch = (uint32_t)v / a.part_w, place = a.part_from + ((uint32_t)v - stretch * a.part_w);
  uint32_t h = stretch * 0x9E3779B1u;
  h = (h ^ (h >> 15)) * 0x85EBCA77u;
  h ^= h >> 13;
  return ((uint64_t)stretch << a.part_log2) + (place ^ (h & ((1u << a.part_log2) - 1u)));
}

// v[i], i in 0 .. 15 (selects: an index into registers would take them through memory)
__device__ __forceinline__ float pick(const floatx16 &v, int i) {
  const bool b0 = i & 1, b1 = i & 2, b2 = i & 4, b3 = i & 8;
  const float a0 = b0 ? v[1] : v[0], a1 = b0 ? v[3] : v[2], a2 = b0 ? v[5] : v[4], a3 = b0 ? v[7] : v[6];
  const float a4 = b0 ? v[9] : v[8], a5 = b0 ? v[11] : v[10], a6 = b0 ? v[13] : v[12], a7 = b0 ? v[15] : v[14];
  const float c0 = b1 ? a1 : a0, c1 = b1 ? a3 : a2, c2 = b1 ? a5 : a4, c3 = b1 ? a7 : a6;
  const float e0 = b2 ? c1 : c0, e1 = b2 ? c3 : c2;
  return b3 ? e1 : e0;
}

// How far the score of a row with |x| <= nx may lie from its value, |q| = nq (of
// the centred vectors where they are).  Each of the kb_n blocks of 16 columns
// takes six matrix instructions, each of which rounds an accumulator that never
// exceeds |q| |x|; 32 roundings more stand for the products left out, the norm,
// the subtraction of the centre and the last addition.  The second term: what
// the instruction may drop of values below the smallest normal number.  The
// largest error seen is 0.13 of it (seven distributions, d = 24 to 2,048).
__device__ __forceinline__ double score_room(double nq, double nx, uint32_t d, uint32_t kb_n, uint32_t metric) {
  const double terms = 6.0 * kb_n + 32.0, size = metric == ANN_L2 ? 2.0 * nq * nx + nx * nx : nq * nx;
  return terms * 0x1p-24 * size + 0x1p-124 * (double)d * (1.0 + nq + nx);
}

// The same for the products of two half-precision parts: three matrix instructions per
// block of 16 columns; a part left over is below 2^-23 of its value or 2^-25 of the
// scaled one's unit (x_unit, q_unit: what 1 in the scaled vectors is worth), and the product of
// two second parts, left out, below 2^-22.
__device__ __forceinline__ double half_room(double nq, double nx, uint32_t d, uint32_t kb_n, uint32_t metric, double x_unit, double q_unit) {
  const double terms = 3.0 * kb_n + 32.0 + 8.0, size = metric == ANN_L2 ? 2.0 * nq * nx + nx * nx : nq * nx;
  const double lost = sqrt((double)d) * (nq * x_unit + nx * q_unit) + (double)d * x_unit * q_unit;
  return terms * 0x1p-24 * size + 0x1p-24 * lost * (1.0 + 0x1p-10) + 0x1p-124 * (double)d * (1.0 + nq + nx);
}

// How far a product of first parts only (bf_screen_kernel) may put the score of a row that can matter from its value,
// where `value` bounds the score of the row in question: |q| times what the row's first part leaves, and the other way
// round (both norms are known: 0.4 of the 2^-11 |x| that a rounding may leave), and what half_room() allows for.  No row
// of the passes so far is larger than max_norm (its square), or leaves more than max_rest (the scaled one's square); L2:
// a row whose score is at most `value` has |x| <= |q| + sqrt(distance) as well, and a rounding leaves it at most 2^-11 |x| and
// 2^-25 per column, scaled, whatever larger rows leave.  (A little more, so that no other row's score seems to be that:
// with |x| = 17/16 |q| + sqrt(distance) + u it is too large by |q|^2 / 256 + |q| sqrt(distance) / 8 + |q| u / 8 at least, and first
// parts take 2^-9 |q| |x| off at most.)  1M x 128, 10,000 queries, norms like exp(z): by the largest row's rest three queries
// in four are lost, so none.
__device__ __forceinline__ float screen_room(float nq, float q_rest, float value, uint32_t d, uint32_t kb_n, uint32_t metric, float x_unit, float unscale,
                                             uint32_t max_norm, uint32_t max_rest) {
  const double more = 1.0 + 0x1p-10;
  double nx = (double)__fsqrt_rn(__uint_as_float(max_norm)) * more;
  if (metric == ANN_L2) {
    const double dist = (double)nq * nq + (double)value;
    nx = fmin(nx, 1.0625 * (double)nq + (double)__fsqrt_rn(fmaxf((float)dist, 0.0f)) * more);
  }
  const double room = half_room((double)nq, nx, d, kb_n, metric, (double)x_unit, (double)unscale / (double)x_unit);
  const double x_rest = fmin((double)__fsqrt_rn(__uint_as_float(max_rest)) * (double)x_unit, 0x1p-11 * nx + 0x1p-25 * (double)__fsqrt_rn((float)d) * (double)x_unit) * more;
  const double rest = x_rest * (double)nq + (nx + x_rest) * (double)q_rest;
  return (float)((room + (metric == ANN_L2 ? 2.0 : 1.0) * rest) * more);
}

// What a wavefront makes of its products: MB x NQ blocks of 32 rows x 32 queries, the
// element i of block (m, f) being row m * 32 + 8 (i / 4) + 4 (lane / 32) + i % 4
// against query f * 32 + lane % 32.  Scores that reach their query's bound collect in
// LDS (with the row's place in the pass) and go to global memory when that is full: one
// atomic addition per entry then, far from the matrix instructions.  The walk over a
// block with hits takes each lane's next hit per turn (a site of code per score made
// 170 KB of instructions; a pass over 90,000 rows 0.95 -> 0.59 ms).
// SCREEN: the products are of first parts only, and what may reach the bound is written.
template <int MB, int NQ, bool SCREEN = false>
struct TileEnd {
  using Args = std::conditional_t<SCREEN, ScreenArgs, ScoreArgs>;
  const Args &a;
  uint32_t q0;        // the wavefront's first query
  uint64_t *hits;     // LDS [kHitList]: (score, row of the pass)
  uint8_t *hits_q;    // LDS [kHitList]: query - q0
  int n_hits = 0;     // the same in all lanes
  float top[NQ], scale[NQ];

  __device__ __forceinline__ TileEnd(const Args &args, uint32_t q0_, uint64_t *hits_, uint8_t *hits_q_) : a(args), q0(q0_), hits(hits_), hits_q(hits_q_) {
    [[maybe_unused]] float x_unit = 1.0f;
    [[maybe_unused]] uint32_t max_norm = 0, max_rest = 0;
    if constexpr (SCREEN) {
      x_unit = ldexpf(1.0f, -half_exponent(rows_sq(a.sample_sq)));
      max_norm = *(volatile uint32_t *)&a.state->max_norm;
      max_rest = *(volatile uint32_t *)&a.state->max_rest;
    }
#pragma unroll
    for (int f = 0; f < NQ; ++f) {
      const uint32_t q = q0 + f * 32 + lane_id() % 32;
      top[f] = a.scores == nullptr && q < a.nq ? unorder_f32((uint32_t)(a.bound[q] >> 32)) : -INFINITY;
      if constexpr (SCREEN) {
        // (no bound, FLT_MAX: everything; a lost query, NaN: nothing; a query whose norm is no float: nothing, its result is found to be uncertain)
        if (top[f] > -INFINITY && top[f] < 0x1.fffffep127f) {
          float room = screen_room(a.q_norm[q], a.q_rest[q], top[f], a.d, a.kb_n, a.metric, x_unit, a.unscale[q], max_norm, max_rest);
          room = screen_room(a.q_norm[q], a.q_rest[q], top[f] + room, a.d, a.kb_n, a.metric, x_unit, a.unscale[q], max_norm, max_rest);
          top[f] = room < INFINITY ? top[f] + 2.0f * room * (1.0f + 0x1p-20f) : -INFINITY;   // (a room for the bound, one for the score)
        }
      }
      scale[f] = a.metric == ANN_L2 ? -2.0f : -1.0f;
      if (a.unscale != nullptr) scale[f] *= q < a.nq ? a.unscale[q] : 0.0f;   // (powers of two)
    }
  }
  __device__ __forceinline__ static void fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  // the collected hits that reach their query's (score, id) bound -> the queries' entries
  __device__ __forceinline__ void flush() {
    fence();
    bool over = false;
    for (int e = lane_id(); e < n_hits; e += kWave) {
      const uint32_t q = q0 + hits_q[e];
      const uint64_t hit = hits[e];
      const uint64_t row = a.first + (uint32_t)hit;
      uint64_t id = a.stretch != 0.0 ? sample_row(row, a.stretch) : row;
      if constexpr (SCREEN)
        if (a.part_w) id = part_row(a, row);
      const uint64_t ent = (hit & 0xFFFFFFFF00000000ull) | (uint32_t)id;
      if (!SCREEN && ent > a.bound[q]) continue;
      const uint32_t pos = atomicAdd(&a.count[q], 1u);
      if (pos < a.cap)
        a.buf[(uint64_t)q * a.cap + pos] = ent;
      else
        over = true;
    }
    fence();
    n_hits = 0;
    // a query with more entries than room has to be treated otherwise: no more of them
    if (__ballot(over) != 0) {
#pragma unroll
      for (int f = 0; f < NQ; ++f) {
        const uint32_t q = q0 + f * 32 + lane_id() % 32;
        if (q < a.nq && *(volatile uint32_t *)&a.count[q] > a.cap) top[f] = -INFINITY;
      }
    }
  }
  // xn: LDS, the rows' squared norms (inner product: 0; +inf: no score); row0: the first row's place in the pass
  __device__ __forceinline__ void finish(floatx16 (&acc)[MB][NQ], const float *xn, uint32_t row0) {
    const int half = lane_id() / 32, l32 = lane_id() % 32;
    float low[MB][NQ];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
#pragma unroll
      for (int f = 0; f < NQ; ++f) low[m][f] = INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x4 = *reinterpret_cast<const float4 *>(xn + m * 32 + 8 * g + 4 * half);
        const float xv[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
        for (int f = 0; f < NQ; ++f)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[m][f][4 * g + e] = fmaf(scale[f], acc[m][f][4 * g + e], xv[e]);
            low[m][f] = fminf(low[m][f], acc[m][f][4 * g + e]);   // (never a NaN)
          }
      }
    }
    if (a.scores) {
#pragma unroll
      for (int f = 0; f < NQ; ++f) {
        const uint32_t q = q0 + f * 32 + l32;
        if (q >= a.nq) continue;
        float *to = a.scores + (uint64_t)q * a.ld + row0;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int g = 0; g < 4; ++g)   // (a NaN becomes +inf: never selected)
            *reinterpret_cast<float4 *>(to + m * 32 + 8 * g + 4 * half) =
                make_float4(fminf(acc[m][f][4 * g], INFINITY), fminf(acc[m][f][4 * g + 1], INFINITY), fminf(acc[m][f][4 * g + 2], INFINITY),
                            fminf(acc[m][f][4 * g + 3], INFINITY));
      }
      return;
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int f = 0; f < NQ; ++f) {
        if (__ballot(low[m][f] <= top[f]) == 0) continue;
        uint32_t mine = 0;   // this lane's scores up to the bound, a bit each
#pragma unroll
        for (int i = 0; i < 16; ++i) mine |= acc[m][f][i] <= top[f] ? 1u << i : 0u;
        for (;;) {
          const uint64_t hm = __ballot(mine != 0);
          if (hm == 0) break;
          const int n_new = __popcll(hm);
          if (n_hits + n_new > kHitList) flush();
          if (mine != 0) {
            const int i = __builtin_ctz(mine);
            const int pos = n_hits + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, 0u));
            hits[pos] = ((uint64_t)order_u32(pick(acc[m][f], i)) << 32) | (row0 + (uint32_t)(m * 32 + 8 * (i / 4) + 4 * half + i % 4));
            hits_q[pos] = (uint8_t)(f * 32 + l32);
            mine &= mine - 1;
          }
          n_hits += n_new;
        }
      }
  }
};

template <bool VEC4, int MB, int NQ, bool CENTRE, int PARTS>
__global__ __launch_bounds__(256, 2) void bf_score_kernel(ScoreArgs a) {
  constexpr int WB = 4 / MB;                   // wavefronts side by side over the base rows
  constexpr int QT32 = 4 / WB * NQ;            // blocks of 32 queries per tile
  static_assert(WB * MB * 32 == kSB, "tile shape");
  constexpr int NR = kSB / 32;                 // base rows per thread
  static_assert(PARTS == 3 || !CENTRE, "centred rows come in three parts");
  __shared__ __align__(16) unsigned char stage_s[2][PARTS * kPlane];
  __shared__ __align__(16) float xn_s[2][kSB];
  __shared__ uint64_t hit_s[4][kHitList];
  __shared__ uint8_t hit_q_s[4][kHitList];

  // on one die: a group of query tiles over all the die's slabs, then the next group
  const uint32_t die = blockIdx.x & 7u, nth = blockIdx.x >> 3, die_slabs = (a.slabs + 7) / 8;
  const uint32_t group = nth / (a.q_group * die_slabs), left = nth % (a.q_group * die_slabs);
  const uint32_t width = a.q_tiles - group * a.q_group < a.q_group ? a.q_tiles - group * a.q_group : a.q_group;
  const uint32_t qt = group * a.q_group + left % width, slab = left / width * 8u + die;
  const uint64_t tiles = (a.rows + kSB - 1) / kSB;
  const uint64_t tile_begin = (uint64_t)slab * a.tiles_per_slab;
  const uint64_t tile_end = tile_begin + a.tiles_per_slab < tiles ? tile_begin + a.tiles_per_slab : tiles;
  if (slab >= a.slabs || tile_begin >= tile_end) return;

  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, half = lane / 32, l32 = lane % 32;
  const int wb = wave % WB, wq = wave / WB;
  const int s_row = tid / 8, s_col = (tid % 8) * 4;
  const uint32_t n_chunks = a.kb_n / 2;
  const uint4 *qf[NQ];
#pragma unroll
  for (int f = 0; f < NQ; ++f) qf[f] = a.qfrag + (uint64_t)(qt * QT32 + wq * NQ + f) * a.kb_n * (PARTS * 64) + lane;
  // two parts: the rows' scale, and the squared norm from which on a row may not fit the format
  float x_scale = 1.0f, far_from = INFINITY;
  if constexpr (PARTS == 2) {
    const int e = __builtin_amdgcn_readfirstlane(half_exponent(rows_sq(a.sample_sq)));
    x_scale = ldexpf(1.0f, e);
    far_from = ldexpf(kFarNorm2, -2 * e);
  }

  // ---- base rows: fetch (four floats of four rows per thread), split, stage.
  // Nothing here branches: the steps below are one block of instructions, in
  // which the splitting fills the issue slots between matrix instructions.
  float4 reg[NR];
  float sq[NR] = {}, sq_other[NR] = {};   // squared norm: the sums over the last chunk and every second before it, and over the others
  float max_norm = 0.f;   // inner product: largest squared norm seen
  const float *row_at[NR];
  auto new_rows = [&](uint64_t tile) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      uint64_t r = tile * kSB + s_row + 32 * i;
      r = r < a.rows ? r : a.rows - 1;
      if (a.stretch != 0.0) r = sample_row(r, a.stretch);
      row_at[i] = a.x + r * a.d;
    }
  };
  auto fetch = [&](uint32_t c) {
    const uint32_t k = c * kSK + s_col;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const float *p = row_at[i];
      if constexpr (VEC4) {
        reg[i] = *reinterpret_cast<const float4 *>(p + (k < a.d ? k : 0));
      } else {
        reg[i] = make_float4(p[k < a.d ? k : 0], p[k + 1 < a.d ? k + 1 : 0], p[k + 2 < a.d ? k + 2 : 0], p[k + 3 < a.d ? k + 3 : 0]);
      }
    }
  };
  // (columns past d hold other values of the row: the queries are zero there, and the norms leave them out)
  auto stage = [&](int b, uint32_t c) {
    const uint32_t k = c * kSK + s_col;
    float4 mid = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (CENTRE) mid = make_float4(a.centre[k < a.d ? k : 0], a.centre[k + 1 < a.d ? k + 1 : 0], a.centre[k + 2 < a.d ? k + 2 : 0], a.centre[k + 3 < a.d ? k + 3 : 0]);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      float4 v = reg[i];
      if constexpr (CENTRE) v = make_float4(__fsub_rn(v.x, mid.x), __fsub_rn(v.y, mid.y), __fsub_rn(v.z, mid.z), __fsub_rn(v.w, mid.w));
      float t;
      if constexpr (VEC4) {
        t = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w)));
        t = k < a.d ? t : 0.f;
      } else {
        const float e[4] = {v.x, v.y, v.z, v.w};
        t = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float u = fmaf(e[j], e[j], t);
          t = k + j < a.d ? u : t;
        }
      }
      const float sum = sq_other[i] + t;
      sq_other[i] = sq[i];
      sq[i] = sum;
      uint32_t w01[PARTS], w23[PARTS];
      if constexpr (PARTS == 3) {
        split3(v.x, v.y, w01);
        split3(v.z, v.w, w23);
      } else {
        split2(v.x, v.y, x_scale, w01);
        split2(v.z, v.w, x_scale, w23);
      }
      const int row = s_row + 32 * i;
      const int at = row * 64 + (((s_col >> 3) ^ (row >> 2)) & 3) * 16 + (s_col & 4) * 2;
#pragma unroll
      for (int p = 0; p < PARTS; ++p)
        *reinterpret_cast<uint2 *>(stage_s[b] + p * kPlane + at) = make_uint2(w01[p], w23[p]);
    }
  };
  // all columns of the tile's rows have been staged: their norms
  auto put_norms = [&](uint64_t tile) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      float t = sq[i] + sq_other[i];
      t += __int_as_float(dpp_i32<kDppQuadXor1>(__float_as_int(t)));
      t += __int_as_float(dpp_i32<kDppQuadXor2>(__float_as_int(t)));
      t += __int_as_float(dpp_i32<kDppRowHalfMirror>(__float_as_int(t)));
      sq[i] = sq_other[i] = 0.f;
      if (tid % 8 == 0) {
        // Rows whose squared norm is no float are left out of the scores.  L2: they are infinitely far.  Inner
        // product: with a NaN they have no score; the others may be near, and are listed for the exact stage.
        const uint64_t r = tile * kSB + s_row + 32 * i;
        const bool in = r < a.rows && t < far_from;
        xn_s[tile & 1][s_row + 32 * i] = in ? (a.metric == ANN_L2 ? t : 0.f) : INFINITY;
        if (a.metric != ANN_L2 && a.state != nullptr) {
          if (in) {
            max_norm = fmaxf(max_norm, t);
          } else if (r < a.rows && t >= far_from && qt == 0 && a.list_far) {
            const uint32_t at = atomicAdd(&a.state->far_rows, 1u);
            if (at < kFarRows) a.state->far_row[at] = (uint32_t)r;
          }
        } else if (PARTS == 2 && a.state != nullptr && r < a.rows && t >= far_from && t < INFINITY) {
          a.state->left_out = 1u;
        }
      }
    }
  };

  TileEnd<MB, NQ> end(a, (qt * QT32 + wq * NQ) * 32, hit_s[wave], hit_q_s[wave]);

  floatx16 acc[MB][NQ];
  auto clear = [&]() {
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int f = 0; f < NQ; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[m][f][i] = 0.f;
  };
  auto load_q = [&](uint4 (&to)[NQ][PARTS], uint32_t kb) {
#pragma unroll
    for (int f = 0; f < NQ; ++f)
#pragma unroll
      for (int p = 0; p < PARTS; ++p) to[f][p] = qf[f][kb * (PARTS * 64) + p * 64];
  };
  auto multiply = [&](const uint4 (&q)[NQ][PARTS], int b, int kbi) {
    uint4 xa[MB][PARTS];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const int row = (wb * MB + m) * 32 + l32;
      const int at = row * 64 + (((kbi * 2 + half) ^ (row >> 2)) & 3) * 16;
#pragma unroll
      for (int p = 0; p < PARTS; ++p) xa[m][p] = *reinterpret_cast<const uint4 *>(stage_s[b] + p * kPlane + at);
    }
    // the small products first
    constexpr int kProducts = PARTS == 3 ? 6 : 3;
    constexpr int pa[6] = {PARTS == 3 ? 2 : 1, 0, PARTS == 3 ? 1 : 0, 1, 0, 0}, pb[6] = {0, PARTS == 3 ? 2 : 1, PARTS == 3 ? 1 : 0, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < kProducts; ++t)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int f = 0; f < NQ; ++f)
          if constexpr (PARTS == 3)
            acc[m][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa[m][pa[t]]), __builtin_bit_cast(bf16x8, q[f][pb[t]]), acc[m][f], 0, 0, 0);
          else
            acc[m][f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, xa[m][pa[t]]), __builtin_bit_cast(halfx8, q[f][pb[t]]), acc[m][f], 0, 0, 0);
  };

  // The next (tile, chunk) to stage and the one after it, which is fetched as soon as its registers are free.
  auto after = [&](uint64_t &tile, uint32_t &c) {
    if (++c == n_chunks) {
      c = 0;
      ++tile;
    }
  };
  uint4 q0[NQ][PARTS], q1[NQ][PARTS];
  uint64_t tile = tile_begin, f_tile = tile_begin;
  uint32_t c = 0, f_c = 0;
  new_rows(tile);
  fetch(0);
  load_q(q0, 0);
  stage(0, 0);
  if (n_chunks == 1) put_norms(tile);
  after(f_tile, f_c);
  if (f_c == 0) new_rows(f_tile);   // (past the end: clamped)
  fetch(f_c);
  clear();
  __syncthreads();
  int cur = 0;
  for (;;) {
    const uint32_t g_c = f_c + 1 == n_chunks ? 0 : f_c + 1;   // the chunk after the one that is staged now
    load_q(q1, 2 * c + 1);
    multiply(q0, cur, 0);
    stage(cur ^ 1, f_c);
    load_q(q0, 2 * f_c);
    multiply(q1, cur, 1);
    // a matrix instruction occupies its unit for eight issue slots: the vector instructions (the
    // splitting, above all) are spread behind them (five each measured best: 13.4 ms, 14.4 with four, 13.8 with seven)
#pragma unroll
    for (int i = 0; i < (PARTS == 3 ? 12 : 6) * MB * NQ; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, MB * NQ == 4 ? 5 : 10, 0);
    }
    if (f_tile < tile_end && f_c + 1 == n_chunks) put_norms(f_tile);
    after(f_tile, f_c);
    if (g_c == 0) new_rows(f_tile);
    fetch(g_c);
    if (c + 1 == n_chunks) {
      end.finish(acc, xn_s[tile & 1] + wb * MB * 32, (uint32_t)(tile * kSB) + wb * MB * 32);
      clear();
    }
    after(tile, c);
    if (tile >= tile_end) break;
    __syncthreads();
    cur ^= 1;
  }
  if (end.n_hits > 0) end.flush();
  if (a.metric != ANN_L2 && a.state != nullptr) {
    max_norm = wave_max_f32(max_norm);
    // (2,000 wavefronts at one address take 8 us; most find a value that is large enough)
    if (lane == 0 && *(volatile uint32_t *)&a.state->max_norm < __float_as_uint(max_norm)) atomicMax(&a.state->max_norm, __float_as_uint(max_norm));
  }
}

// ---------------------------------------------------------------------------
// Many queries: most scores only have to be shown to be too large, which takes the product of the
// first parts alone, a third of the work.  What that leaves is re-evaluated in fp64 before anything is
// selected or bounded by it (bf_range_kernel).
//
// Where that leaves too much (see bf_range_kernel) the call is repeated with both parts of all rows, bf_pair_kernel.
//
// bf_halve_rows_kernel brings the first parts (PLANES 1) or both of a pass' rows, or of a slab of it, into the order
// the matrix instruction wants (16-byte unit (((row / 32) * kb_n + kb) * PLANES + plane) * 64 + lane) and writes
// the rows' squared norms, summed in fp64 (+inf: left out of the scores).  One workgroup per 32 rows, a wavefront
// takes every fourth block of 16 columns.  Both parts: reading and writing 128 MB each way takes 47 us.
template <bool VEC4, int PLANES>
__global__ __launch_bounds__(256) void bf_halve_rows_kernel(std::conditional_t<PLANES == 1, ScreenArgs, ScoreArgs> a, uint4 *__restrict__ frag, float *__restrict__ norm) {
  __shared__ double part_s[8][32];
  __shared__ float rest_s[8][32];
  const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  uint32_t abandoned = 0, n_hopeless = 0;
  if constexpr (PLANES == 1) {   // (both parts: no state but in the last pass)
    abandoned = a.state->abandoned;
    n_hopeless = a.state->n_hopeless;
  }
  const uint64_t at = (uint64_t)blockIdx.x * 32 + lane % 32;
  const int e = __builtin_amdgcn_readfirstlane(half_exponent(rows_sq(a.sample_sq)));
  const float scale = ldexpf(1.0f, e), far_from = ldexpf(kFarNorm2, -2 * e);
  if (abandoned || n_hopeless * (4 * kVoters) > a.nq) {   // (see bf_range_kernel; read with the sample's norms)
    if (blockIdx.x == 0 && tid == 0) a.state->abandoned = 1u;
    return;
  }
  uint64_t r = at < a.rows ? at : a.rows - 1;
  r = a.stretch != 0.0 ? sample_row(a.first + r, a.stretch) : a.first + r;
  bool real = at < a.rows;
  if constexpr (PLANES == 1)
    if (a.part_w) {
      r = part_row(a, r);
      real = real && r < a.n;
      if (!real) r = a.n - 1;
    }
  const float *row = a.x + r * a.d;
  uint4 *to = frag + (uint64_t)blockIdx.x * a.kb_n * (64 * PLANES) + lane;
  double sq = 0.0;
  float rest = 0.0f;
#pragma unroll 2
  for (uint32_t kb = wave; kb < a.kb_n; kb += 4) {
    const uint32_t k0 = kb * 16 + 8 * (lane / 32);
    float v[8];
    if constexpr (VEC4) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t k = k0 + 4 * h;
        float4 w = *reinterpret_cast<const float4 *>(row + (k < a.d ? k : 0));
        if (k >= a.d) w = make_float4(0.f, 0.f, 0.f, 0.f);
        v[4 * h] = w.x, v[4 * h + 1] = w.y, v[4 * h + 2] = w.z, v[4 * h + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = row[k0 + j < a.d ? k0 + j : 0];
        v[j] = k0 + j < a.d ? v[j] : 0.0f;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) sq = fma((double)v[j], (double)v[j], sq);
    uint32_t w[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) split2(v[2 * j], v[2 * j + 1], scale, w[j]);
#pragma unroll
    for (int p = 0; p < PLANES; ++p) to[(uint64_t)kb * (64 * PLANES) + p * 64] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
    if constexpr (PLANES == 2) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const halfx2 hi = __builtin_bit_cast(halfx2, w[j][0]);
      const float l0 = __builtin_fmaf(v[2 * j], scale, -(float)hi.x), l1 = __builtin_fmaf(v[2 * j + 1], scale, -(float)hi.y);
      rest = fmaf(l0, l0, fmaf(l1, l1, rest));
    }
  }
  part_s[wave * 2 + lane / 32][lane % 32] = sq;
  rest_s[wave * 2 + lane / 32][lane % 32] = rest;
  __syncthreads();
  if (tid >= 32) return;
  float t = (float)(((part_s[0][tid] + part_s[1][tid]) + (part_s[2][tid] + part_s[3][tid])) + ((part_s[4][tid] + part_s[5][tid]) + (part_s[6][tid] + part_s[7][tid])));
  const bool in = real && t < far_from;
  norm[at] = in ? (a.metric == ANN_L2 ? t : 0.f) : INFINITY;
  if (PLANES == 2 && a.state == nullptr) return;
  if (a.metric == ANN_L2) {
    if (real && t >= far_from && t < INFINITY) a.state->left_out = 1u;
    if (PLANES == 2) return;
  } else if (real && t >= far_from && a.list_far) {
    const uint32_t n = atomicAdd(&a.state->far_rows, 1u);
    if (n < kFarRows) a.state->far_row[n] = (uint32_t)r;
  }
  t = in ? t : 0.0f;
  rest = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) rest += rest_s[i][tid];
  rest = in ? rest : 0.0f;
#pragma unroll
  for (int m = 1; m < 32; m <<= 1) {
    t = fmaxf(t, __int_as_float(xor_lane_i32(__float_as_int(t), m)));
    rest = fmaxf(rest, __int_as_float(xor_lane_i32(__float_as_int(rest), m)));
  }
  if (tid == 0 && *(volatile uint32_t *)&a.state->max_norm < __float_as_uint(t)) atomicMax(&a.state->max_norm, __float_as_uint(t));
  if (PLANES == 1 && tid == 0 && *(volatile uint32_t *)&a.state->max_rest < __float_as_uint(rest)) atomicMax(&a.state->max_rest, __float_as_uint(rest));
}

// Both parts.  A workgroup of four wavefronts takes 128 rows x 256 queries per tile, a wavefront 128
// x 64: eight accumulators, 128 registers, so that six products of 16 columns come to two
// LDS reads of rows and one global read of queries.  No vector instruction
// stands between the matrix instructions; two wavefronts share a SIMD, and one's
// end of a tile falls into the other's products.  10,000 x 262,144 x 128: 1.75 to 2.0
// ms, by the clock: 3.27 M cycles each time, at 1.86 down to 1.63 GHz as the card warms up,
// the matrix cores busy in 60 % of them = 383 to 336 TFLOP/s of fp32 work (bf_score_kernel with two parts: 2.68
// ms; with three: 3.7).  The rate is the same at 768 columns, so the loop over chunks is what leaves the
// rest idle, not the end of a tile.  128 queries per tile: 7 % slower; first products onto a constant zero instead
// of cleared registers and the rows' parts requested one block ahead: 1.5 %.
constexpr int kPairQueries = 256;
__global__ __launch_bounds__(256, 2) void bf_pair_kernel(ScoreArgs a) {
  constexpr int MB = 4, NQ = 2, QT32 = 4 * NQ;
  static_assert(QT32 * 32 == kPairQueries, "tile shape");
  __shared__ __align__(16) uint4 stage_s[2][4 * 2 * 2 * 64];   // [row / 32][kb][plane][lane]
  __shared__ __align__(16) float xn_s[2][kSB];
  __shared__ uint64_t hit_s[4][kHitList];
  __shared__ uint8_t hit_q_s[4][kHitList];

  // (as bf_score_kernel: a group of query tiles over all of a die's slabs, then the next group)
  const uint32_t die = blockIdx.x & 7u, nth = blockIdx.x >> 3, die_slabs = (a.slabs + 7) / 8;
  const uint32_t group = nth / (a.q_group * die_slabs), left = nth % (a.q_group * die_slabs);
  const uint32_t width = a.q_tiles - group * a.q_group < a.q_group ? a.q_tiles - group * a.q_group : a.q_group;
  const uint32_t qt = group * a.q_group + left % width, slab = left / width * 8u + die;
  const uint32_t tiles = (uint32_t)((a.rows + kSB - 1) / kSB);
  const uint32_t tile_begin = slab * a.tiles_per_slab;
  const uint32_t tile_end = tile_begin + a.tiles_per_slab < tiles ? tile_begin + a.tiles_per_slab : tiles;
  if (slab >= a.slabs || tile_begin >= tile_end) return;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const uint32_t n_chunks = a.kb_n / 2;
  const uint4 *qf[NQ];
#pragma unroll
  for (int f = 0; f < NQ; ++f) qf[f] = a.qfrag + (uint64_t)(qt * QT32 + wave * NQ + f) * a.kb_n * 128 + lane;

  // the chunk (two blocks of 16 columns) that is staged next: 32 rows' four units by each wavefront, and the tile's norms
  uint32_t tile = tile_begin, f_tile = tile_begin, c = 0, f_c = 0;
  uint4 x0, x1, x2, x3;
  float xn_reg;
  const uint4 *xf = a.xfrag + ((uint64_t)tile_begin * 4 + wave) * a.kb_n * 128 + lane;
  auto fetch = [&]() {
    const uint4 *p = xf + f_c * 256;
    x0 = p[0];
    x1 = p[64];
    x2 = p[128];
    x3 = p[192];
    xn_reg = a.norm[(f_tile < tile_end ? f_tile : tile_end - 1) * kSB + tid % kSB];
  };
  auto stage = [&](int b) {
    uint4 *to = &stage_s[b][wave * 256 + lane];
    to[0] = x0;
    to[64] = x1;
    to[128] = x2;
    to[192] = x3;
    xn_s[f_tile & 1][tid % kSB] = xn_reg;   // (the same values with every chunk of a tile)
  };
  auto advance = [&]() {
    if (++f_c == n_chunks) {
      f_c = 0;
      if (++f_tile < tile_end) xf += (uint64_t)4 * a.kb_n * 128;   // (past the end: the last tile again)
    }
  };

  TileEnd<MB, NQ> end(a, (qt * QT32 + wave * NQ) * 32, hit_s[wave], hit_q_s[wave]);
  floatx16 acc[MB][NQ];
  auto load_q = [&](uint4 (&to)[NQ][2], uint32_t kb) {
#pragma unroll
    for (int f = 0; f < NQ; ++f)
#pragma unroll
      for (int p = 0; p < 2; ++p) to[f][p] = qf[f][kb * 128 + p * 64];
  };
  halfx8 xa[2][2];
  auto read_rows = [&](halfx8 (&to)[2], const uint4 *from) {
#pragma unroll
    for (int p = 0; p < 2; ++p) to[p] = __builtin_bit_cast(halfx8, from[p * 64]);
  };
  // 16 columns: the products of 32 rows at a time while the next 32 rows' parts (after the last: those at `next`) are on their way
  auto multiply = [&](const uint4 (&q)[NQ][2], const uint4 *from, const uint4 *next, bool first) {
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      if (m + 1 < MB)
        read_rows(xa[(m + 1) & 1], from + (m + 1) * 256);
      else if (next)
        read_rows(xa[0], next);
      // the small products first
      constexpr int pa[3] = {1, 0, 0}, pb[3] = {0, 1, 0};
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int f = 0; f < NQ; ++f) {
          const floatx16 zero = {};
          acc[m][f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[m & 1][pa[t]], __builtin_bit_cast(halfx8, q[f][pb[t]]), first && t == 0 ? zero : acc[m][f], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  uint4 q0[NQ][2], q1[NQ][2];
  fetch();
  load_q(q0, 0);
  stage(0);
  advance();
  fetch();
  __syncthreads();
  int cur = 0;
  for (;;) {
    const uint4 *from = &stage_s[cur][lane];
    load_q(q1, 2 * c + 1);
    read_rows(xa[0], from);
    __builtin_amdgcn_sched_barrier(0);
    if (c == 0)
      multiply(q0, from, from + 128, true);
    else
      multiply(q0, from, from + 128, false);
    stage(cur ^ 1);
    load_q(q0, 2 * f_c);
    advance();
    fetch();
    __builtin_amdgcn_sched_barrier(0);
    multiply(q1, from + 128, nullptr, false);
    if (++c == n_chunks) {
      end.finish(acc, xn_s[tile & 1], tile * kSB);
      c = 0;
      if (++tile == tile_end) break;
    }
    __syncthreads();
    cur ^= 1;
  }
  if (end.n_hits > 0) end.flush();
}

// First parts.  A workgroup of four wavefronts takes 128 rows x 256 queries per tile, a wavefront 128
// x 64: eight accumulators, 128 registers.  64 columns of rows are staged through LDS at a time; queries
// come from the L2, 32 columns ahead of the products.  No vector instruction stands between the matrix
// instructions; two wavefronts share a SIMD, and one's end of a tile falls into the other's products.
// 524,000 rows x 128 against 10,000 queries: 1.53 ms = 900 TFLOP/s of fp32 work, matrix cores busy 46 % of the cycles
// at 1.89 GHz (three of the four products of two parts 5.1 ms, bound by the power that the matrix cores may draw).  With the chunk
// on its way in an array, which the compiler kept in scratch memory, 2.38; with 64-bit addresses 1.6.
constexpr int kScreenQueries = 256;
constexpr int kScreenKb = 4;   // blocks of 16 columns staged at a time
__global__ __launch_bounds__(256, 2) void bf_screen_kernel(ScreenArgs a) {
  constexpr int MB = 4, NQ = 2, QT32 = 4 * NQ;
  static_assert(QT32 * 32 == kScreenQueries, "tile shape");
  __shared__ __align__(16) uint4 stage_s[2][4 * kScreenKb * 64];   // [row / 32][kb][lane]
  __shared__ __align__(16) float xn_s[2][kSB];
  __shared__ uint64_t hit_s[4][kHitList];
  __shared__ uint8_t hit_q_s[4][kHitList];

  const uint32_t abandoned = a.state->abandoned;
  // (as bf_score_kernel: a group of query tiles over all of a die's slabs, then the next group)
  const uint32_t die = blockIdx.x & 7u, nth = blockIdx.x >> 3, die_slabs = (a.slabs + 7) / 8;
  const uint32_t group = nth / (a.q_group * die_slabs), left = nth % (a.q_group * die_slabs);
  const uint32_t width = a.q_tiles - group * a.q_group < a.q_group ? a.q_tiles - group * a.q_group : a.q_group;
  const uint32_t qt = group * a.q_group + left % width, slab = left / width * 8u + die;
  const uint32_t tiles = (uint32_t)((a.rows + kSB - 1) / kSB);
  const uint32_t tile_begin = slab * a.tiles_per_slab;
  const uint32_t tile_end = tile_begin + a.tiles_per_slab < tiles ? tile_begin + a.tiles_per_slab : tiles;
  if (slab >= a.slabs || tile_begin >= tile_end) return;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const uint32_t n_chunks = (a.kb_n + kScreenKb - 1) / kScreenKb;
  // Loads through buffer descriptors: an offset of the lane, the rest in scalar registers (64-bit addresses take 20 vector
  // registers, which go to scratch memory, and reading them back at a tile's end waits for every load on its way).
  const uint32_t lane16 = lane * 16, block_bytes = a.kb_n * 1024;   // of 32 rows' first parts; queries have two parts
  const auto q_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.qfrag + (uint64_t)(qt * QT32 + wave * NQ) * a.kb_n * 128), 0, NQ * 2 * block_bytes, 0x00027000);
  const auto x_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.xfrag), 0, tiles * 4 * block_bytes, 0x00027000);
  const auto norm_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.norm), 0, tiles * kSB * 4, 0x00027000);
  auto load16 = [&](auto buf, uint32_t at) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(buf, lane16, at, 0));
  };

  // the chunk that is staged next: 32 rows' units by each wavefront, and the tile's norms
  uint32_t tile = tile_begin, f_tile = tile_begin, c = 0, f_c = 0;
  uint4 x0, x1, x2, x3;   // (an array goes to scratch memory, and every load is waited for at once)
  static_assert(kScreenKb == 4, "registers of a chunk");
  float xn_reg;
  uint32_t xf = (tile_begin * 4 + wave) * block_bytes;
  auto fetch = [&]() {
    auto unit = [&](uint32_t j) {   // (past the last block: that one again, never used)
      return load16(x_buf, xf + (f_c * kScreenKb + j < a.kb_n ? f_c * kScreenKb + j : a.kb_n - 1) * 1024);
    };
    x0 = unit(0), x1 = unit(1), x2 = unit(2), x3 = unit(3);
    xn_reg = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(norm_buf, tid % kSB * 4, (f_tile < tile_end ? f_tile : tile_end - 1) * kSB * 4, 0));
  };
  auto stage = [&](int b) {
    uint4 *to = &stage_s[b][wave * kScreenKb * 64 + lane];
    to[0] = x0, to[64] = x1, to[128] = x2, to[192] = x3;
    xn_s[f_tile & 1][tid % kSB] = xn_reg;   // (the same values with every chunk of a tile)
  };
  auto advance = [&]() {
    if (++f_c == n_chunks) {
      f_c = 0;
      if (++f_tile < tile_end) xf += 4 * block_bytes;   // (past the end: the last tile again)
    }
  };

  TileEnd<MB, NQ, true> end(a, (qt * QT32 + wave * NQ) * 32, hit_s[wave], hit_q_s[wave]);
  floatx16 acc[MB][NQ];
  // queries: two blocks of 16 columns
  auto load_q = [&](uint4 (&to)[2][NQ], uint32_t kb) {
#pragma unroll
    for (uint32_t j = 0; j < 2; ++j)
#pragma unroll
      for (int f = 0; f < NQ; ++f) to[j][f] = load16(q_buf, f * 2 * block_bytes + (kb + j < a.kb_n ? kb + j : a.kb_n - 1) * 2048);
  };
  halfx8 xa[2][MB];
  auto read_rows = [&](halfx8 (&to)[MB], const uint4 *from) {
#pragma unroll
    for (int m = 0; m < MB; ++m) to[m] = __builtin_bit_cast(halfx8, from[m * kScreenKb * 64]);
  };
  // two blocks of 16 columns at `from`, the first one's rows in xa[0]; the second's, and those at `next` (if any), are read meanwhile
  auto multiply = [&](const uint4 (&q)[2][NQ], const uint4 *from, const uint4 *next, bool first) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 0)
        read_rows(xa[1], from + 64);
      else if (next)
        read_rows(xa[0], next);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int f = 0; f < NQ; ++f) {
          const floatx16 zero = {};
          acc[m][f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[j][m], __builtin_bit_cast(halfx8, q[j][f]), first && j == 0 ? zero : acc[m][f], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  uint4 q0[2][NQ], q1[2][NQ];
  if (abandoned) return;
  if (blockIdx.x == 0 && tid == 0) a.state->n_hopeless = 0u;
  fetch();
  load_q(q0, 0);
  stage(0);
  advance();
  fetch();
  __syncthreads();
  int cur = 0;
  for (;;) {
    const uint4 *from = &stage_s[cur][lane];
    const bool whole = c * kScreenKb + 2 < a.kb_n;   // (kb_n is even: a last chunk may be half)
    load_q(q1, whole ? c * kScreenKb + 2 : 0);
    read_rows(xa[0], from);
    __builtin_amdgcn_sched_barrier(0);
    if (c == 0)
      multiply(q0, from, from + 128, true);
    else
      multiply(q0, from, from + 128, false);
    stage(cur ^ 1);
    load_q(q0, f_c * kScreenKb);
    advance();
    fetch();
    __builtin_amdgcn_sched_barrier(0);
    if (whole) multiply(q1, from + 128, nullptr, false);
    if (++c == n_chunks) {
      end.finish(acc, xn_s[tile & 1], tile * kSB);
      c = 0;
      if (++tile == tile_end) break;
    }
    __syncthreads();
    cur ^= 1;
  }
  if (end.n_hits > 0) end.flush();
}

// What bf_range_kernel, and the selection from the sample before it, need (see there).
struct RangeArgs {
  const float *x, *q;
  const float *sample_sq, *unscale, *q_norm, *q_rest;
  CallState *state;
  uint32_t d, kb_n, metric, want, most;
  bool last;   // pass
  // what a pass tells of the last (see vote())
  float part, weight, limit;
  uint32_t few;   // entries that a wavefront takes
  uint64_t *buf;
  uint32_t *count;
  uint32_t cap;
  uint64_t *bound;
};
constexpr int kSelThreads = 256;
constexpr uint32_t kFewEntries = 8 * kWave;
constexpr uint32_t range_room(int threads) { return threads == kWave ? kFewEntries : 4 * kSelThreads; }   // entries that may be among the best

// How far the score of an entry up to two rooms beyond a bound may lie from its value.
__device__ __forceinline__ float entry_room(const RangeArgs &a, uint32_t q, float bound) {
  const float x_unit = ldexpf(1.0f, -half_exponent(rows_sq(a.sample_sq))), q_norm = a.q_norm[q], q_rest = a.q_rest[q], unscale = a.unscale[q];
  const uint32_t max_norm = a.state->max_norm, max_rest = a.state->max_rest;
  const float room = screen_room(q_norm, q_rest, bound, a.d, a.kb_n, a.metric, x_unit, unscale, max_norm, max_rest);
  return screen_room(q_norm, q_rest, bound + 3.0f * room, a.d, a.kb_n, a.metric, x_unit, unscale, max_norm, max_rest);
}
// A voting query tells whether the last pass will lose it: whether more than `limit` rows lie up to two rooms beyond the
// bound that all rows will give.  That bound's rank among the rows so far lies between 1 (n_best entries are up to two rooms
// beyond the best) and `want` (n_bound beyond the bound so far): `part` of the way, by its logarithm.  Each entry stands for
// `weight` rows.
__device__ __forceinline__ void vote(const RangeArgs &a, uint32_t q, uint32_t n_best, uint32_t n_bound) {
  const float n = a.part > 0.0f ? __expf((1.0f - a.part) * __logf((float)n_best) + a.part * __logf((float)n_bound)) : (float)n_best;
  if (q % kVoters == 0 && n * a.weight > a.limit) atomicAdd(&a.state->n_hopeless, 1u);
}

// ---------------------------------------------------------------------------
// Selection by bisection on the order-preserving bits of the scores: a bound
// that at least `want` and at most `most` of the workgroup's entries reach.
// Entries lie in registers, EPT per thread; a step counts the entries up to the
// middle (one compare and one population count per register and wavefront).
// With more than `most` equal scores at the bound the ids decide (ascending).
// Entries with an ordered score above kMaxScore (+inf) are none.
constexpr uint32_t kMaxScore = 0xFF7FFFFFu;   // FLT_MAX in score order

// THREADS: of the workgroup; one wavefront needs no LDS and no barriers.
template <int EPT, int THREADS = kSelThreads>
struct Selector {
  uint32_t key[EPT], id[EPT];
  uint32_t *red;   // LDS [2][4]
  int parity = 0;

  __device__ __forceinline__ uint32_t total(uint32_t wave_count) {
    if constexpr (THREADS == kWave) return wave_count;
    if (threadIdx.x % kWave == 0) red[parity * 4 + threadIdx.x / kWave] = wave_count;
    __syncthreads();
    const uint32_t t = red[parity * 4] + red[parity * 4 + 1] + red[parity * 4 + 2] + red[parity * 4 + 3];
    parity ^= 1;
    return t;
  }
  __device__ __forceinline__ uint32_t count_up_to(uint32_t k) {
    uint32_t c = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) c += (uint32_t)__popcll(__ballot(key[e] <= k));
    return total(c);
  }
  // (score << 32 | id) bound; n_kept: entries that reach it
  __device__ __forceinline__ uint64_t run(uint32_t want, uint32_t most, uint32_t &n_kept) {
    n_kept = count_up_to(kMaxScore);
    if (n_kept <= most) return ((uint64_t)kMaxScore << 32) | 0xFFFFFFFFu;
    // count(lo) < want, count(hi) > most
    uint32_t lo = 0, hi = kMaxScore;
    {
      uint32_t mn = 0xFFFFFFFFu;
#pragma unroll
      for (int e = 0; e < EPT; ++e) mn = key[e] < mn ? key[e] : mn;
      uint32_t mx = mn;   // the largest of the threads' minima: as many entries as threads reach it
#pragma unroll
      for (int x = 1; x < kWave; x <<= 1) {
        const uint32_t o = (uint32_t)xor_lane_i32((int)mn, x), p = (uint32_t)xor_lane_i32((int)mx, x);
        mn = o < mn ? o : mn;
        mx = p > mx ? p : mx;
      }
      if constexpr (THREADS > kWave) {
        if (threadIdx.x % kWave == 0) {
          red[parity * 4 + threadIdx.x / kWave] = mn;
          red[8 + threadIdx.x / kWave] = mx;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < THREADS / kWave; ++w) {
          mn = red[parity * 4 + w] < mn ? red[parity * 4 + w] : mn;
          mx = red[8 + w] > mx ? red[8 + w] : mx;
        }
        parity ^= 1;
      }
      if (mn > 0) lo = mn - 1;
      if (most < (uint32_t)THREADS && mx < hi) hi = mx;
    }
    while (hi - lo > 1) {
      const uint32_t mid = lo + (hi - lo) / 2;
      const uint32_t c = count_up_to(mid);
      if (c >= want && c <= most) {
        n_kept = c;
        return ((uint64_t)mid << 32) | 0xFFFFFFFFu;
      }
      if (c < want)
        lo = mid;
      else
        hi = mid;
    }
    // equal scores: `hi` is the score, too few entries are below it and too many reach it
    const uint32_t below = count_up_to(lo);
    uint32_t ilo = 0, ihi = 0xFFFFFFFFu;   // ids up to ilo - 1 are too few, up to ihi too many
    for (;;) {
      const uint32_t mid = ilo + (ihi - ilo) / 2;
      uint32_t c = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) c += (uint32_t)__popcll(__ballot(key[e] == hi && id[e] <= mid));
      c = below + total(c);
      if ((c >= want && c <= most) || ilo >= ihi) {
        n_kept = c;
        return ((uint64_t)hi << 32) | mid;
      }
      if (c < want)
        ilo = mid + 1;
      else
        ihi = mid;
    }
  }
  // The smallest score.
  __device__ __forceinline__ uint32_t lowest() {
    uint32_t mn = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < EPT; ++e) mn = key[e] < mn ? key[e] : mn;
#pragma unroll
    for (int x = 1; x < kWave; x <<= 1) {
      const uint32_t o = (uint32_t)xor_lane_i32((int)mn, x);
      mn = o < mn ? o : mn;
    }
    if constexpr (THREADS > kWave) {
      if (threadIdx.x % kWave == 0) red[parity * 4 + threadIdx.x / kWave] = mn;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < THREADS / kWave; ++w) mn = red[parity * 4 + w] < mn ? red[parity * 4 + w] : mn;
      parity ^= 1;
    }
    return mn;
  }
  // How many entries lie up to two rooms beyond the best.
  __device__ __forceinline__ uint32_t near_best(float room) {
    const float last = unorder_f32(lowest()) + 2.0f * room;
    return count_up_to(last < INFINITY ? order_u32(last) : kMaxScore);
  }
};

// The best of one stretch of a query's scores.  Sample (stretch != 0): the bound
// is all that is wanted (vote, with first parts: and what it tells of the passes to come).  Otherwise the entries go to out[q][blockIdx.y][most],
// padded with all-ones, and the bound is the smallest of the stretches'.
template <int EPT, typename... Vote>
__global__ __launch_bounds__(kSelThreads) void bf_select_scores_kernel(const float *__restrict__ scores, uint32_t ld, uint64_t rows,
                                                                       double stretch, uint32_t want, uint32_t most,
                                                                       uint64_t *__restrict__ bound, uint64_t *__restrict__ out, Vote... range) {
  __shared__ uint32_t red[16], wave_at[4];
  const uint32_t q = blockIdx.x, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const uint64_t r0 = (uint64_t)blockIdx.y * (EPT * kSelThreads);
  Selector<EPT> s;
  s.red = red;
#pragma unroll
  for (int i = 0; i < EPT / 4; ++i) {
    const uint64_t r = r0 + (uint32_t)(i * kSelThreads + tid) * 4;
    // (ld is a multiple of 4 and at least rows; columns from rows on hold +inf up to the end of the last tile)
    float4 v = make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
    if (r < rows) v = *reinterpret_cast<const float4 *>(scores + (uint64_t)q * ld + r);
    const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s.key[4 * i + e] = r + e < rows ? order_u32(vv[e]) : 0xFFFFFFFFu;
      s.id[4 * i + e] = (uint32_t)(stretch != 0.0 ? sample_row(r + e, stretch) : r + e);
    }
  }
  uint32_t n_kept;
  const uint64_t b = s.run(want, most, n_kept);
  if (out == nullptr) {
    if (tid == 0) bound[q] = b;
    auto tell = [&](const RangeArgs &a) {
      if (q % kVoters != 0 || (uint32_t)(b >> 32) >= kMaxScore) return;
      const uint32_t n_near = s.near_best(entry_room(a, q, unorder_f32((uint32_t)(b >> 32))));
      if (tid == 0) vote(a, q, n_near, n_near);
    };
    (tell(range), ...);
    return;
  }
  if (tid == 0) atomicMin(reinterpret_cast<unsigned long long *>(&bound[q]), (unsigned long long)b);
  uint64_t *list = out + ((uint64_t)q * gridDim.y + blockIdx.y) * most;
  uint32_t mine = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const uint64_t ent = ((uint64_t)s.key[e] << 32) | s.id[e];
    mine += (uint32_t)__popcll(__ballot(s.key[e] <= kMaxScore && ent <= b));
  }
  __syncthreads();
  if (lane == 0) wave_at[wave] = mine;
  __syncthreads();
  uint32_t at = 0;
  for (uint32_t w = 0; w < wave; ++w) at += wave_at[w];
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const uint64_t ent = ((uint64_t)s.key[e] << 32) | s.id[e];
    const bool keep = s.key[e] <= kMaxScore && ent <= b;
    const uint64_t m = __ballot(keep);
    if (keep) list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = ent;
    at += (uint32_t)__popcll(m);
  }
  for (uint32_t e = n_kept + tid; e < most; e += kSelThreads) list[e] = ~0ull;
}

// What the last selection of a batch needs to tell how far its result is certain.
struct CertainArgs {
  const float *q;      // [nq][d]
  const float *centre; // [d] what rows (and, L2, queries) were centred by, or NULL
  uint32_t d, kb_n, metric;
  CallState *state;
  const float *sample_sq, *unscale;   // two parts (otherwise NULL): as in ScoreArgs
  float *below;        // [nq] out
  bool screened;       // entries are those of bf_range_kernel: none of a query that is lost
};

// The best of a query's entries.  count == NULL: all `cap` of them (all-ones:
// none).  cand == NULL: only the bound is updated (kept if fewer than `want`
// entries were found) and the count cleared for the next pass; otherwise the
// ids go to cand[q][most], padded, and c.below[q] says up to which distance no
// other row can be nearer: the value of the first pair left out less what its
// score may be too large by.  (A row nearer than a distance D has |x| <= |q| +
// sqrt(D), whatever other rows measure; in an inner product the largest row
// counts.)  Infinity: nothing was left out, or the query has a NaN and no scores.
template <int EPT>
__global__ __launch_bounds__(kSelThreads) void bf_select_entries_kernel(const uint64_t *__restrict__ buf, uint32_t *__restrict__ count,
                                                                        uint32_t cap, uint32_t want, uint32_t most,
                                                                        uint64_t *__restrict__ bound, uint32_t *__restrict__ cand,
                                                                        CertainArgs c) {
  __shared__ uint32_t red[16], n_out;
  __shared__ double norm_s[kSelThreads / kWave], along_s[kSelThreads / kWave];
  const uint32_t q = blockIdx.x, tid = threadIdx.x;
  if (cand != nullptr) {
    double sq = 0.0, along = 0.0;   // (inner product of centred rows: all scores lack q . centre)
    for (uint32_t j = tid; j < c.d; j += kSelThreads) {
      float v = c.q[(uint64_t)q * c.d + j];
      if (c.centre) {
        if (c.metric == ANN_L2)
          v = __fsub_rn(v, c.centre[j]);
        else
          along += (double)v * c.centre[j];
      }
      sq += fabsf(v) < 0x1.fep127f || v != v ? (double)v * v : INFINITY;   // (larger ones have no three parts)
    }
    sq = group_sum_f64<kWave>(sq);
    if (c.centre) along = group_sum_f64<kWave>(along);
    if (tid % kWave == 0) {   // (read after the selection's barriers)
      norm_s[tid / kWave] = sq;
      along_s[tid / kWave] = along;
    }
  }
  const uint32_t found = count ? count[q] : cap;
  const bool repeated = c.screened && c.state->abandoned, lost = repeated || (c.screened && found > cap);   // (repeated: the whole call)
  const uint32_t n_ent = lost ? 0u : (found < cap ? found : cap);
  Selector<EPT> s;
  s.red = red;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const uint32_t i = (uint32_t)e * kSelThreads + tid;
    const uint64_t ent = i < n_ent ? buf[(uint64_t)q * cap + i] : ~0ull;
    s.key[e] = (uint32_t)(ent >> 32);
    s.id[e] = (uint32_t)ent;
  }
  if (tid == 0) n_out = 0;
  uint32_t n_kept;
  const uint64_t b = s.run(want, most, n_kept);   // (a barrier or more: everyone has read the count)
  if (cand == nullptr) {
    if (tid == 0) {
      if (n_kept >= want && b < bound[q]) bound[q] = b;
      count[q] = 0;
    }
    return;
  }
  if (tid == 0) {
    double sq = 0.0, along = 0.0;
    for (int w = 0; w < kSelThreads / kWave; ++w) {
      sq += norm_s[w];
      along += along_s[w];
    }
    const uint64_t out = b < bound[q] ? b : bound[q];
    // (norms in fp32, rounded up: one thread computes this while the others are done)
    const float more = 1.0f + 0x1p-20f, nq = __fsqrt_rn((float)sq) * more;
    const double value = unorder_f32((uint32_t)(out >> 32)), dist = c.metric == ANN_L2 ? sq + value : value - along;
    float nx = (c.metric == ANN_L2 ? nq + __fsqrt_rn(fmaxf((float)dist, 0.0f)) : __fsqrt_rn(__uint_as_float(c.state->max_norm))) * more;
    double room = score_room(nq, nx, c.d, c.kb_n, c.metric);
    if (c.unscale) {
      const double room3 = room;
      float most = 0.0f;
      for (int i = 0; i < 64; ++i) most = fmaxf(most, c.sample_sq[i]);
      const int e = half_exponent(most);
      // (L2: rows that were left out for their size may be as near as this one; where there are none, no row is larger than that)
      const bool beyond = c.metric == ANN_L2 && !(nx * nx < ldexpf(0.99f * kFarNorm2, -2 * e));
      if (beyond && !c.state->left_out) nx = __fsqrt_rn(ldexpf(1.01f * kFarNorm2, -2 * e));
      room = half_room(nq, nx, c.d, c.kb_n, c.metric, ldexpf(1.0f, -e), ldexpf(c.unscale[q], e));
      if (beyond && c.state->left_out) room = INFINITY;
      if (room > room3) atomicAdd(&c.state->n_wide, 1u);
    }
    float below = (float)(dist - room);
    if (found > cap) below = -INFINITY;   // entries were lost
    // (rows left out for their size were not counted)
    if ((uint32_t)(out >> 32) >= kMaxScore) below = c.unscale && c.state->left_out ? -INFINITY : INFINITY;
    // (two parts: from here on the query's squared norm in fp32, which its scale comes from, may be infinite and its scores no numbers)
    if (lost || (c.unscale && sq >= 0x1p127)) below = -INFINITY;
    if (sq != sq) below = INFINITY;
    if (sq == INFINITY) below = -INFINITY;
    if (repeated) below = INFINITY;
    if (lost && below == -INFINITY) atomicAdd(&c.state->n_lost, 1u);
    c.below[q] = below;
  }
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const uint64_t ent = ((uint64_t)s.key[e] << 32) | s.id[e];
    if (s.key[e] <= kMaxScore && ent <= b) cand[(uint64_t)q * most + atomicAdd(&n_out, 1u)] = s.id[e];
  }
  for (uint32_t e = n_kept + tid; e < most; e += kSelThreads) cand[(uint64_t)q * most + e] = ANN_PAD_ID;
}

// A query's entries after a pass of bf_screen_kernel, whose scores may be a room (screen_room) off: the score that `want` to
// `most` of them reach bounds the next pass, and what is more than two rooms beyond it goes (one for the bound, one for the
// entry: it is not among the `want` best).  After the last pass what is left is re-evaluated in fp64, the score rounded
// once, and the best `want` to `most` of that stay.  More than there is room for: the query is lost, and the count says so to the
// last selection.
// Where vectors lie far from the origin for their spread, or in narrow clusters, thousands of rows lie within the room, and
// first parts settle nothing.  A query in kVoters tells, from the sample and each pass, what the last pass will find (see
// select_round).  Once one voter in four will be lost the passes after it do nothing and the call is repeated with two
// parts; below that the lost queries are taken up again by themselves.  10,000 queries x 1M x 128, two parts alone / first
// parts, and centred rows for what these lost / this: 7 spreads from the origin 7.3 / 4.4 / 4.5 ms, 10 7.4 / 21.4 / 7.5, 20
// 7.8 / 21.4 / 8.0; 100 clusters of spread 0.1 7.7 / 5.3 / 5.5, 0.05 7.9 / 21.0 / 8.2.  Where nothing is lost the votes cost
// 0 to 1 %; where the passes are given up, the sample and what is left of them 0.3 ms here, 0.1 with 2,000 queries.
// (Re-evaluating each pass's new entries made the bounds a room tighter and cost more: 200,000 rows, d = 768, k = 100,
// 2,000 queries: these kernels 263 instead of 660 us.)
// A wavefront takes a query with up to 512 entries, a workgroup one with more, in a launch of its own: 10,000 queries with
// about a hundred each, k = 10, d = 128, by workgroups 130 to 205 us a pass, by wavefronts 16 to 57.  After the last pass a workgroup takes every query where there is much
// to read again, want d >= 32,768 elements: d = 768, k = 100 by both kinds 442 us, by workgroups 222 (d = 300, k = 10, 3,000
// queries, whole call: 658 by workgroups, 620 by wavefronts; d = 960, k = 10: no difference).

// Those that may be among the best to best[]; the score that `want` to `most` reach; n_near (but in the last pass): how many lie
// within two rooms of the best.
template <int EPT, int THREADS>
__device__ __forceinline__ uint64_t range_entries(const RangeArgs &a, uint32_t q, uint32_t n_ent, float room, uint64_t *best, uint32_t *n_best, uint32_t *red,
                                                  uint32_t &n_near) {
  const uint32_t tid = threadIdx.x;
  Selector<EPT, THREADS> s;
  s.red = red;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const uint32_t i = (uint32_t)(e * THREADS) + tid;
    const uint64_t ent = i < n_ent ? a.buf[(uint64_t)q * a.cap + i] : ~0ull;
    s.key[e] = (uint32_t)(ent >> 32);
    s.id[e] = (uint32_t)ent;
  }
  uint32_t n_kept;
  const uint64_t b = s.run(a.want, a.most, n_kept);
  const float last = n_ent <= a.most ? INFINITY : unorder_f32((uint32_t)(b >> 32)) + 2.0f * room * (1.0f + 0x1p-20f);
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    if (s.key[e] > kMaxScore || unorder_f32(s.key[e]) > last) continue;
    const uint32_t at = atomicAdd(n_best, 1u);
    if (at < range_room(THREADS)) best[at] = ((uint64_t)s.key[e] << 32) | s.id[e];
  }
  if (!a.last && q % kVoters == 0) n_near = s.near_best(room);
  __syncthreads();
  return b;
}
// VEC4: rows and queries are read 16 bytes at a time (both aligned to that).
template <bool VEC4, int THREADS>
__global__ __launch_bounds__(THREADS) void bf_range_kernel(RangeArgs a) {
  constexpr uint32_t kRoomHere = range_room(THREADS), kLanes = THREADS == kWave ? 4 : 8;   // lanes to a row
  __shared__ uint32_t red[16], n_best[2];
  __shared__ unsigned long long last_s;
  __shared__ uint64_t best[kRoomHere];
  const uint32_t q = blockIdx.x, tid = threadIdx.x;
  const uint32_t found = a.count[q];
  // (none, or taken by the other launch, which may only leave few of many)
  if (found == 0 || (found <= a.few) != (THREADS == kWave)) return;
  if (a.state->abandoned) return;
  if (found > a.cap) {   // entries were lost
    if (!a.last && tid == 0) {
      vote(a, q, found, found);
      a.bound[q] = 0;   // (no number: the query has no more entries)
    }
    return;
  }
  const uint64_t old_bound = a.bound[q];
  if (tid < 2) n_best[tid] = 0;
  if (tid == 0) last_s = 0;
  __syncthreads();
  const float room = entry_room(a, q, unorder_f32((uint32_t)(old_bound >> 32)));
  uint64_t b;
  uint32_t n_near = 0;
  if constexpr (THREADS == kWave)
    b = range_entries<8, THREADS>(a, q, found, room, best, n_best, red, n_near);
  else if (found <= 8 * kSelThreads)
    b = range_entries<8, THREADS>(a, q, found, room, best, n_best, red, n_near);
  else
    b = range_entries<32, THREADS>(a, q, found, room, best, n_best, red, n_near);
  const uint32_t n = n_best[0];
  const bool bounds = found > a.most && b < old_bound;   // (else the selection took all of them)
  if (!a.last) {
    if (n <= kRoomHere && n < found)
      for (uint32_t i = tid; i < n; i += THREADS) a.buf[(uint64_t)q * a.cap + i] = best[i];
    if (tid == 0) {
      if (n <= kRoomHere) a.count[q] = n;
      if (bounds) a.bound[q] = b;
      vote(a, q, n_near, n);
    }
    return;
  }
  if (n > kRoomHere) {
    if (tid == 0) a.count[q] = a.cap + 1;
    return;
  }
  const float *qr = a.q + (uint64_t)q * a.d;
  for (uint32_t i = tid / kLanes; i < n; i += THREADS / kLanes) {
    const uint32_t id = (uint32_t)best[i];
    const float *row = a.x + (uint64_t)id * a.d;
    double dot = 0.0, sq = 0.0;
    if constexpr (VEC4) {
#pragma unroll 8
      for (uint32_t j = tid % kLanes * 4; j < a.d; j += kLanes * 4) {
        const float4 v = *reinterpret_cast<const float4 *>(row + j);
        const float4 w = *reinterpret_cast<const float4 *>(qr + j);
        dot = fma((double)v.x, (double)w.x, dot), dot = fma((double)v.y, (double)w.y, dot);
        dot = fma((double)v.z, (double)w.z, dot), dot = fma((double)v.w, (double)w.w, dot);
        sq = fma((double)v.x, (double)v.x, sq), sq = fma((double)v.y, (double)v.y, sq);
        sq = fma((double)v.z, (double)v.z, sq), sq = fma((double)v.w, (double)v.w, sq);
      }
    } else {
#pragma unroll 8
      for (uint32_t j = tid % kLanes; j < a.d; j += kLanes) {
        const double v = row[j];
        dot = fma(v, (double)qr[j], dot);
        sq = fma(v, v, sq);
      }
    }
    dot = group_sum_f64<kLanes>(dot);
    sq = group_sum_f64<kLanes>(sq);
    if (tid % kLanes == 0) best[i] = ((uint64_t)order_u32((float)(a.metric == ANN_L2 ? sq - 2.0 * dot : -dot)) << 32) | id;
  }
  __syncthreads();
  Selector<(int)kRoomHere / THREADS, THREADS> s;
  s.red = red;
#pragma unroll
  for (int e = 0; e < (int)kRoomHere / THREADS; ++e) {
    const uint32_t i = (uint32_t)(e * THREADS) + tid;
    const uint64_t ent = i < n ? best[i] : ~0ull;
    s.key[e] = (uint32_t)(ent >> 32);
    s.id[e] = (uint32_t)ent;
  }
  uint32_t n_kept;
  const uint64_t kept = s.run(a.want, a.most, n_kept);
#pragma unroll
  for (int e = 0; e < (int)kRoomHere / THREADS; ++e) {
    const uint64_t ent = ((uint64_t)s.key[e] << 32) | s.id[e];
    if (s.key[e] <= kMaxScore && ent <= kept) {
      a.buf[(uint64_t)q * a.cap + atomicAdd(&n_best[1], 1u)] = ent;
      atomicMax(&last_s, (unsigned long long)ent);
    }
  }
  __syncthreads();
  if (tid == 0) {
    // (The last that stays: where no more than `most` were left the selection takes all and gives no bound.  What went or was
    // never noted lies more than a room beyond `from`.)
    const float from = unorder_f32((uint32_t)((bounds ? b : old_bound) >> 32)) + room;
    const uint64_t beyond = from < INFINITY ? (uint64_t)order_u32(from) << 32 : ~0ull;
    if (n_kept >= a.want) a.bound[q] = last_s < beyond ? last_s : beyond;
    a.count[q] = n_kept;
  }
}

// The whole search with fp32 products and a top-k per (query, slab): for batches
// that the split products cannot serve.
static ann_status bruteforce_fp32(const float *x, uint64_t n, uint32_t d, const float *q, uint32_t nq, uint32_t k, uint32_t metric,
                                  uint32_t *out_ids, float *out_dist, uint32_t n_cu, hipStream_t st) {
  const uint32_t kp = k + 8;               // candidates kept per (query, slab): k plus a margin for fp32 score error
  const uint32_t cb = kp + kBT;
  const bool vec4 = d % 4 == 0 && (reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(q)) % 16 == 0;
  const uint32_t q_tiles = (nq + kQT - 1) / kQT;
  const uint64_t tiles = (n + kBT - 1) / kBT;
  // Slabs of base rows: the grid (query tiles x slabs) should fill the chip a
  // whole number of times (two workgroups per compute unit).  Among 3 to 8
  // turns take the one whose last turn is fullest.
  const uint32_t slots = n_cu * 2u;
  uint32_t slabs = 1;
  double best_fill = 0.0;
  for (uint32_t turns = 3; turns <= 8; ++turns) {
    const uint32_t s_ = slots * turns / q_tiles;
    if (s_ == 0) continue;
    const double fill = (double)q_tiles * s_ / ((double)slots * turns);
    if (fill > best_fill + 0.01) {
      best_fill = fill;
      slabs = s_;
    }
  }
  if (slabs > tiles) slabs = (uint32_t)tiles;
  if (slabs * kp > 4096) slabs = 4096 / kp;
  if (slabs < 1) slabs = 1;
  const uint64_t rows_per_slab = ((tiles + slabs - 1) / slabs) * kBT;
  slabs = (uint32_t)((n + rows_per_slab - 1) / rows_per_slab);

  const size_t smem = (size_t)2 * (kQT + kBT) * kLd * sizeof(float) + kQT * (sizeof(float) + sizeof(uint32_t)) +
                      (size_t)kQT * cb * sizeof(uint64_t);
  const void *fn = vec4 ? reinterpret_cast<const void *>(bf_tile_kernel<true>) : reinterpret_cast<const void *>(bf_tile_kernel<false>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute");
  const size_t n_cand_words = (size_t)nq * slabs * kp, n_norms = metric == ANN_L2 ? (size_t)n : 0;
  uint32_t *cand = nullptr;
  ANN_HIP(device_alloc((void **)&cand, (n_cand_words + n_norms) * sizeof(uint32_t)));
  float *xnorm = reinterpret_cast<float *>(cand + n_cand_words);
  if (metric == ANN_L2) row_norm_kernel<<<2048, 256, 0, st>>>(x, n, d, xnorm);
  const dim3 grid(q_tiles, slabs);
  if (vec4)
    bf_tile_kernel<true><<<grid, 256, smem, st>>>(x, xnorm, n, d, q, nq, metric, rows_per_slab, kp, cb, cand);
  else
    bf_tile_kernel<false><<<grid, 256, smem, st>>>(x, xnorm, n, d, q, nq, metric, rows_per_slab, kp, cb, cand);
  e = hipGetLastError();
  ann_status rc = e == hipSuccess ? rerank_device(x, n, d, metric, q, nq, cand, slabs * kp, slabs * kp, k, out_ids, out_dist, n_cu, st)
                                  : hip_fail(e, "brute-force tile kernel launch");
  const hipError_t e2 = hipStreamSynchronize(st);
  device_free(cand, e2 == hipSuccess);
  if (rc != ANN_OK) return rc;
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  return ANN_OK;
}

// Slabs of `tiles` row tiles so that the last turn of workgroups (two per compute unit) is nearly full.
static void choose_slabs(uint64_t tiles, uint32_t q_tiles, uint32_t n_cu, uint32_t &out_slabs, uint32_t &tiles_per_slab) {
  const uint64_t slots = 2ull * n_cu;
  // a workgroup's time in tiles, with half a tile for its start
  double best = 0.0;
  uint64_t slabs = 1, tps = tiles;
  const uint64_t most = 8 * slots / q_tiles + 8;
  for (uint64_t s = 1; s <= most && s <= tiles; s = s < 8 ? s + 1 : s + 8) {
    const uint64_t t = (tiles + s - 1) / s, used = (tiles + t - 1) / t;
    const double cost = (double)((used * q_tiles + slots - 1) / slots) * ((double)t + 0.5);
    if (s == 1 || cost < best * 0.99) {
      best = cost;
      slabs = used;
      tps = t;
    }
  }
  out_slabs = (uint32_t)slabs;
  tiles_per_slab = (uint32_t)tps;
}

// One pass of the score kernel over a.rows rows: tile shape by the number of
// queries, slabs so that the last turn of workgroups (two per compute unit) is
// nearly full.
static ann_status launch_scores(ScoreArgs a, bool vec4, uint32_t n_cu, hipStream_t st) {
  const uint64_t row_tiles = (a.rows + kSB - 1) / kSB;
  uint32_t qt = a.nq > 64 || a.unscale || (a.centre && a.nq > 32) ? 128u : (a.nq > 32 ? 64u : 32u);
  // few rows: smaller query tiles while workgroups of the larger would leave compute units idle
  // (100 queries x 10,000 rows x 128, 79 workgroups / 316: the pass 18.8 / 13 us, the call 71.0 / 65.4)
  while (qt > 32 && !a.unscale && !a.centre && row_tiles * ((a.nq + qt - 1) / qt) < n_cu) qt /= 2;
  a.q_tiles = (a.nq + qt - 1) / qt;
  choose_slabs(row_tiles, a.q_tiles, n_cu, a.slabs, a.tiles_per_slab);
  a.q_group = 16;
  if (a.q_group > a.q_tiles) a.q_group = a.q_tiles;
  const uint32_t grid = a.q_tiles * ((a.slabs + 7) / 8 * 8);
#define ANN_BS(V)                                                     \
  do {                                                                \
    if (a.unscale)                                                    \
      bf_score_kernel<V, 4, 1, false, 2><<<grid, 256, 0, st>>>(a);    \
    else if (a.centre && qt == 128)                                   \
      bf_score_kernel<V, 4, 1, true, 3><<<grid, 256, 0, st>>>(a);     \
    else if (a.centre)                                                \
      bf_score_kernel<V, 1, 1, true, 3><<<grid, 256, 0, st>>>(a);     \
    else if (qt == 128)                                               \
      bf_score_kernel<V, 4, 1, false, 3><<<grid, 256, 0, st>>>(a);    \
    else if (qt == 64)                                                \
      bf_score_kernel<V, 1, 2, false, 3><<<grid, 256, 0, st>>>(a);    \
    else                                                              \
      bf_score_kernel<V, 1, 1, false, 3><<<grid, 256, 0, st>>>(a);    \
  } while (0)
  if (vec4)
    ANN_BS(true);
  else
    ANN_BS(false);
#undef ANN_BS
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

// The same with both parts of the rows ahead, a slab of at most x_rows at a time.  A die's group
// of query tiles is a megabyte of parts, four tiles at least (between 4 and 16 tiles within 1 %).
static ann_status launch_pairs(ScoreArgs a, bool vec4, uint4 *xfrag, float *norm, uint64_t x_rows, uint32_t n_cu, hipStream_t st) {
  const uint64_t n = a.rows;
  a.xfrag = xfrag;
  a.norm = norm;
  a.q_tiles = (a.nq + kPairQueries - 1) / kPairQueries;
  a.q_group = 64 / a.kb_n > 4 ? 64 / a.kb_n : 4;
  if (a.q_group > a.q_tiles) a.q_group = a.q_tiles;
  for (a.first = 0; a.first < n; a.first += x_rows) {
    a.rows = n - a.first < x_rows ? n - a.first : x_rows;
    const uint32_t tiles = (uint32_t)((a.rows + kSB - 1) / kSB);
    if (vec4)
      bf_halve_rows_kernel<true, 2><<<tiles * (kSB / 32), 256, 0, st>>>(a, xfrag, norm);
    else
      bf_halve_rows_kernel<false, 2><<<tiles * (kSB / 32), 256, 0, st>>>(a, xfrag, norm);
    choose_slabs(tiles, a.q_tiles, n_cu, a.slabs, a.tiles_per_slab);
    const uint32_t grid = a.q_tiles * ((a.slabs + 7) / 8 * 8);
    bf_pair_kernel<<<grid, 256, 0, st>>>(a);
  }
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

// One pass of first parts, a slab of at most x_rows rows at a time.  A die's group
// of query tiles is a megabyte of parts, four tiles at least (between 4 and 16 tiles within 1 %).
static ann_status launch_screen(ScreenArgs a, bool vec4, uint4 *xfrag, float *norm, uint64_t x_rows, uint32_t n_cu, hipStream_t st) {
  const uint64_t n = a.rows;
  a.xfrag = xfrag;
  a.norm = norm;
  a.q_tiles = (a.nq + kScreenQueries - 1) / kScreenQueries;
  a.q_group = 128 / a.kb_n > 4 ? 128 / a.kb_n : 4;
  if (a.q_group > a.q_tiles) a.q_group = a.q_tiles;
  for (a.first = 0; a.first < n; a.first += x_rows) {
    a.rows = n - a.first < x_rows ? n - a.first : x_rows;
    const uint32_t tiles = (uint32_t)((a.rows + kSB - 1) / kSB);
    if (vec4)
      bf_halve_rows_kernel<true, 1><<<tiles * (kSB / 32), 256, 0, st>>>(a, xfrag, norm);
    else
      bf_halve_rows_kernel<false, 1><<<tiles * (kSB / 32), 256, 0, st>>>(a, xfrag, norm);
    choose_slabs(tiles, a.q_tiles, n_cu, a.slabs, a.tiles_per_slab);
    const uint32_t grid = a.q_tiles * ((a.slabs + 7) / 8 * 8);
    bf_screen_kernel<<<grid, 256, 0, st>>>(a);
  }
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

// ---------------------------------------------------------------------------
// Queries whose result is not certain (see bf_select_entries_kernel): vectors far
// from the origin, where the squares cancel, or many rows at the same distance.
// Where first parts lost a quarter of them or more (see bf_range_kernel; with so many of a call's queries that the passes
// were given up, all of these), the selection again with two parts.
// After two parts, where these left more room than three for a quarter as many queries as are
// uncertain, the selection again with three parts: rows much smaller or larger than the sample's
// largest lose in half precision, not in bf16.  (300,000 x 128, norms spread like exp(3 z), 2,000
// queries: 12.0 ms with centred rows at once, in which the small ones lose, too; 0.93 so; 1.12 with three parts
// only.  Rows that occur 50 times are uncertain with any scores: 1M x 128, 700 queries 5.0 ms with
// three parts first, 3.57 without.)
// Then the whole selection with centred rows and queries (distances do not
// change, nor does the order of inner products), which brings the scores' error
// down to that of the spread.  What is still uncertain then: the k-th distance
// found so far bounds the score of every row that can be among the k nearest, so
// a pass over all rows, of which everything up to that bound is re-evaluated,
// settles a query if it finds at most kRoom rows; with more, the best of those
// that were found bound the next pass.  What does not settle that way (thousands
// of rows at one distance, infinities in a query) goes to bf_tile_kernel, as
// before there were bounds.
// 10,000 queries x 1M x 128, k = 10, 300 or 2,300 spreads from the origin: 30 ms
// (15.4 if certain at once; fp32 products alone took 25.6 and lost neighbours).

constexpr uint32_t kRoom = 4096;       // rows re-evaluated per uncertain query and pass
constexpr uint32_t kMaxPasses = 4;

// Mean of a sample of the rows, column by column (values that are not of ordinary size left out).
__global__ __launch_bounds__(1024) void bf_centre_kernel(const float *__restrict__ x, uint32_t rows, double stretch, uint32_t d,
                                                         float *__restrict__ centre) {
  __shared__ double sum_s[16][64];
  __shared__ uint32_t n_s[16][64];
  const uint32_t c = threadIdx.x % 64, r = threadIdx.x / 64, j = blockIdx.x * 64 + c;
  double sum = 0.0;
  uint32_t n = 0;
  if (j < d)
    for (uint32_t i = r; i < rows; i += 16) {
      const float v = x[sample_row(i, stretch) * d + j];
      if (fabsf(v) < 0x1p50f) sum += v, ++n;
    }
  sum_s[r][c] = sum;
  n_s[r][c] = n;
  __syncthreads();
  if (r == 0 && j < d) {
    for (int k = 1; k < 16; ++k) sum += sum_s[k][c], n += n_s[k][c];
    centre[j] = n ? (float)(sum / n) : 0.0f;
  }
}

// One wavefront per uncertain query: its coordinates side by side with the
// others', and the bound of the pass.  Zero: no pass can settle it.
__global__ __launch_bounds__(64) void bf_gather_uncertain_kernel(const float *__restrict__ Q, uint32_t d, uint32_t kb_n, uint32_t k, uint32_t metric,
                                                                 const float *__restrict__ centre, const uint32_t *__restrict__ list,
                                                                 const float *__restrict__ out_dist, const CallState *__restrict__ state,
                                                                 float *__restrict__ Qg, uint64_t *__restrict__ bound,
                                                                 uint32_t *__restrict__ count) {
  const uint32_t i = blockIdx.x, q = list[i];
  double sq = 0.0, along = 0.0;
  bool bad = false;
  for (uint32_t j = lane_id(); j < d; j += kWave) {
    const float v = Q[(uint64_t)q * d + j], c = centre ? centre[j] : 0.0f, vc = metric == ANN_L2 ? __fsub_rn(v, c) : v;
    Qg[(uint64_t)i * d + j] = v;
    sq += (double)vc * vc;
    along += (double)v * c;
    bad = bad || !(fabsf(v) < 0x1.fep127f) || !(fabsf(vc) < 0x1.fep127f);
  }
  if (bound == nullptr) return;
  sq = group_sum_f64<kWave>(sq);
  along = group_sum_f64<kWave>(along);
  bad = __ballot(bad) != 0;
  if (lane_id() != 0) return;
  count[i] = 0;
  const double far = out_dist[(uint64_t)q * k + k - 1], up = far + fabs(far) * 0x1p-22 + 0x1p-140;   // (rounded to a float on the way)
  const double nq = sqrt(sq), nx = metric == ANN_L2 ? nq + sqrt(fmax(up, 0.0)) : sqrt((double)__uint_as_float(state->max_norm));
  const double value = (metric == ANN_L2 ? up - sq : up + along) + score_room(nq, nx, d, kb_n, metric);
  uint64_t b = ((uint64_t)kMaxScore << 32) | 0xFFFFFFFFu;
  if (value < 0x1.fffffep127) {
    float f = (float)value;
    if ((double)f < value) f = nextafterf(f, INFINITY);
    b = ((uint64_t)order_u32(f) << 32) | 0xFFFFFFFFu;
  }
  bound[i] = bad ? 0ull : b;
}

// The entries of a pass as candidates, padded; one workgroup per query.
__global__ __launch_bounds__(256) void bf_entries_to_candidates_kernel(const uint64_t *__restrict__ buf, const uint32_t *__restrict__ count,
                                                                       uint32_t *__restrict__ cand, CallState *__restrict__ state) {
  const uint32_t q = blockIdx.x, n = count[q] < kRoom ? count[q] : kRoom;
  for (uint32_t e = threadIdx.x; e < kRoom; e += 256) cand[(uint64_t)q * kRoom + e] = e < n ? (uint32_t)buf[(uint64_t)q * kRoom + e] : ANN_PAD_ID;
  if (threadIdx.x == 0) atomicMax(&state->most_entries, n);
}

// Queries of a selection that are uncertain, by their place in it -> their numbers.
__global__ void bf_next_list_kernel(const uint32_t *__restrict__ places, const uint32_t *__restrict__ list, CallState *__restrict__ state,
                                    uint32_t *__restrict__ next) {
  for (uint32_t i = threadIdx.x; i < state->n_uncertain; i += blockDim.x) next[atomicAdd(&state->n_next, 1u)] = list[places[i]];
  __syncthreads();
  if (threadIdx.x == 0) state->n_uncertain = 0;
}

// Results of a pass to their queries' places; one wavefront per query.  A query
// with more entries than room goes to the next pass if its k-th distance fell.
// bound == NULL: results of the fp32 kernel, taken unless a pass found better.
__global__ __launch_bounds__(64) void bf_scatter_uncertain_kernel(const uint32_t *__restrict__ list, uint32_t k, const uint64_t *__restrict__ bound,
                                                                  const uint32_t *__restrict__ count, const uint32_t *__restrict__ ids,
                                                                  const float *__restrict__ dist, uint32_t *__restrict__ out_ids,
                                                                  float *__restrict__ out_dist, CallState *__restrict__ state,
                                                                  uint32_t *__restrict__ next, uint32_t *__restrict__ fp32) {
  const uint32_t i = blockIdx.x, q = list[i];
  const float was = out_dist[(uint64_t)q * k + k - 1], is = dist[(uint64_t)i * k + k - 1];
  bool take;
  if (bound == nullptr) {
    take = is <= was;
  } else {
    const bool all = bound[i] != 0 && count[i] <= kRoom, better = bound[i] != 0 && is < was;
    take = all || better;
    if (!all && lane_id() == 0) {
      if (better)
        next[atomicAdd(&state->n_next, 1u)] = q;
      else
        fp32[atomicAdd(&state->n_fp32, 1u)] = q;
    }
  }
  __syncthreads();   // (one wavefront: everyone has read the old distance)
  if (!take) return;
  for (uint32_t j = lane_id(); j < k; j += kWave) {
    out_ids[(uint64_t)q * k + j] = ids[(uint64_t)i * k + j];
    out_dist[(uint64_t)q * k + j] = dist[(uint64_t)i * k + j];
  }
}

// Inner product with rows whose squared norm is no float: they are no part of
// the passes.  One wavefront per query: its results so far, and behind them those of
// these rows that fp32 products find near (neither a NaN nor infinitely far).
__global__ __launch_bounds__(64) void bf_far_rows_kernel(const float *__restrict__ x, uint32_t d, const float *__restrict__ Q, uint32_t k,
                                                         const CallState *__restrict__ state, uint32_t n_far, const uint32_t *__restrict__ out_ids,
                                                         uint32_t *__restrict__ cand) {
  const uint32_t q = blockIdx.x, width = k + n_far;
  const uint32_t *mine = out_ids + (uint64_t)q * k;
  uint32_t *to = cand + (uint64_t)q * width;
  for (uint32_t j = lane_id(); j < k; j += kWave) to[j] = mine[j];
  for (uint32_t f = 0; f < n_far; ++f) {
    const uint32_t row = state->far_row[f];
    float acc = 0.0f;
    for (uint32_t j = lane_id(); j < d; j += kWave) acc = fmaf(x[(uint64_t)row * d + j], Q[(uint64_t)q * d + j], acc);
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) acc += __int_as_float(xor_lane_i32(__float_as_int(acc), m));
    bool there = false;   // (bf_tile_kernel knows these rows)
    for (uint32_t j = lane_id(); j < k; j += kWave) there = there || mine[j] == row;
    there = __ballot(there) != 0;
    if (lane_id() == 0) to[k + f] = -acc < INFINITY && !there ? row : ANN_PAD_ID;
  }
}

// Device memory for `items` of something or, when there is not that much, for fewer.
template <typename Bytes>
static hipError_t alloc_some(void **ptr, uint64_t &items, uint64_t least, Bytes bytes) {
  return alloc_some(
      items, least, bytes,
      [ptr](size_t b) {
        const hipError_t e = device_alloc(ptr, b);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
      },
      hipErrorOutOfMemory);
}

struct Truth {
  const float *x;
  uint64_t n;
  uint32_t d;
  const float *q;
  uint32_t k, metric;
  uint32_t *out_ids;
  float *out_dist;
  uint32_t n_cu;
  hipStream_t st;
};

static uint64_t up256(uint64_t v) { return (v + 255) & ~255ull; }

// How a call's candidates are selected, and the buffers for a round of queries.
struct Selection {
  uint32_t want, most, most_bound;   // see ann_bruteforce_topk
  uint32_t kb_n, cap, first, samples;
  uint32_t part_log2, part_cap;   // first parts: passes over 1 / 2^part_log2 of the rows, entries per query
  uint64_t stretches, ld;
  bool vec4, dense, halves;   // halves: scores from two half-precision parts
  double growth;
  uint4 *qfrag;
  float *scores, *below;
  uint64_t *buf, *bound;
  uint32_t *count, *cand;
  CallState *state;
  float *sample_sq, *unscale, *q_norm, *q_rest;
  uint4 *xfrag;        // room for x_rows rows' first parts, or pair_rows rows' parts, and their norms
  float *xnorm;
  uint64_t x_rows, pair_rows;   // first parts; both
};

// One round: the k nearest rows of the m queries at qr.
static ann_status select_round(const Truth &t, const Selection &s, const float *qr, uint32_t m, const float *centre, bool list_far,
                               uint32_t *out_ids, float *out_dist, uint32_t *uncertain, uint32_t first_query) {
  const uint32_t blocks32 = (m + 255) / 256 * 8;
  const uint64_t units = (uint64_t)blocks32 * s.kb_n * 64;
  const bool halves = s.halves && centre == nullptr;
  if (halves)
    bf_halve_queries_kernel<<<dim3(blocks32, (s.kb_n + 15) / 16), 1024, 0, t.st>>>(qr, m, t.d, s.kb_n, s.sample_sq, s.qfrag, s.unscale, s.q_norm, s.q_rest, s.bound, s.count);
  else
    bf_split_queries_kernel<<<(uint32_t)(units / 256 < 4096 ? (units + 255) / 256 : 4096), 256, 0, t.st>>>(
        qr, m, t.d, s.kb_n, blocks32, t.metric == ANN_L2 ? centre : nullptr, s.qfrag, s.bound, s.count,
        list_far && !s.halves ? &s.state->n_uncertain : nullptr);   // (list_far: the first round of a call)
  ScoreArgs a{};
  a.x = t.x;
  a.qfrag = s.qfrag;
  a.d = t.d;
  a.kb_n = s.kb_n;
  a.nq = m;
  a.metric = t.metric;
  a.ld = (uint32_t)s.ld;
  a.bound = s.bound;
  a.buf = s.buf;
  a.count = s.count;
  a.cap = s.cap;
  a.centre = centre;
  a.list_far = list_far;
  a.sample_sq = halves ? s.sample_sq : nullptr;
  a.unscale = halves ? s.unscale : nullptr;
  const CertainArgs certain{qr, centre, t.d, s.kb_n, t.metric, s.state, a.sample_sq, a.unscale, s.below, halves && s.x_rows};
  auto select_entries = [&](uint32_t *cnt, uint32_t *to, uint32_t up_to) {
    if (s.cap <= 2048)
      bf_select_entries_kernel<8><<<m, kSelThreads, 0, t.st>>>(s.buf, cnt, s.cap, s.want, up_to, s.bound, to, certain);
    else if (s.cap <= 4096)
      bf_select_entries_kernel<16><<<m, kSelThreads, 0, t.st>>>(s.buf, cnt, s.cap, s.want, up_to, s.bound, to, certain);
    else
      bf_select_entries_kernel<32><<<m, kSelThreads, 0, t.st>>>(s.buf, cnt, s.cap, s.want, up_to, s.bound, to, certain);
  };
  ann_status rc;
  if (s.dense) {
    a.rows = t.n;
    a.scores = s.scores;
    a.state = s.state;
    rc = launch_scores(a, s.vec4, t.n_cu, t.st);
    if (rc != ANN_OK) return rc;
    bf_select_scores_kernel<kSampleRows / kSelThreads><<<dim3(m, (uint32_t)s.stretches), kSelThreads, 0, t.st>>>(s.scores, a.ld, t.n, 0, s.want, s.most,
                                                                                                                 s.bound, s.buf);
    select_entries(nullptr, s.cand, s.most);
  } else if (halves && s.x_rows) {
    // First parts: a sample, all of whose scores are written, gives the first bounds.  Then all rows in passes over a
    // 2^part_log2-th of them, three times that, four times what there was so far, and so on, each a random sample: what may reach
    // the bounds is a few times a bound's rank per pass, and the best of it gives the next bounds.
    // (A sample of 4,096 rows, one of 64,000 and then all rows in order, three products each: 1M x 128, 10,000 queries 7,640 to
    // 7,940 us, with passes over parts 7,554, with first products only 3,510 to 3,660.)
    ScreenArgs b{a};
    b.rows = kSampleRows;
    b.stretch = (double)t.n / kSampleRows;
    b.scores = s.scores;
    b.state = s.state;   // (the largest norm; the sample's rows come again)
    b.list_far = false;
    b.q_norm = s.q_norm;
    b.q_rest = s.q_rest;
    rc = launch_screen(b, s.vec4, s.xfrag, s.xnorm, s.x_rows, t.n_cu, t.st);
    if (rc != ANN_OK) return rc;
    // What the last pass will leave of a query is the rows up to two rooms beyond the bound that all rows will give, whose rank among
    // those so far is want / all.  Below one, the best so far lies further out than that bound: by as much as the square
    // root of the rank corrects.  Estimate over what was left, after the sample and each pass: 1M x 128, k = 10, 8 spreads from the
    // origin 2.2, 1.5, 1.0, 0.9 (without the root 5.3, 2.4), k = 100, 6 spreads 1.5, 1.1, 0.9, 0.9; 200,000 x 768, k = 100, 5 spreads 0.6,
    // 0.9, 0.9; 100 clusters of spread 0.09 0.8, 0.9, 0.8, 0.9.  The last pass notes up to three times what it leaves.
    RangeArgs range{t.x, qr, s.sample_sq, s.unscale, s.q_norm, s.q_rest, s.state, t.d, s.kb_n, t.metric, s.want, s.most_bound, false, 0.0f, 1.0f, 0.0f, kFewEntries,
                    s.buf, s.count, s.part_cap, s.bound};
    range.limit = (float)(s.part_cap / 3 < range_room(kSelThreads) ? s.part_cap / 3 : range_room(kSelThreads));
    auto rows_so_far = [&](double all) {   // one in `all`
      const double rank = s.want / all;
      range.part = rank > 1.0 ? (float)(log(rank) / log((double)s.want)) : 0.0f;
      range.weight = (float)(rank > 1.0 ? all : all * sqrt(rank));
    };
    rows_so_far(b.stretch);
    bf_select_scores_kernel<kSampleRows / kSelThreads><<<m, kSelThreads, 0, t.st>>>(s.scores, b.ld, b.rows, b.stretch, s.want, s.most_bound, s.bound,
                                                                                    nullptr, range);
    b.scores = nullptr;
    b.stretch = 0.0;
    b.list_far = list_far;
    b.cap = s.part_cap;
    b.n = t.n;
    b.part_log2 = s.part_log2;
    const uint32_t parts = 1u << s.part_log2;
    for (uint32_t from = 0, to = 1; from < parts; from = to, to *= 4) {
      b.part_from = from;
      b.part_w = to - from;
      b.rows = ((t.n + parts - 1) >> s.part_log2) * b.part_w;
      rc = launch_screen(b, s.vec4, s.xfrag, s.xnorm, s.x_rows, t.n_cu, t.st);
      if (rc != ANN_OK) return rc;
      range.last = to == parts;
      rows_so_far((double)parts / to);
      if (range.last && (uint64_t)s.want * t.d >= 32768) range.few = 0;   // (see bf_range_kernel)
      if (s.vec4 && reinterpret_cast<uintptr_t>(qr) % 16 == 0) {
        if (range.few) bf_range_kernel<true, kWave><<<m, kWave, 0, t.st>>>(range);
        bf_range_kernel<true, kSelThreads><<<m, kSelThreads, 0, t.st>>>(range);
      } else {
        if (range.few) bf_range_kernel<false, kWave><<<m, kWave, 0, t.st>>>(range);
        bf_range_kernel<false, kSelThreads><<<m, kSelThreads, 0, t.st>>>(range);
      }
    }
    // (at most most_bound entries now, of queries that are not lost)
    bf_select_entries_kernel<2><<<m, kSelThreads, 0, t.st>>>(s.buf, s.count, s.part_cap, s.want, s.most, s.bound, s.cand, certain);
  } else {
    double rows = (double)s.first;
    for (uint32_t p = 0; p <= s.samples; ++p, rows *= s.growth) {
      const bool last = p == s.samples;
      a.rows = last ? t.n : (p == 0 ? (uint64_t)s.first : (uint64_t)rows);
      a.stretch = last ? 0.0 : (double)t.n / (double)a.rows;
      a.scores = p == 0 ? s.scores : nullptr;
      a.state = last ? s.state : nullptr;
      rc = halves && s.pair_rows && m >= 512 + s.kb_n * 16 ? launch_pairs(a, s.vec4, s.xfrag, s.xnorm, s.pair_rows, t.n_cu, t.st)
                                                           : launch_scores(a, s.vec4, t.n_cu, t.st);
      if (rc != ANN_OK) return rc;
      if (p == 0 && s.first == kSampleRows)
        bf_select_scores_kernel<kSampleRows / kSelThreads><<<m, kSelThreads, 0, t.st>>>(s.scores, a.ld, a.rows, a.stretch, s.want, s.most_bound, s.bound,
                                                                                        nullptr);
      else if (p == 0)
        bf_select_scores_kernel<2 * kSampleRows / kSelThreads><<<m, kSelThreads, 0, t.st>>>(s.scores, a.ld, a.rows, a.stretch, s.want, s.most_bound,
                                                                                            s.bound, nullptr);
      else
        select_entries(s.count, last ? s.cand : nullptr, last ? s.most : s.most_bound);
    }
  }
  ANN_HIP(hipGetLastError());
  return rerank_device(t.x, t.n, t.d, t.metric, qr, m, s.cand, s.most, s.most, t.k, out_ids, out_dist, t.n_cu, t.st, nullptr, 0, 0.0f, nullptr,
                       Certainty{s.below, &s.state->n_uncertain, uncertain, first_query});
}

// The fp32 kernel for the listed queries.
static ann_status fp32_for(const Truth &t, const uint32_t *list, uint32_t m_all) {
  uint64_t m = m_all < 8192 ? m_all : 8192;
  auto bytes = [&](uint64_t c) { return up256(c * t.d * 4) + up256(c * t.k * 4) * 2; };
  unsigned char *base = nullptr;
  const hipError_t e = alloc_some((void **)&base, m, 1, bytes);
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  float *qg = reinterpret_cast<float *>(base);
  uint32_t *ids = reinterpret_cast<uint32_t *>(base + up256(m * t.d * 4));
  float *dist = reinterpret_cast<float *>(base + up256(m * t.d * 4) + up256(m * t.k * 4));
  ann_status rc = ANN_OK;
  for (uint64_t i0 = 0; i0 < m_all && rc == ANN_OK; i0 += m) {
    const uint32_t c = (uint32_t)(m_all - i0 < m ? m_all - i0 : m);
    bf_gather_uncertain_kernel<<<c, 64, 0, t.st>>>(t.q, t.d, 0, t.k, t.metric, nullptr, list + i0, t.out_dist, nullptr, qg, nullptr, nullptr);
    rc = bruteforce_fp32(t.x, t.n, t.d, qg, c, t.k, t.metric, ids, dist, t.n_cu, t.st);
    if (rc == ANN_OK)
      bf_scatter_uncertain_kernel<<<c, 64, 0, t.st>>>(list + i0, t.k, nullptr, nullptr, ids, dist, t.out_ids, t.out_dist, nullptr, nullptr, nullptr);
  }
  const hipError_t e1 = hipGetLastError(), e2 = hipStreamSynchronize(t.st);
  device_free(base, e2 == hipSuccess);
  if (rc != ANN_OK) return rc;
  if (e1 != hipSuccess) return hip_fail(e1, "fp32 kernel for uncertain queries");
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  return ANN_OK;
}

// The uncertain queries list[0 .. n_list), `round` of them at a time in s: the
// selection with centred rows, passes over what that leaves, and the fp32 kernel
// for what these do.
static ann_status settle(const Truth &t, const Selection &s, uint64_t round, uint32_t *list, uint32_t n_list, uint32_t n_wide, uint32_t n_lost) {
  CallState *const state = s.state;
  // buffers for m queries at a time, the other lists and the centre
  uint64_t m = n_list < 2048 ? n_list : 2048;
  if (m > round) m = round;
  auto parts = [&](uint64_t c, uint64_t (&at)[8]) {
    const uint64_t size[8] = {c * kRoom * 8, c * kRoom * 4, c * t.d * 4, c * t.k * 4, c * t.k * 4, c * 4, 2ull * n_list * 4, (uint64_t)t.d * 4};
    uint64_t total = 0;
    for (int i = 0; i < 8; ++i) {
      at[i] = total;
      total += up256(size[i]);
    }
    return total;
  };
  uint64_t at[8];
  unsigned char *base = nullptr;
  hipError_t e = alloc_some((void **)&base, m, 1, [&](uint64_t c) { return parts(c, at); });
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  parts(m, at);
  uint64_t *buf = reinterpret_cast<uint64_t *>(base + at[0]);
  uint32_t *cand = reinterpret_cast<uint32_t *>(base + at[1]), *ids = reinterpret_cast<uint32_t *>(base + at[3]);
  float *qg = reinterpret_cast<float *>(base + at[2]), *dist = reinterpret_cast<float *>(base + at[4]);
  uint32_t *places = reinterpret_cast<uint32_t *>(base + at[5]), *other = reinterpret_cast<uint32_t *>(base + at[6]), *fp32 = other + n_list;
  float *centre = reinterpret_cast<float *>(base + at[7]);

  const uint32_t sample = t.n < kSampleRows ? (uint32_t)t.n : kSampleRows;
  bf_centre_kernel<<<(t.d + 63) / 64, 1024, 0, t.st>>>(t.x, sample, (double)t.n / sample, t.d, centre);
  fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->n_uncertain, 1, 0u);
  fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->max_norm, 1, 0u);   // (each selection finds that of the centred rows)

  Selection two = s, three = s;
  two.x_rows = 0;
  three.halves = false;
  auto select_chunk = [&](uint32_t i0, uint32_t c, const Selection &with, const float *around) -> ann_status {
    bf_gather_uncertain_kernel<<<c, 64, 0, t.st>>>(t.q, t.d, s.kb_n, t.k, t.metric, nullptr, list + i0, t.out_dist, nullptr, qg, nullptr, nullptr);
    const ann_status rc = select_round(t, with, qg, c, around, false, ids, dist, places, 0);
    if (rc != ANN_OK) return rc;
    bf_scatter_uncertain_kernel<<<c, 64, 0, t.st>>>(list + i0, t.k, nullptr, nullptr, ids, dist, t.out_ids, t.out_dist, nullptr, nullptr, nullptr);
    bf_next_list_kernel<<<1, 1024, 0, t.st>>>(places, list + i0, state, other);
    ANN_HIP(hipGetLastError());
    return ANN_OK;
  };
  auto pass_chunk = [&](uint32_t i0, uint32_t c) -> ann_status {
    fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->most_entries, 1, 0u);
    bf_gather_uncertain_kernel<<<c, 64, 0, t.st>>>(t.q, t.d, s.kb_n, t.k, t.metric, centre, list + i0, t.out_dist, state, qg, s.bound, s.count);
    const uint32_t blocks32 = (c + 127) / 128 * 4;
    const uint64_t units = (uint64_t)blocks32 * s.kb_n * 64;
    bf_split_queries_kernel<<<(uint32_t)(units / 256 < 4096 ? (units + 255) / 256 : 4096), 256, 0, t.st>>>(
        qg, c, t.d, s.kb_n, blocks32, t.metric == ANN_L2 ? centre : nullptr, s.qfrag, nullptr, nullptr, nullptr);
    ScoreArgs a{};
    a.x = t.x;
    a.qfrag = s.qfrag;
    a.rows = t.n;
    a.d = t.d;
    a.kb_n = s.kb_n;
    a.nq = c;
    a.metric = t.metric;
    a.bound = s.bound;
    a.buf = buf;
    a.count = s.count;
    a.cap = kRoom;
    a.centre = centre;
    ann_status rc = launch_scores(a, s.vec4, t.n_cu, t.st);
    if (rc != ANN_OK) return rc;
    bf_entries_to_candidates_kernel<<<c, 256, 0, t.st>>>(buf, s.count, cand, state);
    uint32_t most = 0;
    ANN_HIP(read_words(&state->most_entries, &most, 1, t.st));
    rc = rerank_device(t.x, t.n, t.d, t.metric, qg, c, cand, most ? most : 1, kRoom, t.k, ids, dist, t.n_cu, t.st);
    if (rc != ANN_OK) return rc;
    bf_scatter_uncertain_kernel<<<c, 64, 0, t.st>>>(list + i0, t.k, s.bound, s.count, ids, dist, t.out_ids, t.out_dist, state, other, fp32);
    ANN_HIP(hipGetLastError());
    return ANN_OK;
  };
  ann_status rc = ANN_OK;
  uint32_t n_fp32 = 0;
  // pass -2: two parts; -1: three parts; 0: centred rows; then the passes with a bound
  auto three_help = [&]() { return s.halves && n_wide >= (n_list + 3) / 4; };
  int pass = n_lost >= (n_list + 3) / 4 ? -2 : (three_help() ? -1 : 0);
  if (pass == -2) fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->n_wide, 1, 0u);
  for (; n_list > 0 && rc == ANN_OK; ++pass) {
    if (pass > (int)kMaxPasses) {
      rc = fp32_for(t, list, n_list);
      break;
    }
    for (uint64_t i0 = 0; i0 < n_list && rc == ANN_OK; i0 += m) {
      const uint32_t c = (uint32_t)(n_list - i0 < m ? n_list - i0 : m);
      rc = pass <= 0 ? select_chunk((uint32_t)i0, c, pass == -2 ? two : three, pass < 0 ? nullptr : centre) : pass_chunk((uint32_t)i0, c);
    }
    if (rc != ANN_OK) break;
    uint32_t left[2] = {0, 0};
    e = read_words(&state->n_next, left, 2, t.st);
    if (e != hipSuccess) {
      rc = hip_fail(e, "the wait for a pass' counters");
      break;
    }
    n_list = left[0];
    n_fp32 = left[1];
    if (pass == -2) {
      e = read_words(&state->n_wide, &n_wide, 1, t.st);
      if (e != hipSuccess) {
        rc = hip_fail(e, "the wait for a pass' counters");
        break;
      }
      if (!three_help()) pass = -1;
    }
    fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->n_next, 1, 0u);
    if (pass < 0) fill_u32_kernel<<<1, 64, 0, t.st>>>(&state->max_norm, 1, 0u);
    uint32_t *was = list;
    list = other;
    other = was;
  }
  if (rc == ANN_OK && n_fp32 > 0) rc = fp32_for(t, fp32, n_fp32);
  e = hipStreamSynchronize(t.st);
  device_free(base, e == hipSuccess);
  if (rc != ANN_OK) return rc;
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  return ANN_OK;
}

// Adds the listed far rows to every query's results.
static ann_status add_far_rows(const Truth &t, uint32_t nq, uint32_t n_far, const CallState *state) {
  const uint32_t width = t.k + n_far;
  uint64_t m = nq;
  const uint64_t fit = (256ull << 20) / (width * 4);
  if (m > fit) m = fit;
  uint32_t *cand = nullptr;
  const hipError_t e = alloc_some((void **)&cand, m, 1, [&](uint64_t c) { return c * width * 4; });
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  ann_status rc = ANN_OK;
  for (uint64_t q0 = 0; q0 < nq && rc == ANN_OK; q0 += m) {
    const uint32_t c = (uint32_t)(nq - q0 < m ? nq - q0 : m);
    bf_far_rows_kernel<<<c, 64, 0, t.st>>>(t.x, t.d, t.q + q0 * t.d, t.k, state, n_far, t.out_ids + q0 * t.k, cand);
    rc = rerank_device(t.x, t.n, t.d, t.metric, t.q + q0 * t.d, c, cand, width, width, t.k, t.out_ids + q0 * t.k, t.out_dist + q0 * t.k, t.n_cu, t.st);
  }
  const hipError_t e2 = hipStreamSynchronize(t.st);
  device_free(cand, e2 == hipSuccess);
  if (rc != ANN_OK) return rc;
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamSynchronize");
  return ANN_OK;
}

}  // namespace ann

using namespace ann;

extern "C" ann_status ann_bruteforce_topk(const float *x, uint64_t n, uint32_t d, const float *q, uint32_t nq, uint32_t k,
                                          uint32_t metric, uint32_t *out_ids, float *out_dist, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!x || !q || !out_ids || !out_dist) return fail(ANN_EINVAL, "ann_bruteforce_topk: NULL argument");
  if (n == 0 || n >= (1ull << 31) || d == 0 || nq == 0 || k == 0) return fail(ANN_EINVAL, "ann_bruteforce_topk: empty input or n >= 2^31");
  if (metric != ANN_L2 && metric != ANN_IP) return fail(ANN_EINVAL, "ann_bruteforce_topk: unknown metric %u", metric);
  if (k > 256) return fail(ANN_ECAPACITY, "ann_bruteforce_topk: k = %u exceeds 256", k);
  if (d > 2048) return fail(ANN_ECAPACITY, "ann_bruteforce_topk: d = %u exceeds 2048", d);
  const uint32_t n_cu = compute_units();
  // k and a margin for the error of the scores; the selection stops as soon as it has between `want` and `most`
  const uint32_t want = k + 8, most = want + (want / 2 > 14 ? want / 2 : 14);
  // (a bound from a sample is worth a few steps more: what reaches it in the next pass is proportional to it)
  const uint32_t most_bound = want + (want / 8 > 2 ? want / 8 : 2);
  const bool vec4 = d % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
  const uint32_t kb_n = (d + kSK - 1) / kSK * 2;

  // All scores written out: up to four stretches, or up to 2^24 scores (64 MB)
  // whose stretches' best fit one selection workgroup (8,192 entries).  Beyond,
  // bounds from samples: a pass writes about `growth` times the entries of its
  // bound (room for six standard deviations of the sample's order statistic).
  // A first sample of 8,192 rows instead of 4,096 is taken where it saves a pass
  // (2,000 x 200,000 x 768, k = 100: a pass over 28,000 rows, 0.60 ms of 4.9).
  const uint64_t stretches = (n + kSampleRows - 1) / kSampleRows;
  const bool dense = stretches <= 4 || ((uint64_t)nq * n <= (1ull << 24) && stretches * most <= 8192);
  const double spread = (double)most_bound + 6.0 * sqrt((double)most_bound);
  double growth = 1.0;
  uint32_t samples = 0, first = kSampleRows, cap;   // samples: passes before the last one
  if (dense) {
    cap = (uint32_t)(stretches * most);
  } else {
    const double limit = 8192.0 / spread < 32.0 ? 8192.0 / spread : 32.0;
    auto passes = [&](double rows) { return (uint32_t)ceil(log((double)n / rows) / log(limit)); };
    samples = passes(kSampleRows);
    if (samples > 1 && passes(2.0 * kSampleRows) < samples) {
      first = 2 * kSampleRows;
      --samples;
    }
    if (samples < 1) samples = 1;
    growth = pow((double)n / first, 1.0 / samples);
    cap = 2048;
    while ((double)cap < growth * spread && cap < 8192) cap <<= 1;
  }
  const uint64_t ld = dense ? (n + kSB - 1) / kSB * kSB : first;
  // With first parts: passes over a 4^i-th of the rows, at most eight times the first sample, and so on (see select_round).
  uint32_t part_log2 = 0, part_cap = 2048;
  while ((double)(n >> part_log2) > 8.0 * kSampleRows) part_log2 += 2;
  const double part_growth = (double)n / (1u << part_log2) / kSampleRows;
  while ((double)part_cap < (part_growth > 3.0 ? part_growth : 3.0) * spread + most_bound && part_cap < 8192) part_cap <<= 1;
  // (up to 4,096 where that takes no more rounds: a query may then have as many rows within the room as bf_range_kernel takes)
  while (part_cap < 4096 && (512ull << 20) / (ld * 4 + 2ull * part_cap * 8) / 128 * 128 >= nq) part_cap <<= 1;
  const uint32_t room = cap > part_cap ? cap : part_cap;
  // queries per round: at most half a GiB of scores and entries, less if the card has no room
  const uint64_t per_query = ld * 4 + (uint64_t)room * 8;
  uint64_t round = (512ull << 20) / per_query / 128 * 128;
  if (round < 128) round = 128;
  if (round > nq) round = nq;
  // Two parts where products take the time (up to 64 queries a call reads rows, few rows are a matter of
  // launches) and where near rows' scores lose no more than with three: from 65 columns on, see bf_score_kernel.  First parts
  // only where that costs less than it saves: every row is read once more to be rounded, and there are more passes.  That is a
  // question of the queries and, since a pass has a least time, of all scores.  Two parts / first parts, us: 1M x 128, 256 queries
  // 410 / 430, 512 656 / 491; 200,000 x 128, 512 207 / 224, 700 255 / 243; 200,000 x 768, k = 100, 400 743 / 743, 700 1,038 / 852;
  // 200,000 x 960, 512 803 / 795, 1,000 1,452 / 974; 100,000 x 300, 512 224 / 236, 700 274 / 255; 50,000 x 400, 700 235 / 291, 1,000
  // 319 / 317; 30,000 x 96, 700 133 / 132, 2,500 192 / 177.  So up to 512 queries it depends on the rows, and most sets lose; a
  // million rows would gain from somewhere between 256 and 512 queries on, and are kept with the others.
  const bool halves = !dense && nq > 64 && kb_n >= 6;
  uint64_t x_rows = 0, pair_rows = 0;
  if (halves && nq > 512 && ((uint64_t)nq * n >= 50'000'000 || nq >= 512 + kb_n * 16)) {
    x_rows = kScreenBytes / (kb_n * 32) / kSB * kSB;
    if (x_rows > (n + kSB - 1) / kSB * kSB) x_rows = (n + kSB - 1) / kSB * kSB;
    pair_rows = kScreenBytes / (kb_n * 64) / kSB * kSB;
    if (pair_rows > x_rows) pair_rows = x_rows;
  }
  auto parts = [&](uint64_t m, uint64_t (&at)[15]) {
    const uint64_t size[15] = {(m + 255) / 256 * 8 * kb_n * 192 * 16, m * ld * 4, m * room * 8, m * 8, m * 4, m * most * 4, m * 4, sizeof(CallState),
                               (uint64_t)nq * 4, 64 * 4, m * 4, (x_rows > 2 * pair_rows ? x_rows : 2 * pair_rows) * kb_n * 32, x_rows * 4, m * 4, m * 4};
    uint64_t total = 0;
    for (int i = 0; i < 15; ++i) {
      at[i] = total;
      total += up256(size[i]);
    }
    return total;
  };
  uint64_t at[15];
  unsigned char *base = nullptr;
  uint64_t m_fit = round;
  hipError_t e = alloc_some((void **)&base, m_fit, nq < 128 ? nq : 128, [&](uint64_t m) { return parts(m, at); });
  if (e != hipSuccess && x_rows) {   // no room for the rows' first parts
    x_rows = pair_rows = 0;
    m_fit = round;
    e = alloc_some((void **)&base, m_fit, nq < 128 ? nq : 128, [&](uint64_t m) { return parts(m, at); });
  }
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  round = m_fit;
  parts(round, at);
  CallState *const state = reinterpret_cast<CallState *>(base + at[7]);
  uint32_t *const uncertain = reinterpret_cast<uint32_t *>(base + at[8]);
  Selection s{};
  s.want = want;
  s.most = most;
  s.most_bound = most_bound;
  s.kb_n = kb_n;
  s.cap = cap;
  s.first = first;
  s.samples = samples;
  s.part_log2 = part_log2;
  s.part_cap = part_cap;
  s.stretches = stretches;
  s.ld = ld;
  s.vec4 = vec4;
  s.dense = dense;
  s.growth = growth;
  s.qfrag = reinterpret_cast<uint4 *>(base + at[0]);
  s.scores = reinterpret_cast<float *>(base + at[1]);
  s.buf = reinterpret_cast<uint64_t *>(base + at[2]);
  s.bound = reinterpret_cast<uint64_t *>(base + at[3]);
  s.count = reinterpret_cast<uint32_t *>(base + at[4]);
  s.cand = reinterpret_cast<uint32_t *>(base + at[5]);
  s.below = reinterpret_cast<float *>(base + at[6]);
  s.state = state;
  s.sample_sq = reinterpret_cast<float *>(base + at[9]);
  s.unscale = reinterpret_cast<float *>(base + at[10]);
  s.halves = halves;
  s.xfrag = reinterpret_cast<uint4 *>(base + at[11]);
  s.xnorm = reinterpret_cast<float *>(base + at[12]);
  s.x_rows = x_rows;
  s.pair_rows = pair_rows;
  s.q_norm = reinterpret_cast<float *>(base + at[13]);
  s.q_rest = reinterpret_cast<float *>(base + at[14]);
  const Truth t{x, n, d, q, k, metric, out_ids, out_dist, n_cu, st};

  ann_status rc = ANN_OK;
  uint32_t found[5] = {0, 0, 0, 0, 0};   // uncertain queries, far rows, queries that three parts would leave less uncertain, lost ones, passes given up
  bool idle = true;
  for (;;) {
    // the counters are cleared by the first kernel of either path
    if (s.halves) bf_sample_norms_kernel<<<kNormSample / 16, 1024, 0, st>>>(x, d, (double)n / kNormSample, s.sample_sq, &state->n_uncertain);
    for (uint64_t q0 = 0; q0 < nq && rc == ANN_OK; q0 += round) {
      const uint32_t m = (uint32_t)(nq - q0 < round ? nq - q0 : round);
      rc = select_round(t, s, q + q0 * d, m, nullptr, q0 == 0, out_ids + q0 * k, out_dist + q0 * k, uncertain, (uint32_t)q0);
    }
    // (100 queries x 10,000 rows x 128, read through pinned memory and with one launch less at the start: 65.9 -> 55.9 us)
    const hipError_t e2 = rc == ANN_OK ? read_words(&state->n_uncertain, found, 5, st) : hipStreamSynchronize(st);
    if (rc == ANN_OK && e2 != hipSuccess) rc = hip_fail(e2, "the wait for a call's counters");
    idle = e2 == hipSuccess;
    if (rc == ANN_OK && s.x_rows && (found[4] || found[3] > nq / 8 * 3)) {   // (see bf_range_kernel; of so many, 2,048 at a time cost as much)
      s.x_rows = 0;
      continue;
    }
    if (rc != ANN_OK || !s.halves || found[1] <= kFewFarRows) break;
    s.halves = false;   // inner product, more than a few rows outside half precision's range: three parts
  }
  if (rc == ANN_OK && found[1] > kFarRows) {
    rc = bruteforce_fp32(x, n, d, q, nq, k, metric, out_ids, out_dist, n_cu, st);
  } else if (rc == ANN_OK) {
    if (found[0] > 0) rc = settle(t, s, round, uncertain, found[0], found[2], s.x_rows ? found[3] : 0u);
    if (rc == ANN_OK && found[1] > 0) rc = add_far_rows(t, nq, found[1], state);
    if (rc != ANN_OK) idle = hipStreamSynchronize(st) == hipSuccess;
  }
  device_free(base, idle);
  return rc;
}
