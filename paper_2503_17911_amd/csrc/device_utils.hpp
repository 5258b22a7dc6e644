// Wave64 device helpers for gfx950: cross-lane reductions on DPP, the
// order-preserving key transform, and the code-row dot product.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ann {

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// DPP controls (GFX9 encoding).
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm:[1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm:[2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ int xor_lane_i32(int v, int mask) {
  return __builtin_amdgcn_ds_bpermute((lane_id() ^ mask) << 2, v);
}

// A lane's own value and that of the lane 16 (ROWS) or 32 lanes away, the lower lane's first.
struct LanePair {
  uint32_t low, high;
};
template <bool ROWS>
__device__ __forceinline__ LanePair lane_pair(uint32_t v) {
  const auto p = ROWS ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return {p[0], p[1]};
}
__device__ __forceinline__ int half_sum_i32(int v) {
  const LanePair p = lane_pair<false>((uint32_t)v);
  return (int)(p.low + p.high);
}

// Sum over aligned groups of W consecutive lanes; every lane of the group
// ends with the group's total.  W in {1,2,4,8,16,32,64}.  No LDS round trips
// (about 130 cycles each): exchanges inside a row of 16 lanes by DPP - once a
// quad's lanes hold one value, the mirrored lane's is that of the lane 4 or 8 away -
// and between rows by lane swaps.
template <int W>
__device__ __forceinline__ int group_sum_i32(int v) {
  if constexpr (W >= 2) v += dpp_i32<kDppQuadXor1>(v);
  if constexpr (W >= 4) v += dpp_i32<kDppQuadXor2>(v);
  if constexpr (W >= 8) v += dpp_i32<kDppRowHalfMirror>(v);
  if constexpr (W >= 16) v += dpp_i32<kDppRowMirror>(v);
  if constexpr (W >= 32) {
    const LanePair p = lane_pair<true>((uint32_t)v);
    v = (int)(p.low + p.high);
  }
  if constexpr (W >= 64) v = half_sum_i32(v);
  return v;
}

// Inclusive prefix sum over the 64 lanes (row shifts inside each row of 16
// lanes, then the row totals are broadcast to the rows that follow).
__device__ __forceinline__ int wave_inclusive_scan_i32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ double xor_lane_f64(double v, int mask) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = xor_lane_i32(lo, mask);
  hi = xor_lane_i32(hi, mask);
  return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  return __hiloint2double(dpp_i32<CTRL>(__double2hiint(v)), dpp_i32<CTRL>(__double2loint(v)));
}
template <bool ROWS>
__device__ __forceinline__ double pair_sum_f64(double v) {
  const LanePair lo = lane_pair<ROWS>((uint32_t)__double2loint(v)), hi = lane_pair<ROWS>((uint32_t)__double2hiint(v));
  return __hiloint2double((int)hi.low, (int)lo.low) + __hiloint2double((int)hi.high, (int)lo.high);
}
template <int W>
__device__ __forceinline__ double group_sum_f64(double v) {
  if constexpr (W >= 2) v += dpp_f64<kDppQuadXor1>(v);
  if constexpr (W >= 4) v += dpp_f64<kDppQuadXor2>(v);
  if constexpr (W >= 8) v += dpp_f64<kDppRowHalfMirror>(v);
  if constexpr (W >= 16) v += dpp_f64<kDppRowMirror>(v);
  if constexpr (W >= 32) v = pair_sum_f64<true>(v);
  if constexpr (W >= 64) v = pair_sum_f64<false>(v);
  return v;
}

__device__ __forceinline__ float wave_max_f32(float v) {
  v = fmaxf(v, __int_as_float(dpp_i32<kDppQuadXor1>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i32<kDppQuadXor2>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i32<kDppRowHalfMirror>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i32<kDppRowMirror>(__float_as_int(v))));
  LanePair p = lane_pair<true>(__float_as_uint(v));
  v = fmaxf(__uint_as_float(p.low), __uint_as_float(p.high));
  p = lane_pair<false>(__float_as_uint(v));
  return fmaxf(__uint_as_float(p.low), __uint_as_float(p.high));
}

// Where a result is defined as an fp64 sum of `count` terms in a given order,
// rounded once to fp32, the sum may be formed in any order as long as every
// order rounds to the same float.  Two sums of the same terms differ by at most
// 2 (count - 1) u / (1 - (count - 1) u) times the sum of the terms' magnitudes
// (u = 2^-53); `magnitudes` is that sum as computed, and the bound below leaves
// room for its own rounding and for that of the two ends of the interval.
// False (also for sums that are not finite): form the sum in the given order.
__device__ __forceinline__ bool certain_f32(double sum, double magnitudes, uint32_t count, float &rounded) {
  const double room = magnitudes * ((double)(2 * count + 16) * 0x1p-53);
  const float low = (float)(sum - room), high = (float)(sum + room);
  rounded = low;
  return low == high && fabsf(low) < INFINITY && (low != 0.0f || room == 0.0);
}

// acc + the lanes' terms, added one after the other (the whole wavefront takes
// part and all lanes get the result; a lane without a term brings 0).  `room`:
// 64 doubles of LDS that belong to the wavefront.  Through LDS the 64 terms come
// ahead of the chain of additions; lane by lane (v_readlane) an addition took
// 90 cycles.
__device__ __forceinline__ double add_in_order(double acc, double term, double *room) {
  room[lane_id()] = term;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int h = 0; h < 64; h += 32) {
    double t[32];
#pragma unroll
    for (int l = 0; l < 32; ++l) t[l] = room[h + l];
#pragma unroll
    for (int l = 0; l < 32; ++l) acc += t[l];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return acc;
}

// Inner product of two rows, summed in fp64 in dimension order and rounded
// once, by a whole wavefront.
__device__ __forceinline__ float dot_in_order(const float *a, const float *b, uint32_t d, double *room) {
  double acc = 0.0;
  for (uint32_t base = 0; base < d; base += 64) {
    const uint32_t j = base + (uint32_t)lane_id();
    acc = add_in_order(acc, j < d ? (double)a[j] * (double)b[j] : 0.0, room);
  }
  return (float)acc;
}

// Row of x that is row j of a sample: a random one of the j-th stretch of rows
// (the stretches tile the whole set, so the rows are distinct).
__device__ __forceinline__ uint64_t sample_row(uint64_t j, double stretch) {
  uint32_t h = (uint32_t)j * 0x9E3779B1u;
  h = (h ^ (h >> 15)) * 0x85EBCA77u;
  h ^= h >> 13;
  const uint64_t begin = (uint64_t)((double)j * stretch), end = (uint64_t)((double)(j + 1) * stretch);
  return begin + __umulhi(h, (uint32_t)(end - begin));
}

// fp32 -> uint32 such that unsigned order equals numeric order (no NaN).
__device__ __forceinline__ uint32_t order_u32(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unorder_f32(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

// Traversal key from the integer dot product (paper Section 5.2: squared L2 as
// stored norm minus twice the inner product; the per-query ||q||^2 is left out).
// Written with explicit roundings so that it is one multiply (exact), one
// subtract and one fused multiply-add, whatever the compiler's contraction mode.
__device__ __forceinline__ float key_from_idot(uint32_t metric, float s, float qlo, int idot, float norm_term) {
  float key;
  if (metric == ANN_L2) {
    float h = __fsub_rn(norm_term, __fmul_rn(2.0f, qlo));
    key = __fmaf_rn(__fmul_rn(-2.0f, s), (float)idot, h);
  } else {
    key = -__fmaf_rn(s, (float)idot, qlo);
  }
  uint32_t b = __float_as_uint(key);
  if ((b & 0x7FFFFFFFu) == 0) b = 0;  // -0 -> +0
  return __uint_as_float(b);
}

// The same for the 15-bit folded query, whose integer dot product arrives as
// two parts (query value = 128 * hi + lo): they are joined in 64 bits and
// converted to fp32 with one rounding.
__device__ __forceinline__ float key_from_idot15(uint32_t metric, float s, float qlo, int idot_hi, int idot_lo,
                                                 float norm_term) {
  const long long idot = (long long)idot_hi * 128 + (long long)idot_lo;
  const float f = __ll2float_rn(idot);
  float key;
  if (metric == ANN_L2) {
    float h = __fsub_rn(norm_term, __fmul_rn(2.0f, qlo));
    key = __fmaf_rn(__fmul_rn(-2.0f, s), f, h);
  } else {
    key = -__fmaf_rn(s, f, qlo);
  }
  uint32_t b = __float_as_uint(key);
  if ((b & 0x7FFFFFFFu) == 0) b = 0;
  return __uint_as_float(b);
}

// Partial integer dot product of one 16-byte code chunk with this lane's
// share of the folded query.
//   BITS == 8: the chunk holds 16 codes stored as (c ^ 0x80), i.e. c - 128 as
//              int8; tq[0..3] hold the 16 matching query bytes.
//   BITS == 4: the chunk holds 32 codes; tq[0..3] hold the query bytes of the
//              even dimensions (low nibbles), tq[4..7] those of the odd ones.
template <int BITS>
__device__ __forceinline__ int chunk_dot(const uint4 &c, const int *tq) {
  int acc = 0;
  if constexpr (BITS == 8) {
    acc = __builtin_amdgcn_sdot4(tq[0], (int)c.x, acc, false);
    acc = __builtin_amdgcn_sdot4(tq[1], (int)c.y, acc, false);
    acc = __builtin_amdgcn_sdot4(tq[2], (int)c.z, acc, false);
    acc = __builtin_amdgcn_sdot4(tq[3], (int)c.w, acc, false);
  } else {
    const uint32_t m = 0x0F0F0F0Fu;
    acc = __builtin_amdgcn_sdot4(tq[0], (int)(c.x & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[4], (int)((c.x >> 4) & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[1], (int)(c.y & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[5], (int)((c.y >> 4) & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[2], (int)(c.z & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[6], (int)((c.z >> 4) & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[3], (int)(c.w & m), acc, false);
    acc = __builtin_amdgcn_sdot4(tq[7], (int)((c.w >> 4) & m), acc, false);
  }
  return acc;
}

// Dimension that byte e of word w of a folded query holds (the words in the order chunk_dot takes them).
template <int BITS>
__device__ __forceinline__ uint32_t folded_dim(uint32_t w, uint32_t e) {
  return BITS == 8 ? 4 * w + e : w / 8 * 32 + w % 4 * 8 + e * 2 + w % 8 / 4;
}

template <int BITS>
struct TqRegs {
  static constexpr int kWords = BITS == 8 ? 4 : 8;
};

}  // namespace ann
