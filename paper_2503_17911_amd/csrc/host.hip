// Host side of the library: error reporting, index upload/packing, workspace.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <new>
#include <vector>

#include "ann_internal.hpp"
#include "kept_blocks.hpp"

namespace ann {

static thread_local char g_err[512] = "";

ann_status fail(ann_status code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

ann_status hip_fail(hipError_t e, const char *what) {
  ann_status code = (e == hipErrorOutOfMemory) ? ANN_ENOMEM : ANN_EDEVICE;
  return fail(code, "%s: %s", what, hipGetErrorString(e));
}

// ---------------------------------------------------------------- device memory
// The driver clears freed memory before it hands it out again, at about 54 GB/s:
// a program that uploads and frees indexes (or runs exhaustive searches) one
// after the other soon waits for that in every hipFree - 20 ms for the 1.1 GB of a
// 200,000 x 960 index, where the whole build takes 3 - besides about 0.8 ms for
// unmapping.  So freed blocks are kept (kept_blocks.hpp says which and how many);
// all of them are given back when an allocation fails and by ann_trim_memory.
namespace {

std::mutex g_kept_mutex;
KeptBlocks g_kept;

std::mutex g_words_mutex;
uint32_t *g_words[kKeptHostWords];
int g_n_words = 0;

void give_back_kept() {
  for (;;) {
    KeptBlock b;
    {
      std::lock_guard<std::mutex> lock(g_kept_mutex);
      if (!g_kept.take_oldest(b)) return;
    }
    (void)hipFree(b.ptr);
  }
}

}  // namespace

static __global__ void copy_words_kernel(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst, int count) {
  if ((int)threadIdx.x < count) dst[threadIdx.x] = src[threadIdx.x];
}

static uint32_t *host_words_take() {
  {
    std::lock_guard<std::mutex> lock(g_words_mutex);
    if (g_n_words > 0) return g_words[--g_n_words];
  }
  void *p = nullptr;
  if (hipHostMalloc(&p, kHostWords * sizeof(uint32_t), hipHostMallocPortable) == hipSuccess) return static_cast<uint32_t *>(p);
  (void)hipGetLastError();
  return nullptr;
}

static void host_words_give(uint32_t *words) {
  {
    std::lock_guard<std::mutex> lock(g_words_mutex);
    if (g_n_words < kKeptHostWords) {
      g_words[g_n_words++] = words;
      return;
    }
  }
  (void)hipHostFree(words);
}

hipError_t read_words(const uint32_t *src, uint32_t *dst, int count, hipStream_t st) {
  uint32_t *const words = host_words_take();
  hipError_t e;
  if (words) {
    copy_words_kernel<<<1, 64, 0, st>>>(src, words, count);
    e = hipGetLastError();
  } else {
    e = hipMemcpyAsync(dst, src, (size_t)count * sizeof(uint32_t), hipMemcpyDeviceToHost, st);
  }
  const hipError_t e2 = hipStreamSynchronize(st);
  if (!words) return e != hipSuccess ? e : e2;
  if (e == hipSuccess && e2 == hipSuccess)
    for (int i = 0; i < count; ++i) dst[i] = reinterpret_cast<volatile uint32_t *>(words)[i];
  if (e2 == hipSuccess) host_words_give(words);   // (a stream that failed may still write to them)
  return e != hipSuccess ? e : e2;
}

uint32_t compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return (uint32_t)n;
}

hipError_t device_alloc(void **ptr, size_t bytes) {
  *ptr = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const size_t unit = bytes >= ((size_t)1 << 20) ? (size_t)2 << 20 : (size_t)4096;
  const size_t want = (bytes + unit - 1) / unit * unit;
  {
    std::lock_guard<std::mutex> lock(g_kept_mutex);
    KeptBlock b;
    if (g_kept.take(dev, want, b)) {
      *ptr = b.ptr;
      return hipSuccess;
    }
  }
  e = hipMalloc(ptr, want);
  if (e != hipErrorOutOfMemory) return e;
  (void)hipGetLastError();
  give_back_kept();
  return hipMalloc(ptr, want);
}

void device_free(void *ptr, bool idle) {
  if (!ptr) return;
  hipDeviceptr_t base = nullptr;
  KeptBlock b;
  hipPointerAttribute_t at{};
  if (!idle || hipMemGetAddressRange(&base, &b.bytes, (hipDeviceptr_t)ptr) != hipSuccess || hipPointerGetAttributes(&at, ptr) != hipSuccess ||
      !KeptBlocks::fits(b.bytes)) {
    (void)hipFree(ptr);
    return;
  }
  b.ptr = ptr;
  b.device = at.device;
  KeptBlock out[kKeepBlocks];
  int n_out = 0;
  {
    std::lock_guard<std::mutex> lock(g_kept_mutex);
    n_out = g_kept.put(b, out);
  }
  for (int i = 0; i < n_out; ++i) (void)hipFree(out[i].ptr);
}

// ---------------------------------------------------------------- pack kernels
// codes [n][row_bytes] -> [n][row_stride]; 8-bit codes are stored biased by
// 128 (c ^ 0x80 read as int8 is c - 128) so the signed packed-dot instruction
// applies; padding bytes are never multiplied by a non-zero query byte.
// Bound: one read and one write of the codes.  A thread moves 16 bytes of a row
// in units of ALIGN bytes, the largest of 16, 4 and 1 that divides row_bytes and
// the array's address.  (One byte per thread, with a 64-bit division each: 1M x
// 128 in 263 us; now 44 us.)
template <int ALIGN>
__global__ void pack_codes_kernel(const uint8_t *__restrict__ in, uint8_t *__restrict__ out, uint64_t n,
                                  uint32_t row_bytes, uint32_t row_stride, uint32_t flip) {
  const uint32_t pieces = row_stride / 16, flip4 = flip * 0x01010101u;
  const uint64_t total = n * pieces;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < total; e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t i = total <= 0xFFFFFFFFull ? (uint32_t)e / pieces : e / pieces;
    const uint32_t b0 = (uint32_t)(e - i * pieces) * 16;
    const uint8_t *row = in + i * row_bytes;
    uint32_t w[4] = {0, 0, 0, 0};
    if constexpr (ALIGN == 16) {
      if (b0 < row_bytes) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + b0);
        w[0] = v.x, w[1] = v.y, w[2] = v.z, w[3] = v.w;
      }
    } else if constexpr (ALIGN == 4) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (b0 + 4 * j < row_bytes) w[j] = *reinterpret_cast<const uint32_t *>(row + b0 + 4 * j);
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (b0 + j < row_bytes) w[j / 4] |= (uint32_t)row[b0 + j] << (8 * (j % 4));
    }
    reinterpret_cast<uint4 *>(out)[e] = make_uint4(w[0] ^ flip4, w[1] ^ flip4, w[2] ^ flip4, w[3] ^ flip4);
  }
}

// CSR -> [n][degree] with padding; sets *bad if a row is too long.
template <typename T>
__global__ void pack_csr_kernel(const T *__restrict__ cols, const uint64_t *__restrict__ offsets,
                                T *__restrict__ out, uint64_t n, uint32_t degree, T pad, uint32_t *bad) {
  uint64_t total = n * degree;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < total; e += (uint64_t)gridDim.x * blockDim.x) {
    uint64_t i = e / degree;
    uint32_t t = (uint32_t)(e - i * degree);
    uint64_t b = offsets[i], len = offsets[i + 1] - b;
    if (t == 0 && len > degree) atomicOr(bad, 1u);
    out[e] = (t < len) ? cols[b + t] : pad;
  }
}

// Every neighbour id is a node (bad |= 2), and a row names none twice (bad |= 4).
// LANES (a power of two, at least the degree) lanes take a row, one slot each,
// and compare it with the slots up to LANES / 2 places on.  1M rows of 32: 3.6 ms
// (one thread per row, every pair read from memory) -> 91 us.
template <int LANES>
__global__ __launch_bounds__(256) void check_adjacency_kernel(const uint32_t *__restrict__ adj, uint64_t n, uint32_t degree,
                                                              uint32_t *bad) {
  const uint32_t slot = threadIdx.x % LANES;
  const uint64_t step = (uint64_t)gridDim.x * (256 / LANES);
  uint32_t found = 0;
  for (uint64_t row = (uint64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES; row < n; row += step) {
    const uint32_t v = slot < degree ? adj[row * degree + slot] : ANN_PAD_ID;
    if (v != ANN_PAD_ID && v >= n) found |= 2u;
#pragma unroll
    for (int s = 1; s <= LANES / 2; ++s) {
      const uint32_t o = (uint32_t)__shfl((int)v, (int)((slot + s) % LANES), LANES);
      found |= v != ANN_PAD_ID && v == o ? 4u : 0u;
    }
  }
  if (found) atomicOr(bad, found);
}

// Redundant layout: entry (i, t), t < stored, receives a copy of the code row
// (and norm term) of neighbour adjacency[i][t]; padding slots are zero.
__global__ void build_prs_kernel(const uint32_t *__restrict__ adj, const uint8_t *__restrict__ codes,
                                 const float *__restrict__ norm, uint64_t n, uint32_t degree, uint32_t stored,
                                 uint32_t row_stride, uint8_t *__restrict__ out_codes, float *__restrict__ out_norm) {
  const uint32_t cpr = row_stride / 16;
  const uint64_t total = n * stored * cpr;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < total; e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t entry = e / cpr;
    const uint32_t c = (uint32_t)(e - entry * cpr);
    const uint64_t node = entry / stored;
    const uint32_t t = (uint32_t)(entry - node * stored);
    const uint32_t v = adj[node * degree + t];
    const bool real = v != ANN_PAD_ID && v < n;
    reinterpret_cast<uint4 *>(out_codes)[e] =
        real ? reinterpret_cast<const uint4 *>(codes + (uint64_t)v * row_stride)[c] : make_uint4(0, 0, 0, 0);
    if (c == 0 && out_norm) out_norm[entry] = real ? norm[v] : 0.0f;
  }
}

// Adjacency rows with the neighbours' norm terms behind them: row i is
// adjacency[i][0 .. degree) followed by norm[adjacency[i][t]] for t in
// 0 .. degree (zero for padding slots).
__global__ void build_row_norms_kernel(const uint32_t *__restrict__ adj, const float *__restrict__ norm, uint64_t n,
                                       uint32_t degree, uint32_t *__restrict__ out) {
  const uint64_t total = n * degree;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < total; e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t node = e / degree;
    const uint32_t t = (uint32_t)(e - node * degree);
    const uint32_t v = adj[e];
    const bool real = v != ANN_PAD_ID && v < n;
    out[node * 2 * degree + t] = v;
    out[node * 2 * degree + degree + t] = real ? __float_as_uint(norm[v]) : 0u;
  }
}

namespace {

// Device buffer holding a copy of `count` elements from host or device memory.
template <typename T>
ann_status dev_copy(T **dst, const T *src, size_t count, bool src_on_host, hipStream_t st) {
  *dst = nullptr;
  if (count == 0) return ANN_OK;
  ANN_HIP(device_alloc((void **)dst, count * sizeof(T)));
  ANN_HIP(hipMemcpyAsync(*dst, src, count * sizeof(T), src_on_host ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice,
                         st));
  return ANN_OK;
}

void free_workspace(Workspace &w, bool idle) {
  device_free(w.tq, idle);
  device_free(w.s, idle);
  device_free(w.qlo, idle);
  device_free(w.sum_t, idle);
  w = Workspace{};
}

// idle: nothing enqueued on the device can be using the index.
void destroy(ann_index *ix, bool idle) {
  if (!ix) return;
  device_free(ix->vectors, idle);
  device_free(ix->adjacency, idle);
  device_free(ix->labels, idle);
  device_free(ix->adjacency_norms, idle);
  device_free(ix->pivot_codes, idle);
  device_free(ix->prs_codes, idle);
  device_free(ix->prs_norm, idle);
  device_free(ix->pivot_norm, idle);
  device_free(ix->pivot_ids, idle);
  for (int l = 0; l < ANN_MAX_LEVELS; ++l) {
    device_free(ix->level[l].codes, idle);
    device_free(ix->level[l].lo, idle);
    device_free(ix->level[l].delta, idle);
    device_free(ix->level[l].norm_term, idle);
  }
  for (StreamWorkspaces &sw : ix->stream_ws)
    for (Workspace &w : sw.ws) free_workspace(w, idle);
  delete ix;
}

inline int grid_for(uint64_t total, int block) {
  uint64_t g = (total + block - 1) / block;
  return (int)(g > 65535 * 16 ? 65535 * 16 : (g ? g : 1));
}

}  // namespace

uint32_t streams_in_use(const ann_index *ix) {
  uint32_t n = 0;
  for (const StreamWorkspaces &c : ix->stream_ws) n += c.used && ix->ws_clock - c.last_use < kRecentCalls ? 1u : 0u;
  return n > 0 ? n : 1u;
}

ann_status workspace_for(ann_index *ix, uint32_t level, uint32_t nq, hipStream_t st, WorkspaceLease &lease) {
  if (!lease.lock.owns_lock()) lease.lock = std::unique_lock<std::mutex>(ix->ws_mutex);
  StreamWorkspaces *sw = nullptr, *free_slot = nullptr, *oldest = nullptr;
  for (StreamWorkspaces &c : ix->stream_ws) {
    if (c.used && c.stream == st) {
      sw = &c;
      break;
    }
    if (!c.used && !free_slot) free_slot = &c;
    if (c.used && (!oldest || c.last_use < oldest->last_use)) oldest = &c;
  }
  if (!sw) {
    if (free_slot) {
      sw = free_slot;
    } else {
      // every set is taken: hand the least recently used one to this stream,
      // once nothing on the device can still be reading it
      ANN_HIP(hipDeviceSynchronize());
      sw = oldest;
      for (Workspace &w : sw->ws) w.folded_q = nullptr, w.folded_nq = 0;
    }
    sw->used = true;
    sw->stream = st;
  }
  sw->last_use = ++ix->ws_clock;
  Workspace &w = sw->ws[level];
  lease.ws = &w;
  if (nq <= w.nq_cap) return ANN_OK;
  // growth is the only allocation on the search path (ann_reserve_workspace
  // moves it out of the path); it waits for work that may still be using the
  // old buffers
  ANN_HIP(hipDeviceSynchronize());
  free_workspace(w, true);
  uint32_t cap = nq < 1024 ? 1024 : nq;
  w.tq_plane = tq_plane_for(ix->level[level]);
  w.tq_stride = w.tq_plane * (ix->query_bits == 15 ? 2u : 1u);
  ANN_HIP(device_alloc((void **)&w.tq, (size_t)cap * w.tq_stride));
  ANN_HIP(device_alloc((void **)&w.s, (size_t)cap * sizeof(float)));
  ANN_HIP(device_alloc((void **)&w.qlo, (size_t)cap * sizeof(float)));
  ANN_HIP(device_alloc((void **)&w.sum_t, (size_t)cap * 2 * sizeof(int32_t)));
  w.nq_cap = cap;
  return ANN_OK;
}

}  // namespace ann

using namespace ann;

extern "C" {

const char *ann_last_error(void) { return g_err; }
const char *ann_version(void) { return "ann-gfx950 0.1"; }

ann_status ann_upload_index(const ann_index_desc *desc, void *stream, ann_index **out) {
  hipStream_t st = (hipStream_t)stream;
  if (!out) return fail(ANN_EINVAL, "ann_upload_index: out is NULL");
  *out = nullptr;
  if (!desc) return fail(ANN_EINVAL, "ann_upload_index: desc is NULL");
  if (desc->n == 0 || desc->n >= (1ull << 31)) return fail(ANN_EINVAL, "n must be in [1, 2^31), got %llu", (unsigned long long)desc->n);
  if (desc->d == 0) return fail(ANN_EINVAL, "d must be positive");
  if (desc->d > 2048) return fail(ANN_ECAPACITY, "d = %u exceeds the supported maximum 2048", desc->d);
  if (desc->degree == 0) return fail(ANN_EINVAL, "degree must be positive");
  if (desc->degree > ANN_MAX_DEGREE) return fail(ANN_ECAPACITY, "degree = %u exceeds ANN_MAX_DEGREE = %u", desc->degree, ANN_MAX_DEGREE);
  if (desc->metric != ANN_L2 && desc->metric != ANN_IP) return fail(ANN_EINVAL, "unknown metric %u", desc->metric);
  if ((desc->flags & ANN_DESC_UNIT_NORM_L2_KEYS) && desc->metric != ANN_IP)
    return fail(ANN_EINVAL, "ANN_DESC_UNIT_NORM_L2_KEYS is for ANN_IP indexes");
  if (desc->n_levels < 1 || desc->n_levels > ANN_MAX_LEVELS) return fail(ANN_EINVAL, "n_levels must be 1..%d", ANN_MAX_LEVELS);
  if (!desc->adjacency) return fail(ANN_EINVAL, "adjacency is NULL");
  if (desc->entry_point >= desc->n) return fail(ANN_EINVAL, "entry_point %u is not a node", desc->entry_point);
  for (uint32_t l = 0; l < desc->n_levels; ++l) {
    const ann_sq_level &L = desc->level[l];
    if (L.bits != 8 && L.bits != 4) return fail(ANN_EINVAL, "level %u: bits must be 4 or 8, got %u", l, L.bits);
    if (L.bits == 4 && (desc->d & 1)) return fail(ANN_EINVAL, "level %u: 4-bit codes need an even d", l);
    if (!L.codes || !L.lo || !L.delta) return fail(ANN_EINVAL, "level %u: codes, lo and delta must be given", l);
    if ((desc->metric == ANN_L2 || (desc->flags & ANN_DESC_UNIT_NORM_L2_KEYS)) && !L.norm_term)
      return fail(ANN_EINVAL, "level %u: norm_term is required for ANN_L2 and for ANN_DESC_UNIT_NORM_L2_KEYS", l);
  }
  const bool host = (desc->flags & ANN_DESC_HOST_POINTERS) != 0;
  const uint64_t n = desc->n;

  ann_index *ix = new (std::nothrow) ann_index();
  if (!ix) return fail(ANN_ENOMEM, "host allocation failed");
  ix->n = n;
  ix->d = desc->d;
  ix->degree = desc->degree;
  ix->metric = desc->metric;
  ix->query_bits = (desc->flags & ANN_DESC_QUERY_15BIT) ? 15u : 8u;
  ix->key_metric = (desc->flags & ANN_DESC_UNIT_NORM_L2_KEYS) ? (uint32_t)ANN_L2 : desc->metric;
  ix->n_levels = desc->n_levels;
  ix->entry_point = desc->entry_point;
  (void)hipGetDevice(&ix->device);
  ix->n_cu = (int)compute_units();

  ann_status rc = ANN_OK;
  uint32_t *bad_dev = nullptr;
  uint8_t *raw_codes = nullptr;
  uint32_t *raw_cols = nullptr;
  uint64_t *raw_offs = nullptr;
  float *raw_labels = nullptr;
  auto cleanup = [&](ann_status r) {
    // (after a failure what has been enqueued may still use the buffers)
    const bool idle = r == ANN_OK || hipDeviceSynchronize() == hipSuccess;
    device_free(bad_dev, idle);
    device_free(raw_codes, idle);
    device_free(raw_cols, idle);
    device_free(raw_offs, idle);
    device_free(raw_labels, idle);
    if (r != ANN_OK) destroy(ix, idle);
    return r;
  };
#define ANN_TRY(expr)                      \
  do {                                     \
    rc = (expr);                           \
    if (rc != ANN_OK) return cleanup(rc);  \
  } while (0)
#define ANN_TRY_HIP(call)                                         \
  do {                                                            \
    hipError_t e_ = (call);                                       \
    if (e_ != hipSuccess) return cleanup(hip_fail(e_, #call));    \
  } while (0)

  ANN_TRY_HIP(device_alloc((void **)&bad_dev, sizeof(uint32_t)));
  ANN_TRY_HIP(hipMemsetAsync(bad_dev, 0, sizeof(uint32_t), st));

  if (desc->vectors) ANN_TRY(dev_copy(&ix->vectors, desc->vectors, (size_t)n * desc->d, host, st));

  for (uint32_t l = 0; l < desc->n_levels; ++l) {
    const ann_sq_level &S = desc->level[l];
    LevelDev &L = ix->level[l];
    L.bits = S.bits;
    L.row_bytes = S.bits == 8 ? desc->d : desc->d / 2;
    // Rows start on 16-byte boundaries.  Where it costs at most a third more
    // memory they are also laid out so that no row crosses more 128-byte lines
    // than it must: a stride that divides 128 or is a multiple of it (96-byte
    // rows at stride 128 touch one line each instead of one or two; 480-byte
    // rows at stride 512 four instead of four or five).
    L.row_stride = (L.row_bytes + 15u) & ~15u;
    {
      uint32_t aligned = L.row_bytes <= 16 ? 16u : L.row_bytes <= 32 ? 32u : L.row_bytes <= 64 ? 64u : (L.row_bytes + 127u) & ~127u;
      if ((aligned - L.row_bytes) * 3u <= L.row_bytes) L.row_stride = aligned;
    }
    const uint32_t chunks = L.row_stride / 16u;
    if (chunks > 64) return cleanup(fail(ANN_ECAPACITY, "level %u: code rows of %u bytes exceed 1024", l, L.row_bytes));
    uint32_t sl = 1;
    while (sl * 4 < chunks) sl <<= 1;
    L.search_lanes = sl;
    ANN_TRY(dev_copy(&L.lo, S.lo, desc->d, host, st));
    ANN_TRY(dev_copy(&L.delta, S.delta, desc->d, host, st));
    if (S.norm_term) ANN_TRY(dev_copy(&L.norm_term, S.norm_term, (size_t)n, host, st));
    const uint8_t *src = S.codes;
    if (host) {
      ANN_TRY(dev_copy(&raw_codes, S.codes, (size_t)n * L.row_bytes, true, st));
      src = raw_codes;
    }
    ANN_TRY_HIP(device_alloc((void **)&L.codes, (size_t)n * L.row_stride));
    const uint64_t total = n * (L.row_stride / 16);
    const uint32_t flip = S.bits == 8 ? 0x80u : 0u;
    const uintptr_t together = reinterpret_cast<uintptr_t>(src) | L.row_bytes;
    if (together % 16 == 0)
      pack_codes_kernel<16><<<grid_for(total, 256), 256, 0, st>>>(src, L.codes, n, L.row_bytes, L.row_stride, flip);
    else if (together % 4 == 0)
      pack_codes_kernel<4><<<grid_for(total, 256), 256, 0, st>>>(src, L.codes, n, L.row_bytes, L.row_stride, flip);
    else
      pack_codes_kernel<1><<<grid_for(total, 256), 256, 0, st>>>(src, L.codes, n, L.row_bytes, L.row_stride, flip);
    ANN_TRY_HIP(hipGetLastError());
    if (host) {
      ANN_TRY_HIP(hipStreamSynchronize(st));
      device_free(raw_codes, true);
      raw_codes = nullptr;
    }
  }

  const uint64_t total_adj = n * desc->degree;
  if (desc->csr_offsets) {
    const uint64_t *offs = desc->csr_offsets;
    const uint32_t *cols = desc->adjacency;
    uint64_t nnz = 0;
    if (host) {
      nnz = desc->csr_offsets[n];
      ANN_TRY(dev_copy(&raw_offs, desc->csr_offsets, (size_t)n + 1, true, st));
      ANN_TRY(dev_copy(&raw_cols, desc->adjacency, (size_t)nnz, true, st));
      offs = raw_offs;
      cols = raw_cols;
    }
    ANN_TRY_HIP(device_alloc((void **)&ix->adjacency, total_adj * sizeof(uint32_t)));
    pack_csr_kernel<uint32_t><<<grid_for(total_adj, 256), 256, 0, st>>>(cols, offs, ix->adjacency, n, desc->degree,
                                                                         ANN_PAD_ID, bad_dev);
    ANN_TRY_HIP(hipGetLastError());
    if (desc->edge_labels) {
      const float *lab = desc->edge_labels;
      if (host) {
        ANN_TRY(dev_copy(&raw_labels, desc->edge_labels, (size_t)nnz, true, st));
        lab = raw_labels;
      }
      ANN_TRY_HIP(device_alloc((void **)&ix->labels, total_adj * sizeof(float)));
      pack_csr_kernel<float><<<grid_for(total_adj, 256), 256, 0, st>>>(lab, offs, ix->labels, n, desc->degree, 0.0f,
                                                                        bad_dev);
      ANN_TRY_HIP(hipGetLastError());
    }
  } else {
    ANN_TRY(dev_copy(&ix->adjacency, desc->adjacency, (size_t)total_adj, host, st));
    if (desc->edge_labels) ANN_TRY(dev_copy(&ix->labels, desc->edge_labels, (size_t)total_adj, host, st));
  }
  {
    const uint32_t lanes = desc->degree <= 8 ? 8u : (desc->degree <= 16 ? 16u : (desc->degree <= 32 ? 32u : 64u));
    const uint64_t blocks = (n + 256 / lanes - 1) / (256 / lanes);
    const int grid = (int)(blocks < 16384 ? blocks : 16384);
    switch (lanes) {
      case 8: check_adjacency_kernel<8><<<grid, 256, 0, st>>>(ix->adjacency, n, desc->degree, bad_dev); break;
      case 16: check_adjacency_kernel<16><<<grid, 256, 0, st>>>(ix->adjacency, n, desc->degree, bad_dev); break;
      case 32: check_adjacency_kernel<32><<<grid, 256, 0, st>>>(ix->adjacency, n, desc->degree, bad_dev); break;
      default: check_adjacency_kernel<64><<<grid, 256, 0, st>>>(ix->adjacency, n, desc->degree, bad_dev);
    }
  }
  ANN_TRY_HIP(hipGetLastError());
  uint32_t bad = 0;
  ANN_TRY_HIP(read_words(bad_dev, &bad, 1, st));
  if (bad & 1u) return cleanup(fail(ANN_EINVAL, "a CSR row has more than degree = %u neighbours", desc->degree));
  if (bad & 2u) return cleanup(fail(ANN_EINVAL, "adjacency holds a neighbour id >= n"));
  if (bad & 4u) return cleanup(fail(ANN_EINVAL, "an adjacency row names the same neighbour twice"));
#undef ANN_TRY
#undef ANN_TRY_HIP
  cleanup(ANN_OK);
  *out = ix;
  return ANN_OK;
}

ann_status ann_build_prs_ratio(ann_index *index, float ratio, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!index) return fail(ANN_EINVAL, "ann_build_prs_ratio: index is NULL");
  if (!(ratio > 0.0f && ratio <= 1.0f)) return fail(ANN_EINVAL, "ann_build_prs_ratio: the ratio must be in (0, 1]");
  uint32_t stored = (uint32_t)((double)ratio * index->degree + 0.999999);
  if (stored < 1) stored = 1;
  if (stored > index->degree) stored = index->degree;
  if (index->prs_codes && index->prs_slots == stored) return ANN_OK;
  if (index->prs_codes) {
    ANN_HIP(hipDeviceSynchronize());  // a search may still be reading the old copy
    device_free(index->prs_codes, true);
    device_free(index->prs_norm, true);
    index->prs_codes = nullptr;
    index->prs_norm = nullptr;
    index->prs_slots = 0;
  }
  const LevelDev &L = index->level[0];
  const uint64_t entries = index->n * stored;
  ANN_HIP(device_alloc((void **)&index->prs_codes, (size_t)entries * L.row_stride));
  if (index->key_metric == ANN_L2) {
    hipError_t e = device_alloc((void **)&index->prs_norm, (size_t)entries * sizeof(float));
    if (e != hipSuccess) {
      device_free(index->prs_codes, true);
      index->prs_codes = nullptr;
      return hip_fail(e, "hipMalloc");
    }
  }
  const uint64_t total = entries * (L.row_stride / 16);
  build_prs_kernel<<<grid_for(total, 256), 256, 0, st>>>(index->adjacency, L.codes, index->prs_norm ? L.norm_term : nullptr,
                                                         index->n, index->degree, stored, L.row_stride, index->prs_codes,
                                                         index->prs_norm);
  ANN_HIP(hipGetLastError());
  ANN_HIP(hipStreamSynchronize(st));
  index->prs_slots = stored;
  return ANN_OK;
}

ann_status ann_build_row_norms(ann_index *index, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (!index) return fail(ANN_EINVAL, "ann_build_row_norms: index is NULL");
  if (index->adjacency_norms) return ANN_OK;
  const LevelDev &L = index->level[0];
  if (index->key_metric != ANN_L2 || !L.norm_term)
    return fail(ANN_EINVAL, "ann_build_row_norms: the index's keys use no norm term (inner-product keys)");
  ANN_HIP(device_alloc((void **)&index->adjacency_norms, (size_t)index->n * index->degree * 2 * sizeof(uint32_t)));
  build_row_norms_kernel<<<grid_for(index->n * index->degree, 256), 256, 0, st>>>(index->adjacency, L.norm_term, index->n,
                                                                                  index->degree, index->adjacency_norms);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    device_free(index->adjacency_norms, false);
    index->adjacency_norms = nullptr;
    return hip_fail(e, "build_row_norms_kernel");
  }
  return ANN_OK;
}

ann_status ann_build_prs(ann_index *index, void *stream) {
  if (!index) return fail(ANN_EINVAL, "ann_build_prs: index is NULL");
  return ann_build_prs_ratio(index, 1.0f, stream);
}

ann_status ann_reserve_workspace(ann_index *index, uint32_t max_nq, void *stream) {
  if (!index) return fail(ANN_EINVAL, "ann_reserve_workspace: index is NULL");
  if (max_nq == 0) return fail(ANN_EINVAL, "ann_reserve_workspace: max_nq == 0");
  WorkspaceLease lease;
  for (uint32_t l = 0; l < index->n_levels; ++l) {
    ann_status rc = workspace_for(index, l, max_nq, (hipStream_t)stream, lease);
    if (rc != ANN_OK) return rc;
  }
  return ANN_OK;
}

ann_status ann_free_index(ann_index *index) {
  if (!index) return ANN_OK;
  int dev = index->device;
  (void)hipGetDevice(&dev);
  if (dev != index->device) (void)hipSetDevice(index->device);
  const bool idle = hipDeviceSynchronize() == hipSuccess;
  if (dev != index->device) (void)hipSetDevice(dev);
  destroy(index, idle);
  return ANN_OK;
}

ann_status ann_trim_memory(void) {
  give_back_kept();
  for (;;) {
    uint32_t *words = nullptr;
    {
      std::lock_guard<std::mutex> lock(g_words_mutex);
      if (g_n_words > 0) words = g_words[--g_n_words];
    }
    if (!words) return ANN_OK;
    (void)hipHostFree(words);
  }
}

}  // extern "C"
