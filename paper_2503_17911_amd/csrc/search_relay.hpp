// Several expansions per step for small batches: a query's chain of steps shared
// out between a wavefront that keeps the pool and four that evaluate.
//
// A step is selection, adjacency rows, visited filter, code rows, merge.  The
// merge is the longest part, and what is expanded next does not have to wait for
// it: the P closest un-expanded entries of the merged pool are the P smallest of
// the un-expanded entries before and the step's candidates.  So while the workers
// evaluate, the keeper merges the candidates of earlier steps (once there are enough
// to be worth it) and lists the pool's closest un-expanded entries; when the workers are
// done it ranks those together with the few candidates that are closer than the last of
// them, and hands out the first P.  The pool's size is kept: with n candidates pending, a
// node is handed out ahead of the merge only if it comes no later than the pool's entry n
// places before the last; where that fails, or many candidates are closer (at a search's
// start), the merge comes first.
//
// A worker takes every fourth node: adjacency row, visited filter, code rows, keys, and
// what beats the pool's last entry (as of the hand-out: the merge drops the rest) goes to
// LDS.  Two barriers a step, of LDS only.
//
// The visited set is a bit per node where those fit in LDS, else SearchWave's cache.  The workers enter nodes into the cache as
// they come to them, so which node is forgotten, and how many are evaluated again, depends on timing; the pool does not.
//
// Bound: a step's chain, about 3,700 cycles at 1M x 128 (5,600 with search_team_kernel): hand-out and
// barriers 500, adjacency and code rows 1,100 from behind the L2, keys and what goes to LDS 500, ranking 700, a merge
// where it is longer than the workers' part.  Search call, search_team_kernel / this one: one query on 1M x 128, ef =
// 128: 105 / 80 us, 100 queries 327 / 232; 100 x 100,000 x 128, ef = 400: 313 / 198; 100 x 100,000 x 960 4-bit, ef = 256
// 219 / 176; 100 x 10,000 x 128, ef = 64: 57 / 47.
#pragma once
#include "search_kernel.hpp"

namespace ann {

constexpr int kRelayWorkers = 4;
// Wavefronts per SIMD a kernel is compiled for (five: 96 registers; four: 128), and queries to a compute unit: of a
// query's five wavefronts two are on the first SIMD.  96 registers bring a third query and cost spills in most kernels with
// four pool registers or more.  60,000 nodes, search call with 128 / 96: 128-byte rows, ef = 512, 100 queries 215 / 220 us, 512 234 /
// 243, 768 (with 128 not resident: another kernel) 377 / 263; 200 dimensions, 4 bits, ef = 256 119 / 123, 135 / 140, 191 / 152; 400, 8
// bits, ef = 128 115 / 115, 133 / 133, 163 / 140.  128 where 96 cost more than the third query gives: 16 lanes (900, 8 bits, ef =
// 128 136 / 250, 168 / 351, 228 / 415), 4-bit rows of eight lanes (960, ef = 128 129 / 195, 149 / 233, 171 / 263) or with eight pool
// registers (200, ef = 512 228 / 289, 269 / 344, 398 / 388).
__host__ __device__ constexpr int relay_waves(int bits, int lpr, int m) { return (bits == 8 ? lpr <= 8 : lpr <= 4 && m < 8) ? 5 : 4; }
__host__ __device__ constexpr uint32_t relay_queries(int bits, int lpr, int m) { return relay_waves(bits, lpr, m) == 5 ? 3u : 2u; }

// Whether every slot of an adjacency row has lanes of its own: no list of the unvisited neighbours then.  (Built for rows of one
// and two lanes; both the LDS that a launch is granted and the kernel that is launched follow from this.)
__host__ __device__ constexpr bool relay_by_slot(uint32_t lpr, uint32_t degree) { return lpr <= 2 && degree * lpr <= 64u; }
static_assert(relay_by_slot(1, ANN_MAX_DEGREE), "rows of one lane have no kernel with a list");

constexpr int kNear = 32;   // un-expanded pool entries and candidates that the next step's nodes are picked from

struct alignas(16) RelayShared {
  uint64_t near[kNear];
  uint64_t worst;
  uint32_t n_out, n_picks, n_eval, pad;
  uint32_t picks[8];
  float s, qlo;
  int32_t bias;
  uint32_t pad2[3];
};
static_assert(sizeof(RelayShared) % 16 == 0, "what follows it in LDS is read 16 bytes at a time");

__host__ inline size_t relay_smem_bytes(int m, int p, bool by_slot, uint32_t vis_words, uint32_t tq_stride) {
  return (size_t)(merge_buf_entries(m) + stage_area_entries(m, 1, true) + p * 64 + (by_slot ? 0 : p * 64)) * 8 + sizeof(RelayShared) + tq_stride +
         (size_t)vis_words * 4;
}

ann_status launch_search_relay(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, bool wide_step, hipStream_t st);

template <int BITS, int LPR, int M, int P, bool BY_SLOT>
struct SearchRelay : SearchWave<BITS, LPR, M, 1, true, 1, true, false, true> {
  using Base = SearchWave<BITS, LPR, M, 1, true, 1, true, false, true>;
  using Base::a;
  using Base::bias;
  using Base::cand;
  using Base::coff;
  using Base::CPL;
  using Base::ef_q;
  using Base::G;
  using Base::grp;
  using Base::lane;
  using Base::n_dist;
  using Base::n_exp;
  using Base::pk;
  using Base::pv;
  using Base::qlo;
  using Base::s;
  using Base::sub;
  using Base::vis;
  using Base::worst;

  static constexpr int kNodes = P / kRelayWorkers;    // per worker and step
  // Candidates are merged once there are more than this many (8, 16, 24, 40 within 3 %; every step, 100 queries on
  // 1M x 128: 243 against 232 us).  With the cache at every step: a forgotten node must not meet itself with
  // another mark.
  static constexpr int kLazy = 16;

  RelayShared *sh;
  uint64_t *out;    // LDS [64 P]: the step's candidates
  uint64_t *list;   // LDS [64 kNodes] of this worker (not BY_SLOT): unvisited neighbours
  uint32_t n32;

  __device__ __forceinline__ SearchRelay(const SearchArgs &args, uint64_t *smem, int worker) : Base(args, smem) {
    out = this->stage + stage_area_entries(M, 1, true);
    sh = reinterpret_cast<RelayShared *>(out + 64 * P);
    uint64_t *at = reinterpret_cast<uint64_t *>(sh + 1);
    list = at + (worker > 0 ? worker - 1 : 0) * 64 * kNodes;
    if (!BY_SLOT) at += 64 * P;
    this->tql = reinterpret_cast<const int *>(at);
    vis = reinterpret_cast<uint32_t *>(at + a.tq_stride / 8);
    n32 = a.n < 0xFFFFFFFFull ? (uint32_t)a.n : 0xFFFFFFFFu;
  }

  // What was written to LDS before is there for all wavefronts of the query after (global loads stay on their way).
  __device__ __forceinline__ static void meet() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }

  // Marks node id (where `valid`) as visited; true if it was not.
  __device__ __forceinline__ bool mark(bool valid, uint32_t id) {
    if (a.vis_cache) return valid && this->packed_cache_test_and_set(id);
    const uint32_t bit = valid ? 1u << (id & 31u) : 0u;
    return (~atomicOr(&vis[valid ? id >> 5 : 0u], bit) & bit) != 0;
  }

  __device__ __forceinline__ float key_of(const uint4 (&row)[CPL], float nrm) const {
    const int dot = group_sum_i32<LPR>(this->row_dot(row)) + bias;
    return key_from_idot(a.metric, s, qlo, dot, nrm);
  }

  // ---- a worker
  __device__ __forceinline__ void request_row(uint32_t v, uint4 (&row)[CPL], float &nrm) const {
    const uint32_t at = v * a.row_stride;   // (below 2^32)
#pragma unroll
    for (int j = 0; j < CPL; ++j) row[j] = *reinterpret_cast<const uint4 *>(a.codes + (at + coff[j]));
    if (!a.adj_norms && a.norm_term) nrm = a.norm_term[v];
  }
  // Candidates (where `q`) to LDS, behind those of the other workers.
  __device__ __forceinline__ void put(bool q, uint64_t c64, uint64_t qm, int base) {
    if (q) out[base + lanes_below(qm)] = c64;
  }
  __device__ __forceinline__ int reserve(int n) {
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&sh->n_out, (uint32_t)n);
    return (int)__builtin_amdgcn_readfirstlane((int)base);
  }

  __device__ __forceinline__ void work(int worker) {
    uint32_t n_fresh = 0;
    for (;;) {
      meet();   // nodes handed out
      const uint32_t n = __builtin_amdgcn_readfirstlane((int)sh->n_picks);
      if (n == 0) break;
      uint32_t u[kNodes];
#pragma unroll
      for (int i = 0; i < kNodes; ++i) u[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh->picks[worker - 1 + i * kRelayWorkers]);
      const uint64_t last = sh->worst;
      if (worker - 1 < (int)n) {
        // the adjacency rows
        const int slot = BY_SLOT ? grp : lane;
        const uint32_t at = (uint32_t)slot < a.degree ? (uint32_t)slot : a.degree - 1;
        uint32_t id[kNodes], nrm[kNodes];
#pragma unroll
        for (int i = 0; i < kNodes; ++i) {
          const uint32_t *row = a.adjacency + (uint64_t)(u[i] < n32 ? u[i] : 0u) * a.adj_stride;
          id[i] = row[at];
          nrm[i] = a.adj_norms ? row[a.degree + at] : 0u;
        }
        bool want[kNodes], fresh[kNodes];
#pragma unroll
        for (int i = 0; i < kNodes; ++i)
          want[i] = ((uint32_t)slot < a.degree) & (id[i] < n32) & (worker - 1 + i * kRelayWorkers < (int)n);
        if constexpr (BY_SLOT) {
          // all neighbours' rows, visited or not: the filter's round trip is not waited for
          uint4 rows[kNodes][CPL];
          float norm[kNodes];
#pragma unroll
          for (int i = 0; i < kNodes; ++i) {
            norm[i] = __uint_as_float(nrm[i]);
            request_row(want[i] ? id[i] : 0u, rows[i], norm[i]);
          }
#pragma unroll
          for (int i = 0; i < kNodes; ++i) {
            fresh[i] = mark(want[i] & (sub == 0), id[i]);
            n_fresh += (uint32_t)__popcll(__ballot(fresh[i]));
          }
          uint64_t c64[kNodes], qm[kNodes];
          int n_q = 0;
#pragma unroll
          for (int i = 0; i < kNodes; ++i) {
            c64[i] = pack64(order_u32(key_of(rows[i], norm[i])), id[i] << 1);
            qm[i] = __ballot(fresh[i] & (c64[i] < last));
            n_q += __popcll(qm[i]);
          }
          if (n_q > 0) {
            int base = reserve(n_q);
#pragma unroll
            for (int i = 0; i < kNodes; ++i) {
              put(__builtin_amdgcn_inverse_ballot_w64(qm[i]), c64[i], qm[i], base);
              base += __popcll(qm[i]);
            }
          }
        } else {
          int n_list = 0;
#pragma unroll
          for (int i = 0; i < kNodes; ++i) {
            fresh[i] = mark(want[i], id[i]);
            const uint64_t fm = __ballot(fresh[i]);
            if (fresh[i]) list[n_list + lanes_below(fm)] = pack64(id[i], nrm[i]);
            n_list += __popcll(fm);
          }
          n_fresh += (uint32_t)n_list;
          wave_sync();
          constexpr int U = LPR >= 16 ? 4 : (LPR >= 8 ? 3 : (LPR >= 4 ? 2 : 1));
          for (int base = 0; base < n_list; base += G * U) {
            uint4 rows[U][CPL];
            float norm[U];
            uint32_t v[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
              const int ci = base + t * G + grp;
              const uint64_t e = list[ci < n_list ? ci : n_list - 1];
              v[t] = (uint32_t)(e >> 32);
              norm[t] = __uint_as_float((uint32_t)e);
              request_row(v[t], rows[t], norm[t]);
            }
            uint64_t c64[U], qm[U];
            int n_q = 0;
#pragma unroll
            for (int t = 0; t < U; ++t) {
              c64[t] = pack64(order_u32(key_of(rows[t], norm[t])), v[t] << 1);
              qm[t] = __ballot((sub == 0) & (base + t * G + grp < n_list) & (c64[t] < last));
              n_q += __popcll(qm[t]);
            }
            if (n_q > 0) {
              int to = reserve(n_q);
#pragma unroll
              for (int t = 0; t < U; ++t) {
                put(__builtin_amdgcn_inverse_ballot_w64(qm[t]), c64[t], qm[t], to);
                to += __popcll(qm[t]);
              }
            }
          }
        }
      }
      meet();   // candidates are there
    }
    if (lane == 0) atomicAdd(&sh->n_eval, n_fresh);
    meet();
  }

  // ---- the keeper
  uint64_t pend;   // candidates that are not in the pool yet: one per lane, all-ones where there is none
  int n_pend;      // in the lowest lanes

  // Merges up to 64 candidates, in the n lowest lanes, into the pool.
  __device__ __forceinline__ void merge_lanes(uint64_t c, int n) {
    const bool have = c < worst;
    const uint64_t hm = __ballot(have);
    const int n_have = __popcll(hm);
    if (n_have == 0) return;
    if (n_have <= ANN_FEW) {
      // (to the lowest lanes)
      if (have) this->stage[lanes_below(hm)] = c;
      wave_sync();
      const uint64_t few = lane < n_have ? this->stage[lane] : 0;
      wave_sync();
      this->merge_few(n_have, few);
      return;
    }
    int width = kWave;
    if (n <= kWave / 2) {   // each half of the wavefront holds them
      c = pack64((uint32_t)__shfl((int)(uint32_t)(c >> 32), lane & 31), (uint32_t)__shfl((int)(uint32_t)c, lane & 31));
      width = kWave / 2;
    }
    this->merge(c < worst, (uint32_t)(c >> 32), (uint32_t)c, width);
  }
  __device__ __forceinline__ void merge_pending() {
    if (n_pend > 0) merge_lanes(pend, n_pend);
    pend = ~0ull;
    n_pend = 0;
  }

  // The pool's (at most P) closest un-expanded entries, in order, to near[0 .. P); all-ones where there is none.
  // This lane's, and the last of them.
  __device__ __forceinline__ uint64_t closest_open(uint64_t &last) {
    if (lane < P) sh->near[lane] = ~0ull;
    int before = 0;
#pragma unroll
    for (int r = 0; r < M; ++r) {
      const bool open = (pv[r] & 1u) == 0;
      const uint64_t um = __ballot(open);
      const int rank = before + lanes_below(um);
      if (open && rank < P) sh->near[rank] = pack64(pk[r], pv[r]);
      before += __popcll(um);
    }
    wave_sync();
    const uint64_t v = lane < P ? sh->near[lane < P ? lane : 0] : ~0ull;
    last = lane_value(v, P - 1);
    return v;
  }
  __device__ __forceinline__ static uint64_t lane_value(uint64_t v, int l) {
    return pack64((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l), (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l));
  }
  // Hands out n nodes (the lanes' `v` where `is`, as number `rank`), the closest un-expanded ones up to `up_to`.
  __device__ __forceinline__ void hand_out(bool is, uint64_t v, int rank, int n, uint64_t up_to) {
#pragma unroll
    for (int r = 0; r < M; ++r) pv[r] |= pack64(pk[r], pv[r]) <= up_to ? 1u : 0u;   // (entries that are expanded stay so)
    pend |= pend <= up_to ? 1u : 0u;
    if (is) sh->picks[rank] = (uint32_t)v >> 1;
    if (lane == 0) {
      sh->n_picks = (uint32_t)n;
      sh->n_out = 0;
      sh->worst = worst;
    }
    n_exp += (uint32_t)n;
  }

  // The next step's nodes from the pool's closest un-expanded entries (near[0 .. P), the last of them `last`) and the
  // pending candidates, ahead of the merge; false if that cannot be told yet.
  __device__ __forceinline__ bool pick(uint64_t last) {
    bool hot = (pend <= last) & ((pend & 1u) == 0);   // (all-ones: there is none)
    uint64_t hm = __ballot(hot);
    if (a.vis_cache) {
      // A node that the cache has forgotten may be in the pool, or come twice: it goes (with an expanded
      // mark the merge would not find it equal to the pool's entry).
      for (uint64_t left = hm; left != 0; left &= left - 1) {
        const int l = __builtin_ctzll(left);
        const uint64_t c = lane_value(pend, l);
        uint64_t same = __ballot((pend == c) & (lane < l));
#pragma unroll
        for (int r = 0; r < M; ++r) same |= __ballot((pv[r] | 1u) == ((uint32_t)c | 1u));
        if (same != 0) {
          pend = lane == l ? ~0ull : pend;
          hm &= ~(1ull << l);
        }
      }
      hot = __builtin_amdgcn_inverse_ballot_w64(hm);
    }
    const int n_near = P + __popcll(hm);
    const int at = ef_q - 1 - __popcll(__ballot(pend != ~0ull));
    if (n_near > kNear || at < 0) return false;
    if (hot) sh->near[P + lanes_below(hm)] = pend;
    if (lane >= n_near && lane < kNear) sh->near[lane] = ~0ull;
    wave_sync();
    const uint64_t v = sh->near[lane & (kNear - 1)];
    int rank = 0;
    auto count = [&](int from) {
      uint4 two[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) two[t] = reinterpret_cast<const uint4 *>(sh->near + from)[t];
#pragma unroll
      for (int t = 0; t < 8; ++t) rank += (pack64(two[t].y, two[t].x) < v ? 1 : 0) + (pack64(two[t].w, two[t].z) < v ? 1 : 0);
    };
    count(0);
    if (n_near > 16) count(16);
    const bool is = (lane < kNear) & (v != ~0ull) & (rank < P);
    const int got = __popcll(__ballot(is));
    if (got == 0) return false;
    const uint64_t up_to = lane_value(v, __builtin_ctzll(__ballot(is & (rank == got - 1))));
    // the pool's entry as many places before the last as there are candidates
    uint32_t ek = pk[0], ev = pv[0];
#pragma unroll
    for (int r = 1; r < M; ++r) {
      ek = at / kWave == r ? pk[r] : ek;
      ev = at / kWave == r ? pv[r] : ev;
    }
    if (up_to > lane_value(pack64(ek, ev), at % kWave)) return false;
    hand_out(is, v, rank, got, up_to);
    return true;
  }

  __device__ __forceinline__ void keep(uint32_t qi) {
    {   // initial nodes I: into the pool and into V
      uint32_t nb = kEmpty;
      if (a.entry_ids) {
        if (lane < (int)a.n_entry) nb = a.entry_ids[(uint64_t)qi * a.n_entry + lane];
      } else if (lane == 0) {
        nb = a.entry_point;
      }
      uint32_t nrm = 0;
      if (a.adj_norms && nb < n32) nrm = __float_as_uint(a.norm_term[nb]);
      const bool fresh = mark(nb < n32, nb);
      const uint64_t fm = __ballot(fresh);
      if (fresh) cand[lanes_below(fm)] = pack64(nb, nrm);
      this->evaluate_and_merge(__popcll(fm));
    }
    const int lazy = a.vis_cache ? 0 : kLazy;
    pend = ~0ull;
    n_pend = 0;
    int n = 0;             // candidates in out[] that are not in `pend`
    bool handed = false;   // the next step's nodes are with the workers
    for (;;) {
      uint64_t last;
      if (handed) {
        meet();
        if (n_pend > lazy) merge_pending();
      } else {
        merge_pending();
        for (int b = 0; b < n; b += kWave) merge_lanes(b + lane < n ? out[b + lane] : ~0ull, n - b);
        const uint64_t v = closest_open(last);
        const int got = __popcll(__ballot(v != ~0ull));
        if (got == 0) break;
        hand_out(lane < got, v, lane, got, lane_value(v, got - 1));
        meet();
      }
      closest_open(last);
      meet();   // the workers are done

      n = __builtin_amdgcn_readfirstlane((int)sh->n_out);
      handed = false;
      if (n_pend + n <= kWave) {
        const int from = lane - n_pend;
        const uint64_t c = out[from < 0 ? 0 : from];
        if ((from >= 0) & (from < n)) pend = c < worst ? c : ~0ull;
        n_pend += n;
        n = 0;
        handed = pick(last);
      }
    }
    if (lane == 0) sh->n_picks = 0;
    meet();
    meet();
    n_dist += (uint32_t)__builtin_amdgcn_readfirstlane((int)sh->n_eval);
    this->write_results(qi);
  }

  __device__ __forceinline__ void run(uint32_t qi, int wave) {
    if (wave == 0) {
      if (lane == 0) {
        sh->n_eval = 0;
        sh->n_out = 0;
        sh->n_picks = 0;
      }
      if (a.q != nullptr) {
        this->fold(qi);
        if (lane == 0) {
          sh->s = s;
          sh->qlo = qlo;
          sh->bias = bias;
        }
      } else {
        this->load_query_terms(qi);
      }
      this->start_pool(qi);
      meet();   // query folded, visited set empty
      keep(qi);
    } else {
      const uint32_t fill = a.vis_cache ? kEmpty : 0u;
      for (uint32_t i = (wave - 1) * kWave + lane; i < a.vis_words / 4; i += kRelayWorkers * kWave)
        reinterpret_cast<uint4 *>(vis)[i] = make_uint4(fill, fill, fill, fill);
      meet();
      if (a.q != nullptr) {
        s = sh->s;
        qlo = sh->qlo;
        bias = sh->bias;
        this->load_query_part(this->tql);
      } else {
        this->load_query_terms(qi);
      }
      work(wave);
    }
  }
};

template <int BITS, int LPR, int M, int P, bool BY_SLOT>
__global__ __launch_bounds__(64 * (1 + kRelayWorkers)) __attribute__((amdgpu_waves_per_eu(relay_waves(BITS, LPR, M)))) void search_relay_kernel(SearchArgs args) {
  extern __shared__ uint64_t smem[];
  if (blockIdx.x >= args.nq) return;
  const uint32_t qi = args.order ? args.order[blockIdx.x] : blockIdx.x;
  if (qi >= args.nq) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  SearchRelay<BITS, LPR, M, P, BY_SLOT> w(args, smem, wave);
  w.run(qi, wave);
}

template <int BITS, int LPR, int P, bool BY_SLOT>
static ann_status launch_relay_m(const SearchArgs &a, int m, hipStream_t st) {
  const size_t smem = relay_smem_bytes(m, P, BY_SLOT, a.vis_words, a.tq_stride);
  constexpr int kThreads = 64 * (1 + kRelayWorkers);
  switch (m) {
    case 1: search_relay_kernel<BITS, LPR, 1, P, BY_SLOT><<<a.nq, kThreads, smem, st>>>(a); break;
    case 2: search_relay_kernel<BITS, LPR, 2, P, BY_SLOT><<<a.nq, kThreads, smem, st>>>(a); break;
    case 4: search_relay_kernel<BITS, LPR, 4, P, BY_SLOT><<<a.nq, kThreads, smem, st>>>(a); break;
    case 8: search_relay_kernel<BITS, LPR, 8, P, BY_SLOT><<<a.nq, kThreads, smem, st>>>(a); break;
    default: return fail(ANN_EUNSUPPORTED, "no kernel for pool registers per lane = %d", m);
  }
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

template <int BITS, int P>
static ann_status launch_relay(const SearchArgs &a, uint32_t lpr, int m, hipStream_t st) {
  const bool by_slot = relay_by_slot(lpr, a.degree);
  switch (lpr) {
    case 1: return launch_relay_m<BITS, 1, P, true>(a, m, st);
    case 2: return by_slot ? launch_relay_m<BITS, 2, P, true>(a, m, st) : launch_relay_m<BITS, 2, P, false>(a, m, st);
    case 4: return launch_relay_m<BITS, 4, P, false>(a, m, st);
    case 8: return launch_relay_m<BITS, 8, P, false>(a, m, st);
    case 16: return launch_relay_m<BITS, 16, P, false>(a, m, st);
    default: return fail(ANN_EUNSUPPORTED, "no kernel for %u lanes per code row", lpr);
  }
}

}  // namespace ann
