// One expansion per step for small batches: a query's chain of dependent steps.
//
// A batch that leaves compute units idle takes as long as its longest query, and
// that is a chain: adjacency row, code rows, merge, next node.  So a step's node
// is guessed one step ahead (the closest un-expanded pool entry but the one in
// hand: right in two steps of three and more), and the code rows of the guess'
// unvisited neighbours are requested before the merge; the adjacency row of the
// guess after that is requested with them.  Where the guess was right a step has
// no memory round trip, and nothing was marked visited in between, so what was
// unvisited when the rows were requested still is.
//
// Candidates stay in the lanes that hold their rows, and a few are put into the
// pool one after the other by a shift of the pool's registers by a lane (DPP),
// without LDS.  More of them go through SearchWave's merge.
//
// The visited set is a bit per node in LDS: complete, so nothing is evaluated
// twice.  For base sets whose bits fit for all resident queries.
//
// Bound: about 1,500 cycles a step where the guess was right, of instructions of one
// wavefront (selection 350, keys 250, requests 150, a candidate's insertion 150, a
// merge of more than eight 2,000); a wrong guess costs two round trips, 800 cycles from
// the L2, 1,500 from behind it.  Against the kernels before (search_small_kernel; with
// labels or the cap the general kernel): 100 queries on 10,000 x 128, ef = 64: 131 -> 76
// us; 1,000 on 300,000 x 128, ef = 128: 495 -> 300; 100 on 1M x 128: 704 -> 429; 1,000 on
// 100,000 x 960 4-bit, ef = 256: 774 -> 650; labels and cap, 513 on 50,021 x 100: 324 ->
// 188, 10,000 on 50,000 x 100: 2,309 -> 555.  All rows of a node instead of a list of the
// unvisited: as fast for rows of one and two lanes, 960 4-bit 800 us.
#pragma once
#include "search_kernel.hpp"

namespace ann {

constexpr uint64_t kChainNodes = 1u << 21;   // 32-bit offsets into adjacency (512 bytes a row) and codes (1,024)

// Wavefronts per SIMD a kernel is compiled for.
__host__ __device__ constexpr int chain_waves(int lpr, int m) { return lpr <= 2 ? (m < 8 ? 4 : 3) : (lpr == 4 ? 3 : 2); }

// Whether every slot of an adjacency row has lanes of its own: no list of the unvisited neighbours then.
__host__ __device__ constexpr bool chain_by_slot(uint32_t lpr, uint32_t degree) { return degree * lpr <= 64u; }

__host__ inline size_t chain_smem_bytes(int m, uint32_t vis_words, uint32_t tq_stride) {
  return (size_t)(merge_buf_entries(m) + stage_area_entries(m, 1, true) + 64) * 8 + (size_t)vis_words * 4 + tq_stride;
}

ann_status launch_search_chain(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st);
ann_status launch_search_chain_filtered(const SearchArgs &a, uint32_t bits, uint32_t lpr, int m, hipStream_t st);

// BY_SLOT: lane group g holds the neighbour in slot g (chain_by_slot).  Otherwise the unvisited neighbours
// are listed in LDS and group g holds entries g, g + G, ... of the list.
template <int BITS, int LPR, int M, bool BY_SLOT, bool FILTER>
struct SearchChain : SearchWave<BITS, LPR, M, 1, true, 1, true, false, true> {
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
  using Base::mbuf;
  using Base::n_dist;
  using Base::n_exp;
  using Base::pk;
  using Base::pv;
  using Base::qlo;
  using Base::s;
  using Base::stage;
  using Base::sub;
  using Base::vis;
  using Base::worst;

  // Groups of rows requested ahead (the rest of a list, if any, when its step has come).
  static constexpr int K = BY_SLOT || LPR <= 2 ? 1 : (LPR == 4 ? 2 : (LPR == 8 ? 3 : 4));
  // Candidates put in one by one; more are merged at once.
  static constexpr int kOneByOne = M <= 2 ? 8 : (M == 4 ? 4 : 2);

  // An adjacency row: this lane's slot's id, norm term and label.
  struct Slot {
    uint32_t id, nrm;
    float lab;
  };

  uint32_t n32;       // nodes
  uint32_t slot_at;   // byte offset of this lane's slot in an adjacency row
  bool slot_used;     // (one lane of those that share a slot)
  const char *lab_base;   // labels (or the adjacency rows), bytes from one row to the next
  uint32_t lab_stride;
  uint64_t *list;     // LDS [64] (not BY_SLOT): unvisited neighbours, id and norm term
  int n_list;
  // the rows of the guess: BY_SLOT also the word of the visited set that the id's bit is in, and the label
  uint32_t rid[K], rnrm[K], seen;
  float gnrm[K], rlab;
  uint4 rows[K][CPL];

  __device__ __forceinline__ SearchChain(const SearchArgs &args, uint64_t *smem) : Base(args, smem) {
    list = reinterpret_cast<uint64_t *>(vis + a.vis_words);
    this->tql = reinterpret_cast<const int *>(list + 64);
    n32 = (uint32_t)a.n;
    const uint32_t slot = (uint32_t)(BY_SLOT ? grp : lane);
    slot_used = (slot < a.degree) & (!BY_SLOT | (sub == 0));
    slot_at = (slot < a.degree ? slot : a.degree - 1) * 4u;
    lab_base = FILTER && a.labels ? reinterpret_cast<const char *>(a.labels) : reinterpret_cast<const char *>(a.adjacency);
    lab_stride = (FILTER && a.labels ? a.degree : a.adj_stride) * 4u;
    asm volatile("" : "+s"(lab_base));   // (the compiler else makes the second a copy of the id, which it waits for)
    seen = 0;
    rlab = 0.0f;
    n_list = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) rid[i] = rnrm[i] = 0u;
  }

  // Requests node u's adjacency row.  The same number of loads whatever the options are (what is not wanted is
  // read from a line that is on its way anyhow), so that how many are behind the code rows is known when these are
  // waited for.
  __device__ __forceinline__ void request_ids(uint32_t u, Slot &to) {
    const char *adj = reinterpret_cast<const char *>(a.adjacency);
    const uint32_t row = u * a.adj_stride * 4u + slot_at;
    to.id = *reinterpret_cast<const uint32_t *>(adj + row);
    to.nrm = *reinterpret_cast<const uint32_t *>(adj + (row + (a.adj_norms ? a.degree * 4u : 0u)));
    if constexpr (FILTER) to.lab = *reinterpret_cast<const float *>(lab_base + (u * lab_stride + slot_at));
  }
  // Whether this lane stands for a neighbour that may be followed.
  __device__ __forceinline__ bool wanted(uint32_t id, float lab) const {
    bool is = slot_used & (id < n32);
    if constexpr (FILTER) is &= (a.labels == nullptr) | (lab <= a.alpha_s);
    return is;
  }
  // Code row i of node v.
  __device__ __forceinline__ void request_row(int i, uint32_t v) {
    const bool gathered = !a.adj_norms && a.norm_term != nullptr;
    const char *norms = reinterpret_cast<const char *>(gathered ? reinterpret_cast<const uint8_t *>(a.norm_term) : a.codes);
    const uint32_t at = v * a.row_stride;
#pragma unroll
    for (int j = 0; j < CPL; ++j) rows[i][j] = *reinterpret_cast<const uint4 *>(a.codes + (at + coff[j]));
    gnrm[i] = *reinterpret_cast<const float *>(norms + (gathered ? v * 4u : at));
  }
  // Requests the code rows of an adjacency row's neighbours (BY_SLOT all of them: whether they are visited is
  // looked at when they are there; padding: node 0's).
  __device__ __forceinline__ void request_rows(const Slot &from) {
    if constexpr (BY_SLOT) {
      rid[0] = from.id;
      rnrm[0] = from.nrm;
      rlab = from.lab;
      const uint32_t v = rid[0] < n32 ? rid[0] : 0u;
      request_row(0, v);
      seen = vis[v >> 5];
    } else {
      const bool want = wanted(from.id, from.lab);
      const uint32_t v = want ? from.id : 0u;
      bool open = want & ((vis[v >> 5] >> (v & 31u) & 1u) == 0);
      uint64_t om = __ballot(open);
      int rank = lanes_below(om);
      if constexpr (FILTER) {   // the first m_s unvisited neighbours in stored order
        open &= (uint32_t)rank < a.m_s;
        om = __ballot(open);
      }
      n_list = __popcll(om);
      if (open) list[rank] = pack64(from.id, from.nrm);
      wave_sync();
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (i == 0 || i * G < n_list) take_listed(i, i * G + grp);
    }
  }
  // Entry ci of the list (past its end: the last one) as row i.
  __device__ __forceinline__ void take_listed(int i, int ci) {
    const int last = n_list > 0 ? n_list - 1 : 0;
    const uint64_t e = n_list > 0 ? list[ci < last ? ci : last] : 0u;
    rid[i] = (uint32_t)(e >> 32);
    rnrm[i] = (uint32_t)e;
    request_row(i, rid[i]);
  }
  // Marks node id (where `is`) as visited.  (Without a branch: no bit of word 0 otherwise.)
  __device__ __forceinline__ void mark(bool is, uint32_t id) { atomicOr(&vis[is ? id >> 5 : 0u], is ? 1u << (id & 31u) : 0u); }

  // Puts one candidate, the same in all lanes, into the pool: entries above it move up by one, and what passes
  // the pool's end (perhaps the candidate) is dropped.
  __device__ __forceinline__ void insert(uint32_t ck, uint32_t cv) {
    const uint64_t c64 = pack64(ck, cv);
    uint64_t below[M];
#pragma unroll
    for (int r = 0; r < M; ++r) below[r] = __ballot(pack64(pk[r], pv[r]) < c64);
#pragma unroll
    for (int r = M - 1; r >= 0; --r) {
      // entry i's predecessor, and whether that one is below the candidate
      const uint32_t in_k = r > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)pk[r > 0 ? r - 1 : 0], 63) : ck;
      const uint32_t in_v = r > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)pv[r > 0 ? r - 1 : 0], 63) : cv;
      const uint32_t prev_k = (uint32_t)__builtin_amdgcn_update_dpp((int)in_k, (int)pk[r], 0x138, 0xF, 0xF, false);   // wave_shr:1
      const uint32_t prev_v = (uint32_t)__builtin_amdgcn_update_dpp((int)in_v, (int)pv[r], 0x138, 0xF, 0xF, false);
      const uint64_t prev_below = below[r] << 1 | (r > 0 ? below[r > 0 ? r - 1 : 0] >> 63 : 1ull);
      const bool keep = __builtin_amdgcn_inverse_ballot_w64(below[r]), here = __builtin_amdgcn_inverse_ballot_w64(prev_below);
      const bool beyond = r * kWave + lane >= ef_q;
      pk[r] = keep ? pk[r] : (beyond ? kEmpty : (here ? ck : prev_k));
      pv[r] = keep ? pv[r] : (beyond ? kEmpty : (here ? cv : prev_v));
    }
  }

  // Key of row i (key_from_idot: -fma(s, dot, qlo) is fma(-s, dot, -qlo), so both metrics are one multiplication
  // and addition of the same shape).
  __device__ __forceinline__ uint32_t ordered_key(int i) const {
    const float nrm = a.adj_norms ? __uint_as_float(rnrm[i]) : gnrm[i];
    const int dot = group_sum_i32<LPR>(this->row_dot(rows[i])) + bias;
    const float from = a.metric == ANN_L2 ? __fsub_rn(nrm, __fmul_rn(2.0f, qlo)) : -qlo, by = a.metric == ANN_L2 ? -2.0f * s : -s;
    const float key = __fmaf_rn(by, (float)dot, from);
    return order_u32(key == 0.0f ? 0.0f : key);   // -0 -> +0
  }

  __device__ __forceinline__ void run(uint32_t qi) {
    uint32_t r_id = kEmpty, a_id = kEmpty;   // nodes whose code rows, whose adjacency row were requested ahead
    Slot ahead{};
    const uint32_t e = a.entry_point;
    // the entry point's neighbours are requested ahead of the folding
    if (!a.entry_ids) request_ids(e, ahead);
    for (uint32_t i = lane; i < a.vis_words / 4; i += kWave) reinterpret_cast<uint4 *>(vis)[i] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
    if (!a.entry_ids) {
      mark(lane == 0, e);
      wave_sync();
      request_rows(ahead);
      r_id = e;
    }
    if (a.q != nullptr)
      this->fold(qi);
    else
      this->load_query_terms(qi);
    this->start_pool(qi);
    wave_sync();

    // initial nodes I: into the pool and into V
    {
      uint32_t nb = kEmpty;
      bool fresh = false;
      if (a.entry_ids) {
        if (lane < (int)a.n_entry) nb = a.entry_ids[(uint64_t)qi * a.n_entry + lane];
        const uint32_t bit = nb < n32 ? 1u << (nb & 31u) : 0u;
        fresh = (~atomicOr(&vis[nb < n32 ? nb >> 5 : 0u], bit) & bit) != 0;
      } else if (lane == 0) {
        nb = e;
        fresh = true;
      }
      uint32_t nrm = 0;
      if (a.adj_norms && nb < n32) nrm = __float_as_uint(a.norm_term[nb]);
      const uint64_t fm = __ballot(fresh);
      if (fresh) cand[lanes_below(fm)] = pack64(nb, nrm);
      this->evaluate_and_merge(__popcll(fm));
    }
    // (nothing of the above is on its way any more: the compiler else waits for everything at the loop's head)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)

    // the closest un-expanded entry, and the two after it
    uint32_t u, next, after;
    auto select = [&]() {
      uint64_t um[M];
#pragma unroll
      for (int r = 0; r < M; ++r) um[r] = __ballot((pv[r] & 1u) == 0);
      // (large pools by branches: 30 queries x 20,000 x 60, ef = 300: 571 us, without 746)
      auto take = [&](bool expand) {
        uint32_t id = kEmpty;
        bool got = false;
#pragma unroll
        for (int r = 0; r < M; ++r) {
          const bool here = !got && um[r] != 0;
          if (M > 2 && !here) continue;
          const int l = __builtin_ctzll(um[r] | (1ull << 63));
          const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)pv[r], l) >> 1;
          id = here ? v : id;
          if (expand) pv[r] |= here && lane == l ? 1u : 0u;
          um[r] = here ? um[r] & (um[r] - 1) : um[r];
          got = got || here;
        }
        return id;
      };
      u = take(true);
      next = take(false);
      after = take(false);
    };
    for (select(); u != kEmpty; select()) {
      ++n_exp;
      if (r_id != u) {   // the guess was wrong: both round trips
        Slot now;
        if (a_id == u)
          now = ahead;
        else
          request_ids(u, now);
        request_rows(now);
      }
      // the adjacency row of the next guess, where it was not requested ahead
      Slot late;
      const bool in_time = a_id == next;
      if (!in_time && next != kEmpty) request_ids(next, late);

      // keys of the unvisited neighbours, which are marked
      uint32_t ck[K], cv[K];
      uint64_t qm[K];
      int n_q = 0;
      if constexpr (BY_SLOT) {
        bool fresh = wanted(rid[0], rlab) & ((seen >> (rid[0] & 31u) & 1u) == 0);
        uint64_t fm = __ballot(fresh);
        if constexpr (FILTER) {
          fresh &= (uint32_t)lanes_below(fm) < a.m_s;
          fm = __ballot(fresh);
        }
        mark(fresh, rid[0]);
        n_list = __popcll(fm);
        ck[0] = ordered_key(0);
        cv[0] = rid[0] << 1;
        qm[0] = __ballot(fresh & (pack64(ck[0], cv[0]) < worst));
        n_q = __popcll(qm[0]);
      } else {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          qm[i] = 0;
          if (i > 0 && i * G >= n_list) continue;
          const bool fresh = (sub == 0) & (i * G + grp < n_list);
          mark(fresh, rid[i]);
          ck[i] = ordered_key(i);
          cv[i] = rid[i] << 1;
          qm[i] = __ballot(fresh & (pack64(ck[i], cv[i]) < worst));
          n_q += __popcll(qm[i]);
        }
      }
      n_dist += (uint32_t)n_list;
      const bool more = !BY_SLOT && K * G < 64 && n_list > K * G;
      if (more) {   // the rest of a long list
        n_q = stage_candidates(ck, cv, qm);
        for (int base = K * G; base < n_list; base += G) {
          const bool fresh = (sub == 0) & (base + grp < n_list);
          take_listed(0, base + grp);
          mark(fresh, rid[0]);
          const uint64_t c64 = pack64(ordered_key(0), rid[0] << 1);
          const bool q = fresh & (c64 < worst);
          const uint64_t bm = __ballot(q);
          if (q) stage[n_q + lanes_below(bm)] = c64;
          n_q += __popcll(bm);
        }
      }

      // the next step's rows and the adjacency row of the one after, on their way during the merge
      r_id = next;
      if (next != kEmpty) {
        request_rows(in_time ? ahead : late);
        request_ids(after != kEmpty ? after : next, ahead);
        a_id = after;
      }

      if (n_q == 0) {
      } else if (!more && n_q <= kOneByOne) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          while (qm[i] != 0) {
            const int l = __builtin_ctzll(qm[i]);
            qm[i] &= qm[i] - 1;
            insert((uint32_t)__builtin_amdgcn_readlane((int)ck[i], l), (uint32_t)__builtin_amdgcn_readlane((int)cv[i], l));
          }
        }
        this->refresh_worst();
      } else {
        if (!more) stage_candidates(ck, cv, qm);
        // (the merge wants the pool in LDS as well)
#pragma unroll
        for (int r = 0; r < M; ++r) mbuf[r * kWave + lane] = pack64(pk[r], pv[r]);
        this->merge_staged(n_q);
      }
    }
    this->write_results(qi);
  }

  __device__ __forceinline__ int stage_candidates(const uint32_t (&ck)[K], const uint32_t (&cv)[K], const uint64_t (&qm)[K]) {
    int at = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (__builtin_amdgcn_inverse_ballot_w64(qm[i])) stage[at + lanes_below(qm[i])] = pack64(ck[i], cv[i]);
      at += __popcll(qm[i]);
    }
    return at;
  }
};

template <int BITS, int LPR, int M, bool BY_SLOT, bool FILTER>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(chain_waves(LPR, M)))) void search_chain_kernel(SearchArgs args) {
  extern __shared__ uint64_t smem[];
  if (blockIdx.x >= args.nq) return;
  const uint32_t qi = args.order ? args.order[blockIdx.x] : blockIdx.x;
  if (qi >= args.nq) return;
  SearchChain<BITS, LPR, M, BY_SLOT, FILTER> w(args, smem);
  w.run(qi);
}

template <int BITS, int LPR, bool BY_SLOT, bool FILTER>
static ann_status launch_chain_m(const SearchArgs &a, int m, hipStream_t st) {
  const size_t smem = chain_smem_bytes(m, a.vis_words, a.tq_stride);
  switch (m) {
    case 1: search_chain_kernel<BITS, LPR, 1, BY_SLOT, FILTER><<<a.nq, 64, smem, st>>>(a); break;
    case 2: search_chain_kernel<BITS, LPR, 2, BY_SLOT, FILTER><<<a.nq, 64, smem, st>>>(a); break;
    case 4: search_chain_kernel<BITS, LPR, 4, BY_SLOT, FILTER><<<a.nq, 64, smem, st>>>(a); break;
    case 8: search_chain_kernel<BITS, LPR, 8, BY_SLOT, FILTER><<<a.nq, 64, smem, st>>>(a); break;
    default: return fail(ANN_EUNSUPPORTED, "no kernel for pool registers per lane = %d", m);
  }
  ANN_HIP(hipGetLastError());
  return ANN_OK;
}

template <int BITS, bool FILTER>
static ann_status launch_chain(const SearchArgs &a, uint32_t lpr, int m, hipStream_t st) {
  const bool by_slot = chain_by_slot(lpr, a.degree);
  switch (lpr) {
    case 1: return launch_chain_m<BITS, 1, true, FILTER>(a, m, st);
    case 2: return by_slot ? launch_chain_m<BITS, 2, true, FILTER>(a, m, st) : launch_chain_m<BITS, 2, false, FILTER>(a, m, st);
    case 4: return launch_chain_m<BITS, 4, false, FILTER>(a, m, st);
    case 8: return launch_chain_m<BITS, 8, false, FILTER>(a, m, st);
    case 16: return launch_chain_m<BITS, 16, false, FILTER>(a, m, st);
    default: return fail(ANN_EUNSUPPORTED, "no kernel for %u lanes per code row", lpr);
  }
}

}  // namespace ann
