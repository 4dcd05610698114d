// Device side of the search that more than one kernel runs: the retrieve stage from group statistics, and the re-rank
// stage of plain beam search (see kernels_search.hip).
#pragma once
#include "lsq_internal.h"

namespace lsq {

// Total order used everywhere: higher score first, lower index first among equal scores.
__device__ __forceinline__ bool precedes(float s1, int i1, float s2, int i2) {
  return s1 > s2 || (s1 == s2 && i1 < i2);
}

// ---------------------------------------------------------------------------------------------
// The retrieve stage (paper sec. 2.2) from group statistics that the logit product left behind: for every
// row and every group of 32 consecutive tokens the pair (largest logit, sum of exp(logit - largest)).
// One wavefront per row:
//   * softmax normaliser of the row from the G pairs (no pass over the logits);
//   * candidate value of every group's best token, cand = score + ((x - max) - log sum), the same
//     arithmetic as row_topk_kernel token by token (monotone in x, so it is the group's best cand);
//   * R = the k-th largest of the 64 lanes' best group values (each lane holds every 64th group): k distinct
//     tokens reach R, so every token of the row's exact top k has cand >= R, and such tokens only sit
//     in groups whose best reaches R -- the paper's threshold with the product's column groups as
//     the "random" groups;
//   * only those groups' logits are read (k groups of 32 unless values tie), tokens with cand >= R
//     are ranked exactly by (cand descending, token ascending).
// Rows where more than QMAX groups or CMAX tokens reach R (long runs of equal logits) fall back to k
// exact rounds over the whole row.  Same output as row_topk_kernel (no diverse groups); raw: the k largest
// logits themselves (sampling), no score, no normaliser.
// Groups / tokens that may reach the threshold before the fallback, in which one wavefront goes over the row k times (4.5 ms at
// k = 32, 50257 tokens).  With k = 32 of nearly flat logits some 43 groups reach it, 58 to 70 in one row out of 300: a list of 64
// overflowed in every other generation of 32 rows x 128 tokens (33.5 -> 37.8 ms).
constexpr int kTopkGroupsQ = 128, kTopkGroupsC = 160;

// One row by one wavefront; ql, cs, ci: the wavefront's own LDS lists (kTopkGroupsQ, kTopkGroupsC entries); os, oi:
// where the k pairs go (global memory or LDS).
template <int GPL, int PB = 8>
__device__ __forceinline__ void topk_groups_row(const float* __restrict__ logits, const float* __restrict__ stats,
                                                const float* __restrict__ score, const int32_t* __restrict__ fin,
                                                int r, int V, int G, int k, int eos, float* os, int32_t* oi, int lane,
                                                int* ql_w, float* cs_w, int* ci_w, int raw = 0) {
  constexpr int QMAX = kTopkGroupsQ, CMAX = kTopkGroupsC;
  // raw (sampling): the k largest logits themselves, no score, no normaliser, no finished rows
  const float bs = raw ? 0.f : score[r];
  const int f = raw ? 0 : fin[r];
  // the row's statistics, requested before anything is decided
  float gm[GPL], gz[GPL];
#pragma unroll
  for (int q = 0; q < GPL; ++q) {
    const int g = q * 64 + lane;
    if (g < G) {
      const float2 t = *reinterpret_cast<const float2*>(stats + ((size_t)r * G + g) * 2);
      gm[q] = t.x; gz[q] = t.y;
    } else {
      gm[q] = -INFINITY; gz[q] = 0.f;
    }
  }
  if (f) {   // a finished hypothesis offers itself once
    if (lane < k) { os[lane] = lane == 0 ? bs : -INFINITY; oi[lane] = lane == 0 ? eos : -1; }
    return;
  }
  if (bs == -INFINITY) {   // every candidate is -inf: the order is by token alone
    if (lane < k) { os[lane] = -INFINITY; oi[lane] = lane < V ? lane : -1; }
    return;
  }
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < GPL; ++q) m = fmaxf(m, gm[q]);
  m = wave_max(m);
  float zt = 0.f;
#pragma unroll
  for (int q = 0; q < GPL; ++q) zt += gz[q] * __expf(gm[q] - m);   // a group that does not exist: 0 * exp(-inf) = 0
  zt = wave_sum(zt);
  const float logz = logf(zt);
  auto cand_of = [&](float x) { return raw ? x : __fadd_rn(bs, __fsub_rn(__fsub_rn(x, m), logz)); };
  float cg[GPL];
#pragma unroll
  for (int q = 0; q < GPL; ++q) cg[q] = (q * 64 + lane < G) ? cand_of(gm[q]) : -INFINITY;
  // R: every lane's best group value is the value of a distinct token; the k-th largest of those 64 is
  // reached by k tokens, so it is a valid threshold (at most the k-th largest group value, and close to it
  // when there are many more groups than k).
  float lm = -INFINITY;
#pragma unroll
  for (int q = 0; q < GPL; ++q) lm = fmaxf(lm, cg[q]);
  float R = -INFINITY;   // fewer than k groups: -inf, every token passes
  if (k <= LSQ_MAX_BEAM_) {   // k rounds of the wavefront's maximum, one lane leaving each time
    float left = lm;
    for (int i = 0; i < k; ++i) {
      R = wave_max(left);
      if (lane == (int)__builtin_ctzll(__ballot(left == R))) left = -INFINITY;
    }
  } else {
    int lrank = 0;
#pragma unroll
    for (int c = 0; c < 64; ++c) {
      const float o = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lm), c));
      lrank += (o > lm || (o == lm && c < lane)) ? 1 : 0;
    }
    R = wave_max(lrank == k - 1 ? lm : -INFINITY);
  }
  // the groups that reach R
  int nq = 0;
#pragma unroll
  for (int q = 0; q < GPL; ++q) {
    const bool in = q * 64 + lane < G && cg[q] >= R;
    const unsigned long long mask = __ballot(in);
    if (mask == 0) continue;   // nearly always
    if (in) {
      const int at = nq + __popcll(mask & ((1ull << lane) - 1ull));
      if (at < QMAX) ql_w[at] = q * 64 + lane;
    }
    nq += __popcll(mask);
  }
  __builtin_amdgcn_wave_barrier();   // the list is read by other lanes of this wavefront (LDS keeps a wavefront's order)
  const float* row = logits + (size_t)r * V;
  int nc = 0;
  if (nq <= QMAX) {
    // two groups per pass (lanes 0-31 one, lanes 32-63 the next), the logits of PB passes requested together
    for (int p0 = 0; p0 < nq && nc <= CMAX; p0 += 2 * PB) {
      float xs[PB];
      int vs[PB];
#pragma unroll
      for (int u = 0; u < PB; ++u) {
        const int gi = p0 + 2 * u + (lane >> 5);
        vs[u] = gi < nq ? ql_w[min(gi, QMAX - 1)] * 32 + (lane & 31) : V;
        xs[u] = row[min(vs[u], V - 1)];
      }
#pragma unroll
      for (int u = 0; u < PB; ++u) {
        const float c = cand_of(xs[u]);
        const bool in = vs[u] < V && c >= R;
        const unsigned long long mask = __ballot(in);
        if (mask == 0) continue;
        if (in) {
          const int at = nc + __popcll(mask & ((1ull << lane) - 1ull));
          if (at < CMAX) { cs_w[at] = c; ci_w[at] = vs[u]; }
        }
        nc += __popcll(mask);
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  if (nq <= QMAX && nc <= CMAX) {
    if (nc <= 64) {
      const float sc = lane < nc ? cs_w[lane] : -INFINITY;
      const int v = lane < nc ? ci_w[lane] : 0x7fffffff;
      int rank = 0;
      for (int o = 0; o < nc; ++o)
        rank += precedes(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sc), o)), __builtin_amdgcn_readlane(v, o), sc, v) ? 1 : 0;
      if (lane < nc && rank < k) { os[rank] = sc; oi[rank] = v; }
    } else {
      for (int c = lane; c < nc; c += 64) {
        const float sc = cs_w[c];
        const int v = ci_w[c];
        int rank = 0;
        for (int o = 0; o < nc; ++o) rank += precedes(cs_w[o], ci_w[o], sc, v) ? 1 : 0;
        if (rank < k) { os[rank] = sc; oi[rank] = v; }
      }
    }
    if (lane >= nc && lane < k) { os[lane] = -INFINITY; oi[lane] = -1; }   // vocabulary smaller than k
    return;
  }
  // exact fallback: k rounds over the whole row, each the best token strictly after the previous winner
  float ps = INFINITY;
  int pi = -1;
  for (int round = 0; round < k; ++round) {
    float bsc = -INFINITY;
    int bi = 0x7fffffff;
    for (int v = lane; v < V; v += 64) {
      const float c = cand_of(row[v]);
      if (precedes(ps, pi, c, v) && (bi == 0x7fffffff || precedes(c, v, bsc, bi))) { bsc = c; bi = v; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float s2 = __shfl_xor(bsc, o, kWave);
      const int i2 = __shfl_xor(bi, o, kWave);
      if (i2 != 0x7fffffff && (bi == 0x7fffffff || precedes(s2, i2, bsc, bi))) { bsc = s2; bi = i2; }
    }
    if (bi == 0x7fffffff) {
      if (lane == 0) { os[round] = -INFINITY; oi[round] = -1; }
    } else {
      if (lane == 0) { os[round] = bsc; oi[round] = bi; }
      ps = bsc;
      pi = bi;
    }
  }
}

// x[base + i] = E[tok[i]] * scale + pe[pos] for the k rows of a sentence (tok[i] < 0: row left alone), by one
// wavefront: the rows' 16-byte chunks are dealt out over the lanes and requested up to eight per lane at a time, so the
// k gathers travel together instead of one row after the other.  One row of d = 512 is one chunk per lane: eight, seven of them
// repetitions, with the two savings in topk_groups_row, cost 1.0 to 1.3 us of a search kernel of 8.6 to 10.5.
// The arithmetic is embed_row's (scaled_sum).
template <typename T, int U>
__device__ __forceinline__ void next_input_chunks(const NextInput& nx, const int* tok, int base, int k, int pos, int lane) {
  const int d = nx.d;
  const T* E = (const T*)nx.E;
  T* x = (T*)nx.x;
  const float* pe = nx.pe + (size_t)pos * d;
  using raw_t = typename Vec8<T>::raw_t;
  const int cpr = d >> 3, total = k * cpr;
  for (int u0 = 0; u0 < total; u0 += 64 * U) {
    raw_t e[U];
    floatx4 pa[U], pb[U];
    int row[U], col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = u0 + u * 64 + lane;
      const int i = min(idx, total - 1) / cpr;
      col[u] = (min(idx, total - 1) - i * cpr) * 8;
      row[u] = (idx < total && tok[i] >= 0) ? base + i : -1;
      e[u] = Vec8<T>::load_raw(E + (size_t)embedding_row(tok[i]) * d + col[u]);
      pa[u] = *reinterpret_cast<const floatx4*>(pe + col[u]);
      pb[u] = *reinterpret_cast<const floatx4*>(pe + col[u] + 4);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float p[8] = {pa[u][0], pa[u][1], pa[u][2], pa[u][3], pb[u][0], pb[u][1], pb[u][2], pb[u][3]};
      const raw_t y = scaled_sums(e[u], nx.scale, p);
      if (row[u] >= 0) *reinterpret_cast<raw_t*>(x + (size_t)row[u] * d + col[u]) = y;
    }
  }
}
template <typename T>
__device__ __forceinline__ void next_input_rows(const NextInput& nx, const int* tok, int base, int k, int pos, int lane) {
  const int d = nx.d, chunks = k * (d >> 3);
  if ((d & 7) != 0) {
    for (int i = 0; i < k; ++i)
      if (tok[i] >= 0) embed_row<T>((const T*)nx.E + (size_t)tok[i] * d, nx.pe + (size_t)pos * d, (T*)nx.x + (size_t)(base + i) * d, d, nx.scale, lane, 64);
  } else if (chunks <= 64) {
    next_input_chunks<T, 1>(nx, tok, base, k, pos, lane);
  } else if (chunks <= 128) {
    next_input_chunks<T, 2>(nx, tok, base, k, pos, lane);
  } else {
    next_input_chunks<T, 8>(nx, tok, base, k, pos, lane);
  }
}

// ALONE: the wavefront is the whole workgroup (its barriers are the workgroup's); otherwise other wavefronts of the
// workgroup have finished their part, and LDS and memory serve this one's accesses in the order it makes them.
template <bool ALONE>
__device__ __forceinline__ void rerank_sync() {
  if constexpr (ALONE) {
    __syncthreads();
  } else {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

// The end of a unit's part in a step: `unfinished` of its sentences go on.  Arrivals (low half) and unfinished
// sentences (high half) are counted in one word, so that a unit makes one returning atomic; the last of `units` to
// arrive leaves the count in active[t], advances the position counter -- every unit read it at its start, and the only
// other readers are kernels launched later -- and tells the host (report, pinned memory: step number and count in one
// word; nothing else is read on the strength of it).
// In two halves: what is issued in between hides the atomic's way to memory and back.
__device__ __forceinline__ int step_arrive(int32_t* step_state, int unfinished) { return atomicAdd(&step_state[1], 1 + (unfinished << 16)); }
__device__ __forceinline__ void step_finish(int before, int32_t* active, int t, int32_t* step_state, int next_pos, int unfinished,
                                            int units, unsigned long long* report, int fixed_count = -1) {
  if ((before & 0xFFFF) != units - 1) return;
  const int n = fixed_count >= 0 ? fixed_count : (before >> 16) + unfinished;
  step_state[1] = 0;
  active[t] = n;
  step_state[0] = next_pos;
  if (report)
    __hip_atomic_store(report, ((unsigned long long)(t + 1) << 32) | (unsigned)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Rank of candidate `lane` (score s) among a unit's n candidates in LDS: higher score first, lower index first among equal
// scores -- the rows' lists are sorted and stand one behind the other, so that is the lower (beam, token).  Empty slots
// (token -1) do not count.  Every lane reads every candidate: broadcasts, four at a time.
template <int n>
__device__ __forceinline__ int candidate_rank(const float* cand_s, const int* cand_i, float s, int lane) {
  int rank = 0;
#pragma unroll
  for (int c = 0; c < n; c += 4) {
    const floatx4 s4 = *reinterpret_cast<const floatx4*>(cand_s + c);
    const int4 t4 = *reinterpret_cast<const int4*>(cand_i + c);
    const int t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      rank += c + e < n && t[e] >= 0 && (s4[e] > s || (s4[e] == s && c + e < lane)) ? 1 : 0;
  }
  return rank;
}

// What the re-rank stage reads besides the candidates, requested together (one trip to memory instead of one per
// phase) and, where the retrieve stage runs in the same kernel, before that one: the step, the state of the beam a
// candidate continues (lane c continues beam c / k whatever its rank turns out to be), the sentence's length cap and
// this lane's first position of the k token histories and slab tables.
// No request sits behind a test of something that is itself read from memory: lanes past the k*k candidates repeat the
// last one and positions past the step repeat the last position of the histories (both discarded later), so every load
// can leave before the step counter has arrived.
struct RerankState {
  int t, plen, pfin, cap_b;
  int h[LSQ_MAX_BEAM_], ha[LSQ_MAX_BEAM_];
};
__device__ __forceinline__ void rerank_history(RerankState& st, const int32_t* __restrict__ tokens, const int32_t* __restrict__ anc,
                                               int base, int k, int T1, int p) {
  const int pc = min(p, T1 - 1);
#pragma unroll
  for (int i = 0; i < LSQ_MAX_BEAM_; ++i)
    if (i < k) {
      st.h[i] = tokens[(size_t)(base + i) * T1 + pc];
      st.ha[i] = anc ? anc[(size_t)(base + i) * T1 + pc] : 0;
    }
}
__device__ __forceinline__ RerankState rerank_request(const int32_t* __restrict__ tokens, const int32_t* __restrict__ len,
                                                      const int32_t* __restrict__ fin, const int32_t* __restrict__ cap,
                                                      const int32_t* __restrict__ anc, int k, int T1, int t_base,
                                                      const int32_t* __restrict__ step_state, const SearchGroups& gr, int b, int lane) {
  RerankState st;
  const int base = b * (gr.k_all > 1 ? gr.k_all : k) + gr.goff, j = min(lane, k * k - 1) / k;
  st.t = t_base + (step_state ? step_state[0] : 0);
  st.plen = len[base + j];
  st.pfin = fin[base + j];
  st.cap_b = cap[b];
  rerank_history(st, tokens, anc, base, k, T1, lane);
  return st;
}

// Retrieve and re-rank in one launch (plain beam search from the logit product's group statistics): a workgroup
// per sentence, wavefront w retrieves row w's k best into LDS; every wavefront then ranks the sentence's k*k candidates
// (the same in all of them) and settles hypothesis w: its history, state and next decoder input.  A chain of memory trips
// of about a microsecond each -- statistics, logits of the qualifying groups, embedding rows -- with everything else
// requested up front.  Same bookkeeping as rerank_sentence.
// In two parts, so that a kernel that has other work before the logits can make the request (rerank_request) earlier.
struct SearchShared {
  int ql[LSQ_MAX_BEAM_][kTopkGroupsQ];
  float cs[LSQ_MAX_BEAM_][kTopkGroupsC];
  int ci[LSQ_MAX_BEAM_][kTopkGroupsC];
  alignas(16) float cand_s[LSQ_MAX_BEAM_ * LSQ_MAX_BEAM_];
  alignas(16) int cand_i[LSQ_MAX_BEAM_ * LSQ_MAX_BEAM_];
  int sh_tok[LSQ_MAX_BEAM_];
};
// LAST: the kernel ends with this step; otherwise its other steps follow, and what the step counter has to hear is left to the last one.
// Returns whether the sentence goes on.
template <int GPL, int K>
__device__ __forceinline__ bool retrieve_rerank_sentence(
    const float* logits, const float* stats, float* __restrict__ score, int32_t* __restrict__ tokens,
    int32_t* __restrict__ len, int32_t* __restrict__ fin, int32_t* __restrict__ parent,
    int32_t* __restrict__ active, int V, int G, int T1, int32_t* __restrict__ step_state, int eos,
    int32_t* __restrict__ anc, const NextInput& nx, float* __restrict__ cand_out_s, int32_t* __restrict__ cand_out_i,
    unsigned long long* report, int b, SearchShared& sh, RerankState st, bool last = true) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  constexpr int k = K, kk = K * K;   // known to the compiler: a wavefront on its own takes 8 cycles for every instruction
  const int base = b * k, row = base + wave;
  topk_groups_row<GPL, K <= 4 ? 4 : 8>(logits, stats, score, fin, row, V, G, k, eos, sh.cand_s + wave * k, sh.cand_i + wave * k, lane,
                       sh.ql[wave], sh.cs[wave], sh.ci[wave]);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the histories are here before any wavefront of the sentence overwrites them
  __syncthreads();   // blockDim.x = 64 k: every wavefront has a row
  if (cand_out_s && (int)threadIdx.x < kk) {   // the survivors, for whoever inspects them afterwards
    cand_out_s[(size_t)b * kk + threadIdx.x] = sh.cand_s[threadIdx.x];
    cand_out_i[(size_t)b * kk + threadIdx.x] = sh.cand_i[threadIdx.x];
  }
  // the embedding rows this row's candidates would need, touched so that the one that wins is near by then
  int touched = 0;
  if (nx.E) {
    const unsigned row_bytes = (unsigned)nx.d * (nx.dtype == DT_F16 ? 2 : 4);
    for (int i = lane >> 4; i < k; i += 4)
      for (unsigned o = (lane & 15) * 128; o < row_bytes; o += 2048)
        touched += *reinterpret_cast<const int*>(reinterpret_cast<const char*>(nx.E) + (size_t)embedding_row(sh.cand_i[wave * k + i]) * row_bytes + o);
  }
  const int t = st.t, cl = min(lane, kk - 1), j = cl / k;
  const float s = lane < kk ? sh.cand_s[cl] : -INFINITY;
  const int tok = lane < kk ? sh.cand_i[cl] : -1;
  const int rank = candidate_rank<kk>(sh.cand_s, sh.cand_i, s, lane);
  const bool win = tok >= 0 && rank < k;
  const int nlen = st.pfin ? st.plen : st.plen + 1;
  const int nfin = st.pfin || tok == eos || nlen >= st.cap_b ? 1 : 0;
  const int go_on = __any(win && !nfin) ? 1 : 0;
  int before = 0;
  if (wave == 0 && lane == 0) {
    if (last) before = step_arrive(step_state, go_on);
    else if (go_on) __hip_atomic_fetch_add(&active[t], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const unsigned long long mine = __ballot(win && rank == wave);   // at most one lane: hypothesis w's candidate
  const int from = mine ? __builtin_amdgcn_readlane(j, (int)__builtin_ctzll(mine)) : wave;
  if (lane == 0) sh.sh_tok[wave] = -1;
  rerank_sync<false>();
  if (win && rank == wave) {
    sh.sh_tok[wave] = st.pfin ? eos : tok;   // what the row feeds the decoder next (a finished row: anything valid)
    if (!st.pfin) tokens[(size_t)row * T1 + nlen] = tok;
    len[row] = nlen;
    fin[row] = nfin;
    score[row] = s;
    parent[row] = j;
  }
  // token history, positions 0..t, and the table that says which slab holds position p of it (cache refreshing without
  // moving the cache; position t + 1 is written by the row itself)
  for (int p = lane, p0 = 0; p0 <= t && p0 < T1; p0 += 64, p += 64) {
    if (p0 > 0) {   // a history longer than 64 positions: one more trip per 64
      rerank_history(st, tokens, anc, base, k, T1, p);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    int val = 0, vala = 0;
#pragma unroll
    for (int i = 0; i < LSQ_MAX_BEAM_; ++i)
      if (i == from) { val = st.h[i]; vala = st.ha[i]; }
    if (from != wave && p <= t && p < T1) {
      tokens[(size_t)row * T1 + p] = val;
      if (anc) anc[(size_t)row * T1 + p] = vala;
    }
  }
  if (anc && lane == 0 && t + 1 < T1) anc[(size_t)row * T1 + t + 1] = wave;
  rerank_sync<false>();
  // The next step's decoder input of this row (one launch less per step).  A row that no candidate won
  // (fewer live candidates than beams) embeds nothing: it is dead and stays so.
  if (nx.E && t + 1 < T1 - 1) {
    if (nx.dtype == DT_F16) next_input_rows<half_t>(nx, &sh.sh_tok[wave], row, 1, t + 1, lane);
    else next_input_rows<float>(nx, &sh.sh_tok[wave], row, 1, t + 1, lane);
  }
  asm volatile("" ::"v"(touched));
  if (last && wave == 0 && lane == 0) step_finish(before, active, t, step_state, t + 1, go_on, (int)gridDim.x, report);
  return go_on;
}

}  // namespace lsq
