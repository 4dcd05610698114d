// Decoder layers of one step in one launch, each group of rows on a die of its own (float16, heads of 64, FFN of 4d).
//
// The chip is eight dies with 32 compute units and an L2 each.  What the workgroups of one die hand each other need not leave
// its L2: it is stored with workgroup scope and read with agent-scope loads.  Workgroup scope is enough to reach another compute
// unit of the die: the wavefronts of a workgroup may be spread over several of them (threadgroup split mode, -mtgsplit), for which the
// compiler's stores of that scope carry the same bit, sc0, and nothing is done to the L2, which all compute units that a workgroup can be on
// share.  An agent-scope load includes workgroup scope and passes the reader's own L1 by.  A store without a scope promises nothing before
// the kernel ends, and is no faster (whole translations, 4 to 32 rows: 1.00 times).
// Measured, 32 workgroups that all write a slice and read all of 8 KB: 0.50 us per exchange, against 0.99 with agent-scope
// stores and 1.16 among 128 workgroups all over the chip (kernels_stack.hip).  The price is that every die reads all weights:
// 1.34 TB/s for one die or two, 1.0 for four, 0.92 for all eight (7.4 TB/s together, from the memory-side cache).  So this is for
// models whose layers are small (d = 512: 44 MB, 48 us; d = 256, of which nothing is known, stays with kernels_stack.hip).
//
// Not explained: a kernel that was not kept, with 32 to 64 rows a die (129 to 512 in all), 16 KB per poll and stores without a
// scope, had a wait that ran out once in 1500 to 7000 launches: a value was published and not seen.  An earlier form of this one, with 16 rows
// a die at most and other waits and barriers than now, had none in 187 500 launches with the same stores.  Those stores are the only thing
// found in it that no memory model covers; whether they were the cause is not known.  If a wait does run out no result is lost: the translation is decoded again,
// and the model keeps to the kernels that go by agent scope alone (lsq_runtime.hip, decode_again).
//
// A compute unit's loads come back in the order in which they were issued, whoever issued them: one that finds its line in the
// L2 takes 240 clocks on an idle unit, 560 / 790 / 1590 / 2640 behind 8 / 16 / 32 / 64 KB of weights.  When weights are
// requested therefore decides how long an exchange takes: each time a wait has ended and there is something to compute.
//
// Workgroups are dealt to the dies in turn, eight after one another to eight different ones, but which die is first is another one
// for another stream, and changes for a stream when the process opens others (seen: 0 1 2 .. 7, then 7 0 1 .., then 5 6 7 ..).  So a group is
// the die it finds itself on, and workgroup b's place in it is b / 8.  die_placement() looks whether eight in a row are on different dies when a
// model is loaded.  A launch in which they are not lacks a workgroup of some group.  The others of that group find out when a wait for it
// runs out, half a second later; of a group that lacks them all, the last workgroup of the launch (die_count.h).  Either ends as any wait that runs
// out here does.
// The exchange itself is that of kernels_stack.hip too: data that is its own flag.
#include "die_count.h"
#include "stack_attend.h"
#include "vocabulary_block.h"

namespace lsq {

namespace {

constexpr int kVocabularyRows = 8;     // largest group, and most rows in all, of a launch that takes the vocabulary product along (die_takes_vocabulary)
constexpr int kVocabularyMax = 32;
constexpr int kVocabularyPace = 20;    // 64 clocks between two of a wavefront's requests: launches of 4 rows 72.3 us with 0, 71.7 with 20, 71.9 with 64
constexpr int kDieThreads = 1024;      // eight wavefronts that multiply, eight that exchange
constexpr int kDieLead = 6;            // as kLead: layers of a step in us with 0 / 4 / 6 / 8 / 12: 4 rows 73.0 72.4 70.4 71.6 73.1, 32 rows 85.9 85.4 85.0
                                       // 84.7 85.3, 64 rows 92.9 89.9 90.6 91.3 92.7, 128 rows 109.7 106.7 105.9 106.0 108.5

__device__ __forceinline__ unsigned die_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)); }   // XCC_ID, 4 bits
__global__ void die_of_workgroup_kernel(unsigned* out) {
  if (threadIdx.x == 0) out[blockIdx.x] = die_id();
}

__device__ __forceinline__ void workgroup_barrier() {   // LDS only: loads stay in flight
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void pin() { asm volatile("" ::: "memory"); }   // requests stay where they are written

// ---------------------------------------------------------------------------------------------
// Few rows, d = 512: up to 16 a die.  Eight wavefronts hold the matrices in registers (an eighth of k each), ask for the next
// ones and multiply; the other eight look for the exchanged values, normalise, attend, add the eight partial sums up and
// publish.  Nobody waits for a value behind weights of its own this way, and 128 registers are enough for either.
// Measured, layers of one step in us at positions up to 60, sources of 30 (groups of 8 or 16 rows all over the chip): 4 rows 69 (94),
// 8 rows 69 (100), 32 rows 83 (106), 64 rows 89 (113), 128 rows 104 (130).  Every layer is a chain of eight exchanges and products,
// 9 us of its 11 on one die or two; the rest is what exchanges queue behind weights (with all of them in the L2, on wrong numbers: 59, 59, 59, 70,
// 93).  The chain is made of instructions that wait for one another: what a wavefront does on it has no branches, asks LDS for all it
// needs at once, and what can be done while somebody else works is done then: 77, 78, 94, 101, 118 before.
template <int R, bool PRE>
__global__ void __launch_bounds__(kDieThreads) decoder_die_kernel(const StackArgs a) {
  constexpr int DK = 2, D = 256 * DK, H = D / 64, W = kDieGroup, NT = D / W;
  constexpr int TEAMS = R * H / W, NSH = kWaves / TEAMS;         // wavefronts that share a (row, head) pair
  using Rg = Region<PRE>;
  constexpr int ES = PRE ? 2 : 4;                                // bytes of a residual sum
  constexpr int VP = 16 / ES, NP = D / (64 * VP);                // values of a 16-byte piece, pieces of a row per lane
  constexpr int RW = (R + kWaves - 1) / kWaves;                  // rows of a wavefront
  using sum_t = std::conditional_t<PRE, half_t, float>;
  static_assert(NT == 16, "one unit of columns per workgroup");

  __shared__ __attribute__((aligned(16))) half_t xs[R][D + 8];             // normalised rows
  __shared__ __attribute__((aligned(16))) half_t us[PRE ? R : 1][D + 8];   // pre-LN: the residual stream
  __shared__ __attribute__((aligned(16))) half_t st[R][4 * D + 8];         // contexts, FFN activations
  __shared__ __attribute__((aligned(16))) float part[kWaves][4][R][16];
  __shared__ __attribute__((aligned(16))) Shares shares;
  __shared__ int arrived[kWaves];   // exchanges that a wavefront has seen the end of
  __shared__ unsigned first_key[kWaves][kTrip][64];
  __shared__ __attribute__((aligned(16))) half_t vec[2][7][D];   // of a layer: gains and shifts, biases

  __shared__ uint64_t word;
  constexpr bool VOC = R <= kVocabularyRows;   // group sizes with which dies may be left over
  __shared__ __attribute__((aligned(16))) half_t voc_rows[VOC ? kVocabularyMax : 1][D + 8];
  __shared__ float voc_part[VOC ? kWaves : 1][16][64];
  __shared__ int launch_seq, ticket, in_vain;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, grp = die_id();
  int j = blockIdx.x >> 3;
  const int seq = a.state[0], parity = seq & 1;
  if (tid == 0) word = die_word(grp, j);
  // the last workgroup of the launch to get here: all have read the counters
  auto leave = [&] {
    int32_t* const state = now()->state;
    uint64_t* const count = reinterpret_cast<uint64_t*>(state + 6);
    const uint64_t n = __hip_atomic_fetch_add(count, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (die_launch_ends(n)) {
      *count = 0;
      state[1 + parity] = now()->groups * R + (VOC && now()->V ? 1 : 0);   // the rows for the vocabulary product: in the place of one row more
      __hip_atomic_fetch_xor(state, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool helped = !VOC || !now()->V || __hip_atomic_exchange(state + 5, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (kDies - now()->groups) * kDieGroup;
      if (!helped || !die_groups_there(n + word, now()->groups)) give_up(state, now()->error);
    }
  };
  const int row_bytes = a.layers * Rg::size * D;
  const int hidden_at = G * R * row_bytes;   // of the exchange: the rows for the vocabulary product, [row][d], agent scope
  if (grp >= G) {
    if constexpr (VOC) {
      if (a.V > 0) {
        // ================ A die to spare: its workgroups have the vocabulary's columns, in blocks of 32.  A pair of wavefronts has a block, either
        // half of its k-steps, which wait in registers for the rows: nothing is left to be fetched once these are there.  Which workgroup has which
        // blocks is drawn, so that it does not depend on how the workgroups were dealt out.  4 rows, 32000 columns: launch 67.3 -> 71.5 us instead of a
        // product of 6.2 behind it; what is left of it is an exchange over the whole chip, the products' eight dependent steps and the statistics.
        // (the other wavefronts' own `seq` may be of any age by now: what this launch exchanges in is what the first thread saw)
        if (tid == 0)
          die_spare_signs_off(
              [&] {
                asm volatile("" ::"s"(seq) : "memory");   // here
                return seq;
              },
              [&] {
                const int mine = __hip_atomic_fetch_add(now()->state + 5, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::"v"(mine) : "memory");
                return mine;
              },
              [&](int launch, int columns) {
                launch_seq = launch;
                ticket = columns;
                in_vain = 0;
              },
              leave);
        workgroup_barrier();
        const int of_launch = __builtin_amdgcn_readfirstlane(launch_seq);
        const int lane = tid & 63, half = wave & 1, pair = wave >> 1, helpers = (kDies - G) * kDieGroup;
        const int V = a.V, blocks = (V + 31) / 32, block = __builtin_amdgcn_readfirstlane(ticket) + pair * helpers;
        const half_t* wp = global(a.Ep) + ((size_t)min(block, blocks - 1) * (D / 16) + half * 2) * 512 + lane * 8;
        half8_t w[D / 32];   // k-steps 4 q + 2 half + e
        // (all at once they would be in the way of what the other dies wait for)
        if (block < blocks) {
#pragma unroll
          for (int i = 0; i < D / 32; ++i) {
            w[i] = *reinterpret_cast<const half8_t*>(wp + ((i >> 1) * 4 + (i & 1)) * 512);
            pin();
            __builtin_amdgcn_s_sleep(kVocabularyPace);
          }
        }
        pin();
        Exchange<> ex;
        ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange + (size_t)(of_launch & 1) * a.set_bytes, (short)0, (int)a.set_bytes, 0x00027000);
        ex.polls = of_launch < 0 ? 1 : kSpinLimit;
        const int M = a.M;
        if (wave == 0) {   // a look now and then, until the rows are nearly there
          u32x4 one;
          for (int left = ex.polls;;) {
            one = __builtin_amdgcn_raw_buffer_load_b128(ex.rsrc, M * (D * 2), hidden_at, kAgent);
            if (__all(max(max(one.x, one.y), max(one.z, one.w)) != kSentinel)) break;
            if (--left == 0) {
              in_vain = 1;
              break;
            }
            __builtin_amdgcn_s_sleep(16);
            asm volatile("" ::: "memory");
          }
        }
        workgroup_barrier();
        if (in_vain) ex.polls = 1;
        const int pieces = M * (D / 8);
        for (int p0 = 0; p0 < pieces; p0 += kDieThreads) {
          if (p0 + wave * 64 >= pieces) break;
          const int p = min(p0 + tid, pieces - 1);
          u32x4 raw[1];
          ex.wait<0>([&](int) { return hidden_at; }, [&](int) { return p * 16; }, raw);
          *reinterpret_cast<u32x4*>(&voc_rows[p / (D / 8)][p % (D / 8) * 8]) = raw[0];
        }
        workgroup_barrier();
        // the sums of gemm_f16_skinny_kernel: four of them take the k-steps in turn and are added in pairs
        const int m = lane & 31;
        const half_t* xr = &voc_rows[min(m, M - 1)][(lane >> 5) * 8];
        floatx16 acc[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc[0][e] = 0.f; acc[1][e] = 0.f; }
        if (block < blocks) {
#pragma unroll
          for (int i = 0; i < D / 32; ++i)
            acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[i], *reinterpret_cast<const half8_t*>(xr + ((i >> 1) * 4 + half * 2 + (i & 1)) * 16), acc[i & 1], 0, 0, 0);
          acc[0] += acc[1];
          if (half)
#pragma unroll
            for (int e = 0; e < 16; ++e) voc_part[pair][e][lane] = acc[0][e];
        }
        workgroup_barrier();
        if (!half && block < blocks) {
          float other[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) other[e] = voc_part[pair][e][lane];
          float* const out = global(now()->logits) + (size_t)m * V;
          vocabulary_block<true>([&](int vg, int e) { return acc[0][vg * 4 + e] + other[vg * 4 + e]; },
                           [&](int n, const float (&v)[4]) {
                             if ((V & 3) == 0) {
                               *reinterpret_cast<floatx4*>(out + n) = floatx4{v[0], v[1], v[2], v[3]};
                             } else {
#pragma unroll
                               for (int e = 0; e < 4; ++e)
                                 if (n + e < V) out[n + e] = v[e];
                             }
                           },
                           global(now()->stats), blocks, m, block, M, V, lane);
        }
        ex.report(now()->state, now()->error);
        return;
      }
    }
    if (tid == 0) leave();
    return;
  }
  const int r0 = grp * a.rows_per_group, rows = min(a.rows_per_group, a.M - r0);
  const int dirty = a.state[2 - parity], pos = *a.tpos;

  Exchange<kWorkgroup> ex;   // stores that end in the die's L2, where the readers' agent-scope loads look
  ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange + (size_t)parity * a.set_bytes, (short)0, (int)a.set_bytes, 0x00027000);
  ex.polls = seq < 0 ? 1 : kSpinLimit;
  const int layer_bytes = Rg::size * D * R;
  auto at = [&](int l, int region) { return __builtin_amdgcn_readfirstlane(grp * a.layers * layer_bytes + l * layer_bytes + region * D * R); };
  if (tid < kWaves) { arrived[tid] = 0; shares.left[tid] = 0; }
  workgroup_barrier();

  if (wave < kWaves) {
    // ================ products: wavefront w has an eighth of k; matrices wait in registers
    const int lane = tid & 63, kc = lane >> 4, fm = lane & (R - 1);
    const unsigned lane16 = (unsigned)(kc >> 1) * 1024 + ((lane & 15) + 32 * (kc & 1)) * 16;
    // the first of this wavefront's S k-steps of a unit of 16 columns
    auto slice = [&](const half_t* Wp, int unit, int S) {
      return reinterpret_cast<const char*>(global(Wp)) + (size_t)(unit >> 1) * (S * 16384) + (unit & 1) * 256 + wave * S * 2048;
    };
    const char* p_q[3] = {slice(a.Wqkv, j, DK), slice(a.Wqkv, j + W, DK), slice(a.Wqkv, j + 2 * W, DK)};
    const char* p_1[4] = {slice(a.W1, j, DK), slice(a.W1, j + W, DK), slice(a.W1, j + 2 * W, DK), slice(a.W1, j + 3 * W, DK)};
    const char *p_o = slice(a.Wo, j, DK), *p_2 = slice(a.W2, j, 4 * DK);
    const char *p_c = PRE ? nullptr : slice(a.Wq, j, DK), *p_e = PRE ? nullptr : slice(a.Woc, j, DK);
    auto frag = [&](const char* p, int s) { return *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16); };
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const half8_t* w, auto units, auto steps, const half_t* in, int ld) {
      constexpr int N = decltype(units)::value, S = decltype(steps)::value;
      floatx4 acc[N];
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = zero4;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const half8_t x8 = *reinterpret_cast<const half8_t*>(in + fm * ld + (wave * S + s) * 32 + kc * 8);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i * S + s], x8, acc[i], 0, 0, 0);
      }
      if ((lane & 15) < R) {
#pragma unroll
        for (int i = 0; i < N; ++i) *reinterpret_cast<floatx4*>(&part[wave][i][lane & 15][kc * 4]) = acc[i];
      }
    };
    using n1 = std::integral_constant<int, 1>;
    using n3 = std::integral_constant<int, 3>;
    using n4 = std::integral_constant<int, 4>;
    using k1 = std::integral_constant<int, DK>;
    using k4 = std::integral_constant<int, 4 * DK>;
    // w1: the second half of it Wo's until that is used; q: Wq and Woc once Wqkv is used
    half8_t w1[8], q[6], w2[8], wo[PRE ? 2 : 1];
    auto some = [&](half8_t* w, const char* p, size_t o, int s, int n) {
#pragma unroll
      for (int i = 0; i < n; ++i) w[i] = frag(p + o, s + i);
    };
    half8_t* const o_at = PRE ? wo : w1 + 6;
    size_t o = 0;   // of the layer
    for (int i = 0; i < 3; ++i) some(q + 2 * i, p_q[i], 0, 0, 2);
    if constexpr (PRE) some(o_at, p_o, 0, 0, 2);
    pin();
    const half_t* const x = &xs[0][0];
    const half_t* const y = &st[0][0];
    // Each time the exchanging wavefronts have what they looked for there is nothing to wait for in memory for a
    // while, and the next matrices are requested.
    int exchanges = 0;
    auto values_here = [&] {
      for (++exchanges; !__all(__hip_atomic_load(&arrived[lane & (kWaves - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= exchanges);) __builtin_amdgcn_s_sleep(1);
      pin();
    };
    for (int l = 0; l < a.layers; ++l, o += a.packed_stride) {
      // Past the last layer: pieces that are in the L2 already, instead of 64 KB that nobody wants and the last exchange would queue
      // behind.  (A branch around the requests would cost more: the compiler no longer knows how many are in flight.)
      const bool more = l + 1 < a.layers;
      const size_t next = more ? o + a.packed_stride : o;
      const char* const n_q[3] = {more ? p_q[0] : p_2, more ? p_q[1] : p_2, more ? p_q[2] : p_2};
      if constexpr (!PRE) {
        // How many pieces go where: a compute unit takes in one (8 KB of its 224 of a layer) in 460 clocks where one die reads, 670 where all do, the
        // first after 1200, and what it looks for meanwhile arrives behind them.
        values_here();                                                    // sums of the layer before
        some(o_at, p_o, o, 0, 2); some(w1, p_1[0], o, 0, 2); some(w1 + 2, p_1[1], o, 0, 1);
        pin();
        workgroup_barrier();                                              // 1: input rows
        multiply(q, n3{}, k1{}, x, D + 8);
        workgroup_barrier();                                              // 2
        values_here();                                                    // q, k, v
        some(q, p_c, o, 0, 2); some(q + 2, p_e, o, 0, 2);
        pin();
        workgroup_barrier();                                              // 3: context
        some(w1 + 3, p_1[1], o, 1, 1); some(w1 + 4, p_1[2], o, 0, 1);
        pin();
        multiply(o_at, n1{}, k1{}, y, 4 * D + 8);
        pin();
        workgroup_barrier();                                              // 4
        values_here();                                                    // sums
        some(w1 + 5, p_1[2], o, 1, 1); some(w1 + 6, p_1[3], o, 0, 2); some(w2, p_2, o, 0, 1);
        pin();
        workgroup_barrier();                                              // 5: rows
        multiply(q, n1{}, k1{}, x, D + 8);
        workgroup_barrier();                                              // 6
        values_here();                                                    // queries
        some(w2 + 1, p_2, o, 1, 2);
        pin();
        workgroup_barrier();                                              // 7: context
        some(w2 + 3, p_2, o, 3, 2);
        pin();
        multiply(q + 2, n1{}, k1{}, y, 4 * D + 8);
        pin();
        workgroup_barrier();                                              // 8
        values_here();                                                    // sums
        some(w2 + 5, p_2, o, 5, 3);
        some(q, n_q[0], next, 0, 2); some(q + 2, n_q[1], next, 0, 1);
        pin();
        workgroup_barrier();                                              // 9: rows
        multiply(w1, n4{}, k1{}, x, D + 8);
        workgroup_barrier();                                              // 10
        workgroup_barrier();                                              // 11: activations
        some(q + 3, n_q[1], next, 1, 1); some(q + 4, n_q[2], next, 0, 2);
        pin();
        multiply(w2, n1{}, k4{}, y, 4 * D + 8);
        pin();
        workgroup_barrier();                                              // 12
      } else {
        values_here();                                                    // sums of the layer before
        some(w1, p_1[0], o, 0, 2); some(w1 + 2, p_1[1], o, 0, 2);
        some(w1 + 4, p_1[2], o, 0, 1);
        pin();
        workgroup_barrier();                                              // 1: input rows
        multiply(q, n3{}, k1{}, x, D + 8);
        workgroup_barrier();                                              // 2
        values_here();                                                    // q, k, v
        some(w1 + 5, p_1[2], o, 1, 1); some(w1 + 6, p_1[3], o, 0, 2); some(w2, p_2, o, 0, 2);
        pin();
        workgroup_barrier();                                              // 3: context
        some(w2 + 2, p_2, o, 2, 5);
        multiply(o_at, n1{}, k1{}, y, 4 * D + 8);
        pin();
        workgroup_barrier();                                              // 4
        values_here();                                                    // sums
        some(w2 + 7, p_2, o, 7, 1);
        some(q, n_q[0], next, 0, 2); some(q + 2, n_q[1], next, 0, 2);
        pin();
        workgroup_barrier();                                              // 9: rows
        multiply(w1, n4{}, k1{}, x, D + 8);
        workgroup_barrier();                                              // 10
        workgroup_barrier();                                              // 11: activations
        some(q + 4, n_q[2], next, 0, 2);
        some(o_at, more ? p_o : p_2, next, 0, 2);
        multiply(w2, n1{}, k4{}, y, 4 * D + 8);
        pin();
        workgroup_barrier();                                              // 12
      }
    }
    if (tid == 0) leave();
    return;
  }

  // ================ exchange, LayerNorm, attention
  int xt = tid - kWaves * 64, lane = tid & 63, xw = wave - kWaves;
  // gains, shifts and this workgroup's biases: 16 bytes of one of them per lane, on their way to LDS
  const char* vec_at;   // of the next layer
  if (xw < 6) {
    const half_t* v = xw == 0 ? a.ln1g : xw == 1 ? a.ln1b : xw == 2 ? a.ln2g : xw == 3 || PRE ? a.ln2b : xw == 4 ? a.ln3g : a.ln3b;
    vec_at = reinterpret_cast<const char*>(v + lane * 8);
  } else {
    const int u = min(lane >> 1, 10);   // units: q k v | o | c | e | w1 x 4 | w2
    const half_t* v = u < 3 ? a.bqkv : u == 3 || (PRE && u < 6) ? a.bo : u == 4 ? a.bq : u == 5 ? a.boc : u < 10 ? a.b1 : a.b2;
    vec_at = reinterpret_cast<const char*>(v + (u < 3 ? j + W * u : u < 6 || u == 10 ? j : j + W * (u - 6)) * 16 + (lane & 1) * 8);
  }
  auto vectors = [&] { const half8_t v = *reinterpret_cast<const half8_t*>(global(vec_at)); vec_at += a.plain_stride; return v; };
  auto keep_vectors = [&](int l, const half8_t& v) {
    if (xw < 6) *reinterpret_cast<half8_t*>(&vec[l & 1][xw][lane * 8]) = v;
    else if (xw == 6 && lane < 22) *reinterpret_cast<half8_t*>(&vec[l & 1][6][lane * 8]) = v;
  };
  half8_t ahead = vectors();
  // an exchange has ended for this wavefront: the others may request weights
  int exchanges = 0;
  auto seen = [&] {
    ++exchanges;
    __hip_atomic_store(&arrived[xw], exchanges, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // ---- What the products leave: unit, row and pair of columns that this thread finishes.  Everything it needs besides is read
  // while the products run.  With 4 rows other wavefronts than those that look for the rows next.
  constexpr int SKIP = R == 4 ? 256 : 0;
  int ui = (xt ^ SKIP) / (8 * R), um = xt / 8 % R, un = xt % 8 * 2;
  half2_t bi = {0, 0}, xr = {0, 0};
  auto prepare = [&](int l, int units, int first) {
    if (ui < units) bi = *reinterpret_cast<const half2_t*>(&vec[l & 1][6][(first + ui) * 16 + un]);
    if (units == 1) xr = *reinterpret_cast<const half2_t*>(PRE ? &us[um][j * 16 + un] : &xs[um][j * 16 + un]);
  };
  auto total = [&](float& v0, float& v1) {   // + bias
    floatx2 p[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) p[w] = *reinterpret_cast<const floatx2*>(&part[w][ui][um][un]);
    // all of them requested before the first is added: left to itself the compiler takes a trip to LDS for each
    asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]), "+v"(p[4]), "+v"(p[5]), "+v"(p[6]), "+v"(p[7]));
    v0 = p[0][0]; v1 = p[0][1];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) { v0 += p[w][0]; v1 += p[w][1]; }
    v0 += (float)bi[0]; v1 += (float)bi[1];
  };
  auto residual = [&](int l, int region) {
    if (ui < 1 && um < rows) {
      float v0, v1;
      total(v0, v1);
      const float s0 = (float)xr[0] + v0, s1 = (float)xr[1] + v1;
      if constexpr (PRE) ex.put2(at(l, region), (j * R + um) * 32 + un * 2, (half_t)s0, (half_t)s1);
      else ex.put2(at(l, region), (j * R + um) * 64 + un * 4, s0, s1);
    }
  };
  // ---- rows: wavefront w normalises rows w and w + 8 into xs
  auto normalise = [&](float (&v)[NP][VP], const half_t (&g)[NP][VP], const half_t (&b)[NP][VP], half_t (&o)[NP][VP]) {
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int i = 0; i < VP; ++i) sum += v[q][i];
    const float mean = wave_sum(sum) * (1.0f / D);
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int i = 0; i < VP; ++i) { v[q][i] -= mean; sq += v[q][i] * v[q][i]; }
    // 1 / sqrt by one Newton step: worst 1.53, mean 0.30 units in the last place against 64 bits (division by the root: 1.96, 0.38)
    const float var = wave_sum(sq) * (1.0f / D) + a.eps, r = __builtin_amdgcn_rsqf(var);
    const float rstd = r * (1.5f - 0.5f * var * r * r);
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int i = 0; i < VP; ++i) o[q][i] = (half_t)((float)g[q][i] * (v[q][i] * rstd) + (float)b[q][i]);
  };
  typedef half_t piece_t __attribute__((ext_vector_type(VP)));
  auto pieces = [&](const half_t* p, half_t (&o)[NP][VP]) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const piece_t h = *reinterpret_cast<const piece_t*>(p + (q * 64 + lane) * VP);
#pragma unroll
      for (int i = 0; i < VP; ++i) o[q][i] = h[i];
    }
  };
  auto put_pieces = [&](half_t* p, const half_t (&o)[NP][VP]) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      piece_t h;
#pragma unroll
      for (int i = 0; i < VP; ++i) h[i] = o[q][i];
      *reinterpret_cast<piece_t*>(p + (q * 64 + lane) * VP) = h;
    }
  };
  auto gather_norm = [&](int l, int region, const half_t* g, const half_t* b, half_t* out_x, half_t* out_y, bool publish = false) {
    half_t g8[NP][VP], b8[NP][VP];
    u32x4 raw[RW * NP];
    const int base = at(l, region);
    if (xw < rows) {
    pieces(g, g8);
    pieces(b, b8);
    ex.wait<kDieLead>([&](int) { return base; },
            [&](int i) {
              const int m = min(xw + i / NP * kWaves, rows - 1), q = i % NP * 64 + lane;   // a writer has NT ES bytes of a row
              return (q / (NT * ES / 16) * R + m) * (NT * ES) + q % (NT * ES / 16) * 16;
            }, raw);
    }
    seen();
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const int m = xw + rr * kWaves;
      if (m >= rows) break;
      float v[NP][VP];
      half_t o[NP][VP];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        typedef sum_t vec_t __attribute__((ext_vector_type(VP)));
        const vec_t s = __builtin_bit_cast(vec_t, raw[rr * NP + q]);
#pragma unroll
        for (int i = 0; i < VP; ++i) v[q][i] = (float)s[i];
        if constexpr (PRE) {
          *reinterpret_cast<vec_t*>(&us[m][(q * 64 + lane) * VP]) = s;
          if (out_x) *reinterpret_cast<vec_t*>(out_x + (size_t)(r0 + m) * D + (q * 64 + lane) * VP) = s;
        }
      }
      normalise(v, g8, b8, o);
      if (publish) {   // to the other dies
        Exchange<> all;
        all.rsrc = ex.rsrc;
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
          for (int i = 0; i < VP; i += 2) all.put2(hidden_at, (r0 + m) * (D * 2) + ((q * 64 + lane) * VP + i) * 2, o[q][i], o[q][i + 1]);
      }
      put_pieces(xs[m], o);
      if (out_y) put_pieces(out_y + (size_t)(r0 + m) * D, o);
    }
  };
  // ---- staging of what the products without LayerNorm read
  auto stage_ctx = [&](int l, int region) {
    constexpr int N = (R * D / 8 + 511) / 512;
    const int first = xt ^ SKIP;   // with 4 rows not the wavefronts that attend first
    if ((xw ^ (SKIP / 64)) * 64 >= rows * (D / 8)) return;
    u32x4 raw[N];
    const int base = at(l, region);
    ex.wait<kDieLead>([&](int) { return base; }, [&](int i) { return min(i * 512 + first, rows * (D / 8) - 1) * 16; }, raw);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = i * 512 + first;
      if (p < rows * (D / 8)) *reinterpret_cast<u32x4*>(&st[p / (D / 8)][p % (D / 8) * 8]) = raw[i];
    }
  };
  auto stage_ff = [&](int l) {
    constexpr int N = R * D / 2 / 512;   // 16-byte pieces of units of 16 columns
    u32x4 raw[N];
    const int base = at(l, Rg::ff);
    auto row = [&](int p) { return min(p / 2 % R, rows - 1); };
    ex.wait<kDieLead>([&](int) { return base; },
            [&](int i) { const int p = i * 512 + xt; return (p / (2 * R) * R + row(p)) * 32 + (p & 1) * 16; }, raw);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = i * 512 + xt;
      *reinterpret_cast<u32x4*>(&st[p / 2 % R][p / (2 * R) * 16 + (p & 1) * 8]) = raw[i];
    }
  };
  // ---- attention of one (row, head) pair per team of NSH wavefronts, of which n have keys to look at (stack_attend.h)
  const int team = xw / NSH, ash = xw % NSH;
  int gk = lane >> 3, c8 = (lane & 7) * 8;
  const int pair = j + W * team, am = min(pair / H, rows - 1), ah = pair % H;
  const int arow = r0 + am, sent = arow / a.beam;
  auto team_of = [&](int nkeys) { return pair < rows * H ? team_for<NSH>(nkeys) : 0; };
  int n_self = 0, n_cross = 0, src_off = 0, src_len = 0;
  const bool table = !PRE && a.anc != nullptr;
  const int32_t* slots = table ? a.anc + (size_t)arow * a.anc_ld : nullptr;
  auto slot_of = [&](int p) { return table ? min(max(slots[p], 0), a.beam - 1) : 0; };   // of the sentence's rows
  auto key_offset = [&](int slot, int p) { return ((slot * a.T + p) * D + c8) * 2; };
  // what attention goes by, looked up while the first product runs
  auto look_up = [&] {
    n_self = team_of(pos);
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {   // the first trip's places in the cache, the same in all layers
      const int p = max(min(ash + (gk + u * 8) * n_self, pos - 1), 0);
      first_key[xw][u][lane] = key_offset(slot_of(p), p);
    }
    if constexpr (!PRE) {
      src_off = a.src_off[sent]; src_len = a.src_len[sent];
      n_cross = team_of(src_len);
    }
  };
  half8_t kn[kTrip], vn[kTrip];
  auto request = [&](bool self, const half_t* Kb, const half_t* Vb, int nkeys, int n, int jb, auto first) {
    const size_t own = self ? (size_t)(table ? sent * a.beam : arow) * a.T * D : 0;
    const char* Kh = reinterpret_cast<const char*>(Kb + own + ah * 64);
    const char* Vh = reinterpret_cast<const char*>(Vb + own + ah * 64);
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {   // past the last key: that one again
      unsigned o;
      if (self && first) {
        o = first_key[xw][u][lane];
      } else {
        const int p = max(min(jb + (gk + u * 8) * n, nkeys - 1), 0);
        o = self ? key_offset(slot_of(p), p) : (p * (2 * D) + c8) * 2;
      }
      kn[u] = *reinterpret_cast<const half8_t*>(Kh + o);
      vn[u] = *reinterpret_cast<const half8_t*>(Vh + o);
    }
  };
  int attentions = 0;
  auto attend = [&](int l, auto of_self, const half_t* Kb, const half_t* Vb, int nkeys, int n) {
    constexpr bool self = decltype(of_self)::value;
    half8_t q, knew = {}, vnew = {};
    ++attentions;
    if (ash < n) {
      const int lo = (c8 >> 4) * R * 32 + (c8 & 8) * 2;
      if constexpr (self) {
        u32x4 raw[3];
        const int base = at(l, Rg::qkv) + (ah * 4 * R + am) * 32;
        ex.wait<kDieLead>([&](int i) { return base + i * (D / 16 * 32) * R; }, [&](int) { return lo; }, raw);
        q = __builtin_bit_cast(half8_t, raw[0]); knew = __builtin_bit_cast(half8_t, raw[1]); vnew = __builtin_bit_cast(half8_t, raw[2]);
      } else {
        u32x4 raw[1];
        const int base = at(l, Rg::q2) + (ah * 4 * R + am) * 32;
        ex.wait<kDieLead>([&](int) { return base; }, [&](int) { return lo; }, raw);
        q = __builtin_bit_cast(half8_t, raw[0]);
      }
    }
    seen();
    if (ash >= n) return;
    Attention t;
    auto live = [&](int jb) { return [&, jb](int u) { return jb + (gk + u * 8) * n < nkeys; }; };
    const int span = kTripKeys * n;
    if (nkeys <= span) {
      t.first<self>(q, kn, vn, knew, nkeys == 0, live(ash), [] {});
    } else {
      t.first<self>(q, kn, vn, knew, false, live(ash), [&] { request(self, Kb, Vb, nkeys, n, ash + span, std::false_type{}); });
      for (int jb = ash + span; jb < nkeys; jb += span)   // the same trips in every lane of the wavefront
        t.more(q, kn, vn, live(jb), [&] { if (jb + span < nkeys) request(self, Kb, Vb, nkeys, n, jb + span, std::false_type{}); });
    }
    if (self && ash == n - 1) t.add(vnew, gk == 0);
    t.sum<true>();
    const int base = at(l, self ? Rg::ctx : Rg::ctx2), lo = am * (D * 2) + ah * 128;
    if (n == 1) {
      const half2_t v = context_of(t.acc[0], t.acc[1], t.z);
      if ((lane & 8) == 0) ex.put2(base, lo + own_column<true>(lane) * 2, v[0], v[1]);
      return;
    }
    shares.leave<true>(xw, lane, t);
    if (ash > 0) return shares.tell(xw, attentions);
    const int c = (lane & 31) * 2;   // in both halves of the wavefront alike
    const half2_t v = shares.collect<NSH>(team * NSH, n, attentions, lane, c);
    if (lane < 32) ex.put2(base, lo + c * 2, v[0], v[1]);
  };

  for (int l = 0; l < a.layers; ++l) {
    // what is derived from a thread's place is derived anew in every layer instead of waiting in registers
    asm volatile("" : "+v"(xt), "+v"(lane), "+v"(ui), "+v"(um), "+v"(un), "+v"(gk), "+v"(c8));
    asm volatile("" : "+s"(xw), "+s"(j));
    const half_t* Kc = reinterpret_cast<const half_t*>(global(now()->cache) + (size_t)(2 * l) * now()->cache_stride);
    const half_t* Vc = reinterpret_cast<const half_t*>(global(now()->cache) + (size_t)(2 * l + 1) * now()->cache_stride);
    if (l == 0) {
      seen();
#pragma unroll
      for (int rr = 0; rr < RW; ++rr) {
        const int m = xw + rr * kWaves, r = r0 + m;
        if (m >= rows) break;
        if constexpr (PRE) {
          half_t g8[NP][VP], b8[NP][VP], o[NP][VP];
          float v[NP][VP];
          pieces(a.ln1g, g8);
          pieces(a.ln1b, b8);
          const half_t* e = a.E + (size_t)embedding_row(a.tokens[(size_t)r * (a.T + 1) + a.len[r]]) * D;
          embed_whole_row<half_t, D>(e, a.pe + (size_t)pos * D, us[m], 1.0f, lane);   // the lane's own pieces
          pieces(us[m], o);
#pragma unroll
          for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int i = 0; i < VP; ++i) v[q][i] = (float)o[q][i];
          normalise(v, g8, b8, o);
          put_pieces(xs[m], o);
        } else {
          half_t o[NP][VP];
          pieces(a.x0 + (size_t)r * D, o);
          put_pieces(xs[m], o);
        }
      }
      keep_vectors(0, ahead);
    } else {
      if (ash < n_self) request(true, Kc, Vc, pos, n_self, ash, std::true_type{});
      pin();
      if constexpr (PRE) gather_norm(l - 1, Rg::u3, vec[l & 1][0], vec[l & 1][1], nullptr, nullptr);
      else gather_norm(l - 1, Rg::u3, vec[(l - 1) & 1][4], vec[(l - 1) & 1][5], nullptr, nullptr);
    }
    // Between two barriers of a pair the products run, and there is time for what need not wait for them.
    workgroup_barrier();                                                  // 1
    prepare(l, 3, 0);
    if (l + 1 < a.layers) ahead = vectors();
    pin();
    workgroup_barrier();                                                  // 2
    if (ui < 3 && um < rows) {
      float v0, v1;
      total(v0, v1);
      const half_t h0 = (half_t)v0, h1 = (half_t)v1;
      ex.put2(at(l, Rg::qkv), ((j + W * ui) * R + um) * 32 + un * 2, h0, h1);
      if (ui >= 1) *reinterpret_cast<half2_t*>(const_cast<half_t*>(ui == 1 ? Kc : Vc) + ((size_t)(r0 + um) * a.T + pos) * D + j * 16 + un) = half2_t{h0, h1};
    }
    if (l == 0) {
      look_up();
      if (ash < n_self) request(true, Kc, Vc, pos, n_self, ash, std::true_type{});
      pin();
    }
    attend(l, std::true_type{}, Kc, Vc, pos, n_self);
    if (l + 1 < a.layers) keep_vectors(l + 1, ahead);
    stage_ctx(l, Rg::ctx);
    workgroup_barrier();                                                  // 3
    prepare(l, 1, 3);
    pin();
    workgroup_barrier();                                                  // 4
    residual(l, Rg::u1);
    if constexpr (!PRE) {
      const half_t* kvb = reinterpret_cast<const half_t*>(global(now()->cross) + (size_t)l * now()->cross_stride) + (size_t)src_off * 2 * D;
      if (ash < n_cross) request(false, kvb, kvb + D, src_len, n_cross, ash, std::true_type{});
      pin();
      gather_norm(l, Rg::u1, vec[l & 1][0], vec[l & 1][1], nullptr, nullptr);
      workgroup_barrier();                                                // 5
      prepare(l, 1, 4);
      pin();
      workgroup_barrier();                                                // 6
      if (ui < 1 && um < rows) {
        float v0, v1;
        total(v0, v1);
        ex.put2(at(l, Rg::q2), (j * R + um) * 32 + un * 2, (half_t)v0, (half_t)v1);
      }
      attend(l, std::false_type{}, kvb, kvb + D, src_len, n_cross);
      stage_ctx(l, Rg::ctx2);
      workgroup_barrier();                                                // 7
      prepare(l, 1, 5);
      pin();
      workgroup_barrier();                                                // 8
      residual(l, Rg::u2);
    }
    gather_norm(l, PRE ? Rg::u1 : Rg::u2, vec[l & 1][2], vec[l & 1][3], nullptr, nullptr);
    if (VOC && l + 1 == a.layers && now()->V > 0 && grp == 0 && j == 1 && xt < 4) {   // the rows for the vocabulary product are two exchanges away
      Exchange<> all;
      all.rsrc = ex.rsrc;
      all.put(hidden_at, now()->M * (D * 2) + xt * 4, 0);
    }
    workgroup_barrier();                                                  // 9
    prepare(l, 4, 6);
    pin();
    workgroup_barrier();                                                  // 10
    if (ui < 4 && um < rows) {
      float v0, v1;
      total(v0, v1);
      if constexpr (PRE) { v0 = tanh_gelu(v0); v1 = tanh_gelu(v1); }
      else { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); }
      ex.put2(at(l, Rg::ff), ((j + W * ui) * R + um) * 32 + un * 2, (half_t)v0, (half_t)v1);
    }
    stage_ff(l);
    workgroup_barrier();                                                  // 11
    prepare(l, 1, 10);
    {   // the other set is for the next launch
      const size_t n16 = (size_t)dirty * a.layers * (Rg::size * D) / 16, all = (size_t)(G * W) * (kWaves * 64);
      const u32x4 s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
      for (size_t i = (size_t)(grp * W + j) * (kWaves * 64) + xt + l * all; i < n16; i += a.layers * all)
        reinterpret_cast<u32x4*>(a.exchange + (size_t)(1 - parity) * a.set_bytes)[i] = s4;
    }
    pin();
    workgroup_barrier();                                                  // 12
    residual(l, Rg::u3);
  }
  if (j == 0) {   // the rows for the vocabulary product
    const bool publish = VOC && now()->V > 0;
    if constexpr (PRE) gather_norm(a.layers - 1, Rg::u3, a.lnfg, a.lnfb, a.x_out, a.hidden, publish);
    else gather_norm(a.layers - 1, Rg::u3, vec[(a.layers - 1) & 1][4], vec[(a.layers - 1) & 1][5], nullptr, a.hidden, publish);
  }
  ex.report(a.state, a.error);
}

}  // namespace

// How M rows are dealt out.  Short histories, whole translations of 75 steps in ms, groups of 4 / 8 rows, each in a process of its own (two machines
// within 0.5 %; beam 1 and 4 or 5): 12 rows 7.36 / 7.58, 13 rows 7.85 / 7.67, 16 rows 8.2 / 7.9, 20 rows 8.3 / 7.95, 24 rows 8.35 / 8.2, 25 rows 8.36 /
// 8.45 and 8.53 / 8.55, 28 rows 8.4 / 8.85, 30 rows 8.49 / 8.69 and 8.63 / 8.84, 32 rows 8.6 / 9.0: a fourth die that reads weights costs
// more than the longer chain of 8 rows; groups of 4 need it from 13 rows on, groups of 8 from 25 on, where the shorter chain is ahead again.
// (Where the weights lie in memory weighs as much: behind a dozen models in one process groups of 8 took 7.9 to 8.9 ms at 25 to
// 32 rows, those of 4 8.4 to 8.7.)  More than 32 rows are more than eight groups of 4.
// Long ones: over as many dies as there are sentences for, since a die reads its rows' histories at its own rate
// (one row per sentence, us a step at positions 240 / 1008: 16 pre-LN rows on two dies 201 / 361, on eight 170 / 256; 4 rows of a post-LN model
// on one 100 / 139, on four 97 / 124).
struct DieChoice { int R, rows, groups; };
static DieChoice choose_die(int M, int beam, int len) {
  DieChoice c = {M <= 12 || (M > 24 && M <= 32) ? 4 : M <= 64 ? 8 : 16, 0, 0};
  if (len > 128) {
    const int each = (M + kDies - 1) / kDies, whole = (each + beam - 1) / beam * beam;
    c.rows = whole <= 16 ? whole : each;
    c.R = c.rows <= 4 ? 4 : c.rows <= 8 ? 8 : 16;
  } else {
    const int n = (M + c.R - 1) / c.R;
    c.rows = (M + n - 1) / n;
  }
  c.groups = (M + c.rows - 1) / c.rows;
  return c;
}

static const void* die_kernel_of(int R, bool pre) {
  return R == 4 ? (pre ? (const void*)decoder_die_kernel<4, true> : (const void*)decoder_die_kernel<4, false>)
       : R == 8 ? (pre ? (const void*)decoder_die_kernel<8, true> : (const void*)decoder_die_kernel<8, false>)
                : (pre ? (const void*)decoder_die_kernel<16, true> : (const void*)decoder_die_kernel<16, false>);
}

// Against the kernels of kernels_stack.hip (the one of its two that is ahead), whole steps in us, V = 16 000:
//   positions                  16-60      60-112     112-200    200-280    280-400    400-560    560-940
//   post-LN, 4 rows, beam 4    80 / 90    81 / 91    84 / 94    89 / 98   101 / 106  105 / 111  118 / 124
//   32 rows, beam 4            99 / 102  100 / 103  102 / 106  107 / 110  118 / 118  122 / 123  133 / 138
//   64 rows, beam 4           107 / 105  110 / 106  122 / 115  129 / 122  137 / 132  152 / 151  196 / 191
//   128 rows, beam 4          124 / 137  139 / 141  148 / 148  173 / 161  206 / 185  as the others from 400 on
//   128 rows, one per sentence 129 / 140 148 / 158  180 / 182  212 / 210  240 / 242  281 / 284  364 / 365
//   pre-LN, 12 layers, 16 rows 125 / 120 132 / 122  145 / 127  152 / 133  as the others from 300 on
//   pre-LN, 32 rows           145 / 124  149 / 129  155 / 139  169 / 157
//   pre-LN, 64 rows           159 / 136  169 / 151  196 / 180  as the others from 160 on
//   pre-LN, 128 rows          192 / 185  as the others from 56 on
// The lines stand where earlier forms of the kernels crossed; products of paired k-steps have brought groups of 8 rows (pre-LN and 64 rows) and keys through
// LDS groups of 32 (128 rows) past this one since, by what the table says.  A source key counts as half of one of the history (128 rows,
// sources of 500 and 2000: 232 463, 229 446, earlier forms).
bool die_supported(int arch, int M, int d, int beam, int pos, int src) {
  if (d != 512 || M < 1 || M > 16 * kDies) return false;
  const int most = arch == 1 ? (M <= 32 ? 300 : M <= 64 ? 160 : 56) : M > 64 && beam > 1 ? 400 : 1 << 30;
  return pos + src / 2 <= most && resident(die_kernel_of(choose_die(M, beam, pos).R, arch == 1), kDieThreads);
}

// Groups that leave dies over, whose registers hold the vocabulary: eight blocks of 32 columns a workgroup.  Whole steps in us, a product of its own / here, V = 32 000,
// sources of 30 tokens:
//   positions                  5-25           25-50          50-75          75-110         110-200        200-300
//    4 rows, beam 4         82.1 / 79.4    81.1 / 79.2    81.7 / 79.7    82.9 / 80.8    85.9 / 83.8    92.5 / 90.3
//   12 rows, beam 4         85.6 / 84.0    85.7 / 84.0    86.2 / 84.6    86.8 / 85.2    89.8 / 88.0    96.7 / 95.4
//   24 rows, beam 4         93.4 / 90.5    93.7 / 91.1    95.4 / 92.4    97.6 / 94.6   102.6 / 101.5  109.6 / 109.4
//   24 rows, one per sentence 92.3 / 89.9  94.0 / 91.8    96.4 / 94.6    99.4 / 97.7
// (1 row 75.7 / 74.1.)  Past position 128, where rows go to as many dies as there are sentences, 28 and 32 rows of beams 7 and 8 are four groups as well (positions
// 132-160, 160-200, 200-250: 119 / 117, 121 / 117, 122 / 118; 123 / 121, 128 / 123, 129 / 125).  Pre-LN, 12 layers, up to position 110: 4 rows 116 / 114 ...
// 123 / 121, 12 rows 129 / 128 ... 136 / 135, 24 rows 139 / 138 ... 150 / 149; level behind 128.
// More than four groups: the dies left over would hold 24 576, 16 384 and 8192 columns.  Seven (25 to 28 rows) are behind with V = 8000, post-LN 91.9 / 92.9,
// 93.1 / 93.8, pre-LN 136.9 / 138.1, 143.3 / 144.6: one die has the whole product then.  Five and six, which there are past position 128 only,
// would be 1 to 1.5 us of 90 to 98 ahead; the line does not tell them apart.
bool die_takes_vocabulary(int arch, int M, int layers, int beam, int pos, int V) {
  const DieChoice c = choose_die(M, beam, pos);
  const int places = layers * (arch == 1 ? Region<true>::size : Region<false>::size) / 2;   // rows of d float16 that the exchange region of one row has room for
  return M <= min(places - 1, kVocabularyMax) && c.R <= kVocabularyRows && c.groups <= kDies / 2 && (V + 31) / 32 <= kWaves * (kDies - c.groups) * kDieGroup;
}

size_t die_exchange_bytes(int arch, int M, int d, int layers) {
  // groups of 4 rows: at most M and 8 of them; of 8 and 16: more than half full, and the 8-row groups of kernels_stack.hip
  // one row more: what the vocabulary product reads
  const int rows = min(16 * kDies, max(4 * min(kDies, M), 2 * M + 16)) + 1;
  return d == 512 ? (size_t)rows * layers * (arch == 1 ? Region<true>::size : Region<false>::size) * d : 0;
}

hipError_t launch_decoder_die(int arch, const StackArgs& args, int pos, hipStream_t s) {
  StackArgs a = args;
  const DieChoice c = choose_die(a.M, a.beam, pos);
  a.groups = c.groups;
  a.rows_per_group = c.rows;
  void* kargs[] = {&a};
  return hipLaunchKernel(die_kernel_of(c.R, arch == 1), dim3(kDies * kDieGroup), dim3(kDieThreads), kargs, 0, s);
}

hipError_t die_placement(unsigned* scratch, bool* dies, hipStream_t s) {
  unsigned id[kDies * kDieGroup] = {};
  die_of_workgroup_kernel<<<kDies * kDieGroup, kDieThreads, 0, s>>>(scratch);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(id, scratch, sizeof(id), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  *dies = e == hipSuccess;
  for (int b = 0; b < kDies * kDieGroup; b += kDies) {
    unsigned found = 0;
    for (int i = 0; i < kDies; ++i) found |= 1u << (id[b + i] & 15);
    if (found != (1u << kDies) - 1) *dies = false;
  }
  return e;
}

}  // namespace lsq
