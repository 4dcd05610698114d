// All decoder layers of one step in ONE launch, for few rows (float16, heads of 64, FFN of 4d).
//
// A step of few rows is a chain of products and attentions each of which is over in well under a microsecond of work;
// as launches of their own they cost 4..7 us each (kernel boundary 1.7 us, then input rows, weights and reduction one
// after the other).  Here the chain runs inside one resident grid: every workgroup owns a slice of the columns of every
// product, keeps its weights coming while it waits, and hands its results to the others through memory without a
// grid-wide barrier.
//
// Exchange.  Every intermediate (one region per row, layer and stage) is written exactly once per launch with agent-
// scope stores and read with agent-scope loads that repeat until no 32-bit word of the value is the sentinel 0xFFFFFFFF:
// the data is its own flag.  A written word never equals the sentinel (publish_word).  The regions exist twice; launch n
// uses set n % 2, which holds nothing but sentinels when it starts, and refills the other set for launch n + 1.
// Measured on this chip, 128 workgroups that all write a slice and read all of 16 KB: 1.2 us per exchange, against
// 2.3 us for a grid barrier followed by cached reads, and 1.7 us + load latency for a kernel boundary.
//
// Rows.  A group of W workgroups takes at most 8 rows through all layers; rows are independent between a step's start
// and end, so up to 256 / W groups work next to each other on rows of their own.  Workgroup j of every group sits on
// the same XCD (blockIdx % 8), so that the groups share the weights they stream through that XCD's L2.
//
// All workgroups must be resident at once: the launcher checks the occupancy, and every wait is bounded (kSpinLimit
// polls, then the error flag is set, nothing is waited for any more, and this launch and those queued behind it run to their
// end).
#include <cstdlib>

#include "stack_attend.h"

namespace lsq {

namespace {

constexpr int kRows = 8;               // rows of a group
constexpr int kMinRows = 4;            // a writer's piece is at least as large as for these: several writers in one line slow each other down

// DK: d / 256.  X: workgroups of a group per 16 columns of d (W = d / 16 * X): the products with d columns take 16 / X
// columns per workgroup, those with 3d and 4d columns ceil(3 / X) and 4 / X units of 16.  PRE: pre-LN, no cross-attention.
//
// Layout of the exchanged values: what one workgroup writes for all rows of its group is contiguous ([writer][row][its
// columns]); row-major regions, where 4..16 writers share every 128-byte line, take 0.3..0.7 us longer per exchange.
template <int DK, int X, bool PRE>
__global__ void __launch_bounds__(kThreads) decoder_stack_kernel(const StackArgs a) {
  constexpr int D = 256 * DK, H = D / 64, W = D / 16 * X, NT = 16 / X;
  constexpr int NU = 4 / X, UQ = X == 2 ? 3 : (3 + X - 1) / X;   // X = 2: three units of 8 columns of q, k, v
  constexpr int QT = NT < 8 ? 8 : NT;                          // query columns of the cross-attention per workgroup
  constexpr int TEAMS = X == 1 ? 2 : 1, NSH = kWaves / TEAMS;   // wavefronts that share a (row, head) pair
  using Rg = Region<PRE>;
  constexpr int NV = (D + 511) / 512;
  constexpr int ES = PRE ? 2 : 4;                              // bytes of a residual sum
  constexpr int CH = (kRows * D * ES / 16 + kThreads - 1) / kThreads;   // 16-byte pieces of all rows' sums per thread
  using sum_t = std::conditional_t<PRE, half_t, float>;

  __shared__ __attribute__((aligned(16))) half_t xs[kRows][D + 8];    // normalised rows
  __shared__ __attribute__((aligned(16))) sum_t us[kRows][D + 16 / ES];   // residual sums (pre-LN: the residual stream)
  __shared__ __attribute__((aligned(16))) float part[kWaves][NU > UQ ? NU : UQ][kRows][16];
  __shared__ __attribute__((aligned(16))) float part2[kWaves][kRows][16];
  __shared__ __attribute__((aligned(16))) Shares shares;
  __shared__ unsigned first_key[kWaves][kTrip][8];   // of the first trip, per lane group: places in the cache, the same in all layers

  int tid = threadIdx.x, lane = tid & 63;
  int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, bid = blockIdx.x;
  int grp = (bid >> 3) % G, j = (bid >> 3) / G * 8 + (bid & 7);
  int r0 = grp * a.rows_per_group, rows = min(a.rows_per_group, a.M - r0);
  const int seq = a.state[0], parity = seq & 1, dirty = a.state[2 - parity];
  int pos = *a.tpos;

  Exchange ex;
  ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange + (size_t)parity * a.set_bytes, (short)0, (int)a.set_bytes, 0x00027000);
  ex.polls = seq < 0 ? 1 : kSpinLimit;
  const int row_bytes = a.layers * Rg::size * D;
  const int rp = max(a.rows_per_group, kMinRows);   // rows a writer's piece has room for
  auto at = [&](int l, int region) { return (grp * row_bytes + (l * Rg::size + region) * D) * rp; };

  // ---- matrix fragments: lane (n = lane & 15, kc = lane >> 4) of a 32-wide k-step holds W[col + n][32 s + 8 kc ..]
  // The 16 x 16 products have room for twice the rows of a group: rows 0..7 of the one operand hold k-step 2 i, rows 8..15 k-step 2 i + 1 of the
  // same rows, and of the columns' side the matrices that have only 8 columns here do the same (PAIR).  Of the product the
  // quadrants in which both are the same k-step are what is wanted (fold): half the requests for exchanged values, which a wavefront
  // waits for, and for those matrices; a CU takes 16 clocks for any request, whether its lanes ask for the same lines or not.  Products that add
  // one k-step to the next move the odd ones' columns over instead (multiply_pairs, as fast: 10.75 / 10.75 ms, 9.23 / 9.16).  Whole translations
  // in ms with this and the sums of sum_of: d = 1024, 4 rows 10.6 -> 10.1, 8 rows 14.2 -> 13.2; d = 768 pre-LN, 8 rows 10.2 -> 9.8, 32 rows 29.3 -> 28.8.
  int fm = lane & 7, kc = lane >> 4, odd = lane >> 3 & 1;
  constexpr bool PAIR = NT == 8, PAIRQ = QT == 8;
  constexpr int DKP = (DK + 1) / 2;
  auto frag_lane = [&](int nt) { return (unsigned)(kc >> 1) * 1024 + ((lane & (nt - 1)) + 32 * (kc & 1)) * 16; };
  unsigned lane16 = frag_lane(16), lane_nt = frag_lane(NT), lane_qt = frag_lane(QT);
  auto frag_col = [&](const half_t* Wp, int K, int col) {   // its first k-step, in bytes
    return reinterpret_cast<const char*>(Wp) + (size_t)(col >> 5) * (K / 16) * 1024 + (col & 31) * 16;
  };
  half8_t wq[UQ][PAIR ? DKP : DK], wo[PAIR ? DKP : DK], wc[PRE ? 1 : PAIRQ ? DKP : DK], we[PRE ? 1 : PAIR ? DKP : DK], w1[NU][DK], w2[PAIR ? 2 * DK : 4 * DK];
  auto load_units = [&](auto& w, const half_t* Wp, int total) {
    constexpr int N = sizeof(w) / sizeof(w[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const char* p = frag_col(Wp, D, min(j + W * i, total - 1) * 16) + wave * (DK * 2048);
#pragma unroll
      for (int s = 0; s < DK; ++s) w[i][s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16);
    }
  };
  // `steps` k-steps of this wavefront; in pairs: of an odd number the last one again
  auto load_steps = [&](auto& w, const char* p, unsigned lo, auto steps, auto paired) {
    constexpr int N = decltype(steps)::value;
    if constexpr (decltype(paired)::value) {
#pragma unroll
      for (int s = 0; s < (N + 1) / 2; ++s) w[s] = *reinterpret_cast<const half8_t*>(p + s * 4096 + (2 * s + 1 < N ? lo + odd * 2048 : lo));
    } else {
#pragma unroll
      for (int s = 0; s < N; ++s) w[s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lo);
    }
  };
  using k1 = std::integral_constant<int, DK>;
  using k4 = std::integral_constant<int, 4 * DK>;
  auto load_cols = [&](auto& w, const half_t* Wp, auto steps, auto columns) {   // columns of d (the last ones again where there are none left)
    constexpr int S = decltype(steps)::value, C = decltype(columns)::value;
    load_steps(w, frag_col(Wp, S * 256, min(j * C, D - C)) + wave * (S * 2048), C == QT ? lane_qt : lane_nt, steps, std::bool_constant<C == 8>{});
  };
  using cn = std::integral_constant<int, NT>;
  using cq = std::integral_constant<int, QT>;
  auto load_qkv = [&](auto& w, const half_t* Wp) {
    if constexpr (PAIR) {
#pragma unroll
      for (int i = 0; i < 3; ++i) load_steps(w[i], frag_col(Wp, D, (j + W * i) * 8) + wave * (DK * 2048), lane_nt, k1{}, std::true_type{});
    } else {
      load_units(w, Wp, 3 * (D / 16));
    }
  };
  // two biases, unconverted: a conversion here would wait for everything requested before them
  auto bias_pair = [](const half_t* b, unsigned col) { return *reinterpret_cast<const half2_t*>(reinterpret_cast<const char*>(b) + col * 2u); };
  auto pin = [] { asm volatile("" ::: "memory"); };   // requests stay where they are written
  auto layer_w = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(global(p)) + (size_t)l * now()->packed_stride); };
  auto layer_p = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(global(p)) + (size_t)l * now()->plain_stride); };

  // ---- rows: all threads bring the residual sums of all rows into us, then wavefront m normalises row m into xs
  int piece_row[CH], piece_col[CH], piece_at[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int p = min(i * kThreads + tid, rows * (D * ES / 16) - 1);   // 16 bytes each, a writer's one after the other
    const int w = p / (rows * (NT * ES / 16)), in = p - w * (rows * (NT * ES / 16));
    piece_row[i] = in / (NT * ES / 16);
    piece_col[i] = w * NT + in % (NT * ES / 16) * (16 / ES);
    piece_at[i] = w * rp * (NT * ES) + in * 16;
  }
  auto normalise = [&](const half8_t (&g8)[NV], const half8_t (&b8)[NV], half_t* out_x, half_t* out_y) {
    float v[NV][8], gv[NV][8], bv[NV][8], o[NV][8];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      Vec8<sum_t>::load(&us[wave][min((q * 64 + lane) * 8, D - 8)], v[q]);
      Vec8<half_t>::unpack(g8[q], gv[q]);
      Vec8<half_t>::unpack(b8[q], bv[q]);
    }
    if (PRE && out_x) {
#pragma unroll
      for (int q = 0; q < NV; ++q)
        if ((q * 64 + lane) * 8 < D) Vec8<half_t>::store(out_x + (size_t)(r0 + wave) * D + (q * 64 + lane) * 8, v[q]);
    }
    // as layernorm_row (lsq_internal.h): mean, then centred variance
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((q * 64 + lane) * 8 < D) sum += v[q][i];
    const float mean = wave_sum(sum) * (1.0f / D);
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[q][i] -= mean;
        if ((q * 64 + lane) * 8 < D) sq += v[q][i] * v[q][i];
      }
    // 1 / sqrt by one Newton step: worst 1.53, mean 0.30 units in the last place against 64 bits (division by the root: 1.96, 0.38)
    const float var = wave_sum(sq) * (1.0f / D) + a.eps, r = __builtin_amdgcn_rsqf(var);
    const float rstd = r * (1.5f - 0.5f * var * r * r);
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i) o[q][i] = gv[q][i] * (v[q][i] * rstd) + bv[q][i];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int c = (q * 64 + lane) * 8;
      if (c < D) {
        Vec8<half_t>::store(&xs[wave][c], o[q]);
        if (out_y) Vec8<half_t>::store(out_y + (size_t)(r0 + wave) * D + c, o[q]);
      }
    }
  };
  auto load_gain = [&](half8_t (&g8)[NV], half8_t (&b8)[NV], const half_t* g, const half_t* b) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const unsigned c = min((q * 64 + lane) * 8, D - 8) * 2;   // bytes
      g8[q] = *reinterpret_cast<const half8_t*>(reinterpret_cast<const char*>(g) + c);
      b8[q] = *reinterpret_cast<const half8_t*>(reinterpret_cast<const char*>(b) + c);
    }
  };
  auto gather_norm = [&](int l, int region, const half_t* g, const half_t* b, half_t* out_x, half_t* out_y) {
    half8_t g8[NV], b8[NV];
    load_gain(g8, b8, g, b);
    u32x4 raw[CH];
    const int base = at(l, region);
    ex.wait<kLead>([&](int) { return base; }, [&](int i) { return piece_at[i]; }, raw);
#pragma unroll
    for (int i = 0; i < CH; ++i) *reinterpret_cast<u32x4*>(&us[piece_row[i]][piece_col[i]]) = raw[i];
    __syncthreads();
    if (wave < rows) normalise(g8, b8, out_x, out_y);
    __syncthreads();
  };

  // ---- products: wavefront w multiplies k in [w K/8, (w+1) K/8); acc: D[n][m], lane (m = lane & 15, n = 4 (lane >> 4) ..)
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  auto multiply_units = [&](const auto& w) {   // input rows from xs, 16-column units
    constexpr int N = sizeof(w) / sizeof(w[0]);
    floatx4 acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = zero4;
#pragma unroll
    for (int s = 0; s < DK; ++s) {
      const half8_t x8 = *reinterpret_cast<const half8_t*>(&xs[fm][(wave * DK + s) * 32 + kc * 8]);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i][s], x8, acc[i], 0, 0, 0);
    }
    if ((lane & 15) < kRows) {
#pragma unroll
      for (int i = 0; i < N; ++i) *reinterpret_cast<floatx4*>(&part[wave][i][lane & 15][kc * 4]) = acc[i];
    }
  };
  auto other_half = [](const half8_t& v) {   // of lane ^ 8
    u32x4 r = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned x = r[i];
      r[i] = __builtin_bit_cast(unsigned, lane_xor<8>(__builtin_bit_cast(float, x)));
    }
    return __builtin_bit_cast(half8_t, r);
  };
  // both halves of k of rows 0..7, in the lanes of the even one: a: of both, or of the even k-steps only, b: of the odd ones
  auto fold = [&](const floatx4& a, const floatx4& b, auto paired) {
    floatx4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (decltype(paired)::value) {
        float lower, upper;
        lane_pair<32>(a[i], lower, upper);
        v[i] = lower + lane_xor<8>(upper);
      } else {
        v[i] = a[i] + lane_xor<8>(b[i]);
      }
    }
    return v;
  };
  auto multiply_pairs = [&](const auto& w) {   // input rows from xs, units of 8 columns; k-step after k-step, as in multiply_units
    constexpr int N = sizeof(w) / sizeof(w[0]);
    floatx4 acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = zero4;
#pragma unroll
    for (int s = 0; s < DK; ++s) {   // the odd ones' columns lie in lanes 8..15
      const half8_t x8 = *reinterpret_cast<const half8_t*>(&xs[fm][(wave * DK + s) * 32 + kc * 8]);
#pragma unroll
      for (int i = 0; i < N; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(s & 1 ? other_half(w[i][s / 2]) : w[i][s / 2], x8, acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((lane & 15) < kRows && kc < 2) *reinterpret_cast<floatx4*>(&part[wave][i][lane & 15][kc * 4]) = acc[i];
  };
  auto sum_of = [&](const float (&p)[kRows][16], int stride, int m, int n, float& v0, float& v1) {   // columns n, n + 1, over the wavefronts in order
    floatx2 t[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t[w] = *reinterpret_cast<const floatx2*>(&p[m][n] + w * stride);
    // all of them requested before the first is added: left to itself the compiler takes a trip to LDS for each
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]));
    v0 = t[0][0]; v1 = t[0][1];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) { v0 += t[w][0]; v1 += t[w][1]; }
  };
  auto total_of = [&](int i, int m, int n, float& v0, float& v1) { sum_of(part[0][i], sizeof(part[0]) / 4, m, n, v0, v1); };

  // ---- attention of one (row, head) pair per team of NSH wavefronts (stack_attend.h).  All of them share the keys, however few there are:
  // which has which is part of the order of the sums.  (As many as have 32 keys each: Transformer-big, 1 sentence 10.19 -> 10.01 ms, decoder-only,
  // d = 768, 1 row 8.92 -> 8.75, and other tokens now and then.)
  const int team = wave / NSH, ash = wave % NSH;
  int gk = lane >> 3, c8 = (lane & 7) * 8;
  const int pair = j + W * team, am = min(pair / H, rows - 1), ah = pair % H;
  const int arow = r0 + am, sent = arow / a.beam;
  const bool table = !PRE && a.anc != nullptr;
  const int32_t* slots = table ? a.anc + (size_t)arow * a.anc_ld : nullptr;
  auto slot_of = [&](int p) { return table ? min(max(slots[p], 0), a.beam - 1) : 0; };   // of the sentence's rows
  auto key_offset = [&](int p) { return (unsigned)((slot_of(p) * a.T + p) * D) * 2u; };
  const bool attends = pair < rows * H;
#pragma unroll
  for (int u = 0; u < kTrip; ++u) first_key[wave][u][gk] = key_offset(max(min(ash + (gk + u * 8) * NSH, pos - 1), 0));
  int src_off = 0, src_len = 0;
  if constexpr (!PRE) { src_off = a.src_off[sent]; src_len = a.src_len[sent]; }
  if (tid < kWaves) shares.left[tid] = 0;   // the first rows' barrier is ahead
  int attentions = 0;

  // Wavefronts that have nothing to look at go on to wait for the context.
  auto attend = [&](int l, auto of_self, const half_t* Kb, const half_t* Vb, int nkeys) {
    constexpr bool self = decltype(of_self)::value;
    ++attentions;
    if (!attends) return;
    half8_t kn[kTrip], vn[kTrip];
    const size_t own = self ? (size_t)(table ? sent * a.beam : arow) * a.T * D : 0;
    const char* Kh = reinterpret_cast<const char*>(Kb + own + ah * 64);
    const char* Vh = reinterpret_cast<const char*>(Vb + own + ah * 64);
    auto request = [&](int jb, auto first, auto keys) {   // past the last key: that one again
#pragma unroll
      for (int u = 0; u < decltype(keys)::value; ++u) {
        const int p = max(min(jb + (gk + u * 8) * NSH, nkeys - 1), 0);
        const unsigned o = (!self ? (unsigned)(p * (2 * D)) * 2u : first ? first_key[wave][u][gk] : key_offset(p)) + c8 * 2;
        kn[u] = *reinterpret_cast<const half8_t*>(Kh + o);
        vn[u] = *reinterpret_cast<const half8_t*>(Vh + o);
      }
    };
    // Eight wavefronts have 64 keys with one per lane group and 128 with two, and request no more: four each time cost 0.5 ms of 10.8 (Transformer-big,
    // 1 sentence).  Four wavefronts (X = 1) have 32 and 64: three forms of the trip spill there, and gained nothing.
    using c1 = std::integral_constant<int, 1>;
    using c2 = std::integral_constant<int, 2>;
    using c4 = std::integral_constant<int, kTrip>;
    const bool one = NSH == 8 && nkeys <= 8 * NSH, two = NSH == 8 && nkeys <= 16 * NSH;
    if (one) request(ash, std::true_type{}, c1{});
    else if (two) request(ash, std::true_type{}, c2{});
    else request(ash, std::true_type{}, c4{});
    pin();
    half8_t q, knew = {}, vnew = {};
    if constexpr (self) {
      u32x4 raw[3];
      constexpr int UC = PAIR ? 8 : 16;   // columns of a unit
      const int base = at(l, Rg::qkv) + (ah * (64 / UC) * rp + am) * (UC * 2);
      ex.wait<kLead>([&](int i) { return base + i * (D * 2) * rp; }, [&](int) { return c8 / UC * rp * (UC * 2) + c8 % UC * 2; }, raw);
      q = __builtin_bit_cast(half8_t, raw[0]); knew = __builtin_bit_cast(half8_t, raw[1]); vnew = __builtin_bit_cast(half8_t, raw[2]);
    } else {
      u32x4 raw[1];
      const int base = at(l, Rg::q2) + (ah * 64 / QT * rp + am) * (QT * 2);
      ex.wait<kLead>([&](int) { return base; }, [&](int) { return c8 / QT * rp * (QT * 2) + c8 % QT * 2; }, raw);
      q = __builtin_bit_cast(half8_t, raw[0]);
    }
    Attention t;
    auto live = [&](int jb) { return [&, jb](int u) { return jb + (gk + u * 8) * NSH < nkeys; }; };
    constexpr int span = kTripKeys * NSH;
    if (one) {
      t.first<self, 1>(q, kn, vn, knew, nkeys == 0, live(ash), [] {});
    } else if (two) {
      t.first<self, 2>(q, kn, vn, knew, false, live(ash), [] {});
    } else {
      t.first<self>(q, kn, vn, knew, nkeys == 0, live(ash), [&] { if (nkeys > span) request(ash + span, std::false_type{}, c4{}); });
      for (int jb = ash + span; jb < nkeys; jb += span)   // the same trips in every lane of the wavefront
        t.more(q, kn, vn, live(jb), [&] { if (jb + span < nkeys) request(jb + span, std::false_type{}, c4{}); });
    }
    if (self && ash == NSH - 1) t.add(vnew, gk == 0);
    t.sum<false>();
    shares.leave<false>(wave, lane, t);
    if (ash > 0) return shares.tell(wave, attentions);
    const int c = (lane & 31) * 2;
    const half2_t v = shares.collect<NSH>(team * NSH, NSH, attentions, lane, c);
    if (lane < 32) ex.put2(at(l, self ? Rg::ctx : Rg::ctx2) + am * (D * 2) + ah * 128, c * 2, v[0], v[1]);
  };

  // ---- a product whose input rows (N k-steps of 32 per wavefront) come straight from the exchange (row-major or units of
  // 16 columns), this workgroup's NT columns; then the residual: region_out <- x + (in . W + bias).  `request`: what is
  // wanted next.
  auto project = [&](const auto& w, auto steps, int l, int region_in, bool units, int region_out, const half_t* bias, auto request) {
    constexpr int N = decltype(steps)::value, NB = (N + 1) / 2;
    const int om = tid / (NT / 2), on = tid % (NT / 2) * 2;
    half2_t bi = {0, 0};
    if (om < rows) bi = bias_pair(bias, j * NT + on);
    u32x4 raw[NB];
    const int step = units ? 64 * rp : 64, base = at(l, region_in) + wave * N * step;
    const int lo = units ? ((kc >> 1) * rp + min(fm, rows - 1)) * 32 + (kc & 1) * 16 : min(fm, rows - 1) * (D * 2) + kc * 16;
    const int lo2 = lo + odd * step;
    ex.wait<kLead>([&](int i) { return base + 2 * i * step; }, [&](int i) { return 2 * i + 1 < N ? lo2 : lo; }, raw);
    floatx4 acc[2] = {zero4, zero4};
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      half8_t x8 = __builtin_bit_cast(half8_t, raw[i]);
      if constexpr (PAIR) {
        if (2 * i + 1 >= N && odd) x8 = half8_t{};
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i], x8, acc[0], 0, 0, 0);
      } else {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[2 * i], x8, acc[0], 0, 0, 0);
        if (2 * i + 1 < N) acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[min(2 * i + 1, N - 1)], x8, acc[1], 0, 0, 0);
      }
    }
    const floatx4 sum = fold(acc[0], acc[1], std::bool_constant<PAIR>{});
    if ((lane & 15) < kRows && kc * 4 < NT) *reinterpret_cast<floatx4*>(&part2[wave][lane & 15][kc * 4]) = sum;
    request();
    pin();
    half2_t x = {0, 0};
    if (om < rows) x = *reinterpret_cast<const half2_t*>(PRE ? reinterpret_cast<const half_t*>(&us[om][j * NT + on]) : &xs[om][j * NT + on]);
    __syncthreads();
    if (om < rows) {
      float v0, v1;
      sum_of(part2[0], kRows * 16, om, on, v0, v1);
      const int base_out = at(l, region_out) + j * rp * (NT * ES), o = om * (NT * ES) + on * ES;
      if constexpr (PRE) {
        ex.put2(base_out, o, (half_t)((float)x[0] + (v0 + (float)bi[0])), (half_t)((float)x[1] + (v1 + (float)bi[1])));
      } else {
        ex.put2(base_out, o, (float)x[0] + (v0 + (float)bi[0]), (float)x[1] + (v1 + (float)bi[1]));
      }
    }
  };

  // What is derived from a workgroup's place (row offsets, bounds, bases) is derived anew in every stage instead of waiting in scalar
  // registers: 32 to 59 of them were spilled into lanes.  Whole translations: d = 1024, 4 rows 11.21 -> 10.99 ms (75 steps); d = 768 pre-LN,
  // 8 rows 8.45 -> 8.18, 32 rows 10.61 -> 10.43 (104 steps).
  auto renew = [&] { asm volatile("" : "+s"(wave), "+s"(j), "+s"(grp), "+s"(r0), "+s"(rows), "+s"(pos)); };
  // The same for a thread's place, once a layer; twice where the cross-attention's registers come on top of four k-steps' in whole units.
  // Without it d = 1024 spills (32 rows 204 -> 174 us a step's layers); d = 512 gains 2 %, d = 768 would lose 1 to 2 % (8 rows 8.82 -> 8.92 ms, 32 rows
  // 9.55 -> 9.76; decoder-only, 32 rows 25.98 -> 26.25), and needs it for one number only.  No vector register is spilled this way.
  auto renew_lane = [&] {
    asm volatile("" : "+v"(tid), "+v"(lane), "+v"(fm), "+v"(kc), "+v"(odd), "+v"(lane16), "+v"(lane_nt), "+v"(lane_qt));
    asm volatile("" : "+v"(gk), "+v"(c8));
  };

  // ======== the layers.  Every matrix slice is requested at least one exchange before it is multiplied.
  load_qkv(wq, layer_w(now()->Wqkv, 0));
  for (int l = 0; l < a.layers; ++l) {
    if constexpr (DK != 3) renew_lane();
    else if constexpr (X == 1 && !PRE) asm volatile("" : "+v"(c8));
    renew();
    half_t* Kc = reinterpret_cast<half_t*>(global(now()->cache) + (size_t)(2 * l) * now()->cache_stride);
    half_t* Vc = reinterpret_cast<half_t*>(global(now()->cache) + (size_t)(2 * l + 1) * now()->cache_stride);
    // A. the layer's input rows; q, k, v
    const int qi = tid >> 6, qm = (tid >> 3) & 7, qn = (tid & 7) * 2;   // unit, row, pair of columns this thread finishes
    const half_t* bq3 = layer_p(now()->bqkv, l);
    half2_t qb = {0, 0};
    const int qu = PAIR ? 8 : 16, qcol = (j + W * qi) * qu + qn;   // columns of a unit
    const bool qlive = qi < UQ && qn < qu && qcol < 3 * D && qm < rows;
    if (qlive) qb = bias_pair(bq3, qcol);
    if (l == 0) {
      if (wave < rows) {
        const int r = r0 + wave;
        if constexpr (PRE) {
          half8_t g8[NV], b8[NV];
          load_gain(g8, b8, a.ln1g, a.ln1b);
          const half_t* e = a.E + (size_t)embedding_row(a.tokens[(size_t)r * (a.T + 1) + a.len[r]]) * D;
          embed_whole_row<half_t, D>(e, a.pe + (size_t)pos * D, us[wave], 1.0f, lane);
          normalise(g8, b8, nullptr, nullptr);   // reads what this wavefront wrote
        } else {
#pragma unroll
          for (int q = 0; q < NV; ++q)
            if ((q * 64 + lane) * 8 < D)
              *reinterpret_cast<half8_t*>(&xs[wave][(q * 64 + lane) * 8]) = *reinterpret_cast<const half8_t*>(a.x0 + (size_t)r * D + (q * 64 + lane) * 8);
        }
      }
      __syncthreads();
    } else {
      if constexpr (PRE) gather_norm(l - 1, Rg::u3, layer_p(now()->ln1g, l), layer_p(now()->ln1b, l), nullptr, nullptr);
      else gather_norm(l - 1, Rg::u3, layer_p(now()->ln3g, l - 1), layer_p(now()->ln3b, l - 1), nullptr, nullptr);
    }
    if constexpr (PAIR) multiply_pairs(wq);
    else multiply_units(wq);
    load_cols(wo, layer_w(now()->Wo, l), k1{}, cn{});
    if constexpr (PRE) load_units(w1, layer_w(now()->W1, l), 4 * (D / 16));
    else load_cols(wc, layer_w(now()->Wq, l), k1{}, cq{});
    pin();
    __syncthreads();
    if (qlive) {
      float v0, v1;
      total_of(qi, qm, qn, v0, v1);
      const half_t h0 = (half_t)(v0 + (float)qb[0]), h1 = (half_t)(v1 + (float)qb[1]);
      ex.put2(at(l, Rg::qkv) + j * rp * (qu * 2), (W * qi * rp + qm) * (qu * 2) + qn * 2, h0, h1);
      if (qcol >= D) {
        char* cache = reinterpret_cast<char*>((qcol < 2 * D ? Kc : Vc) + ((size_t)r0 * a.T + pos) * D);
        *reinterpret_cast<half2_t*>(cache + (unsigned)(qm * a.T * D + (qcol < 2 * D ? qcol - D : qcol - 2 * D)) * 2u) = half2_t{h0, h1};
      }
    }
    // B, C. self-attention, its output projection
    renew();
    attend(l, std::true_type{}, Kc, Vc, pos);
    renew();
    project(wo, k1{}, l, Rg::ctx, false, Rg::u1, layer_p(now()->bo, l), [&] {
      if constexpr (PRE) load_cols(w2, layer_w(now()->W2, l), k4{}, cn{});
      else load_cols(we, layer_w(now()->Woc, l), k1{}, cn{});
    });
    if constexpr (!PRE) {
      // D. LayerNorm, query product of the cross-attention
      const int pm = tid / (QT / 2), pn = tid % (QT / 2) * 2;
      const bool plive = pm < rows && j * QT < D;
      half2_t pb = {0, 0};
      if (plive) pb = bias_pair(layer_p(now()->bq, l), j * QT + pn);
      gather_norm(l, Rg::u1, layer_p(now()->ln1g, l), layer_p(now()->ln1b, l), nullptr, nullptr);
      if constexpr (PAIRQ) {
        multiply_pairs(reinterpret_cast<const half8_t (&)[1][PRE ? 1 : DKP]>(wc));
      } else {
        floatx4 acc = zero4;
#pragma unroll
        for (int s = 0; s < DK; ++s)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wc[PRE ? 0 : s], *reinterpret_cast<const half8_t*>(&xs[fm][(wave * DK + s) * 32 + kc * 8]), acc, 0, 0, 0);
        if ((lane & 15) < kRows) *reinterpret_cast<floatx4*>(&part[wave][0][lane & 15][kc * 4]) = acc;
      }
      load_units(w1, layer_w(now()->W1, l), 4 * (D / 16));
      pin();
      __syncthreads();
      if (plive) {
        float v0, v1;
        total_of(0, pm, pn, v0, v1);
        ex.put2(at(l, Rg::q2) + j * rp * (QT * 2), pm * (QT * 2) + pn * 2, (half_t)(v0 + (float)pb[0]), (half_t)(v1 + (float)pb[1]));
      }
      // E, F. cross-attention, its output projection
      const half_t* kvb = reinterpret_cast<const half_t*>(global(now()->cross) + (size_t)l * now()->cross_stride) + (size_t)src_off * 2 * D;
      renew();
      attend(l, std::false_type{}, kvb, kvb + D, src_len);
      project(we, k1{}, l, Rg::ctx2, false, Rg::u2, layer_p(now()->boc, l), [&] { load_cols(w2, layer_w(now()->W2, l), k4{}, cn{}); });
    }
    renew();
    if constexpr (DK == 4 && X == 1 && !PRE) renew_lane();
    // G. LayerNorm, first FFN product
    const int fcol = (j + W * qi) * 16 + qn;
    half2_t fb = {0, 0};
    if (qi < NU && qm < rows) fb = bias_pair(layer_p(now()->b1, l), fcol);
    gather_norm(l, PRE ? Rg::u1 : Rg::u2, layer_p(now()->ln2g, l), layer_p(now()->ln2b, l), nullptr, nullptr);
    multiply_units(w1);
    __syncthreads();
    if (qi < NU && qm < rows) {
      float v0, v1;
      total_of(qi, qm, qn, v0, v1);
      v0 += (float)fb[0]; v1 += (float)fb[1];
      if constexpr (PRE) { v0 = tanh_gelu(v0); v1 = tanh_gelu(v1); }
      else { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); }
      ex.put2(at(l, Rg::ff) + j * rp * 32, (W * qi * rp + qm) * 32 + qn * 2, (half_t)v0, (half_t)v1);
    }
    // H. second FFN product
    project(w2, k4{}, l, Rg::ff, true, Rg::u3, layer_p(now()->b2, l), [&] {
      if (l + 1 < a.layers) load_qkv(wq, layer_w(now()->Wqkv, l + 1));
    });
  }
  // ======== the rows for the vocabulary product; everything else ends here
  if (j == 0) {
    if constexpr (PRE) gather_norm(a.layers - 1, Rg::u3, a.lnfg, a.lnfb, a.x_out, a.hidden);
    else gather_norm(a.layers - 1, Rg::u3, layer_p(now()->ln3g, a.layers - 1), layer_p(now()->ln3b, a.layers - 1), nullptr, a.hidden);
  }
  {
    char* other = a.exchange + (size_t)(1 - parity) * a.set_bytes;
    const size_t n16 = (size_t)dirty * row_bytes / 16;
    const u32x4 s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
    for (size_t i = (size_t)bid * kThreads + tid; i < n16; i += (size_t)gridDim.x * kThreads) reinterpret_cast<u32x4*>(other)[i] = s4;
  }
  ex.report(a.state, a.error);
  if (tid == 0) {   // the last workgroup to get here: all have read the counters
    const int n = __hip_atomic_fetch_add(a.state + 4, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n == (int)gridDim.x - 1) {
      a.state[4] = 0;
      a.state[1 + parity] = G * rp;
      __hip_atomic_fetch_xor(a.state, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The same for more rows: a group takes up to 16 MB rows through all layers with W = d / 16 workgroups.
//
// What every workgroup has to read decides here, not the number of exchanges, so the work is cut differently:
//   * workgroup r of a group owns row r: it alone adds up the partial sums of the sublayers' projections, keeps the
//     residual row and publishes the normalised one (float16) -- one exchange more, but the 16 KB of partial sums of a row
//     are read once and not by everybody;
//   * products with d columns are split 4-fold over k (64 columns and a quarter of k per workgroup): each reads a quarter
//     of the input rows and leaves a float slab; the query product's slabs are added by the attention that needs them;
//   * a product with columns for every workgroup takes its input rows straight from the exchange, an eighth of k per wavefront; the split ones
//     stage their quarter in LDS.
// Exchange regions exist for two layers; a workgroup that publishes into layer l's resets what it wrote for layer l - 1
// at the same place (consumed by then: it could not have got here otherwise) and has waited for the acknowledgement
// before its next publication but one, on which everybody's way to layer l + 1 depends.  A launch starts with the slot
// after the one the last launch ended with, and cleans that one first.
template <bool PRE> struct RowsRegion {   // bytes per row / d
  static constexpr int xi = 0, qkv = 2, ctx = 8, os = 10, x1 = 26, ff = 28, fs = 36;
  static constexpr int qs = PRE ? 0 : 52, ctx2 = PRE ? 0 : 68, cs = PRE ? 0 : 70, x2 = PRE ? 0 : 86, size = PRE ? 52 : 88;
};

template <int DK, int MB, bool PRE>
__global__ void __launch_bounds__(kThreads) decoder_stack_rows_kernel(const StackArgs a) {
  constexpr int D = 256 * DK, H = D / 64, W = D / 16, R = 16 * MB, CG = D / 64;
  constexpr int TEAMS = R / 4, NSH = kWaves / TEAMS;
  constexpr int KS = 2 * DK;                        // k-steps of a quarter of k
  constexpr int CHQ = (MB * DK + 3) / 4;            // 16-byte pieces per thread of a quarter of R rows of d halves
  using Rg = RowsRegion<PRE>;
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

  // Staged quarters of input rows, and the second FFN product's sums over the wavefronts; the other products' sums.  Between a product and the
  // next, 8 KB of either are a wavefront's: its second trip of keys.
  constexpr int kKeyBytes = 2 * kTrip * 1024, kParts = kWaves * 4 * R * 16 * 4, kRoom = kParts > kWaves * kKeyBytes ? kParts : kWaves * kKeyBytes;
  using sums_t = float[kWaves][4][R][16];
  __shared__ __attribute__((aligned(16))) char st_room[kRoom];
  __shared__ __attribute__((aligned(16))) char part_room[kRoom];
  half_t (&st)[R][D / 4 + 8] = *reinterpret_cast<half_t (*)[R][D / 4 + 8]>(st_room);
  sums_t &part = *reinterpret_cast<sums_t*>(part_room), &part2 = *reinterpret_cast<sums_t*>(st_room);
  static_assert(sizeof(st) <= kRoom && sizeof(sums_t) <= kRoom, "");
  __shared__ __attribute__((aligned(16))) half_t xrow[D];                  // the residual of the row this workgroup owns
  __shared__ float stat[DK][2];
  __shared__ __attribute__((aligned(16))) Shares shares;
  __shared__ unsigned first_key[kWaves][2][kTrip][8];   // of the first two trips, per lane group: places in the cache, the same in all layers

  int tid = threadIdx.x, lane = tid & 63;
  int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, bid = blockIdx.x;
  int grp = (bid >> 3) % G, j = (bid >> 3) / G * 8 + (bid & 7);
  int cg = j >> 2, ks = j & 3;
  int rp = a.rows_per_group, r0 = grp * rp, rows = min(rp, a.M - r0);
  const int seq = a.state[0], dirty = a.state[1];
  int start = seq & 1, pos = *a.tpos;
  const bool owner = j < rows;

  Exchange ex;
  ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange, (short)0, (int)(2 * a.set_bytes), 0x00027000);
  ex.polls = seq < 0 ? 1 : kSpinLimit;
  const int group_bytes = Rg::size * D * rp;
  auto at = [&](int l, int region) { return ((start + l) & 1) * (int)a.set_bytes + grp * group_bytes + region * D * rp; };
  const u32x4 s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
  auto other = [&](int l) { return ((start + l) & 1) ? -(int)a.set_bytes : (int)a.set_bytes; };   // from layer l's slot to the other
  auto put4 = [&](int l, int base, int lo, float v0, float v1, float v2, float v3) {
    const u32x4 w = {publish_word(__builtin_bit_cast(unsigned, v0)), publish_word(__builtin_bit_cast(unsigned, v1)),
                     publish_word(__builtin_bit_cast(unsigned, v2)), publish_word(__builtin_bit_cast(unsigned, v3))};
    __builtin_amdgcn_raw_buffer_store_b128(w, ex.rsrc, lo, base, kAgent);
    __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, lo, base + other(l), kAgent);
  };
  auto put4h = [&](int l, int base, int lo, half_t h0, half_t h1, half_t h2, half_t h3) {
    const u32x2 w = {publish_word(__builtin_bit_cast(unsigned, half2_t{h0, h1})), publish_word(__builtin_bit_cast(unsigned, half2_t{h2, h3}))};
    __builtin_amdgcn_raw_buffer_store_b64(w, ex.rsrc, lo, base, kAgent);
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{kSentinel, kSentinel}, ex.rsrc, lo, base + other(l), kAgent);
  };

  auto put2h = [&](int l, int base, int lo, half_t h0, half_t h1) {
    ex.put2(base, lo, h0, h1);
    __builtin_amdgcn_raw_buffer_store_b32(kSentinel, ex.rsrc, lo, base + other(l), kAgent);
  };

  {   // the slot the last launch ended with: this group's part (needed from layer 1 on), and what no group of this launch has
    char* old = a.exchange + ((start + 1) & 1) * a.set_bytes;
    const int mine_end = min(dirty, (grp + 1) * group_bytes);
    for (int o = grp * group_bytes + (j * kThreads + tid) * 16; o < mine_end; o += W * kThreads * 16)
      __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, o, (int)(old - a.exchange), kAgent);
    for (int o = G * group_bytes + (bid * kThreads + tid) * 16; o < dirty; o += (int)gridDim.x * kThreads * 16)
      __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, o, (int)(old - a.exchange), kAgent);
  }

  // ---- matrix fragments (see decoder_stack_kernel)
  int fm = lane & 15, kc = lane >> 4;
  unsigned lane16 = (unsigned)(kc >> 1) * 1024 + (fm + 32 * (kc & 1)) * 16;
  auto frag = [&](const half_t* Wp, int K, int col, int kstep) {
    return reinterpret_cast<const char*>(Wp) + (size_t)(col >> 5) * (K / 16) * 1024 + (col & 31) * 16 + (size_t)kstep * 2048;
  };
  half8_t wq[3][DK], wo[KS], w1[4][DK], w2[4][DK];
  auto load_units = [&](auto& w, const half_t* Wp) {   // units j + W i of 16 columns, this wavefront's eighth of k
    constexpr int N = sizeof(w) / sizeof(w[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const char* p = frag(Wp, D, (j + W * i) * 16, wave * DK);
#pragma unroll
      for (int s = 0; s < DK; ++s) w[i][s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16);
    }
  };
  auto load_quarter = [&](auto& w, const half_t* Wp) {   // 16 columns (wave & 3) of this workgroup's 64, its quarter of k
    constexpr int N = sizeof(w) / sizeof(w[0]);
    const char* p = frag(Wp, D, cg * 64 + (wave & 3) * 16, ks * KS);
#pragma unroll
    for (int s = 0; s < N; ++s) w[s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16);
  };
  auto load_ffn2 = [&](auto& w, const half_t* Wp) {   // this workgroup's 64 columns, this wavefront's eighth of its quarter of 4d
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* p = frag(Wp, 4 * D, cg * 64 + i * 16, ks * (D / 32) + wave * DK);
#pragma unroll
      for (int s = 0; s < DK; ++s) w[i][s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16);
    }
  };
  auto pin = [] { asm volatile("" ::: "memory"); };

  auto layer_w = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(global(p)) + (size_t)l * now()->packed_stride); };
  auto layer_p = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(global(p)) + (size_t)l * now()->plain_stride); };
  auto half4_at = [](const half_t* b, unsigned col) { return *reinterpret_cast<const half4_t*>(reinterpret_cast<const char*>(b) + col * 2u); };

  // ---- the owner's part: residual row + partial sums of a projection -> normalised row.  Thread t has columns 4t .. 4t+3.
  unsigned oc = min(tid * 4, D - 4);
  const bool oact = tid * 4 < D;
  auto own_publish = [&](float (&v)[4], half4_t g4, half4_t b4, int l, int region_out, half_t* out_y) {
    // mean and centred sum of squares of each wavefront's 256 values, then of the row
    float sm = (v[0] + v[1]) + (v[2] + v[3]);
    sm = wave_sum(sm) * (1.0f / 256);
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) q += (v[i] - sm) * (v[i] - sm);
    q = wave_sum(q);
    if (lane == 0 && wave < DK) { stat[wave][0] = sm; stat[wave][1] = q; }
    __syncthreads();
    float mean = 0.f, m2 = 0.f;
#pragma unroll
    for (int w = 0; w < DK; ++w) mean += stat[w][0];
    mean *= 1.0f / DK;
#pragma unroll
    for (int w = 0; w < DK; ++w) m2 += stat[w][1] + 256.0f * (stat[w][0] - mean) * (stat[w][0] - mean);
    const float var = m2 * (1.0f / D) + a.eps, rs = __builtin_amdgcn_rsqf(var), rstd = rs * (1.5f - 0.5f * var * rs * rs);
    if (oact) {
      half_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = (half_t)((float)g4[i] * ((v[i] - mean) * rstd) + (float)b4[i]);
      if (region_out >= 0) put4h(l, at(l, region_out) + j * (D * 2), oc * 2, h[0], h[1], h[2], h[3]);
      if (!PRE) *reinterpret_cast<half4_t*>(&xrow[oc]) = half4_t{h[0], h[1], h[2], h[3]};
      if (out_y) *reinterpret_cast<half4_t*>(out_y + (size_t)(r0 + j) * D + oc) = half4_t{h[0], h[1], h[2], h[3]};
    }
    __syncthreads();
  };
  auto own_norm = [&](int lin, int region_in, const half_t* bias, const half_t* g, const half_t* b, int l, int region_out,
                      half_t* out_x, half_t* out_y) {
    if (!owner) return;
    const half4_t bi = half4_at(bias, oc), g4 = half4_at(g, oc), b4 = half4_at(b, oc);
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (wave < DK) {
      u32x4 raw[4];
      const int base = at(lin, region_in) + j * 256;
      const int lo = (int)(oc >> 6) * (rp * 256) + (int)(oc & 63) * 4;
      ex.wait<kLead>([&](int i) { return base + i * (CG * 256) * rp; }, [&](int) { return lo; }, raw);
      const half4_t x4 = *reinterpret_cast<const half4_t*>(&xrow[oc]);
      const floatx4 f0 = __builtin_bit_cast(floatx4, raw[0]), f1 = __builtin_bit_cast(floatx4, raw[1]),
                    f2 = __builtin_bit_cast(floatx4, raw[2]), f3 = __builtin_bit_cast(floatx4, raw[3]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = (float)x4[i] + ((((f0[i] + f1[i]) + f2[i]) + f3[i]) + (float)bi[i]);
        if (PRE) v[i] = (float)(half_t)v[i];
      }
      if constexpr (PRE) {
        const half4_t h = {(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
        *reinterpret_cast<half4_t*>(&xrow[oc]) = h;
        if (out_x) *reinterpret_cast<half4_t*>(out_x + (size_t)(r0 + j) * D + oc) = h;
      }
    }
    own_publish(v, g4, b4, l, region_out, out_y);
  };

  // ---- a quarter of the input rows into LDS; all of a workgroup's accesses so far are acknowledged on the way
  auto stage_quarter = [&](int base) {
    u32x4 raw[CHQ];
    const int t = tid;
    constexpr int per_row = D / 32;   // rows the group does not have: its last one again
    ex.wait<kLead>([&](int) { return base + ks * (D / 2); },
            [&](int i) { const int p = i * kThreads + t; return min(p / per_row, rows - 1) * (D * 2) + p % per_row * 16; }, raw);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CHQ; ++i) {
      const int p = i * kThreads + t;
      if (p < R * per_row) *reinterpret_cast<u32x4*>(&st[p / per_row][p % per_row * 8]) = raw[i];
    }
    __syncthreads();
  };

  // ---- products.  An eighth of k per wavefront, so nobody else needs what a wavefront reads of the input rows: straight from the exchange
  // to the matrix cores (through LDS: two barriers and 128 KB of traffic more).  Whole translations in ms: d = 1024, 32 sentences
  // 25.96 -> 25.30, 8 sentences 18.3 -> 17.2; d = 512, 60 sentences 19.5 -> 18.7; d = 768 pre-LN, 64 rows 15.65 -> 14.87.
  // Accesses so far are acknowledged on the way, and the barrier between the sums and their readers is passed before anything that
  // depends on them is published.
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  auto multiply_units = [&](const auto& w, auto lead, int base, auto units, sums_t& sums) {
    constexpr int N = sizeof(w) / sizeof(w[0]);
    constexpr bool U = decltype(units)::value;   // rows in units of 16 columns; otherwise row by row
    u32x4 raw[DK * MB];
    int lo[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int m = min(b * 16 + fm, rows - 1);
      lo[b] = U ? ((kc >> 1) * rp + m) * 32 + (kc & 1) * 16 : m * (D * 2) + kc * 16;
    }
    const int step = U ? rp * 64 : 64, first = base + wave * DK * step;
    ex.wait<decltype(lead)::value>([&](int i) { return first + i / MB * step; }, [&](int i) { return lo[i % MB]; }, raw);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    floatx4 acc[N][MB];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int b = 0; b < MB; ++b) acc[i][b] = zero4;
#pragma unroll
    for (int s = 0; s < DK; ++s)
#pragma unroll
      for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int i = 0; i < N; ++i)
          acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i][s], __builtin_bit_cast(half8_t, raw[s * MB + b]), acc[i][b], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int b = 0; b < MB; ++b) *reinterpret_cast<floatx4*>(&sums[wave][i][b * 16 + fm][kc * 4]) = acc[i][b];
  };
  using lead_t = std::integral_constant<int, kLead>;
  using late_t = std::integral_constant<int, kLead + 6>;
  // four columns of a unit and row per thread: unit tid / (4 R), row, columns
  int ui = tid / (4 * R), um = tid % (4 * R) / 4, un = tid % 4 * 4;
  auto total4 = [&](const sums_t& sums, int i) {
    floatx4 t[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t[w] = *reinterpret_cast<const floatx4*>(&sums[w][i][um][un]);
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]));   // all requested before the first is added
    floatx4 v = t[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += t[w];
    return v;
  };
  auto project_quarter = [&](const auto& w, int l, int region_in, int region_out, auto request) {   // ks-th quarter of k, 64 columns
    stage_quarter(at(l, region_in));
    if (wave < 4 * MB) {
      floatx4 acc[2] = {zero4, zero4};
      const int b = wave >> 2;
#pragma unroll
      for (int s = 0; s < KS; ++s)
        acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[s], *reinterpret_cast<const half8_t*>(&st[b * 16 + fm][s * 32 + kc * 8]), acc[s & 1], 0, 0, 0);
      acc[0] += acc[1];
      const int m = b * 16 + fm;
      if (m < rows)
        put4(l, at(l, region_out) + (ks * CG + cg) * rp * 256, m * 256 + (wave & 3) * 64 + kc * 16, acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
    }
    request();
    pin();
  };

  // ---- attention (see decoder_stack_kernel).  A team has one wavefront or two, so from 33 or 65 positions on a wavefront makes several trips:
  // 9900 of the 94 000 clocks of a layer of 128 rows at d = 1024 and 45 positions, 2400 where one trip is enough.
  const int team = wave / NSH, ash = wave % NSH;
  int gk = lane >> 3, c8 = (lane & 7) * 8;
  const int pair = j + W * team, am = min(pair / H, rows - 1), ah = pair % H;
  const int arow = r0 + am, sent = arow / a.beam;
  const bool table = !PRE && a.anc != nullptr;
  const int32_t* slots = table ? a.anc + (size_t)arow * a.anc_ld : nullptr;
  auto key_at = [&](int jb, int u, int nkeys) { return max(min(jb + (gk + u * 8) * NSH, nkeys - 1), 0); };   // past the last key: that one again
  auto key_offset = [&](int slot, int p) { return (unsigned)((min(max(slot, 0), a.beam - 1) * a.T + p) * D) * 2u; };
  const bool attends = pair < rows * H;
  constexpr int span = kTripKeys * NSH;
  {
    int s0[2][kTrip];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < kTrip; ++u) s0[t][u] = table ? slots[key_at(ash + t * span, u, pos)] : 0;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < kTrip; ++u) first_key[wave][t][u][gk] = key_offset(s0[t][u], key_at(ash + t * span, u, pos));
  }
  int src_off = 0, src_len = 0;
  if constexpr (!PRE) { src_off = a.src_off[sent]; src_len = a.src_len[sent]; }
  if (tid < kWaves) shares.left[tid] = 0;   // the first rows' barrier is ahead
  int attentions = 0;
  auto base_of = [&](bool self, const half_t* b) {
    return reinterpret_cast<const char*>(b + (self ? (size_t)(table ? sent * a.beam : arow) * a.T * D : 0) + ah * 64);
  };
  half8_t kn[kTrip], vn[kTrip];
  auto request_keys = [&](auto of_self, const half_t* Kb, const half_t* Vb, int nkeys) {   // the first trip, into registers
    constexpr bool self = decltype(of_self)::value;
    if (!attends) return;
    const char *Kh = base_of(self, Kb), *Vh = base_of(self, Vb);
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const unsigned o = (self ? first_key[wave][0][u][gk] : (unsigned)(key_at(ash, u, nkeys) * (2 * D)) * 2u) + c8 * 2;
      kn[u] = *reinterpret_cast<const half8_t*>(Kh + o);
      vn[u] = *reinterpret_cast<const half8_t*>(Vh + o);
    }
  };
  // The second trip and those behind it go straight into LDS, the second requested when the wavefront begins to wait for its query: a
  // trip requested when the one before is multiplied came 3 us later, places in the cache first, and there are no registers to request it
  // earlier (eight keys per lane group: 38 to 64 spilled, 128 rows 13 % slower).  Whole translations in ms with this and attention without
  // branches and barriers: d = 1024, 32 sentences 27.6 -> 26.0; d = 512, 60 sentences 20.1 -> 19.2.  slot: of the trip after it; 0 without a table, where a row's history is its own.
  int slot[kTrip] = {};
  auto keys_to_lds = [&](auto of_self, const half_t* Kb, const half_t* Vb, int nkeys, int jb, char* room, auto second) {
    constexpr bool self = decltype(of_self)::value;
    const char *Kh = base_of(self, Kb) + c8 * 2, *Vh = base_of(self, Vb) + c8 * 2;
    char* mine = room + wave * kKeyBytes;
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const int p = key_at(jb, u, nkeys);
      const unsigned o = !self ? (unsigned)(p * (2 * D)) * 2u : second ? first_key[wave][1][u][gk] : key_offset(slot[u], p);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Kh + o), (__attribute__((address_space(3))) void*)(mine + u * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Vh + o), (__attribute__((address_space(3))) void*)(mine + (kTrip + u) * 1024), 16, 0, 0);
    }
    if (self && table && jb + span < nkeys) {
#pragma unroll
      for (int u = 0; u < kTrip; ++u) slot[u] = slots[key_at(jb + span, u, nkeys)];
    }
  };
  // the first keys and values have been requested (request_keys) an exchange earlier; room: of the keys behind them
  auto attend = [&](int l, auto of_self, const half_t* Kb, const half_t* Vb, int nkeys, const half_t* bias_q, char* room) {
    constexpr bool self = decltype(of_self)::value;
    ++attentions;
    if (!attends) return;
    if (nkeys > span) keys_to_lds(of_self, Kb, Vb, nkeys, ash + span, room, std::true_type{});
    half8_t bq8 = {};
    if (!self) bq8 = *reinterpret_cast<const half8_t*>(reinterpret_cast<const char*>(bias_q) + (unsigned)(ah * 64 + c8) * 2u);
    pin();
    half8_t q, knew = {}, vnew = {};
    if constexpr (self) {
      u32x4 raw[3];
      const int base = at(l, Rg::qkv) + (ah * 4 * rp + am) * 32;
      ex.wait<kLead + 6>([&](int i) { return base + i * (D / 16 * 32) * rp; }, [&](int) { return (c8 >> 4) * rp * 32 + (c8 & 8) * 2; }, raw);
      q = __builtin_bit_cast(half8_t, raw[0]); knew = __builtin_bit_cast(half8_t, raw[1]); vnew = __builtin_bit_cast(half8_t, raw[2]);
    } else {
      u32x4 raw[8];   // four slabs of the head's 64 columns
      const int base = at(l, Rg::qs) + (ah * rp + am) * 256;
      ex.wait<kLead>([&](int i) { return base + (i >> 1) * (CG * 256) * rp; }, [&](int i) { return c8 * 4 + (i & 1) * 16; }, raw);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float v = __builtin_bit_cast(floatx4, raw[i >> 2])[i & 3];
#pragma unroll
        for (int sl = 1; sl < 4; ++sl) v += __builtin_bit_cast(floatx4, raw[sl * 2 + (i >> 2)])[i & 3];
        q[i] = (half_t)(v + (float)bq8[i]);
      }
    }
    Attention t;
    auto live = [&](int jb) { return [&, jb](int u) { return jb + (gk + u * 8) * NSH < nkeys; }; };
    t.first<self>(q, kn, vn, knew, nkeys == 0, live(ash), [] {});
    for (int jb = ash + span; jb < nkeys; jb += span) {   // the same trips in every lane of the wavefront
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const char* mine = room + wave * kKeyBytes + lane * 16;
#pragma unroll
      for (int u = 0; u < kTrip; ++u) {
        kn[u] = *reinterpret_cast<const half8_t*>(mine + u * 1024);
        vn[u] = *reinterpret_cast<const half8_t*>(mine + (kTrip + u) * 1024);
      }
      asm volatile("" : "+v"(kn[0]), "+v"(kn[1]), "+v"(kn[2]), "+v"(kn[3]), "+v"(vn[0]), "+v"(vn[1]), "+v"(vn[2]), "+v"(vn[3]) :: "memory");
      if (jb + span < nkeys) keys_to_lds(of_self, Kb, Vb, nkeys, jb + span, room, std::false_type{});
      t.more(q, kn, vn, live(jb), [] {});
    }
    if (self && ash == NSH - 1) t.add(vnew, gk == 0);
    t.sum<false>();
    const int base = at(l, self ? Rg::ctx : Rg::ctx2) + am * (D * 2) + ah * 128;
    if constexpr (NSH == 1) {
      const half2_t v = context_of(t.acc[0], t.acc[1], t.z);
      if ((lane & 8) == 0) put2h(l, base, own_column<false>(lane) * 2, v[0], v[1]);
    } else {
      shares.leave<false>(wave, lane, t);
      if (ash > 0) return shares.tell(wave, attentions);
      const int c = (lane & 31) * 2;
      const half2_t v = shares.collect<NSH>(team * NSH, NSH, attentions, lane, c);
      if (lane < 32) put2h(l, base, c * 2, v[0], v[1]);
    }
  };

  // What is derived from a workgroup's place is derived anew in every stage, and pointers are read where they are used, instead of
  // waiting in scalar registers (69 to 157 of them were spilled; 2 to 4 are left of pre-LN models, 9 to 29 of post-LN ones).  d = 1024 needs it for what is derived from a thread's
  // place as well (it spills otherwise); narrower models would lose 3 to 7 %.  Whole translations of 75 steps: d = 1024, 128 rows
  // 21.4 -> 21.1 ms; d = 512, 200 rows 15.1 -> 14.7, one per sentence 16.6 -> 16.1; d = 768 pre-LN, 120 rows 17.15 -> 16.9 (104 steps).
  auto renew = [&] {
    asm volatile("" : "+s"(wave), "+s"(j), "+s"(cg), "+s"(ks), "+s"(grp), "+s"(rp), "+s"(r0), "+s"(rows), "+s"(pos), "+s"(start));
    if constexpr (DK == 4) {
      asm volatile("" : "+v"(tid), "+v"(lane), "+v"(fm), "+v"(kc), "+v"(lane16), "+v"(oc), "+v"(ui), "+v"(um), "+v"(un));
      asm volatile("" : "+v"(gk), "+v"(c8));
    }
  };

  // ======== the layers
  load_units(wq, layer_w(now()->Wqkv, 0));
  for (int l = 0; l < a.layers; ++l) {
    renew();
    half_t* Kc = reinterpret_cast<half_t*>(global(now()->cache) + (size_t)(2 * l) * now()->cache_stride);
    half_t* Vc = reinterpret_cast<half_t*>(global(now()->cache) + (size_t)(2 * l + 1) * now()->cache_stride);
    // the layer's input rows
    if (l == 0) {
      if (owner) {
        const int r = r0 + j;
        half4_t h = {};
        if constexpr (PRE) {
          const half4_t g4 = half4_at(a.ln1g, oc), b4 = half4_at(a.ln1b, oc);
          const half4_t e4 = half4_at(a.E + (size_t)embedding_row(a.tokens[(size_t)r * (a.T + 1) + a.len[r]]) * D, oc);
          const floatx4 p4 = *reinterpret_cast<const floatx4*>(a.pe + (size_t)pos * D + oc);
          float v[4];
          h = scaled_sums(e4, 1.0f, p4);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = (float)h[i];
          if (oact) *reinterpret_cast<half4_t*>(&xrow[oc]) = h;
          own_publish(v, g4, b4, l, Rg::xi, nullptr);
        } else {
          h = half4_at(a.x0 + (size_t)r * D, oc);
          if (oact) {
            *reinterpret_cast<half4_t*>(&xrow[oc]) = h;
            put4h(l, at(l, Rg::xi) + j * (D * 2), oc * 2, h[0], h[1], h[2], h[3]);
          }
          __syncthreads();
        }
      }
    } else {
      if constexpr (PRE) own_norm(l - 1, Rg::fs, layer_p(now()->b2, l - 1), layer_p(now()->ln1g, l), layer_p(now()->ln1b, l), l, Rg::xi, nullptr, nullptr);
      else own_norm(l - 1, Rg::fs, layer_p(now()->b2, l - 1), layer_p(now()->ln3g, l - 1), layer_p(now()->ln3b, l - 1), l, Rg::xi, nullptr, nullptr);
    }
    // q, k, v
    {
      const int qcol = (j + W * ui) * 16 + un;
      half4_t qb = {};
      const bool qlive = ui < 3 && um < rows;
      if (qlive) qb = half4_at(layer_p(now()->bqkv, l), qcol);
      request_keys(std::true_type{}, Kc, Vc, pos);   // needs nothing of this step
      pin();
      multiply_units(wq, lead_t{}, at(l, Rg::xi), std::false_type{}, part);
      load_quarter(wo, layer_w(now()->Wo, l));
      pin();
      __syncthreads();
      if (qlive) {
        const floatx4 v = total4(part, ui);
        half_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = (half_t)(v[i] + (float)qb[i]);
        put4h(l, at(l, Rg::qkv) + j * rp * 32, (W * ui * rp + um) * 32 + un * 2, h[0], h[1], h[2], h[3]);
        if (qcol >= D) {
          char* cache = reinterpret_cast<char*>((qcol < 2 * D ? Kc : Vc) + ((size_t)r0 * a.T + pos) * D);
          *reinterpret_cast<half4_t*>(cache + (unsigned)(um * a.T * D + (qcol < 2 * D ? qcol - D : qcol - 2 * D)) * 2u) = half4_t{h[0], h[1], h[2], h[3]};
        }
      }
    }
    renew();
    attend(l, std::true_type{}, Kc, Vc, pos, nullptr, st_room);
    renew();
    project_quarter(wo, l, Rg::ctx, Rg::os, [&] {
      if constexpr (PRE) load_units(w1, layer_w(now()->W1, l));
      else load_quarter(wo, layer_w(now()->Wq, l));
    });
    if constexpr (PRE) {
      own_norm(l, Rg::os, layer_p(now()->bo, l), layer_p(now()->ln2g, l), layer_p(now()->ln2b, l), l, Rg::x1, nullptr, nullptr);
    } else {
      const half_t* kvb = reinterpret_cast<const half_t*>(global(now()->cross) + (size_t)l * now()->cross_stride) + (size_t)src_off * 2 * D;
      own_norm(l, Rg::os, layer_p(now()->bo, l), layer_p(now()->ln1g, l), layer_p(now()->ln1b, l), l, Rg::x1, nullptr, nullptr);
      request_keys(std::false_type{}, kvb, kvb + D, src_len);
      pin();
      project_quarter(wo, l, Rg::x1, Rg::qs, [&] { load_quarter(wo, layer_w(now()->Woc, l)); });
      renew();
      attend(l, std::false_type{}, kvb, kvb + D, src_len, layer_p(now()->bq, l), part_room);
      project_quarter(wo, l, Rg::ctx2, Rg::cs, [&] { load_units(w1, layer_w(now()->W1, l)); });
      own_norm(l, Rg::cs, layer_p(now()->boc, l), layer_p(now()->ln2g, l), layer_p(now()->ln2b, l), l, Rg::x2, nullptr, nullptr);
    }
    // first FFN product
    renew();
    {
      const int fcol = (j + W * ui) * 16 + un;
      const bool flive = ui < 4 && um < rows;
      half4_t fb = {};
      if (flive) fb = half4_at(layer_p(now()->b1, l), fcol);
      multiply_units(w1, lead_t{}, at(l, PRE ? Rg::x1 : Rg::x2), std::false_type{}, part);
      load_ffn2(w2, layer_w(now()->W2, l));
      pin();
      __syncthreads();
      if (flive) {
        const floatx4 v = total4(part, ui);
        half_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float t = v[i] + (float)fb[i];
          h[i] = (half_t)(PRE ? tanh_gelu(t) : fmaxf(t, 0.f));
        }
        put4h(l, at(l, Rg::ff) + j * rp * 32, (W * ui * rp + um) * 32 + un * 2, h[0], h[1], h[2], h[3]);
      }
    }
    // Second FFN product.  The first one's sums may still be read by wavefronts whose activations nobody here waits for.
    multiply_units(w2, late_t{}, at(l, Rg::ff) + ks * (D / 16) * rp * 32, std::true_type{}, part2);
    if (l + 1 < a.layers) load_units(wq, layer_w(now()->Wqkv, l + 1));
    pin();
    __syncthreads();
    if (ui < 4 && um < rows) {
      const floatx4 v = total4(part2, ui);
      put4(l, at(l, Rg::fs) + (ks * CG + cg) * rp * 256, um * 256 + (ui * 16 + un) * 4, v[0], v[1], v[2], v[3]);
    }
  }
  const int last = a.layers - 1;
  if constexpr (PRE) own_norm(last, Rg::fs, layer_p(now()->b2, last), a.lnfg, a.lnfb, last, -1, a.x_out, a.hidden);
  else own_norm(last, Rg::fs, layer_p(now()->b2, last), layer_p(now()->ln3g, last), layer_p(now()->ln3b, last), last, -1, nullptr, a.hidden);
  ex.report(a.state, a.error);
  if (tid == 0) {   // the last workgroup to get here: all have read the counters
    const int n = __hip_atomic_fetch_add(a.state + 4, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n == (int)gridDim.x - 1) {
      a.state[4] = 0;
      a.state[1] = G * group_bytes;
      __hip_atomic_fetch_xor(a.state, a.layers & 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

struct Choice { int dk, x, groups, rows; };

// Groups of at most 8 rows each; then as many workgroups per group as 256 CUs hold, but not more than 128 (an exchange
// among 256 workgroups takes 0.4 us longer than among 128).
Choice choose(int arch, int M, int d) {
  Choice c = {d / 256, 0, 0, 0};
  c.groups = (M + kRows - 1) / kRows;
  c.rows = (M + c.groups - 1) / c.groups;
  c.groups = (M + c.rows - 1) / c.rows;
  for (int x : {4, 2, 1})
    if ((x < 4 || arch == 0) && d / 16 * x <= 128 && d / 16 * x * c.groups <= 256) { c.x = x; break; }
  return c;
}

const void* kernel_of(int dk, int x, int pre) {
#define LSQ_STACK(DKV, XV) if (dk == DKV && x == XV) return pre ? (const void*)decoder_stack_kernel<DKV, XV, true> : (const void*)decoder_stack_kernel<DKV, XV, false>
  if (!pre && x == 4)
    return dk == 1 ? (const void*)decoder_stack_kernel<1, 4, false> : dk == 2 ? (const void*)decoder_stack_kernel<2, 4, false> : nullptr;
  LSQ_STACK(1, 1); LSQ_STACK(1, 2);
  LSQ_STACK(2, 1); LSQ_STACK(2, 2);   // post-LN: where the die kernel cannot run
  LSQ_STACK(3, 1); LSQ_STACK(3, 2);
  LSQ_STACK(4, 1); LSQ_STACK(4, 2);
#undef LSQ_STACK
  return nullptr;
}

// the variant for more rows: groups of 16 or 32
Choice choose_rows(int M, int d) {
  Choice c = {d / 256, 0, 0, 0};
  const int most = 256 / (d / 16);
  for (int mb : {1, 2}) {
    if ((M + 16 * mb - 1) / (16 * mb) > most) continue;
    c.x = mb;
    c.groups = min(most, M);
    c.rows = (M + c.groups - 1) / c.groups;
    c.groups = (M + c.rows - 1) / c.rows;
    break;
  }
  return c;
}

const void* rows_kernel_of(int dk, int mb, int pre) {
#define LSQ_ROWS(DKV, MBV) if (dk == DKV && mb == MBV) return pre ? (const void*)decoder_stack_rows_kernel<DKV, MBV, true> : (const void*)decoder_stack_rows_kernel<DKV, MBV, false>
  LSQ_ROWS(2, 1); LSQ_ROWS(2, 2); LSQ_ROWS(3, 1); LSQ_ROWS(3, 2); LSQ_ROWS(4, 1); LSQ_ROWS(4, 2);
#undef LSQ_ROWS
  return nullptr;
}

}  // namespace

size_t stack_exchange_bytes(int arch, int M, int d, int layers) {
  if (const size_t n = die_exchange_bytes(arch, M, d, layers)) return n;
  return (size_t)(min(M, kStackRowsMax) + kRows) * layers * (arch == 1 ? Region<true>::size : Region<false>::size) * d;
}

size_t stack_rows_bytes(int arch, int M, int d) {
  if (!rows_kernel_of(d / 256, 1, arch == 1)) return 0;
  const int most = 32 * (256 / (d / 16));
  return (size_t)(min(M, most) + 16) * (arch == 1 ? RowsRegion<true>::size : RowsRegion<false>::size) * d;
}

bool stack_shape_supported(int dtype, int arch, int H, int d, int F, int layers) {
  return dtype == DT_F16 && d % 256 == 0 && d <= 1024 && H * 64 == d && F == 4 * d &&
         stack_exchange_bytes(arch, kStackRowsMax, d, layers) < (1u << 30);
}

// Which kernel takes M rows on the current device.  A (row, head) pair has 256 keys in flight in groups of 8 rows (128 with X = 1), 64 or 32
// in groups of 16 or 32; the separate kernels give it four wavefronts and read a history that the rows of a sentence share once.  So the order
// changes with the length.  Whole steps in us, beam 4 and sources of 30 tokens, six layers (pre-LN: twelve, one row per prompt), V = 16 000;
// 8-row groups / more rows:
//   positions                 20-60          60-120         120-200        200-320        320-440
//   d = 1024,   8 rows        125 / 132      128 / 136      131 / 141      139 / 148      152 / 160
//              12 rows        127 / 135      129 / 139      133 / 144      142 / 153      156 / 167
//              16 rows        134 / 137      136 / 141      140 / 147      149 / 158      164 / 175
//              24 rows        144 / 142      149 / 149      164 / 159      182 / 173      206 / 193
//              32 rows        146 / 146      154 / 154      171 / 164      190 / 180      214 / 200
//   one per sentence, 8       127 / 132      130 / 136      135 / 142      144 / 153      153 / 168
//              16 rows        137 / 139      142 / 146      150 / 157      161 / 171      171 / 184
//   d = 768,   16 rows        115 / 123      117 / 126      119 / 130      126 / 136      133 / 143
//              24 rows        118 / 126      119 / 130      129 / 134      137 / 140      148 / 148
//              32 rows        122 / 128      123 / 132      133 / 136      142 / 142      155 / 152
//              40 rows        124 / 132      126 / 136      136 / 140      147 / 148      162 / 159
//   d = 768, pre-LN, 16       149 / 160      155 / 169      168 / 187      186 / 206      198 / 226
//              32 rows        173 / 175      190 / 192      208 / 208      228 / 230      255 / 257
//              40 rows        177 / 183      195 / 200      216 / 219      239 / 243      271 / 274
//   d = 512,   12 rows         97 / 108       98 / 112      101 / 116      107 / 122      115 / 129     (where the die kernel does not run)
//              32 rows        102 / 113      103 / 116      106 / 120      112 / 126      119 / 133
//              64 rows        105 / 120      107 / 123      116 / 127      125 / 135      137 / 145
//   d = 512, pre-LN, 40       130 / 149      137 / 155      157 / 172      187 / 205      221 / 235
// and more rows / separate launches:
//   positions                 440-560        560-940        940-1060       1060-1180      1180-1300
//   d = 1024,  16 rows        187 / 307      209 / 314      233 / 337      246 / 342      257 / 351
//              64 rows        276 / 433      321 / 484      372 / 535      399 / 561      423 / 586
//             128 rows        416 / 545      510 / 627      604 / 721      647 / 763      693 / 808
//   d = 768,   48 rows        187 / 364      220 / 397      253 / 445      266 / 459      279 / 477
//             160 rows        341 / 482      415 / 543      488 / 614      522 / 639      558 / 668
//   d = 512,  128 rows        226 / 377      272 / 421      315 / 462      335 / 483      358 / 505
//             256 rows        348 / 472      428 / 541      507 / 606      546 / 639      589 / 679
// d = 768 has groups of 8 as long as they fit the chip: ahead or level to position 320, 2 % behind from there on.  d = 1024 has them up to
// 8 rows; 24 and 32 rows are level at first and behind later.  The lines for 9 to 16 rows of d = 1024 and for d = 512, and those to the separate
// launches (1300, 1120, 960 and 1100), were drawn where earlier forms of these kernels crossed: the present ones cross later or not at all, so a
// line costs what the table says between it and there, 3 to 7 % of a step for 9 to 16 rows of d = 1024 up to position 112.
// Older, of those earlier forms: groups of 8 against separate launches at positions 1008 and 1900, d = 1024, 8 rows 245 / 357, 324 / 388, 32 rows
// 383 / 469, 523 / 538; one row per sentence, which shares nothing, d = 1024, 128 rows on more rows / separate launches 898 / 958, 1418 / 1391.  A source
// key counts as a quarter or half of one of the history (position 16, sources of 2000: d = 512, 128 rows 460 / 458, 256 rows 791 / 784; d = 1024,
// 32 rows 363 / 433, 128 rows 862 / 825).
StackKind stack_kind(int arch, int M, int d, int beam, int pos, int src, bool dies) {
  if (M < 1) return kStackNone;
  if (dies && die_supported(arch, M, d, beam, pos, src)) return kStackDie;
  const Choice c = choose(arch, M, d), r = choose_rows(M, d);
  bool few = c.x != 0 && M <= kStackRowsMax && kernel_of(c.dk, c.x, arch == 1) && resident(kernel_of(c.dk, c.x, arch == 1));
  bool many = r.x != 0 && rows_kernel_of(r.dk, r.x, arch == 1) && resident(rows_kernel_of(r.dk, r.x, arch == 1));
  constexpr int never = 1 << 30;
  const int len = pos + src / 4;
  // 8-row groups against separate launches (extrapolated past 1900; 1 sentence of d = 1024 460 / 464 at 3900), more rows against
  // them, 8-row groups against more rows
  if (beam > 1 && d > 512 && len > (c.x == 1 ? 2000 : 2700)) few = false;
  if (r.x == 1 && beam > 1 && len > 1300) many = false;
  if (r.x == 2 && pos + src / 2 > (beam > 1 ? (d == 512 ? 1120 : d == 768 ? 960 : 1100) : (d == 1024 ? 1600 : never))) many = false;
  const int few_from = d == 768    ? (M <= 40 ? 0 : never)
                       : d == 1024 ? (M <= 8 ? 0 : M <= 16 ? (beam > 1 ? 112 : 352) : never)
                                   : (M <= 8 ? 0 : beam > 1 ? 112 : 240);
  if (few && (!many || len >= few_from)) return kStackFew;
  return many ? kStackMany : kStackNone;
}

// More rows than `stack_kind` has a kernel for as two launches, one after the other, of the kernel for 17 to 128 of them.  d = 1024, sources of 30 tokens, whole
// steps in us, two launches / separate launches:
//   positions          5-25        25-50       50-75
//   beam 4, 132 rows   351 / 409   361 / 414   374 / 427
//           160        374 / 415   393 / 425   408 / 437
//           192        394 / 431   418 / 440   434 / 455
//           208        412 / 434   439 / 444   453 / 461
//           224        424 / 441   450 / 453   463 / 466
//           256        444 / 445   469 / 459   484 / 474
//   beam 5, 160        370 / 432   387 / 440   400 / 452
//           200        402 / 441   426 / 451   441 / 466
//   beam 2, 160        392 / 425   407 / 435   423 / 446
//           200        417 / 436   442 / 446   458 / 459
// A position costs two launches 0.8 us and the separate ones 0.55; the rows of a sentence share less of their history where there are two of
// them.  The lines are where these lead to; a source key counts as half a position.  Past 208 rows what is left of it is short-lived: 4 % at 224 rows in the
// first 25 positions, under 1 % behind them.  Fewer than 129 rows fit one launch: where stack_kind has none for them it is because the separate ones
// are ahead of it, or because the caller wants it so.
bool stack_twice(int arch, int M, int d, int beam, int pos, int src) {
  return arch == 0 && d == 1024 && beam >= 2 && M > 128 && M <= 208 && pos + src / 2 <= 105 + 2 * (208 - M) - (beam == 2 ? 40 : 0);
}

bool stream_has_every_cu(hipStream_t s) {
  for (const char* name : {"HSA_CU_MASK", "ROC_GLOBAL_CU_MASK"}) {   // masks for every queue of the process
    const char* v = std::getenv(name);
    if (v && *v) return false;
  }
  int dev = 0, cus = 0;
  uint32_t mask[32] = {};
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus > 32 * 32 || hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  for (int i = 0; i < cus; ++i)
    if (!(mask[i / 32] >> (i % 32) & 1)) return false;
  return true;
}

hipError_t launch_stack_reset(char* exchange, size_t bytes, int32_t* state, hipStream_t s) {
  hipError_t e = hipMemsetAsync(exchange, 0xFF, bytes, s);
  return e == hipSuccess ? hipMemsetAsync(state, 0, 8 * 4, s) : e;
}

hipError_t launch_stack_end_waits(int32_t* state, hipStream_t s) { return hipMemsetAsync(reinterpret_cast<char*>(state) + 3, 0x80, 1, s); }

hipError_t launch_decoder_stack_rows(int arch, const StackArgs& args, int d, hipStream_t s) {
  const Choice c = choose_rows(args.M, d);
  if (!c.x) return hipErrorInvalidValue;
  StackArgs a = args;
  a.groups = c.groups;
  a.rows_per_group = c.rows;
  void* kargs[] = {&a};
  return hipLaunchKernel(rows_kernel_of(c.dk, c.x, arch == 1), dim3(d / 16 * c.groups), dim3(kThreads), kargs, 0, s);
}

hipError_t launch_decoder_stack(int arch, const StackArgs& args, int d, hipStream_t s) {
  const Choice c = choose(arch, args.M, d);
  StackArgs a = args;
  a.groups = c.groups;
  a.rows_per_group = c.rows;
  void* kargs[] = {&a};
  return hipLaunchKernel(kernel_of(c.dk, c.x, arch == 1), dim3(d / 16 * c.x * c.groups), dim3(kThreads), kargs, 0, s);
}

}  // namespace lsq
