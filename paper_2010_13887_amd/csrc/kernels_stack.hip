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
// polls, then the error flag is set, nothing is waited for any more and the launch runs to its end).
#include "lsq_internal.h"

namespace lsq {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned kSentinel = 0xFFFFFFFFu;
constexpr int kAgent = 16;             // cache policy of agent scope: sc1
constexpr int kSpinLimit = 1 << 19;    // polls of about a microsecond
constexpr int kRows = 8;               // rows of a group
constexpr int kMinRows = 4;            // a writer's piece is at least as large as for these: several writers in one line slow each other down
constexpr int kThreads = 512, kWaves = 8;

// Byte offsets of a row's intermediates inside one layer's region (d: row width)
template <bool PRE> struct Region {
  static constexpr int qkv = 0, ctx = 6, u1 = 8;
  static constexpr int q2 = PRE ? 0 : 12, ctx2 = PRE ? 0 : 14, u2 = PRE ? 0 : 16;   // cross-attention: post-LN models
  static constexpr int ff = PRE ? 10 : 20, u3 = PRE ? 18 : 28, size = PRE ? 20 : 32;
};

__device__ __forceinline__ unsigned publish_word(unsigned v) { return v == kSentinel ? 0x7FFF7FFFu : v; }   // one NaN for another

struct Exchange {
  __amdgpu_buffer_rsrc_t rsrc;
  int* error;
  bool dead;

  // v[i] = the 16 bytes at base(i) + lane(i) once all of them have been written (base: the same in all lanes)
  template <int N, typename B, typename L>
  __device__ __forceinline__ void wait(B base, L lane, u32x4 (&v)[N]) {
    for (int left = dead ? 1 : kSpinLimit;;) {
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane(i), base(i), kAgent);
      unsigned worst = 0;
#pragma unroll
      for (int i = 0; i < N; ++i) worst = max(max(worst, max(v[i].x, v[i].y)), max(v[i].z, v[i].w));
      if (__all(worst != kSentinel)) return;
      if (--left == 0) break;
      __builtin_amdgcn_s_sleep(1);
      asm volatile("" ::: "memory");
    }
    dead = true;
    __hip_atomic_store(error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  __device__ __forceinline__ void put(int base, int lane, unsigned v) {
    __builtin_amdgcn_raw_buffer_store_b32(publish_word(v), rsrc, lane, base, kAgent);
  }
  __device__ __forceinline__ void put(int base, int lane, float v) { put(base, lane, __builtin_bit_cast(unsigned, v)); }
  __device__ __forceinline__ void put2(int base, int lane, half_t a, half_t b) {
    typedef half_t half2_t __attribute__((ext_vector_type(2)));
    put(base, lane, __builtin_bit_cast(unsigned, half2_t{a, b}));
  }
};

__device__ __forceinline__ float tanh_gelu(float v) {
  return 0.5f * v * (1.0f + tanhf(0.7978845608028654f * (v + 0.044715f * v * v * v)));
}

// DK: d / 256.  X: workgroups of a group per 16 columns of d (W = d / 16 * X): the products with d columns take 16 / X
// columns per workgroup, those with 3d and 4d columns ceil(3 / X) and 4 / X units of 16.  PRE: pre-LN, no cross-attention.
//
// Layout of the exchanged values: what one workgroup writes for all rows of its group is contiguous ([writer][row][its
// columns]); row-major regions, where 4..16 writers share every 128-byte line, take 0.3..0.7 us longer per exchange.
template <int DK, int X, bool PRE>
__global__ void __launch_bounds__(kThreads) decoder_stack_kernel(const StackArgs a) {
  constexpr int D = 256 * DK, H = D / 64, W = D / 16 * X, NT = 16 / X;
  constexpr int NU = 4 / X, UQ = (3 + X - 1) / X;
  constexpr int QT = NT < 8 ? 8 : NT;                          // query columns of the cross-attention per workgroup
  constexpr int TEAMS = X == 1 ? 2 : 1, NSH = kWaves / TEAMS;   // wavefronts that share a (row, head) pair
  constexpr int U = 4;                                         // keys of a lane group in flight
  using Rg = Region<PRE>;
  constexpr int NV = (D + 511) / 512;
  constexpr int ES = PRE ? 2 : 4;                              // bytes of a residual sum
  constexpr int CH = (kRows * D * ES / 16 + kThreads - 1) / kThreads;   // 16-byte pieces of all rows' sums per thread
  using sum_t = std::conditional_t<PRE, half_t, float>;
  typedef half_t half2_t __attribute__((ext_vector_type(2)));

  __shared__ __attribute__((aligned(16))) half_t xs[kRows][D + 8];    // normalised rows
  __shared__ __attribute__((aligned(16))) sum_t us[kRows][D + 16 / ES];   // residual sums (pre-LN: the residual stream)
  __shared__ __attribute__((aligned(16))) float part[kWaves][NU > UQ ? NU : UQ][kRows][16];
  __shared__ __attribute__((aligned(16))) float part2[kWaves][kRows][16];
  __shared__ float att_o[kWaves][64], att_m[kWaves], att_l[kWaves];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, bid = blockIdx.x;
  const int grp = (bid >> 3) % G, j = (bid >> 3) / G * 8 + (bid & 7);
  const int r0 = grp * a.rows_per_group, rows = min(a.rows_per_group, a.M - r0);
  const int seq = a.state[0], parity = seq & 1, dirty = a.state[2 - parity], pos = *a.tpos;

  Exchange ex;
  ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange + (size_t)parity * a.set_bytes, (short)0, (int)a.set_bytes, 0x00027000);
  ex.error = a.error;
  ex.dead = false;
  const int row_bytes = a.layers * Rg::size * D;
  const int rp = max(a.rows_per_group, kMinRows);   // rows a writer's piece has room for
  auto at = [&](int l, int region) { return (grp * row_bytes + (l * Rg::size + region) * D) * rp; };

  // ---- matrix fragments: lane (n = lane & 15, kc = lane >> 4) of a 32-wide k-step holds W[col + n][32 s + 8 kc ..]
  const int fm = lane & 7, kc = lane >> 4;
  auto frag_lane = [&](int nt) { return (unsigned)(kc >> 1) * 1024 + ((lane & (nt - 1)) + 32 * (kc & 1)) * 16; };
  const unsigned lane16 = frag_lane(16), lane_nt = frag_lane(NT), lane_qt = frag_lane(QT);
  auto frag_col = [&](const half_t* Wp, int K, int col) {   // its first k-step, in bytes
    return reinterpret_cast<const char*>(Wp) + (size_t)(col >> 5) * (K / 16) * 1024 + (col & 31) * 16;
  };
  half8_t wq[UQ][DK], wo[DK], wc[PRE ? 1 : DK], we[PRE ? 1 : DK], w1[NU][DK], w2[4 * DK];
  auto load_units = [&](auto& w, const half_t* Wp, int total) {
    constexpr int N = sizeof(w) / sizeof(w[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const char* p = frag_col(Wp, D, min(j + W * i, total - 1) * 16) + wave * (DK * 2048);
#pragma unroll
      for (int s = 0; s < DK; ++s) w[i][s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lane16);
    }
  };
  auto load_cols = [&](auto& w, const half_t* Wp, int K, int nt) {   // nt of d columns (the last ones again where there are none left)
    constexpr int N = sizeof(w) / sizeof(w[0]);
    const char* p = frag_col(Wp, K, min(j * nt, D - nt)) + wave * (N * 2048);
    const unsigned lo = nt == QT ? lane_qt : lane_nt;
#pragma unroll
    for (int s = 0; s < N; ++s) w[s] = *reinterpret_cast<const half8_t*>(p + s * 2048 + lo);
  };
  // two biases, unconverted: a conversion here would wait for everything requested before them
  auto bias_pair = [](const half_t* b, unsigned col) { return *reinterpret_cast<const half2_t*>(reinterpret_cast<const char*>(b) + col * 2u); };
  auto pin = [] { asm volatile("" ::: "memory"); };   // requests stay where they are written
  auto layer_w = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(p) + (size_t)l * a.packed_stride); };
  auto layer_p = [&](const half_t* p, int l) { return reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(p) + (size_t)l * a.plain_stride); };

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
    ex.wait([&](int) { return base; }, [&](int i) { return piece_at[i]; }, raw);
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
  auto total_of = [&](int i, int m, int n, float& v0, float& v1) {   // columns n, n + 1, over the wavefronts in order
    v0 = part[0][i][m][n]; v1 = part[0][i][m][n + 1];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) { v0 += part[w][i][m][n]; v1 += part[w][i][m][n + 1]; }
  };

  // ---- attention of one (row, head) pair per team of NSH wavefronts; a lane group of 8 holds a key's 64 values
  const int team = wave / NSH, ash = wave % NSH, gk = lane >> 3, c8 = (lane & 7) * 8;
  const int pair = j + W * team, am = min(pair / H, rows - 1), ah = pair % H;
  const bool attends = pair < rows * H;
  const int arow = r0 + am, sent = arow / a.beam;
  const int jfirst = ash + gk * NSH, jstep = 8 * NSH;
  int slot0[U];
  const bool table = !PRE && a.anc != nullptr;
  const int32_t* slots = table ? a.anc + (size_t)arow * a.anc_ld : nullptr;
  auto slot_of = [&](int p) { return table ? min(max(slots[p], 0), a.beam - 1) : 0; };   // of the sentence's rows
#pragma unroll
  for (int u = 0; u < U; ++u) slot0[u] = slot_of(max(min(jfirst + u * jstep, pos - 1), 0));
  int src_off = 0, src_len = 0;
  if constexpr (!PRE) { src_off = a.src_off[sent]; src_len = a.src_len[sent]; }

  auto dot8 = [](const half8_t& x, const half8_t& y) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_fdot2(half2_t{x[2 * i], x[2 * i + 1]}, half2_t{y[2 * i], y[2 * i + 1]}, s, false);
    return s;
  };
  auto attend = [&](int l, bool self, const half_t* Kb, const half_t* Vb, int nkeys) {
    if (attends) {
      half8_t kn[U], vn[U];
      const size_t own = self ? (size_t)(table ? sent * a.beam : arow) * a.T * D : 0;
      const char* Kh = reinterpret_cast<const char*>(Kb + own + ah * 64);
      const char* Vh = reinterpret_cast<const char*>(Vb + own + ah * 64);
      auto request = [&](int jb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (u > 0 && jb - gk * NSH + u * jstep >= nkeys) continue;   // nobody in this wavefront has such a key
          const int p = max(min(jb + u * jstep, nkeys - 1), 0);
          const unsigned o = ((self ? ((jb == jfirst ? slot0[u] : slot_of(p)) * a.T + p) * D : p * (2 * D)) + c8) * 2u;
          kn[u] = *reinterpret_cast<const half8_t*>(Kh + o);
          vn[u] = *reinterpret_cast<const half8_t*>(Vh + o);
        }
      };
      request(jfirst);
      pin();
      constexpr float qscale = 0.125f * 1.44269504088896340736f;   // scores in units of log 2
      half8_t q, knew, vnew;
      if (self) {
        u32x4 raw[3];
        const int base = at(l, Rg::qkv) + (ah * 4 * rp + am) * 32;
        ex.wait([&](int i) { return base + i * (D / 16 * 32) * rp; }, [&](int) { return (c8 >> 4) * rp * 32 + (c8 & 8) * 2; }, raw);
        q = __builtin_bit_cast(half8_t, raw[0]); knew = __builtin_bit_cast(half8_t, raw[1]); vnew = __builtin_bit_cast(half8_t, raw[2]);
      } else {
        u32x4 raw[1];
        const int base = at(l, Rg::q2) + (ah * 64 / QT * rp + am) * (QT * 2);
        ex.wait([&](int) { return base; }, [&](int) { return c8 / QT * rp * (QT * 2) + c8 % QT * 2; }, raw);
        q = __builtin_bit_cast(half8_t, raw[0]);
      }
      float m = -INFINITY, z = 0.f, acc[8];   // m: of the wavefront
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.f;
      for (int jb = jfirst; jb - gk * NSH < nkeys; jb += U * jstep) {   // the same trips in every lane of the wavefront
        float sc[U], mx = m;
        half8_t vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          sc[u] = -INFINITY;
          if (jb - gk * NSH + u * jstep >= nkeys) continue;
          const float s = group_sum<8>(dot8(q, kn[u])) * qscale;
          if (jb + u * jstep < nkeys) sc[u] = s;
          vv[u] = vn[u];
          mx = fmaxf(mx, sc[u]);
        }
        const int jn = jb + U * jstep;
        if (jn - gk * NSH < nkeys) request(jn);
        for_lane_bits<8>([&](auto bit) { mx = max_lane_xor<decltype(bit)::value>(mx); });
        const float corr = __builtin_amdgcn_exp2f(m - mx);   // mx is finite: the wavefront has a key in this trip
        m = mx;
        z *= corr;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] *= corr;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (jb - gk * NSH + u * jstep >= nkeys) continue;
          const bool live = jb + u * jstep < nkeys;
          const float p = live ? __builtin_amdgcn_exp2f(sc[u] - mx) : 0.f;
          z += p;
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] += p * (live ? (float)vv[u][i] : 0.f);
        }
      }
      if (self && ash == NSH - 1) {   // the new position, counted once: by the team's last wavefront
        const float s = group_sum<8>(dot8(q, knew)) * qscale, mx = fmaxf(m, s);
        const float corr = __builtin_amdgcn_exp2f(m - mx), p = gk == 0 ? __builtin_amdgcn_exp2f(s - mx) : 0.f;
        m = mx;
        z = z * corr + p;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = acc[i] * corr + p * (float)vnew[i];
      }
      for_lane_bits<8>([&](auto bit) {
        constexpr int O = decltype(bit)::value;
        z = add_lane_xor<O>(z);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = add_lane_xor<O>(acc[i]);
      });
      if (gk == 0) {
        *reinterpret_cast<floatx4*>(&att_o[wave][c8]) = floatx4{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<floatx4*>(&att_o[wave][c8 + 4]) = floatx4{acc[4], acc[5], acc[6], acc[7]};
        if (lane == 0) { att_m[wave] = m; att_l[wave] = z; }
      }
    }
    __syncthreads();
    const int tm = tid >> 5, c = (tid & 31) * 2, pr = j + W * tm;   // two values of a pair's context each
    if (tm < TEAMS && pr < rows * H) {
      float mx = -INFINITY, z = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
      for (int w = 0; w < NSH; ++w) mx = fmaxf(mx, att_m[tm * NSH + w]);
#pragma unroll
      for (int w = 0; w < NSH; ++w) {
        const float cw = __builtin_amdgcn_exp2f(att_m[tm * NSH + w] - mx);
        z += att_l[tm * NSH + w] * cw;
        o0 += att_o[tm * NSH + w][c] * cw;
        o1 += att_o[tm * NSH + w][c + 1] * cw;
      }
      const float inv = 1.0f / z;
      ex.put2(at(l, self ? Rg::ctx : Rg::ctx2), pr / H * (D * 2) + (pr % H * 64 + c) * 2, (half_t)(o0 * inv), (half_t)(o1 * inv));
    }
  };

  // ---- a product whose input rows (N k-steps of 32 per wavefront) come straight from the exchange (row-major or units of
  // 16 columns), this workgroup's NT columns; then the residual: region_out <- x + (in . W + bias).  `request`: what is
  // wanted next.
  auto project = [&](const auto& w, int l, int region_in, bool units, int region_out, const half_t* bias, auto request) {
    constexpr int N = sizeof(w) / sizeof(w[0]);
    const int om = tid / (NT / 2), on = tid % (NT / 2) * 2;
    half2_t bi = {0, 0};
    if (om < rows) bi = bias_pair(bias, j * NT + on);
    u32x4 raw[N];
    const int step = units ? 64 * rp : 64, base = at(l, region_in) + wave * N * step;
    const int lo = units ? ((kc >> 1) * rp + min(fm, rows - 1)) * 32 + (kc & 1) * 16 : min(fm, rows - 1) * (D * 2) + kc * 16;
    ex.wait([&](int i) { return base + i * step; }, [&](int) { return lo; }, raw);
    floatx4 acc[2] = {zero4, zero4};
#pragma unroll
    for (int s = 0; s < N; ++s)
      acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[s], __builtin_bit_cast(half8_t, raw[s]), acc[s & 1], 0, 0, 0);
    if ((lane & 15) < kRows && kc * 4 < NT) *reinterpret_cast<floatx4*>(&part2[wave][lane & 15][kc * 4]) = acc[0] + acc[1];
    request();
    pin();
    __syncthreads();
    if (om < rows) {
      float v0 = part2[0][om][on], v1 = part2[0][om][on + 1];
#pragma unroll
      for (int q = 1; q < kWaves; ++q) { v0 += part2[q][om][on]; v1 += part2[q][om][on + 1]; }
      const int base_out = at(l, region_out) + j * rp * (NT * ES), o = om * (NT * ES) + on * ES;
      if constexpr (PRE) {
        const half_t* x = &us[om][j * NT + on];
        ex.put2(base_out, o, (half_t)((float)x[0] + (v0 + (float)bi[0])), (half_t)((float)x[1] + (v1 + (float)bi[1])));
      } else {
        const half_t* x = &xs[om][j * NT + on];
        ex.put(base_out, o, (float)x[0] + (v0 + (float)bi[0]));
        ex.put(base_out, o + 4, (float)x[1] + (v1 + (float)bi[1]));
      }
    }
  };

  // ======== the layers.  Every matrix slice is requested at least one exchange before it is multiplied.
  load_units(wq, layer_w(a.Wqkv, 0), 3 * (D / 16));
  for (int l = 0; l < a.layers; ++l) {
    half_t* Kc = reinterpret_cast<half_t*>(a.cache + (size_t)(2 * l) * a.cache_stride);
    half_t* Vc = reinterpret_cast<half_t*>(a.cache + (size_t)(2 * l + 1) * a.cache_stride);
    // A. the layer's input rows; q, k, v
    const int qi = tid >> 6, qm = (tid >> 3) & 7, qn = (tid & 7) * 2;   // unit, row, pair of columns this thread finishes
    const half_t* bq3 = layer_p(a.bqkv, l);
    half2_t qb = {0, 0};
    const int qcol = (j + W * qi) * 16 + qn;
    const bool qlive = qi < UQ && qcol < 3 * D && qm < rows;
    if (qlive) qb = bias_pair(bq3, qcol);
    if (l == 0) {
      if (wave < rows) {
        const int r = r0 + wave;
        if constexpr (PRE) {
          half8_t g8[NV], b8[NV];
          load_gain(g8, b8, a.ln1g, a.ln1b);
          const half_t* e = a.E + (size_t)a.tokens[(size_t)r * (a.T + 1) + a.len[r]] * D;
          embed_row<half_t>(e, a.pe + (size_t)pos * D, us[wave], D, 1.0f, lane, 64);
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
      if constexpr (PRE) gather_norm(l - 1, Rg::u3, layer_p(a.ln1g, l), layer_p(a.ln1b, l), nullptr, nullptr);
      else gather_norm(l - 1, Rg::u3, layer_p(a.ln3g, l - 1), layer_p(a.ln3b, l - 1), nullptr, nullptr);
    }
    multiply_units(wq);
    load_cols(wo, layer_w(a.Wo, l), D, NT);
    if constexpr (PRE) load_units(w1, layer_w(a.W1, l), 4 * (D / 16));
    else load_cols(wc, layer_w(a.Wq, l), D, QT);
    pin();
    __syncthreads();
    if (qlive) {
      float v0, v1;
      total_of(qi, qm, qn, v0, v1);
      const half_t h0 = (half_t)(v0 + (float)qb[0]), h1 = (half_t)(v1 + (float)qb[1]);
      ex.put2(at(l, Rg::qkv) + j * rp * 32, (W * qi * rp + qm) * 32 + qn * 2, h0, h1);
      if (qcol >= D) {
        char* cache = reinterpret_cast<char*>((qcol < 2 * D ? Kc : Vc) + ((size_t)r0 * a.T + pos) * D);
        *reinterpret_cast<half2_t*>(cache + (unsigned)(qm * a.T * D + (qcol < 2 * D ? qcol - D : qcol - 2 * D)) * 2u) = half2_t{h0, h1};
      }
    }
    // B, C. self-attention, its output projection
    attend(l, true, Kc, Vc, pos);
    project(wo, l, Rg::ctx, false, Rg::u1, layer_p(a.bo, l), [&] {
      if constexpr (PRE) load_cols(w2, layer_w(a.W2, l), 4 * D, NT);
      else load_cols(we, layer_w(a.Woc, l), D, NT);
    });
    if constexpr (!PRE) {
      // D. LayerNorm, query product of the cross-attention
      const int pm = tid / (QT / 2), pn = tid % (QT / 2) * 2;
      const bool plive = pm < rows && j * QT < D;
      half2_t pb = {0, 0};
      if (plive) pb = bias_pair(layer_p(a.bq, l), j * QT + pn);
      gather_norm(l, Rg::u1, layer_p(a.ln1g, l), layer_p(a.ln1b, l), nullptr, nullptr);
      floatx4 acc = zero4;
#pragma unroll
      for (int s = 0; s < DK; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wc[PRE ? 0 : s], *reinterpret_cast<const half8_t*>(&xs[fm][(wave * DK + s) * 32 + kc * 8]), acc, 0, 0, 0);
      if ((lane & 15) < kRows) *reinterpret_cast<floatx4*>(&part[wave][0][lane & 15][kc * 4]) = acc;
      load_units(w1, layer_w(a.W1, l), 4 * (D / 16));
      pin();
      __syncthreads();
      if (plive) {
        float v0, v1;
        total_of(0, pm, pn, v0, v1);
        ex.put2(at(l, Rg::q2) + j * rp * (QT * 2), pm * (QT * 2) + pn * 2, (half_t)(v0 + (float)pb[0]), (half_t)(v1 + (float)pb[1]));
      }
      // E, F. cross-attention, its output projection
      const half_t* kvb = reinterpret_cast<const half_t*>(a.cross + (size_t)l * a.cross_stride) + (size_t)src_off * 2 * D;
      attend(l, false, kvb, kvb + D, src_len);
      project(we, l, Rg::ctx2, false, Rg::u2, layer_p(a.boc, l), [&] { load_cols(w2, layer_w(a.W2, l), 4 * D, NT); });
    }
    // G. LayerNorm, first FFN product
    const int fcol = (j + W * qi) * 16 + qn;
    half2_t fb = {0, 0};
    if (qi < NU && qm < rows) fb = bias_pair(layer_p(a.b1, l), fcol);
    gather_norm(l, PRE ? Rg::u1 : Rg::u2, layer_p(a.ln2g, l), layer_p(a.ln2b, l), nullptr, nullptr);
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
    project(w2, l, Rg::ff, true, Rg::u3, layer_p(a.b2, l), [&] {
      if (l + 1 < a.layers) load_units(wq, layer_w(a.Wqkv, l + 1), 3 * (D / 16));
    });
  }
  // ======== the rows for the vocabulary product; everything else ends here
  if (j == 0) {
    if constexpr (PRE) gather_norm(a.layers - 1, Rg::u3, a.lnfg, a.lnfb, a.x_out, a.hidden);
    else gather_norm(a.layers - 1, Rg::u3, layer_p(a.ln3g, a.layers - 1), layer_p(a.ln3b, a.layers - 1), nullptr, a.hidden);
  }
  {
    char* other = a.exchange + (size_t)(1 - parity) * a.set_bytes;
    const size_t n16 = (size_t)dirty * row_bytes / 16;
    const u32x4 s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
    for (size_t i = (size_t)bid * kThreads + tid; i < n16; i += (size_t)gridDim.x * kThreads) reinterpret_cast<u32x4*>(other)[i] = s4;
  }
  if (tid == 0) {   // the last workgroup to get here: all have read the counters
    const int n = __hip_atomic_fetch_add(a.state + 4, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n == (int)gridDim.x - 1) {
      a.state[4] = 0;
      a.state[1 + parity] = G * rp;
      a.state[0] = seq + 1;
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
  if (!pre && x == 4) return dk == 1 ? (const void*)decoder_stack_kernel<1, 4, false> : dk == 2 ? (const void*)decoder_stack_kernel<2, 4, false> : nullptr;
  LSQ_STACK(1, 1); LSQ_STACK(1, 2);
  LSQ_STACK(2, 1); LSQ_STACK(2, 2);
  LSQ_STACK(3, 1); LSQ_STACK(3, 2);
  LSQ_STACK(4, 1); LSQ_STACK(4, 2);
#undef LSQ_STACK
  return nullptr;
}

// Whether every workgroup of the largest launch of this kernel is resident at once on the current device.
bool resident(int dk, int x, int pre) {
  static int known[5][5][2];   // 0 not asked yet, 1 no, 2 yes
  int& k = known[dk][x][pre];
  if (k == 0) {
    int dev = 0, cus = 0, per_cu = 0;
    const bool ok = hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel_of(dk, x, pre), kThreads, 0) == hipSuccess;
    k = ok && cus * per_cu >= 256 ? 2 : 1;
  }
  return k == 2;
}

}  // namespace

size_t stack_exchange_bytes(int arch, int M, int d, int layers) {
  return (size_t)(min(M, kStackRowsMax) + kRows) * layers * (arch == 1 ? Region<true>::size : Region<false>::size) * d;
}

bool stack_shape_supported(int dtype, int arch, int H, int d, int F, int layers) {
  return dtype == DT_F16 && d % 256 == 0 && d <= 1024 && H * 64 == d && F == 4 * d &&
         stack_exchange_bytes(arch, kStackRowsMax, d, layers) < (1u << 30);
}

bool stack_supported(int arch, int M, int d) {
  if (M < 1 || M > kStackRowsMax) return false;
  const Choice c = choose(arch, M, d);
  return c.x != 0 && kernel_of(c.dk, c.x, arch == 1) != nullptr && resident(c.dk, c.x, arch == 1);
}

hipError_t launch_stack_reset(char* exchange, size_t bytes, int32_t* state, hipStream_t s) {
  hipError_t e = hipMemsetAsync(exchange, 0xFF, bytes, s);
  return e == hipSuccess ? hipMemsetAsync(state, 0, 8 * 4, s) : e;
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
