// All decoder layers of one step in ONE launch, float32 (encoder-decoder models, heads of 64, FFN of 4d, d = 256 or 512).
// Exchange, residency and bounded waits: kernels_stack.hip, whose variant for more rows this follows in the cut of the work
// (row owners for residual and LayerNorm, k split fourfold where there are d columns, exchange regions for two layers).
//
// As separate launches a step at d = 512 and 32 rows took 470 us: 37 products of 10 us, 18 LayerNorms and 12 attentions
// of 5 us, each of which is a microsecond of work.  In this launch: 136 us, 2.1 us per exchange and what follows it; the
// weights (88 MB) come from the caches behind HBM at 0.65 TB/s, so the chain bounds it, not the stream.
//
// Products run on v_mfma_f32_4x4x1 (16 blocks of 4 rows x 4 columns, one k): a group has only 1..32 rows, and the wider
// float32 instructions would spend 16 or 32 rows of matrix time on each 4 (6.7 us per layer and 16 rows; this: 1.7 us per
// 4 rows).  Lane l holds column l of 64 for 4 consecutive k; 4 rows of input for 64 k are one 16-byte read per lane, of
// which an instruction broadcasts the block that has its k.
#include "stack_exchange.h"

namespace lsq {

namespace {

// bytes per row / d
struct RegionF32 {
  static constexpr int xi = 0, qkv = 4, ctx = 16, os = 20, x1 = 36, qs = 40, ctx2 = 56, cs = 60, x2 = 76, ff = 80, fs = 96, size = 112;
};

// Weights [N][K] -> [N / 16][K / 4][16 columns][4 k]: what the wavefronts below load is contiguous.  Rows past N: zeros.
__global__ void __launch_bounds__(256) pack_f32_kernel(const floatx4* __restrict__ src, floatx4* __restrict__ dst, int N, int K4, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const size_t row = i / 16 / K4 * 16 + i % 16, k4 = i / 16 % K4;
  dst[i] = row < (size_t)N ? src[row * K4 + k4] : floatx4{0.f, 0.f, 0.f, 0.f};
}

// DK: d / 256.  NB: blocks of 4 rows a group has at most.
template <int DK, int NB>
__global__ void __launch_bounds__(kThreads) decoder_stack_f32_kernel(const StackArgs a) {
  constexpr int D = 256 * DK, H = D / 64, W = D / 16, R = 4 * NB, CG = D / 64;
  constexpr int TEAMS = NB, NSH = kWaves / TEAMS;                            // (row, head) pairs at once; wavefronts of each
  constexpr int U = 2;                                                       // keys of a lane group in flight
  constexpr int WE = D / 32, WQ = D / 128;                                   // 16-byte pieces per lane: an eighth of d of k, a 32nd
  constexpr int CHX = (R * D / 4 + kThreads - 1) / kThreads;                 // ... per thread: R rows of d floats
  constexpr int CHQ = (R * D / 16 + kThreads - 1) / kThreads;                // ... a quarter of them
  constexpr int EARLY = NB < 8 ? WE / 2 : 0;                                 // pieces of the second FFN matrix requested before the first one's product
  using Rg = RegionF32;

  __shared__ __attribute__((aligned(16))) float st[R][D + 16];               // staged input rows
  __shared__ __attribute__((aligned(16))) float part[kWaves][R][64];
  __shared__ __attribute__((aligned(16))) float xrow[D];                     // the residual of the row this workgroup owns
  __shared__ float stat[DK][2];
  __shared__ __attribute__((aligned(16))) float att_o[kWaves][64];
  __shared__ float att_m[kWaves], att_l[kWaves];

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, bid = blockIdx.x;
  const int grp = (bid >> 3) % G, jx = (bid >> 3) / G;
  const int j = (bid & 7) * (W / 8) + jx;   // neighbouring columns on one XCD: its L2 reads whole lines
  const int cg = j >> 2, ks = j & 3;
  const int rp = a.rows_per_group, r0 = grp * rp, rows = min(rp, a.M - r0);
  const int seq = a.state[0], start = seq & 1, dirty = a.state[1], pos = *a.tpos;
  const bool owner = j < rows;

  Exchange<> ex;
  ex.rsrc = __builtin_amdgcn_make_buffer_rsrc(a.exchange, (short)0, (int)(2 * a.set_bytes), 0x00027000);
  ex.polls = seq < 0 ? 1 : kSpinLimit;
  const int group_bytes = Rg::size * D * rp;
  auto at = [&](int l, int region) { return ((start + l) & 1) * (int)a.set_bytes + grp * group_bytes + region * D * rp; };
  const u32x4 s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
  auto put4 = [&](int l, int base, int lo, floatx4 v) {   // and reset the same place of the other slot
    u32x4 w = __builtin_bit_cast(u32x4, v);
    w = u32x4{publish_word(w.x), publish_word(w.y), publish_word(w.z), publish_word(w.w)};
    __builtin_amdgcn_raw_buffer_store_b128(w, ex.rsrc, lo, base, kAgent);
    __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, lo, base + (((start + l) & 1) ? -(int)a.set_bytes : (int)a.set_bytes), kAgent);
  };

  {   // the slot the last launch ended with: this group's part (needed from layer 1 on), and what no group of this launch has
    const int old = ((start + 1) & 1) * (int)a.set_bytes;
    const int mine_end = min(dirty, (grp + 1) * group_bytes);
    for (int o = grp * group_bytes + (j * kThreads + tid) * 16; o < mine_end; o += W * kThreads * 16)
      __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, o, old, kAgent);
    for (int o = G * group_bytes + (bid * kThreads + tid) * 16; o < dirty; o += (int)gridDim.x * kThreads * 16)
      __builtin_amdgcn_raw_buffer_store_b128(s4, ex.rsrc, o, old, kAgent);
  }

  // ---- weights: pieces of 4 k of column `lane` of 64
  floatx4 wq[WE], wo[WQ], w1[WE], w2[WE];
  auto layer_w = [&](const half_t* p, int l) { return reinterpret_cast<const char*>(p) + (size_t)l * a.packed_stride; };
  auto layer_p = [&](const half_t* p, int l) { return reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + (size_t)l * a.plain_stride); };
  unsigned l16 = (lane & 15) * 16, lq = lane >> 4;
  auto load = [&](auto& w, int first, int count, const char* Wp, int K, int unit, int unit_stride, int k4) {   // w[first..] from k = 4 (k4 + first)
    const char* p = Wp + (size_t)unit * K * 64 + (k4 + first) * 256;
    const unsigned lo = min((int)lq, unit_stride == 1 ? 3 : 2) * (unsigned)(unit_stride * K * 64) + l16;
#pragma unroll
    for (int i = 0; i < count; ++i) w[first + i] = *reinterpret_cast<const floatx4*>(p + i * 256 + lo);
  };
  auto load_qkv = [&](int l) { load(wq, 0, WE, layer_w(a.Wqkv, l), D, j, W, wave * WE); };   // 16 columns each of q, k, v
  auto load_quarter = [&](const half_t* Wp, int l) { load(wo, 0, WQ, layer_w(Wp, l), D, cg * 4, 1, ks * (D / 16) + wave * WQ); };
  auto load_ffn1 = [&](int l, int first, int count) { load(w1, first, count, layer_w(a.W1, l), D, j * 4, 1, wave * WE); };
  auto load_ffn2 = [&](int l, int first, int count) { load(w2, first, count, layer_w(a.W2, l), 4 * D, cg * 4, 1, ks * (D / 4) + wave * WE); };
  auto pin = [] { asm volatile("" ::: "memory"); };

  // ---- the owner's part: residual row + partial sums of a projection -> normalised row.  Thread t has columns 4t .. 4t+3.
  int oc = min(tid * 4, D - 4);
  auto own_norm = [&](int l, int region_in, const float* bias, const float* g, const float* b, int lout, int region_out, float* out_y) {
    if (!owner) return;
    const floatx4 bi = *reinterpret_cast<const floatx4*>(bias + oc), g4 = *reinterpret_cast<const floatx4*>(g + oc),
                  b4 = *reinterpret_cast<const floatx4*>(b + oc);
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    if (wave < DK) {
      u32x4 raw[4];
      const int base = at(l, region_in) + j * 256;
      const int lo = (oc >> 6) * (rp * 256) + (oc & 63) * 4;
      ex.wait<kLeadF32>([&](int i) { return base + i * (CG * 256) * rp; }, [&](int) { return lo; }, raw);
      v = *reinterpret_cast<const floatx4*>(&xrow[oc]) +
          ((((__builtin_bit_cast(floatx4, raw[0]) + __builtin_bit_cast(floatx4, raw[1])) + __builtin_bit_cast(floatx4, raw[2])) +
            __builtin_bit_cast(floatx4, raw[3])) + bi);
    }
    // mean and centred sum of squares of each wavefront's 256 values, then of the row
    const float sm = wave_sum((v[0] + v[1]) + (v[2] + v[3])) * (1.0f / 256);
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
    if (tid * 4 < D) {
      const floatx4 y = g4 * ((v - mean) * rstd) + b4;
      if (region_out >= 0) put4(lout, at(lout, region_out) + j * (D * 4), oc * 4, y);
      *reinterpret_cast<floatx4*>(&xrow[oc]) = y;
      if (out_y) *reinterpret_cast<floatx4*>(out_y + (size_t)(r0 + j) * D + oc) = y;
    }
    __syncthreads();
  };

  // ---- staging: all of a workgroup's accesses so far are acknowledged on the way
  auto stage = [&](auto& raw, int pieces, auto from, auto to) {   // piece p of 16 bytes: from(p) in the exchange, to(p) in LDS
    constexpr int N = sizeof(raw) / sizeof(raw[0]);
    ex.wait<kLeadF32>([&](int) { return 0; }, [&](int i) { return from(min(i * kThreads + tid, pieces - 1)); }, raw);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i * kThreads + tid < pieces) *reinterpret_cast<u32x4*>(to(i * kThreads + tid)) = raw[i];
    __syncthreads();
  };
  auto stage_rows = [&](auto& raw, int base, int cols) {   // rows of d floats, `cols` columns; rows the group does not have: its last one again
    const int per_row = cols / 4;
    stage(raw, R * per_row, [&](int p) { return base + min(p / per_row, rows - 1) * (D * 4) + p % per_row * 16; },
          [&](int p) { return &st[p / per_row][p % per_row * 4]; });
  };

  // ---- products: columns 0..63 of this workgroup's, staged columns from k0 on
  auto multiply = [&](const auto& w, int k0) {
    constexpr int N = sizeof(w) / sizeof(w[0]);
    floatx4 acc[NB];
    const float* src = &st[lane & 3][k0 + min(lane >> 2, N - 1) * 4];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
      const floatx4 x = *reinterpret_cast<const floatx4*>(src + b * 4 * (D + 16));
#define LSQ_K4(I) if constexpr (I < N) {                                                   \
        acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[0], w[I][0], acc[b], 4, I, 0);        \
        acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[1], w[I][1], acc[b], 4, I, 0);        \
        acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[2], w[I][2], acc[b], 4, I, 0);        \
        acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[3], w[I][3], acc[b], 4, I, 0); }
      LSQ_K4(0) LSQ_K4(1) LSQ_K4(2) LSQ_K4(3) LSQ_K4(4) LSQ_K4(5) LSQ_K4(6) LSQ_K4(7)
      LSQ_K4(8) LSQ_K4(9) LSQ_K4(10) LSQ_K4(11) LSQ_K4(12) LSQ_K4(13) LSQ_K4(14) LSQ_K4(15)
#undef LSQ_K4
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave][b * 4 + i][lane] = acc[b][i];
  };
  int um = tid >> 4, un = (tid & 15) * 4;   // four columns of a row per thread
  auto total = [&] {
    floatx4 v = *reinterpret_cast<const floatx4*>(&part[0][um][un]);
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += *reinterpret_cast<const floatx4*>(&part[w][um][un]);
    return v;
  };
  auto project_quarter = [&](int l, int region_in, int region_out, auto request) {   // ks-th quarter of k, 64 columns
    u32x4 raw[CHQ];
    stage_rows(raw, at(l, region_in) + ks * D, D / 4);
    multiply(wo, wave * (D / 32));
    request();
    pin();
    __syncthreads();
    if (um < rows) put4(l, at(l, region_out) + (ks * CG + cg) * rp * 256, um * 256 + un * 4, total());
  };

  // ---- attention: 16 lanes per key, four columns of the head each
  const int team = wave / NSH, ash = wave % NSH;
  int gk = lane >> 4, c4 = (lane & 15) * 4;
  const int pair = j + W * team, am = min(pair / H, rows - 1), ah = pair % H;
  const bool attends = pair < rows * H;
  const int arow = r0 + am, sent = arow / a.beam;
  const int jstep = 4 * NSH;
  int jfirst = ash + gk * NSH;
  const bool table = a.anc != nullptr;
  const int32_t* slots = table ? a.anc + (size_t)arow * a.anc_ld : nullptr;
  auto slot_of = [&](int p) { return table ? min(max(slots[p], 0), a.beam - 1) : 0; };
  int slot0[U];
#pragma unroll
  for (int u = 0; u < U; ++u) slot0[u] = slot_of(max(min(jfirst + u * jstep, pos - 1), 0));
  const int src_off = a.src_off[sent], src_len = a.src_len[sent];
  auto dot4 = [](const floatx4& x, const floatx4& y) { return (x[0] * y[0] + x[1] * y[1]) + (x[2] * y[2] + x[3] * y[3]); };
  floatx4 kn[U], vn[U];
  auto request_keys = [&](bool self, const float* Kb, const float* Vb, int nkeys, int jb) {
    const size_t own = self ? (size_t)(table ? sent * a.beam : arow) * a.T * D : 0;
    const char* Kh = reinterpret_cast<const char*>(Kb + own + ah * 64);
    const char* Vh = reinterpret_cast<const char*>(Vb + own + ah * 64);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && jb - gk * NSH + u * jstep >= nkeys) continue;
      const int p = max(min(jb + u * jstep, nkeys - 1), 0);
      const unsigned o = ((self ? ((jb == jfirst ? slot0[u] : slot_of(p)) * a.T + p) * D : p * (2 * D)) + c4) * 4u;
      kn[u] = *reinterpret_cast<const floatx4*>(Kh + o);
      vn[u] = *reinterpret_cast<const floatx4*>(Vh + o);
    }
  };
  // the first keys and values have been requested (request_keys from jfirst on) an exchange earlier
  auto attend = [&](int l, bool self, const float* Kb, const float* Vb, int nkeys, const float* bias_q) {
    if (attends) {
      constexpr float qscale = 0.125f * 1.44269504088896340736f;
      floatx4 q, knew, vnew;
      if (self) {
        u32x4 raw[3];
        const int base = at(l, Rg::qkv) + (ah * 4 * rp + am) * 192;
        ex.wait<kLeadF32>([&](int i) { return base + i * 64; }, [&](int) { return (c4 >> 4) * rp * 192 + (c4 & 15) * 4; }, raw);
        q = __builtin_bit_cast(floatx4, raw[0]); knew = __builtin_bit_cast(floatx4, raw[1]); vnew = __builtin_bit_cast(floatx4, raw[2]);
      } else {
        const floatx4 bq = *reinterpret_cast<const floatx4*>(bias_q + ah * 64 + c4);
        u32x4 raw[4];   // four slabs of the head's 64 columns
        const int base = at(l, Rg::qs) + (ah * rp + am) * 256;
        ex.wait<kLeadF32>([&](int i) { return base + i * (CG * 256) * rp; }, [&](int) { return c4 * 4; }, raw);
        q = (((__builtin_bit_cast(floatx4, raw[0]) + __builtin_bit_cast(floatx4, raw[1])) + __builtin_bit_cast(floatx4, raw[2])) +
             __builtin_bit_cast(floatx4, raw[3])) + bq;
      }
      float m = -INFINITY, z = 0.f;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      for (int jb = jfirst; jb - gk * NSH < nkeys; jb += U * jstep) {
        float sc[U], mx = m;
        floatx4 vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          sc[u] = -INFINITY;
          if (jb - gk * NSH + u * jstep >= nkeys) continue;
          const float s = group_sum<16>(dot4(q, kn[u])) * qscale;
          if (jb + u * jstep < nkeys) sc[u] = s;
          vv[u] = vn[u];
          mx = fmaxf(mx, sc[u]);
        }
        const int jn = jb + U * jstep;
        if (jn - gk * NSH < nkeys) request_keys(self, Kb, Vb, nkeys, jn);
        for_lane_bits<16>([&](auto bit) { mx = max_lane_xor<decltype(bit)::value>(mx); });
        const float corr = __builtin_amdgcn_exp2f(m - mx);
        m = mx;
        z *= corr;
        acc *= corr;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (jb - gk * NSH + u * jstep >= nkeys) continue;
          const bool live = jb + u * jstep < nkeys;
          const float p = live ? __builtin_amdgcn_exp2f(sc[u] - mx) : 0.f;
          z += p;
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] += p * (live ? vv[u][i] : 0.f);
        }
      }
      if (self && ash == NSH - 1) {
        const float s = group_sum<16>(dot4(q, knew)) * qscale, mx = fmaxf(m, s);
        const float corr = __builtin_amdgcn_exp2f(m - mx), p = gk == 0 ? __builtin_amdgcn_exp2f(s - mx) : 0.f;
        m = mx;
        z = z * corr + p;
        acc = acc * corr + p * vnew;
      }
      for_lane_bits<16>([&](auto bit) {
        constexpr int O = decltype(bit)::value;
        z = add_lane_xor<O>(z);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = add_lane_xor<O>(acc[i]);
      });
      if (gk == 0) {
        *reinterpret_cast<floatx4*>(&att_o[wave][c4]) = acc;
        if (lane == 0) { att_m[wave] = m; att_l[wave] = z; }
      }
    }
    __syncthreads();
    const int tm = tid >> 4, pr = j + W * tm;   // four values of a pair's context each
    if (tm < TEAMS && pr < rows * H) {
      float mx = -INFINITY, z = 0.f;
      floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NSH; ++w) mx = fmaxf(mx, att_m[tm * NSH + w]);
#pragma unroll
      for (int w = 0; w < NSH; ++w) {
        const float cw = __builtin_amdgcn_exp2f(att_m[tm * NSH + w] - mx);
        z += att_l[tm * NSH + w] * cw;
        o += *reinterpret_cast<const floatx4*>(&att_o[tm * NSH + w][un]) * cw;
      }
      const float inv = 1.0f / z;
      put4(l, at(l, self ? Rg::ctx : Rg::ctx2), pr / H * (D * 4) + (pr % H * 64 + un) * 4, o * inv);
    }
  };

  // ======== the layers.  A product's weights are requested in pieces between the exchanges before it: a poll is answered
  // after everything that was requested before it.
  load_qkv(0);
  for (int l = 0; l < a.layers; ++l) {
    // what is derived from a thread's place is derived anew in every layer instead of waiting in registers (it spills otherwise)
    asm volatile("" : "+v"(tid), "+v"(lane), "+v"(l16), "+v"(lq), "+v"(oc), "+v"(um), "+v"(un));
    asm volatile("" : "+v"(gk), "+v"(c4), "+v"(jfirst));
    float* Kc = reinterpret_cast<float*>(a.cache + (size_t)(2 * l) * a.cache_stride);
    float* Vc = reinterpret_cast<float*>(a.cache + (size_t)(2 * l + 1) * a.cache_stride);
    const float* kvb = reinterpret_cast<const float*>(a.cross + (size_t)l * a.cross_stride) + (size_t)src_off * 2 * D;
    if (l > 0) {
      own_norm(l - 1, Rg::fs, layer_p(a.b2, l - 1), layer_p(a.ln3g, l - 1), layer_p(a.ln3b, l - 1), l, Rg::xi, nullptr);
    } else if (owner) {
      if (tid * 4 < D) {
        const floatx4 h = *reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(a.x0) + (size_t)(r0 + j) * D + oc);
        *reinterpret_cast<floatx4*>(&xrow[oc]) = h;
        put4(l, at(l, Rg::xi) + j * (D * 4), oc * 4, h);
      }
      __syncthreads();
    }
    // q, k, v
    {
      const int seg = un >> 4, qc = j * 16 + (un & 15);
      const bool qlive = seg < 3 && um < rows;
      floatx4 qb = {0.f, 0.f, 0.f, 0.f};
      if (qlive) qb = *reinterpret_cast<const floatx4*>(layer_p(a.bqkv, l) + seg * D + qc);
      if (attends) request_keys(true, Kc, Vc, pos, jfirst);   // needs nothing of this step
      pin();
      u32x4 raw[CHX];
      stage_rows(raw, at(l, Rg::xi), D);
      multiply(wq, wave * (D / 8));
      load_quarter(a.Wo, l);
      load_ffn1(l, 0, WE / 4);
      pin();
      __syncthreads();
      if (qlive) {
        const floatx4 v = total() + qb;
        put4(l, at(l, Rg::qkv) + j * rp * 192, um * 192 + un * 4, v);
        if (seg > 0) *reinterpret_cast<floatx4*>((seg == 1 ? Kc : Vc) + ((size_t)(r0 + um) * a.T + pos) * D + qc) = v;
      }
    }
    attend(l, true, Kc, Vc, pos, nullptr);
    project_quarter(l, Rg::ctx, Rg::os, [&] { load_quarter(a.Wq, l); load_ffn1(l, WE / 4, WE / 4); });
    own_norm(l, Rg::os, layer_p(a.bo, l), layer_p(a.ln1g, l), layer_p(a.ln1b, l), l, Rg::x1, nullptr);
    if (attends) request_keys(false, kvb, kvb + D, src_len, jfirst);
    pin();
    project_quarter(l, Rg::x1, Rg::qs, [&] { load_quarter(a.Woc, l); load_ffn1(l, WE / 2, WE / 4); });
    attend(l, false, kvb, kvb + D, src_len, layer_p(a.bq, l));
    project_quarter(l, Rg::ctx2, Rg::cs, [&] { load_ffn1(l, WE * 3 / 4, WE / 4); load_ffn2(l, 0, EARLY); });
    own_norm(l, Rg::cs, layer_p(a.boc, l), layer_p(a.ln2g, l), layer_p(a.ln2b, l), l, Rg::x2, nullptr);
    // FFN
    {
      floatx4 fb = {0.f, 0.f, 0.f, 0.f};
      if (um < rows) fb = *reinterpret_cast<const floatx4*>(layer_p(a.b1, l) + j * 64 + un);
      u32x4 raw[CHX];
      stage_rows(raw, at(l, Rg::x2), D);
      multiply(w1, wave * (D / 8));
      load_ffn2(l, EARLY, WE - EARLY);
      pin();
      __syncthreads();
      if (um < rows) {
        floatx4 v = total() + fb;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
        put4(l, at(l, Rg::ff) + j * rp * 256, um * 256 + un * 4, v);
      }
    }
    {
      u32x4 raw[CHX];   // [64 columns][row]: the d columns of this workgroup's quarter
      const int base = at(l, Rg::ff) + ks * (W / 4) * rp * 256;
      stage(raw, R * D / 4, [&](int p) { return base + p / (16 * R) * (rp * 256) + min(p % (16 * R) >> 4, rows - 1) * 256 + (p & 15) * 16; },
            [&](int p) { return &st[p % (16 * R) >> 4][p / (16 * R) * 64 + (p & 15) * 4]; });
      multiply(w2, wave * (D / 8));
      if (l + 1 < a.layers) load_qkv(l + 1);
      pin();
      __syncthreads();
      if (um < rows) put4(l, at(l, Rg::fs) + (ks * CG + cg) * rp * 256, um * 256 + un * 4, total());
    }
  }
  const int last = a.layers - 1;
  own_norm(last, Rg::fs, layer_p(a.b2, last), layer_p(a.ln3g, last), layer_p(a.ln3b, last), last, -1, reinterpret_cast<float*>(a.hidden));
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

struct ChoiceF32 { const void* kernel; int groups, rows, nb; };

// As many groups as 256 CUs hold: they share the weights through the L2 of their XCD, and a row costs matrix time.
// A whole translation at d = 512, beam 4, against separate launches (ms): 1 sentence 14.3 / 38.2, 8 19.7 / 53.7, 32 32.9 / 83.3,
// 50 with beam 5 (250 rows) 49.9 / 94.4: at short histories it wins wherever it fits.
ChoiceF32 choose_f32(int M, int d) {
  ChoiceF32 c = {};
  c.groups = min(256 / (d / 16), M);
  c.rows = (M + c.groups - 1) / c.groups;
  c.groups = (M + c.rows - 1) / c.rows;
  const int nb = c.nb = c.rows <= 4 ? 1 : c.rows <= 8 ? 2 : c.rows <= 16 ? 4 : c.rows <= min(32, d / 16) ? 8 : 0;
#define LSQ_F32(DKV, NBV) if (d == 256 * DKV && nb == NBV) c.kernel = (const void*)decoder_stack_f32_kernel<DKV, NBV>
  LSQ_F32(1, 1); LSQ_F32(1, 2); LSQ_F32(1, 4); LSQ_F32(2, 1); LSQ_F32(2, 2); LSQ_F32(2, 4); LSQ_F32(2, 8);
#undef LSQ_F32
  return c;
}

}  // namespace

size_t stack_f32_bytes(int M, int d) { return (size_t)(min(M, 8192 / (d / 16)) + 32) * RegionF32::size * d; }

bool stack_f32_shape_supported(int dtype, int arch, int H, int d, int F) {
  return dtype == DT_F32 && arch == 0 && (d == 256 || d == 512) && H * 64 == d && F == 4 * d;
}

// Where the attention of long histories makes it fall behind: a (row, head) pair has 64 / NB keys in flight, the separate
// kernels have more and read what the rows of a sentence share once.  Whole steps in us, this kernel / separate launches, beam 4
// (position 16, 496, 1008, 1900):
//   d = 512:   4 rows 149 / 427, 218 / 495, 297 / 544, 467 / 600 (2900: 665 / 683); 64 rows 216 / 802, 422 / 956, 633 / 1098, 970 / 1246
//            128 rows 298 / 762, 684 / 1071, 1097 / 1344, 1723 / 1651; 192 rows 425 / 827, 1138 / 1286, 1877 / 1716, 3078 / 2279
//            256 rows 489 / 869, 1284 / 1410, 2085 / 1932, 3349 / 2569; position 16, sources of 500 885 / 1016, of 2000 2196 / 1435
//   d = 256:  64 rows 140 / 469, 216 / 561, 313 / 623, 483 / 698; 256 rows 251 / 546, 569 / 716, 916 / 857, 1535 / 1109
// One row per sentence (nothing shared), d = 512: 128 rows 303 / 774 .. 1455 / 1760, 200 rows 457 / 797, 1014 / 1222, 1580 / 1636, 2543 / 2340
bool stack_f32_supported(int M, int d, int beam, int pos, int src) {
  if (M < 1) return false;
  const ChoiceF32 c = choose_f32(M, d);
  if (!c.kernel || !resident(c.kernel)) return false;
  const int len = pos + src * c.nb / 8;
  if (beam > 1) return len <= (c.nb <= 2 ? 3000 : c.nb == 8 ? 730 : d == 512 ? 1650 : 850);
  return c.nb < 8 || len <= 1200;
}

size_t pack_f32_bytes(int N, int K) { return (size_t)(N + 63) / 64 * 64 * K * 4; }

hipError_t launch_pack_f32(const void* plain, void* packed, int N, int K, hipStream_t s) {
  const size_t n = pack_f32_bytes(N, K) / 16;
  pack_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const floatx4*)plain, (floatx4*)packed, N, K / 4, n);
  return hipGetLastError();
}

hipError_t launch_decoder_stack_f32(const StackArgs& args, int d, hipStream_t s) {
  const ChoiceF32 c = choose_f32(args.M, d);
  if (!c.kernel) return hipErrorInvalidValue;
  StackArgs a = args;
  a.groups = c.groups;
  a.rows_per_group = c.rows;
  void* kargs[] = {&a};
  return hipLaunchKernel(c.kernel, dim3(d / 16 * c.groups), dim3(kThreads), kargs, 0, s);
}

}  // namespace lsq
