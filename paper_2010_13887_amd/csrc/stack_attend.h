// Attention of one row and head over up to eight wavefronts, as the decoder stack kernels do it: a lane group of 8 holds a key's
// 64 values, a wavefront has 32 keys in flight, four per lane group.
#pragma once
#include "stack_exchange.h"

namespace lsq {

namespace {

typedef half_t half2_t __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kTrip = 4;               // keys of a lane group in flight
constexpr int kTripKeys = 8 * kTrip;   // ... of a wavefront

// error against 64 bits: that of a chain of float multiply-adds
__device__ __forceinline__ float dot8(const half8_t& x, const half8_t& y) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_fdot2(half2_t{x[2 * i], x[2 * i + 1]}, half2_t{y[2 * i], y[2 * i + 1]}, s, false);
  return s;
}

// Sums over the eight lane groups of values that belong to columns c8 .. c8 + 7 in each: a lane is left with two of them,
// own_column() and the next, in v[0] and v[1].  FAR: lane groups 32 lanes apart first (14 instructions; all eight in every lane
// would be 72), otherwise neighbours first (20).  The two round differently; which is whose: see Attention.
template <bool FAR>
__device__ __forceinline__ void column_sums(float (&v)[8]) {
  auto add32 = [&](int i, int k) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v[i]), __builtin_bit_cast(unsigned, v[k]), false, false);
    const unsigned x = r[0], y = r[1];
    v[i] = __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
  };
  auto add16 = [&](int i, int k) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v[i]), __builtin_bit_cast(unsigned, v[k]), false, false);
    const unsigned x = r[0], y = r[1];
    v[i] = __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
  };
  if constexpr (FAR) {
#pragma unroll
    for (int i = 0; i < 4; ++i) add32(i, i + 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) add16(i, i + 2);
    v[0] = add_lane_xor<8>(v[0]);
    v[1] = add_lane_xor<8>(v[1]);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = add_lane_xor<8>(v[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) add16(i, i + 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) add32(i, i + 2);
  }
}
template <bool FAR>
__device__ __forceinline__ int own_column(int lane) {   // of the head's 64
  return (lane & 7) * 8 + (FAR ? (lane >> 4 & 1) * 2 + (lane >> 5) * 4 : (lane >> 4 & 1) * 4 + (lane >> 5) * 2);
}

// Wavefronts of a team of NSH that look at keys, die kernel: 32 keys each, as long as there are enough of them.
template <int NSH>
__device__ __forceinline__ int team_for(int nkeys) { return min(nkeys <= 32 ? 1 : nkeys <= 64 ? 2 : nkeys <= 128 ? 4 : 8, NSH); }

// A wavefront's share: maximum of its scores (in units of log 2), sum of their exponentials, weighted sum of its values.  The chain of
// instructions, not their number, is what counts for a wavefront that has its SIMD to itself, so a trip is code without branches: keys past
// the last are that one again, and weigh nothing.  live(u): whether key u of the lane group's four is one of the history.
//
// The order of every sum is part of what a kernel gives: a context's last bit turns a draw between two tokens whose cumulative
// weights meet the random number, and that row's text is another one from there on (2 of 30 requests of 60 rows of GPT-2-small's shape,
// top-8, with sums of the same precision in another order).  So it is written out, with multiply-adds in so many words: keys in
// order within a lane group, the new position last and against the maximum so far, lane groups as the kernel says (FAR), wavefronts in
// order, and one division.
struct Attention {
  static constexpr float kScale = 0.125f * 1.44269504088896340736f;
  static constexpr float kLowest = -3.0e38f;   // of a wavefront without a key: finite, so that nothing weighs 0 and not NaN
  float m, z, acc[8], fresh;

  // The first trip, of N keys per lane group.  SELF: also the score of the new position, which is not in the cache yet; `empty`: there is
  // nothing else, and what the cache holds was never written.  next(): once the keys are not needed any more.
  template <bool SELF, int N = kTrip, typename L, typename F>
  __device__ __forceinline__ void first(const half8_t& q, const half8_t (&kn)[kTrip], const half8_t (&vn)[kTrip], const half8_t& knew, bool empty, L live,
                                        F next) {
#pragma clang fp contract(off)
    float sc[N], p[N];
    half8_t vv[N];
    scores<N>(q, kn, vn, live, sc, vv);
    if constexpr (SELF) fresh = group_sum<8>(dot8(q, knew));
    next();
    m = kLowest;
#pragma unroll
    for (int u = 0; u < N; ++u) m = fmaxf(m, sc[u]);
    if constexpr (SELF) {
      if (empty) {
#pragma unroll
        for (int u = 0; u < N; ++u) vv[u] = half8_t{};
      }
    }
    for_lane_bits<8>([&](auto bit) { m = max_lane_xor<decltype(bit)::value>(m); });
#pragma unroll
    for (int u = 0; u < N; ++u) p[u] = __builtin_amdgcn_exp2f(sc[u] - m);
    z = p[0];
#pragma unroll
    for (int u = 1; u < N; ++u) z += p[u];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = p[0] * (float)vv[0][i];
#pragma unroll
      for (int u = 1; u < N; ++u) acc[i] = fmaf(p[u], (float)vv[u][i], acc[i]);
    }
  }
  template <typename L, typename F>
  __device__ __forceinline__ void more(const half8_t& q, const half8_t (&kn)[kTrip], const half8_t (&vn)[kTrip], L live, F next) {
#pragma clang fp contract(off)
    float sc[kTrip], p[kTrip];
    half8_t vv[kTrip];
    scores<kTrip>(q, kn, vn, live, sc, vv);
    next();
    float mx = fmaxf(fmaxf(m, fmaxf(sc[0], sc[1])), fmaxf(sc[2], sc[3]));
    for_lane_bits<8>([&](auto bit) { mx = max_lane_xor<decltype(bit)::value>(mx); });
    const float corr = __builtin_amdgcn_exp2f(m - mx);
    m = mx;
#pragma unroll
    for (int u = 0; u < kTrip; ++u) p[u] = __builtin_amdgcn_exp2f(sc[u] - m);
    z = ((fmaf(z, corr, p[0]) + p[1]) + p[2]) + p[3];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = fmaf(acc[i], corr, p[0] * (float)vv[0][i]);
#pragma unroll
      for (int u = 1; u < kTrip; ++u) acc[i] = fmaf(p[u], (float)vv[u][i], acc[i]);
    }
  }
  // the new position, by one wavefront of the team and behind its last trip; mine: one of the lane groups, which counts it
  __device__ __forceinline__ void add(const half8_t& vnew, bool mine) {
#pragma clang fp contract(off)
    const float mx = fmaxf(m, fresh * kScale), corr = __builtin_amdgcn_exp2f(m - mx);
    const float p = mine ? __builtin_amdgcn_exp2f(fmaf(fresh, kScale, -mx)) : 0.f;
    m = mx;
    z = fmaf(z, corr, p);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = fmaf(acc[i], corr, p * (float)vnew[i]);
  }
  // over the lane groups: columns own_column() and the next in acc[0] and acc[1]
  template <bool FAR>
  __device__ __forceinline__ void sum() {
    column_sums<FAR>(acc);
    for_lane_bits<8>([&](auto bit) { z = add_lane_xor<decltype(bit)::value>(z); });
  }

 private:
  template <int N, typename L>
  static __device__ __forceinline__ void scores(const half8_t& q, const half8_t (&kn)[kTrip], const half8_t (&vn)[kTrip], L live, float (&sc)[N],
                                                half8_t (&vv)[N]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int u = 0; u < N; ++u) sc[u] = dot8(q, kn[u]);
#pragma unroll
    for (int u = 0; u < N; ++u) sc[u] = group_sum<8>(sc[u]) * kScale;
#pragma unroll
    for (int u = 0; u < N; ++u) { sc[u] = live(u) ? sc[u] : -INFINITY; vv[u] = vn[u]; }
  }
};

// Two values of a context.  Product and rounding are two steps: left to itself the compiler makes them one instruction here and
// there, which rounds once.
__device__ __forceinline__ half2_t context_of(float a, float b, float z) {
  const float inv = 1.0f / z;
  float v0 = a * inv, v1 = b * inv;
  asm("" : "+v"(v0), "+v"(v1));
  return half2_t{(half_t)v0, (half_t)v1};
}

// What the wavefronts of a team leave each other in LDS: the first of them adds the shares up.  Nobody else waits: a word per
// wavefront says how many attentions it has left its share of.
struct Shares {
  float o[kWaves][64], m[kWaves], l[kWaves];
  int left[kWaves];

  template <bool FAR>
  __device__ __forceinline__ void leave(int w, int lane, const Attention& t) {
    *reinterpret_cast<floatx2*>(&o[w][own_column<FAR>(lane)]) = floatx2{t.acc[0], t.acc[1]};
    if (lane == 0) { m[w] = t.m; l[w] = t.z; }
  }
  __device__ __forceinline__ void tell(int w, int attentions) {   // LDS takes a wavefront's stores in order
    __hip_atomic_store(&left[w], attentions, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // the team's first wavefront w; n: 2, 4 or 8.  Columns c and c + 1.
  template <int NSH>
  __device__ __forceinline__ half2_t collect(int w, int n, int attentions, int lane, int c) {
    while (!__all(__hip_atomic_load(&left[w + max(min(lane, n - 1), 1)], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= attentions)) {}
    float v0 = 0.f, v1 = 0.f, zt = 0.f;
    auto merge = [&](auto parts) {
#pragma clang fp contract(off)
      constexpr int P = decltype(parts)::value;
      if constexpr (P <= NSH) {
        float pm[P], pl[P], mx = -INFINITY;
        floatx2 po[P];
#pragma unroll
        for (int i = 0; i < P; ++i) { pm[i] = m[w + i]; pl[i] = l[w + i]; po[i] = *reinterpret_cast<const floatx2*>(&o[w + i][c]); }
#pragma unroll
        for (int i = 0; i < P; ++i) asm volatile("" : "+v"(pm[i]), "+v"(pl[i]), "+v"(po[i]));   // all requested before the first is used
#pragma unroll
        for (int i = 0; i < P; ++i) mx = fmaxf(mx, pm[i]);
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const float cw = __builtin_amdgcn_exp2f(pm[i] - mx);
          zt = fmaf(pl[i], cw, zt);
          v0 = fmaf(po[i][0], cw, v0);
          v1 = fmaf(po[i][1], cw, v1);
        }
      }
    };
    if (n == 2) merge(std::integral_constant<int, 2>{});
    else if (n == 4) merge(std::integral_constant<int, 4>{});
    else merge(std::integral_constant<int, 8>{});
    return context_of(v0, v1, zt);
  }
};

}  // namespace

}  // namespace lsq
