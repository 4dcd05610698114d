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
// own_column() and the next, in v[0] and v[1] (14 instructions; all eight in every lane would be 72).
__device__ __forceinline__ void column_sums(float (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v[i]), __builtin_bit_cast(unsigned, v[i + 4]), false, false);
    const unsigned x = r[0], y = r[1];
    v[i] = __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v[i]), __builtin_bit_cast(unsigned, v[i + 2]), false, false);
    const unsigned x = r[0], y = r[1];
    v[i] = __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
  }
  v[0] = add_lane_xor<8>(v[0]);
  v[1] = add_lane_xor<8>(v[1]);
}
__device__ __forceinline__ int own_column(int lane) { return (lane & 7) * 8 + (lane >> 4 & 1) * 2 + (lane >> 5) * 4; }   // of the head's 64

// Wavefronts of a team of NSH that look at keys: 32 keys each, as long as there are enough of them.
template <int NSH>
__device__ __forceinline__ int team_for(int nkeys) { return min(nkeys <= 32 ? 1 : nkeys <= 64 ? 2 : nkeys <= 128 ? 4 : 8, NSH); }

__device__ __forceinline__ float inverse(float v) {   // one Newton step; v is at least 1
  const float r = __builtin_amdgcn_rcpf(v);
  return fmaf(fmaf(-v, r, 1.0f), r, r);
}

// A wavefront's share: maximum of its scores (in units of log 2), sum of their exponentials, weighted sum of its values.  The chain of
// instructions, not their number, is what counts for a wavefront that has its SIMD to itself, so a trip is code without branches: keys past
// the last are that one again, and weigh nothing.  live(u): whether key u of the lane group's four is one of the history.
struct Attention {
  static constexpr float kScale = 0.125f * 1.44269504088896340736f;
  float m, z, acc[8];

  // The first trip.  SELF: also the new position, which is not in the cache yet, where `add` (one lane group of one wavefront);
  // `empty`: there is nothing else, and what the cache holds was never written.  next(): once the keys are not needed any more.
  template <bool SELF, typename L, typename F>
  __device__ __forceinline__ void first(const half8_t& q, const half8_t (&kn)[kTrip], const half8_t (&vn)[kTrip], const half8_t& knew, const half8_t& vnew,
                                        bool add, bool empty, L live, F next) {
    float sc[kTrip + 1], p[kTrip + 1];
    half8_t vv[kTrip];
#pragma unroll
    for (int u = 0; u < kTrip; ++u) sc[u] = dot8(q, kn[u]);
    if constexpr (SELF) sc[kTrip] = dot8(q, knew);
#pragma unroll
    for (int u = 0; u < kTrip + SELF; ++u) sc[u] = group_sum<8>(sc[u]) * kScale;
#pragma unroll
    for (int u = 0; u < kTrip; ++u) { sc[u] = live(u) ? sc[u] : -INFINITY; vv[u] = vn[u]; }
    next();
    m = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    if constexpr (SELF) {
      sc[kTrip] = add ? sc[kTrip] : -INFINITY;
      m = fmaxf(m, sc[kTrip]);
      if (empty) {
#pragma unroll
        for (int u = 0; u < kTrip; ++u) vv[u] = half8_t{};
      }
    }
    for_lane_bits<8>([&](auto bit) { m = max_lane_xor<decltype(bit)::value>(m); });   // finite: the wavefront has a key
#pragma unroll
    for (int u = 0; u < kTrip + SELF; ++u) p[u] = __builtin_amdgcn_exp2f(sc[u] - m);
    z = (p[0] + p[1]) + (p[2] + p[3]);
    if constexpr (SELF) z += p[kTrip];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = p[0] * (float)vv[0][i];
#pragma unroll
      for (int u = 1; u < kTrip; ++u) acc[i] += p[u] * (float)vv[u][i];
      if constexpr (SELF) acc[i] += p[kTrip] * (float)vnew[i];
    }
  }
  template <typename L, typename F>
  __device__ __forceinline__ void more(const half8_t& q, const half8_t (&kn)[kTrip], const half8_t (&vn)[kTrip], L live, F next) {
    float sc[kTrip], p[kTrip];
    half8_t vv[kTrip];
#pragma unroll
    for (int u = 0; u < kTrip; ++u) sc[u] = dot8(q, kn[u]);
#pragma unroll
    for (int u = 0; u < kTrip; ++u) sc[u] = group_sum<8>(sc[u]) * kScale;
#pragma unroll
    for (int u = 0; u < kTrip; ++u) { sc[u] = live(u) ? sc[u] : -INFINITY; vv[u] = vn[u]; }
    next();
    float mx = fmaxf(fmaxf(m, fmaxf(sc[0], sc[1])), fmaxf(sc[2], sc[3]));
    for_lane_bits<8>([&](auto bit) { mx = max_lane_xor<decltype(bit)::value>(mx); });
    const float corr = __builtin_amdgcn_exp2f(m - mx);
    m = mx;
#pragma unroll
    for (int u = 0; u < kTrip; ++u) p[u] = __builtin_amdgcn_exp2f(sc[u] - m);
    z = z * corr + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] *= corr;
#pragma unroll
      for (int u = 0; u < kTrip; ++u) acc[i] += p[u] * (float)vv[u][i];
    }
  }
  // over the lane groups: columns own_column() and the next in acc[0] and acc[1]
  __device__ __forceinline__ void sum() {
    column_sums(acc);
    for_lane_bits<8>([&](auto bit) { z = add_lane_xor<decltype(bit)::value>(z); });
  }
};

// What the wavefronts of a team leave each other in LDS: the first of them adds the shares up.  Nobody else waits: a word per
// wavefront says how many attentions it has left its share of.
struct Shares {
  float o[kWaves][64], m[kWaves], l[kWaves];
  int left[kWaves];

  __device__ __forceinline__ void leave(int w, int lane, const Attention& t) {
    *reinterpret_cast<floatx2*>(&o[w][own_column(lane)]) = floatx2{t.acc[0], t.acc[1]};
    if (lane == 0) { m[w] = t.m; l[w] = t.z; }
  }
  __device__ __forceinline__ void tell(int w, int attentions) {   // LDS takes a wavefront's stores in order
    __hip_atomic_store(&left[w], attentions, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // the team's first wavefront w; n: 2, 4 or 8.  Columns c and c + 1.
  template <int NSH>
  __device__ __forceinline__ void collect(int w, int n, int attentions, int lane, int c, float& v0, float& v1) {
    while (!__all(__hip_atomic_load(&left[w + max(min(lane, n - 1), 1)], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= attentions)) {}
    auto merge = [&](auto parts) {
      constexpr int P = decltype(parts)::value;
      if constexpr (P <= NSH) {
        float pm[P], pl[P], mx = -INFINITY, zt = 0.f;
        floatx2 po[P];
        v0 = 0.f; v1 = 0.f;
#pragma unroll
        for (int i = 0; i < P; ++i) { pm[i] = m[w + i]; pl[i] = l[w + i]; po[i] = *reinterpret_cast<const floatx2*>(&o[w + i][c]); }
#pragma unroll
        for (int i = 0; i < P; ++i) asm volatile("" : "+v"(pm[i]), "+v"(pl[i]), "+v"(po[i]));   // all requested before the first is used
#pragma unroll
        for (int i = 0; i < P; ++i) mx = fmaxf(mx, pm[i]);
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const float cw = __builtin_amdgcn_exp2f(pm[i] - mx);
          zt += pl[i] * cw;
          v0 += po[i][0] * cw;
          v1 += po[i][1] * cw;
        }
        const float inv = inverse(zt);
        v0 *= inv; v1 *= inv;
      }
    };
    if (n == 2) merge(std::integral_constant<int, 2>{});
    else if (n == 4) merge(std::integral_constant<int, 4>{});
    else merge(std::integral_constant<int, 8>{});
  }
};

}  // namespace

}  // namespace lsq
