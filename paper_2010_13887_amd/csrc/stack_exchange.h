// What the decoder stack kernels hand each other intermediates with (see kernels_stack.hip).
#pragma once
#include <unordered_map>

#include "lsq_internal.h"

namespace lsq {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned kSentinel = 0xFFFFFFFFu;
constexpr int kAgent = 16;             // cache policy of agent scope: sc1
constexpr int kWorkgroup = 1;          // ... of workgroup scope: sc0
constexpr int kSpinLimit = 1 << 19;    // polls of about a microsecond
constexpr int kThreads = 512, kWaves = 8;
// A wait starts when there is nothing left to do, long before the value can be there: what is looked for too early is in the way of the stores it
// waits for and of the weights, and comes back behind them.  So the first look is LEAD times 64 clocks late.  Whole passes in ms with 0 / 4 / 8 / 12 / 16 /
// 20: Transformer-big, 1 sentence 11.76 11.51 11.10 10.90 10.85 10.90, 32 sentences 28.7 28.2 28.0 27.7 27.7 27.8; decoder-only, d = 768, 1 row 10.2 9.98
// 9.56 9.45 9.6 10.1, 32 rows 30.95 30.4 29.5 29.3 29.2 29.4.  Stage by stage the groups of 16 and 32 rows gain 0.5 to 1 % with 18 where
// keys of a large group or the FFN's activations are waited for.  float32, whose layers are 135 us of products, has little to gain: 0 against 4, two runs
// of each within 0.1 %: d = 512, 32 rows 17.89 -> 17.77 and 12.40 -> 12.30 ms, 64 rows 15.03 -> 14.95, 128 rows level, 1 row 11.10 -> 11.14; d = 256, 32 rows
// 9.31 -> 9.36, 132 rows 14.29 -> 14.25; with 8 and more 17.9 to 18.4.
constexpr int kLead = 12, kLeadF32 = 4;

__device__ __forceinline__ unsigned publish_word(unsigned v) { return v == kSentinel ? 0x7FFF7FFFu : v; }   // one NaN for another

// The pointers of a layer are read where they are used (see arguments): 60 scalar registers less to spill.  Layers of a step
// in groups of 8 rows: d = 512, 4 rows 92.9 -> 91.6 us, 32 rows 114.3 -> 112.3; the kernel for float32 lost up to 1 % by it and
// keeps its own.
__device__ __forceinline__ const __attribute__((address_space(4))) StackArgs* now() { return arguments<StackArgs>(); }

// Set in the first word of StackArgs::state at the end of a launch in which a wait ran out (the word the kernels read first
// anyway: a word of its own cost 0.5 us a step).  A launch that finds it set looks once where it would wait: the steps queued
// behind the one that gave up end at once instead of each waiting out the limit.
constexpr int kGaveUp = (int)0x80000000u;

__device__ __forceinline__ void give_up(int32_t* state, int* error) {   // tells the launches behind this one, and the host
  __hip_atomic_fetch_or(state, kGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Byte offsets of a row's intermediates inside one layer's region (d: row width): kernels in which every workgroup normalises
template <bool PRE> struct Region {
  static constexpr int qkv = 0, ctx = 6, u1 = 8;
  static constexpr int q2 = PRE ? 0 : 12, ctx2 = PRE ? 0 : 14, u2 = PRE ? 0 : 16;   // cross-attention: post-LN models
  static constexpr int ff = PRE ? 10 : 20, u3 = PRE ? 18 : 28, size = PRE ? 20 : 32;
};

// STORE: cache policy of what is published; kWorkgroup where all readers are on the writer's die (kernels_stack_die.hip)
template <int STORE = kAgent>
struct Exchange {
  static_assert(STORE == kAgent || STORE == kWorkgroup, "a store without a scope need not reach another compute unit before the kernel ends");
  __amdgpu_buffer_rsrc_t rsrc;
  int polls;   // of a wait; 1: one has run out, what this wavefront reads from now on may be missing

  // v[i] = the 16 bytes at base(i) + lane(i) once all of them have been written (base: the same in all lanes).  LEAD: units of
  // 64 clocks before the first look, see kLead.
  template <int LEAD, int N, typename B, typename L>
  __device__ __forceinline__ void wait(B base, L lane, u32x4 (&v)[N]) {
    if constexpr (LEAD > 0) {
      __builtin_amdgcn_s_sleep(LEAD);
      asm volatile("" ::: "memory");
    }
    for (int left = polls;;) {
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
    polls = 1;
  }
  // at the end of the kernel
  __device__ __forceinline__ void report(int32_t* state, int* error) {
    if (polls == 1) give_up(state, error);
  }
  __device__ __forceinline__ void put(int base, int lane, unsigned v) {
    __builtin_amdgcn_raw_buffer_store_b32(publish_word(v), rsrc, lane, base, STORE);
  }
  __device__ __forceinline__ void put2(int base, int lane, float a, float b) {   // 8 bytes
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 w = {publish_word(__builtin_bit_cast(unsigned, a)), publish_word(__builtin_bit_cast(unsigned, b))};
    __builtin_amdgcn_raw_buffer_store_b64(w, rsrc, lane, base, STORE);
  }
  __device__ __forceinline__ void put2(int base, int lane, half_t a, half_t b) {
    typedef half_t half2_t __attribute__((ext_vector_type(2)));
    put(base, lane, __builtin_bit_cast(unsigned, half2_t{a, b}));
  }
};

// Whether every workgroup of a launch of 256 is resident at once on the current device, as far as the device goes; whether
// the stream has all of it: stream_has_every_cu.
inline bool resident(const void* kernel, int threads = kThreads) {
  static std::unordered_map<const void*, bool> known;
  const auto it = known.find(kernel);
  if (it != known.end()) return it->second;
  int dev = 0, cus = 0, per_cu = 0;
  const bool ok = hipGetDevice(&dev) == hipSuccess &&
                  hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                  hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) == hipSuccess && cus * per_cu >= 256;
  known[kernel] = ok;
  return ok;
}

}  // namespace

}  // namespace lsq
