// One step of beam search with a small model as ONE launch: decoder layers, vocabulary product, retrieve and re-rank.
// (Encoder-decoder, d and d_ffn multiples of 64 up to 128 and 512, heads of 16 or 32, vocabulary matrix up to 128 K values.)
//
// A sentence's hypotheses meet no other sentence within a step, and all weights of such a model (230 KB a layer at d = 64,
// float32) pass through one CU's load path in a few microseconds.  So a workgroup takes a sentence through the whole step
// with its rows in LDS: no exchange between workgroups, no launch boundary.  As 15 launches a step of the model with
// d = 64 took 58 us, 4.8 us per product and 5.4 us from one to the next.  Here: 27 us, of which the vocabulary 5 (one CU's load
// path), the search 5, the attentions 2.3 each and the products with what follows them 1.5 to 2 each; bound by the length of
// the chain of instructions.  A translation of 8 steps (2 sentences, beam 4, float32) 535 -> 392 us.
// The steps of a translation share launches: a workgroup goes from one to the next by itself, until its sentence is finished, and
// finds its weights, histories and keys where it left them (8 steps 329 -> 310 us: what lay between two launches).
//
// Products: 4x4 matrix instructions of 16 blocks (one row block: 4 hypotheses; a lane holds one of 64 columns), k split
// over the wavefronts that 64-column units leave idle, added through LDS.  The next product's weights are requested before
// the current one's results are awaited.
#include "search_device.h"

namespace lsq {

namespace {

constexpr int kThreads = 512, kWaves = 8, kParts = 8;
constexpr int kD = 128, kF = 512;   // widest rows

template <typename T> struct Piece;   // consecutive k of one column
template <> struct Piece<float> {
  using vec = floatx4;
  static constexpr int n = 4, stride = 64;   // next piece of the same column in the copy of launch_pack_f32
  __device__ static __forceinline__ const float* at(const float* W, int K, int unit, int k, int lane, int = 0) {
    return W + ((size_t)(unit * 4 + (lane >> 4)) * (K / 4) + k / 4) * 64 + (lane & 15) * 4;
  }
  __device__ static __forceinline__ floatx4 mul(const vec& x, const vec& w, floatx4 acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x[i], w[i], acc, 0, 0, 0);
    return acc;
  }
};
template <> struct Piece<half_t> {
  using vec = half8_t;
  static constexpr int n = 8, stride = 256;   // ... of launch_pack_weights
  __device__ static __forceinline__ const half_t* at(const half_t* W, int K, int unit, int k, int lane, int blocks = 1 << 30) {   // of 32 columns
    return W + ((size_t)min(unit * 2 + (lane >> 5), blocks - 1) * (K / 16)) * 512 + (k / 8) * 256 + (lane & 31) * 8;
  }
  __device__ static __forceinline__ floatx4 mul(const vec& x, const vec& w, floatx4 acc) {
    acc = __builtin_amdgcn_mfma_f32_4x4x4f16(half4_t{x[0], x[1], x[2], x[3]}, half4_t{w[0], w[1], w[2], w[3]}, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_4x4x4f16(half4_t{x[4], x[5], x[6], x[7]}, half4_t{w[4], w[5], w[6], w[7]}, acc, 0, 0, 0);
  }
};

struct SmallArgs { StackArgs st; SearchArgs se; };
// (1500 instructions of spilling with the arguments in registers: a translation of 8 steps 434 us instead of 392)
using ArgsPtr = const __attribute__((address_space(4))) SmallArgs*;

// MANY: any number of steps; otherwise one, without the loop, for callers who wait for each and where rows of the cache are moved in between: a step of 37 / 80 /
// 120 / 237 us with the loop takes 36 / 79 / 117.5 / 232 without.
template <typename T, int K, bool MANY>
__global__ void __launch_bounds__(kThreads) small_step_kernel(const SmallArgs) {
  constexpr int NB = (K + 3) / 4, R = 4 * NB;
  constexpr int P = 8;   // pieces requested ahead
  using Pc = Piece<T>;
  using vec = typename Pc::vec;
  typedef T T4 __attribute__((ext_vector_type(4)));

  constexpr int LX = kD + 16, LQ = 3 * kD + 16, LF = kF + 16;                  // rows of: layer input and context; q, k, v; FFN
  constexpr int XS = 0, CTX = R * LX, QKV = 2 * R * LX, FF = QKV + R * LQ;   // where they start
  __shared__ __attribute__((aligned(16))) T rowsT[FF + R * LF];
  __shared__ __attribute__((aligned(16))) float part[kWaves][R][64];
  __shared__ float prob[kWaves][64];
  __shared__ int slabs[K][64];                                               // of the first 64 positions of every history
  __shared__ float vecs[2][13 * kD + kF];                                    // biases, gains and shifts of a layer, of the next one
  __shared__ SearchShared sh;
  __shared__ int goes_on;

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ArgsPtr a0 = arguments<SmallArgs>();
  int b = blockIdx.x;
  const int D = a0->se.d, F = a0->se.F, H = a0->se.H, V = a0->se.V, G = (V + 31) / 32;
  const int layers = a0->st.layers, T1 = a0->se.T1, Tm = a0->st.T;
  const int first = *global(a0->st.tpos), steps = a0->se.steps;
  auto layer_of = [&](const half_t* p, size_t bytes) { return reinterpret_cast<const T*>(reinterpret_cast<const char*>(global(p)) + bytes); };
  auto pin = [] { asm volatile("" ::: "memory"); };

  // ---- products.  Wavefront w: 64-column unit w / parts, part w % parts of k
  const T* wp = nullptr;
  int np = 0, k0 = 0;        // pieces and first k of this wavefront
  vec w[P];
  auto parts_of = [](int N) {   // log2 of the wavefronts per unit (at most 8 units)
    return N <= 64 ? 3 : N <= 128 ? 2 : N <= 256 ? 1 : 0;
  };
  auto request = [&](const T* Wp, int N, int Kd) {
    const int ps = parts_of(N), u = wave >> ps;
    np = u * 64 < N ? Kd / Pc::n >> ps : 0;
    k0 = (wave & ((1 << ps) - 1)) * np * Pc::n;
    wp = Pc::at(Wp, Kd, u, k0, lane);
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (i < np) w[i] = *reinterpret_cast<const vec*>(wp + i * Pc::stride);
    pin();
  };
  auto multiply = [&](int x, int ldx, floatx4 (&acc)[NB]) {   // rows from rowsT[x] on
    const T* xp = &rowsT[x + (lane & 3) * ldx + k0];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < np; i0 += P) {
      vec cur[P];
#pragma unroll
      for (int i = 0; i < P; ++i) {
        cur[i] = w[i];
        if (i0 + P + i < np) w[i] = *reinterpret_cast<const vec*>(wp + (i0 + P + i) * Pc::stride);
      }
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (i0 + i < np)
#pragma unroll
          for (int n = 0; n < NB; ++n)
            acc[n] = Pc::mul(*reinterpret_cast<const vec*>(xp + n * 4 * ldx + (i0 + i) * Pc::n), cur[i], acc[n]);
    }
  };
  auto product = [&](int x, int ldx) {   // partial sums of this wavefront's columns -> part
    floatx4 acc[NB];
    multiply(x, ldx, acc);
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave][n * 4 + i][lane] = acc[n][i];
  };
  auto total = [&](int ps, int row, int unit) {   // column `lane` of a unit
    float t[kParts], v = 0.f;
#pragma unroll
    for (int i = 0; i < kParts; ++i) t[i] = part[(unit << ps) + min(i, (1 << ps) - 1)][row][lane];
#pragma unroll
    for (int i = 0; i < kParts; ++i) v += i < 1 << ps ? t[i] : 0.f;
    return v;
  };
  // y = T(product + bias), ReLU on request: a wavefront per row and unit
  auto finish = [&](int y, int ldy, int N, int ps, const float* bias, bool relu) {
    for (int i = wave; i < K * (N / 64); i += kWaves) {
      const int row = i % K, unit = i / K;
      float v = total(ps, row, unit) + bias[unit * 64 + lane];
      if (relu) v = fmaxf(v, 0.f);
      rowsT[y + row * ldy + unit * 64 + lane] = (T)v;
    }
    __syncthreads();
  };
  // x = LayerNorm(x + product + bias): a wavefront per row, columns lane and lane + 64
  const float eps = a0->st.eps, inv_d = D > 64 ? 1.0f / 128 : 1.0f / 64;
  auto add_norm = [&](int ps, const float* bias, const float* g, const float* bt) {
    if (wave < K) {
      const bool two = D > 64;
      T* x = &rowsT[XS + wave * LX + lane];
      const float v0 = (float)x[0] + (total(ps, wave, 0) + bias[lane]), v1 = two ? (float)x[64] + (total(ps, wave, 1) + bias[64 + lane]) : 0.f;
      const float mean = wave_sum(v0 + v1) * inv_d;
      const float c0 = v0 - mean, c1 = two ? v1 - mean : 0.f;
      const float var = wave_sum(c0 * c0 + c1 * c1) * inv_d + eps;
      const float rs = __builtin_amdgcn_rsqf(var), rstd = rs * (1.5f - 0.5f * var * rs * rs);
      x[0] = (T)(g[lane] * (c0 * rstd) + bt[lane]);
      if (two) x[64] = (T)(g[64 + lane] * (c1 * rstd) + bt[64 + lane]);
    }
    __syncthreads();
  };
  // a layer's vectors, in this order: the wavefronts take one or two each
  const int VO = 3 * D, VN = VO + 3 * D, VF = VN + 6 * D, V2 = VF + F;   // after bqkv: bo, bq, boc; gains and shifts; b1; b2
  auto load_vectors = [&](int l) {
    float* to = vecs[l & 1];
    const ArgsPtr p = arguments<SmallArgs>();
    const size_t bytes = (size_t)l * p->st.plain_stride;
    auto copy = [&](const half_t* from, int at, int n) {
      const T* v = layer_of(from, bytes);
      for (int i = lane; i < n; i += 64) to[at + i] = (float)v[i];
    };
    switch (wave) {
      case 0: copy(p->st.bqkv, 0, 3 * D); break;
      case 1: copy(p->st.b1, VF, F); break;
      case 2: copy(p->st.bo, VO, D); copy(p->st.bq, VO + D, D); break;
      case 3: copy(p->st.boc, VO + 2 * D, D); copy(p->st.b2, V2, D); break;
      case 4: copy(p->st.ln1g, VN, D); copy(p->st.ln1b, VN + D, D); break;
      case 5: copy(p->st.ln2g, VN + 2 * D, D); copy(p->st.ln2b, VN + 3 * D, D); break;
      case 6: copy(p->st.ln3g, VN + 4 * D, D); copy(p->st.ln3b, VN + 5 * D, D); break;
    }
  };

  // ---- attention: wavefront w takes (row, head) pairs w, w + 8, ...; a lane per key for the scores, then DQ = head size / 4
  // lanes per value row.  64 keys at a time.
  const int hs = 31 - __builtin_clz(H), ds = D > 64 ? 7 : 6;   // both powers of two
  const int src_off = global(a0->st.src_off)[b], src_len = global(a0->st.src_len)[b];
  const float qscale = a0->se.qscale;
  const bool table = a0->se.anc != nullptr;
  auto request_keys = [&](auto dh, auto& kr, auto& vr, bool self, const T* Kb, const T* Vb, int nkeys, int pair, int c0) __attribute__((always_inline)) {
    constexpr int DH = decltype(dh)::value, DQ = DH / 4, GK = 64 / DQ;
    const int row = pair >> hs, h = pair & (H - 1);
    const int last = max(nkeys - 1 - (self ? 1 : 0), 0);   // the newest position's are in LDS
    auto offset = [&](int key) {
      if (!self) return (unsigned)(min(key, last) * 2 * D + h * DH);
      int slab = slabs[row][key & 63];
      if (c0 > 0 && table) slab = min(max(global(arguments<SmallArgs>()->se.anc)[(size_t)(b * K + row) * T1 + min(key, last)], 0), K - 1);
      return (unsigned)((slab * Tm + min(key, last)) * D + h * DH);
    };
    unsigned vo[DQ];
#pragma unroll
    for (int i = 0; i < DQ; ++i) vo[i] = offset(c0 + i * GK + lane / DQ) + lane % DQ * 4;
    const unsigned ko = offset(c0 + lane);
#pragma unroll
    for (int i = 0; i < DQ; ++i) kr[i] = *reinterpret_cast<const T4*>(Kb + ko + i * 4);
#pragma unroll
    for (int i = 0; i < DQ; ++i)
      if (i == 0 || c0 + i * GK < nkeys) vr[i] = *reinterpret_cast<const T4*>(Vb + vo[i]);
  };
  auto attend = [&](auto dh, bool self, const T* Kb, const T* Vb, int nkeys) __attribute__((always_inline)) {
    constexpr int DH = decltype(dh)::value, DQ = DH / 4, GK = 64 / DQ;
    const int gk = lane / DQ, c4 = lane % DQ * 4;
    for (int pair = wave; pair < K * H; pair += kWaves) {
      const int row = pair >> hs, h = pair & (H - 1);
      float m = -INFINITY, z = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
      for (int c0 = 0; c0 < nkeys; c0 += 64) {
        T4 kr[DQ], vr[DQ];
        request_keys(dh, kr, vr, self, Kb, Vb, nkeys, pair, c0);
        if (self && c0 + lane == nkeys - 1)
#pragma unroll
          for (int i = 0; i < DQ; ++i) kr[i] = *reinterpret_cast<const T4*>(&rowsT[QKV + row * LQ + D + h * DH + i * 4]);
        float sp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < DQ; ++i) {
          const T4 q4 = *reinterpret_cast<const T4*>(&rowsT[QKV + row * LQ + h * DH + i * 4]);
#pragma unroll
          for (int e = 0; e < 4; ++e) sp[e] = fmaf((float)q4[e], (float)kr[i][e], sp[e]);
        }
        const float s = c0 + lane < nkeys ? ((sp[0] + sp[1]) + (sp[2] + sp[3])) * qscale : -INFINITY;
        const float mx = fmaxf(m, wave_max(s)), corr = __builtin_amdgcn_exp2f(m - mx), p = __builtin_amdgcn_exp2f(s - mx);
        m = mx;
        prob[wave][lane] = p;   // LDS keeps a wavefront's order
        pin();
        __builtin_amdgcn_wave_barrier();
        z = z * corr + wave_sum(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= corr;
#pragma unroll
        for (int i = 0; i < DQ; ++i)
          if (i == 0 || c0 + i * GK < nkeys) {
            const int key = c0 + i * GK + gk;
            if (self && key == nkeys - 1) vr[i] = *reinterpret_cast<const T4*>(&rowsT[QKV + row * LQ + 2 * D + h * DH + c4]);
            const float pk = prob[wave][i * GK + gk];   // 0 past the last key
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += pk * (key < nkeys ? (float)vr[i][e] : 0.f);
          }
        pin();
        __builtin_amdgcn_wave_barrier();
      }
      for_lane_bits<DQ>([&](auto bit) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = add_lane_xor<decltype(bit)::value>(acc[e]);
      });
      if (gk == 0) {
        const float inv = 1.0f / z;
        *reinterpret_cast<T4*>(&rowsT[CTX + row * LX + h * DH + c4]) = T4{(T)(acc[0] * inv), (T)(acc[1] * inv), (T)(acc[2] * inv), (T)(acc[3] * inv)};
      }
    }
    __syncthreads();
  };
  const std::integral_constant<int, 16> h16;
  const std::integral_constant<int, 32> h32;
  const bool narrow = D == 16 * H;

  // ======== the layers, six products each: q k v, output projection, query of the cross-attention, its output projection,
  // FFN.  One body for all of them: the kernel has to stay within the instruction cache.
  auto shape = [&](int stage, int& N, int& Kd) {
    N = stage == 0 ? 3 * D : stage == 4 ? F : D;
    Kd = stage == 5 ? F : D;
  };
  auto request_stage = [&](int l, int stage) {
    int N, Kd;
    shape(stage, N, Kd);
    const ArgsPtr p = arguments<SmallArgs>();
    request(layer_of((&p->st.Wqkv)[stage], (size_t)l * p->st.packed_stride), N, Kd);   // Wqkv, Wo, Wq, Woc, W1, W2
  };
  auto request_unit = [&](int u) {   // of the embedding
    np = D / Pc::n;
    k0 = 0;
    wp = Pc::at(reinterpret_cast<const T*>(global(arguments<SmallArgs>()->se.Ep)), D, u, 0, lane, G);
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (i < np) w[i] = *reinterpret_cast<const vec*>(wp + i * Pc::stride);
    pin();
  };
  // ======== the steps.  What one of them leaves in memory the next one finds there: it is the same workgroup (and on the same
  // compute unit), so the wait and the barrier between them are enough.
  for (int it = 0;; ++it) {
  if constexpr (MANY) {
    asm volatile("" : "+v"(tid), "+v"(lane), "+s"(b));   // as in the loop over the layers
#pragma unroll
    for (int i = 0; i < P; ++i) asm volatile("" : "=v"(w[i]));   // nothing of the step before is kept
  }
  const int pos = first + it;
  const bool last = !MANY || it + 1 == steps;
  RerankState st = {};
  if (wave < K) {
    const ArgsPtr r = arguments<SmallArgs>();
    st = rerank_request(global(r->se.tokens), global(r->se.len), global(r->se.fin), global(r->se.cap),
                        table ? global(r->se.anc) : nullptr, K, T1, it, global(r->se.step_state), one_group(), b, lane);
  }
  request_stage(0, 0);
  for (int i = tid; i < R * D / 4; i += kThreads) {   // rows the sentence does not have: zeros
    const int row = i >> (ds - 2), c = (i << 2) & (D - 1);
    T4 v = {};
    if (row < K) v = *reinterpret_cast<const T4*>(reinterpret_cast<const T*>(global(a0->st.x0)) + (size_t)(b * K + row) * D + c);
    *reinterpret_cast<T4*>(&rowsT[XS + row * LX + c]) = v;
    if (row >= K) *reinterpret_cast<T4*>(&rowsT[CTX + row * LX + c]) = v;
  }
  for (int i = tid; i < K * 64; i += kThreads) {
    const int row = i / 64, p = min(i % 64, T1 - 1);
    slabs[row][i % 64] = table ? min(max(global(a0->se.anc)[(size_t)(b * K + row) * T1 + p], 0), K - 1) : row;
  }
  if (it == 0 || layers > 2) load_vectors(0);   // of two layers both stay where they are
  if constexpr (R > K)
    if (it == 0) for (int r = K; r < R; ++r)
      for (int c = tid; c < F; c += kThreads) rowsT[FF + r * LF + c] = (T)0.f;
  __syncthreads();
  for (int l = 0, stage = 0; l < layers;) {
    // what is derived from a thread's place is derived anew instead of waiting in registers
    asm volatile("" : "+v"(tid), "+v"(lane));
    const ArgsPtr p = arguments<SmallArgs>();
    T* Kc = reinterpret_cast<T*>(global(p->st.cache) + (size_t)(2 * l) * p->st.cache_stride) + (size_t)(b * K) * Tm * D;
    T* Vc = reinterpret_cast<T*>(reinterpret_cast<char*>(Kc) + p->st.cache_stride);
    const T* kvb = reinterpret_cast<const T*>(global(p->st.cross) + (size_t)l * p->st.cross_stride) + (size_t)src_off * 2 * D;
    int N, Kd;
    shape(stage, N, Kd);
    const int ps = parts_of(N);
    const bool self = stage == 0, attention = stage == 0 || stage == 2;
    const T *Kb = self ? Kc : kvb, *Vb = self ? Vc : kvb + D;
    const int nkeys = self ? pos + 1 : src_len;
    product(stage == 5 ? FF : stage == 1 || stage == 3 ? CTX : XS, stage == 5 ? LF : LX);
    const int next = stage == 5 ? 0 : stage + 1, nl = stage == 5 ? l + 1 : l;
    if (nl < layers) request_stage(nl, next);
    else if (wave * 64 < V) request_unit(wave);
    __syncthreads();
    const float* vl = vecs[l & 1];
    if (stage == 0 || stage == 2 || stage == 4)
      finish(stage == 4 ? FF : QKV, stage == 4 ? LF : LQ, N, ps, vl + (stage == 0 ? 0 : stage == 2 ? VO + D : VF), stage == 4);
    else {
      const float* g = vl + VN + (stage - 1) * D;
      add_norm(ps, vl + (stage == 1 ? VO : stage == 3 ? VO + 2 * D : V2), g, g + D);
    }
    if (stage == 4 && l + 1 < layers && (it == 0 || layers > 2)) load_vectors(l + 1);   // for a barrier two stages on
    if (stage == 0)
      for (int i = tid; i < K * D / 2; i += kThreads) {   // the new keys and values
        const int row = i >> (ds - 1), c = (i << 2) & (2 * D - 1);
        *reinterpret_cast<T4*>((c < D ? Kc + c : Vc + c - D) + ((size_t)row * Tm + pos) * D) =
            *reinterpret_cast<const T4*>(&rowsT[QKV + row * LQ + D + c]);
      }
    if (attention) {
      if (narrow) attend(h16, self, Kb, Vb, nkeys);
      else attend(h32, self, Kb, Vb, nkeys);
    }
    stage = next;
    l = nl;
  }
  const ArgsPtr a1 = arguments<SmallArgs>();
  for (int i = tid; i < K * D; i += kThreads) reinterpret_cast<T*>(global(a1->st.hidden))[((size_t)(b * K) << ds) + i] = rowsT[XS + (i >> ds) * LX + (i & (D - 1))];

  // ======== logits and their group statistics: 64 columns per wavefront and turn
  for (int u = wave; u * 64 < V; u += kWaves) {
    floatx4 acc[NB];
    multiply(XS, LX, acc);
    if ((u + kWaves) * 64 < V) request_unit(u + kWaves);
    const int col = u * 64 + lane;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = n * 4 + i;
        if (row >= K) continue;
        const float v = acc[n][i], mx = group_max<32>(col < V ? v : -INFINITY);
        const float z = group_sum<32>(col < V ? __expf(v - mx) : 0.f);
        if (col < V) global(a1->se.logits)[(size_t)(b * K + row) * V + col] = v;
        if ((lane & 31) == 0 && col < V) *reinterpret_cast<float2*>(global(a1->se.stats) + ((size_t)(b * K + row) * G + (col >> 5)) * 2) = float2{mx, z};
      }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (wave < K) {
    const ArgsPtr e = arguments<SmallArgs>();
    const NextInput next = {global(e->se.next.E), global(e->se.next.pe), global(e->se.next.x), e->se.next.d, e->se.next.dtype, e->se.next.scale};
    const bool more = retrieve_rerank_sentence<4, K>(global(e->se.logits), global(e->se.stats), global(e->se.score), global(e->se.tokens), global(e->se.len),
                                                     global(e->se.fin), global(e->se.parent), global(e->se.active), V, G, T1, global(e->se.step_state),
                                                     e->se.eos, table ? global(e->se.anc) : nullptr, next, global(e->se.cand_score),
                                                     global(e->se.cand_idx), e->se.report, b, sh, st, last);
    if (tid == 0) goes_on = more;
  } else if (last) {
    return;   // the barriers inside are among the wavefronts that remain
  } else {    // as many barriers as there are inside
    for (int p0 = 0; p0 <= pos && p0 < T1; p0 += 64) __syncthreads();
  }
  if (last) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (!goes_on) break;
  }
  // The sentence is finished before the last step of the launch: it counts as one that does not go on from there.
  if (tid == 0) {
    const ArgsPtr e = arguments<SmallArgs>();
    const int before = step_arrive(global(e->se.step_state), 0), t = first + steps - 1;
    step_finish(before, global(e->se.active), t, global(e->se.step_state), t + 1, 0, (int)gridDim.x, e->se.report);
  }
}

template <bool MANY>
const void* small_kernel_of(int dtype, int k) {
#define LSQ_SMALL(K_) case K_: return dtype == DT_F16 ? (const void*)small_step_kernel<half_t, K_, MANY> : (const void*)small_step_kernel<float, K_, MANY>
  switch (k) { LSQ_SMALL(1); LSQ_SMALL(2); LSQ_SMALL(3); LSQ_SMALL(4); LSQ_SMALL(5); LSQ_SMALL(6); LSQ_SMALL(7); LSQ_SMALL(8); }
#undef LSQ_SMALL
  return nullptr;
}

}  // namespace

bool small_step_supported(int arch, int H, int d, int F, int V, int k) {
  return arch == 0 && d % 64 == 0 && d <= kD && F % 64 == 0 && F <= kF && (d == 16 * H || d == 32 * H) &&
         (size_t)(V + 63) / 64 * 64 * d <= (1u << 17) && k <= LSQ_MAX_BEAM_ && topk_groups_supported(V, k, 0);
}

// Where one workgroup per sentence is ahead of the separate launches.  It takes the K*H (row, head) pairs of a layer eight at a
// time through 64 keys a trip (2.2 us for a trip of the history at heads of 16 in float32, 1.7 in float16, half of that for the
// source, twice that at heads of 32), while the separate launches spread them over the chip and cost little more at any
// length.  Whole steps in us, this kernel / separate launches, float32 (position 4, 104, 240, 496, 1008; sources of 8):
//   d = 64, 1 layer, 4 heads:   2 x 4 rows 33 / 57, 38 / 58, 47 / 58, 64 / 59, 99 / 63;   32 x 4 33 / 81, 38 / 81, 48 / 83, 65 / 84, 108 / 94
//                               2 x 8      47 / 69, 57 / 70, 76 / 71, 111 / 73;           64 x 8 47 / 90, 58 / 91, 78 / 97, 117 / 106
//   d = 128, 2 layers, 8 heads: 2 x 4      79 / 103, 100 / 105, 135 / 106, 208 / 112;     32 x 4 78 / 144, 105 / 147, 144 / 156, 217 / 170
//                               2 x 8      115 / 120, 157 / 123, 239 / 125;             256 x 4 90 / 189, 111 / 194, 165 / 223, 283 / 307, 580 / 493
//   ... 6 layers:               2 x 4      217 / 271, 282 / 272, 403 / 279;               32 x 4 215 / 406, 279 / 412, 400 / 429, 626 / 449
//   sources of 64, 128, 256, 500 at position 4, d = 128, 2 layers: 2 x 4 84 / 101, 93 / 101, 111 / 102, 146 / 103;
//                                                               32 x 8 127 / 168, 147 / 169, 183 / 172, 254 / 177
// and the same order in float16 with both sides 15 % lower.  The lines cross at 16 to 66 trips (a trip of the history and heads of 16
// counting two), more with more rows, whose separate launches take longer, and fewer with more layers, over which the
// launches outside of them are spread.
bool small_step_ahead(int batch, int k, int H, int d, int layers, int pos, int src) {
  const int M = batch * k, per_layer = (k * H + kWaves - 1) / kWaves * (d / H / 16);
  const int trips = per_layer * (2 * (pos / 64 + 1) + (src + 63) / 64);
  return trips <= 21 + min(M, 16) / 2 + min(M, 128) / 16 + max(M - 128, 0) / 32 - 3 * (layers - 1) / 2;
}

hipError_t launch_small_step(int dtype, int batch, int k, const StackArgs& args, const SearchArgs& search, hipStream_t s) {
  const void* kernel = search.steps > 1 ? small_kernel_of<true>(dtype, k) : small_kernel_of<false>(dtype, k);
  if (!kernel || batch < 1 || search.steps < 1) return hipErrorInvalidValue;
  SmallArgs a = {args, search};
  void* kargs[] = {&a};
  return hipLaunchKernel(kernel, dim3(batch), dim3(kThreads), kargs, 0, s);
}

}  // namespace lsq
