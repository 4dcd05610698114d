// The encoder of a small model (the shapes of kernels_small.hip) as ONE launch, with what a translation starts from: embedding, encoder
// layers, keys and values of the cross-attention, hypotheses before the first step and their decoder input.
//
// Sentences meet nowhere in it, so a workgroup takes one through all of it with its rows in LDS, as the decoder does: as launches of
// their own (12 for one layer) every product of a few rows was 5 us and as much again to the next.  Bound by the length of the chain: four
// products a layer, each a trip to memory for its weights and a barrier.  The ids come straight from pinned host memory.
// Up to 48 source tokens; longer ones go to the separate launches, where rows of a sentence are spread over the chip.
// A translation of 8 steps (2 sentences of 5 and 8 tokens, d = 64, one layer each, float32), whose encoding was 88 of 309 us, 274 us with 35.
//
// Products: 16 x 16 matrix instructions, rows of the weight matrix as they are (a lane has 16 bytes of its column: k 16 s + 4 (lane >> 4) + i in float32,
// 32 s + 8 (lane >> 4) + i in float16, the same of the input row, so the order of k inside a step is free), the next 64 of k but two in flight.
#include "lsq_internal.h"

namespace lsq {

namespace {

constexpr int kThreads = 512, kWaves = 8;
constexpr int kF = 512;       // widest feed-forward row
constexpr int kQ = 4;         // query rows that a wavefront attends for at a time

template <typename T> struct Step;
template <> struct Step<float> {
  using vec = floatx4;
  static constexpr int n = 4, sums = 8;   // vectors per lane for 64 k; sums side by side, of 8 products each
  __device__ static __forceinline__ void mul(const vec& x, const vec& w, int s, floatx4 (&acc)[sums]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[(s & 1) * 4 + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], w[i], acc[(s & 1) * 4 + i], 0, 0, 0);
  }
  __device__ static __forceinline__ floatx4 total(const floatx4 (&a)[sums]) { return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])); }
};
template <> struct Step<half_t> {
  using vec = half8_t;
  static constexpr int n = 2, sums = 2;
  __device__ static __forceinline__ void mul(const vec& x, const vec& w, int s, floatx4 (&acc)[sums]) {
    acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, w, acc[s], 0, 0, 0);
  }
  __device__ static __forceinline__ floatx4 total(const floatx4 (&acc)[sums]) { return acc[0] + acc[1]; }
};

// MB: blocks of 16 rows
template <typename T, int D, int MB>
__global__ void __launch_bounds__(kThreads) small_encoder_kernel(const SmallEncoderArgs) {
  using St = Step<T>;
  using vec = typename St::vec;
  constexpr int R = 16 * MB, VN = 16 / sizeof(T), PAD = VN;
  constexpr int LX = D + PAD, LQ = 3 * D + PAD, LF = kF + PAD, LT = D + 4;   // rows of: layer input; q, k, v; FFN; float sums
  // one region for q, k, v or the FFN's hidden rows or the sums of the attention's output projection, one for contexts or the sums of the FFN
  constexpr int BIG = R * (LF > LQ ? LF : LQ) * (int)sizeof(T), CTX = R * LT * 4;
  static_assert(BIG >= CTX && LT * 4 >= LX * (int)sizeof(T), "regions shared by floats and rows");
  __shared__ __attribute__((aligned(16))) T xs[R * LX];
  __shared__ __attribute__((aligned(16))) char big[BIG], ctx[CTX];
  __shared__ float prob[kWaves][kQ][64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const auto* a = arguments<SmallEncoderArgs>();
  const int b = blockIdx.x, F = a->F, H = a->H, k = a->k, T1 = a->T1;
  T* const bigT = reinterpret_cast<T*>(big);
  T* const ctxT = reinterpret_cast<T*>(ctx);
  float* const bigF = reinterpret_cast<float*>(big);
  float* const ctxF = reinterpret_cast<float*>(ctx);

  // ---- the request, from host memory: everything in one trip.  Rows past the sentence: token 0, thrown away.
  const int n = min(global(a->h_len)[b], R), off = global(a->h_off)[b];
  const int id = lane < a->id_stride ? global(a->h_ids)[(size_t)b * a->id_stride + lane] : 0;
  if (tid == 0) {
    global(a->src_off)[b] = off;
    global(a->src_len)[b] = n;
    global(a->cap)[b] = global(a->h_cap)[b];
    global(a->order)[b] = global(a->h_order)[b];
    if (b == (int)gridDim.x - 1) global(a->src_off)[b + 1] = off + n;
  }
  // ---- hypotheses before the first step (beam_reset_kernel) and their decoder input
  for (int i = tid; i < k * T1; i += kThreads) global(a->tokens)[(size_t)b * k * T1 + i] = i % T1 == 0 ? a->bos : a->pad;
  if (tid < k) {
    const int r = b * k + tid;
    global(a->score)[r] = tid % a->kg == 0 ? 0.f : -INFINITY;
    global(a->len)[r] = 0;
    global(a->fin)[r] = 0;
    if (a->anc) global(a->anc)[(size_t)r * T1] = tid;
  }
  if (tid == 0) global(a->pen_n)[b] = 0;
  if (b == 0) {
    for (int i = tid; i < T1; i += kThreads) global(a->active)[i] = 0;
    if (tid < 3) global(a->step_state)[tid] = 0;
  }
  const T* E = reinterpret_cast<const T*>(global(a->E));
  const float* pe = global(a->pe);
  if (wave < k) embed_whole_row<T, D>(E + (size_t)a->bos * D, pe, reinterpret_cast<T*>(global(a->x0)) + (size_t)(b * k + wave) * D, a->scale, lane);
  for (int r = wave; r < R; r += kWaves) {
    const int tok = __builtin_amdgcn_readlane(id, r);
    embed_whole_row<T, D>(E + (size_t)(r < n ? tok : 0) * D, pe + (size_t)(r < n ? r : 0) * D, &xs[r * LX], a->scale, lane);
  }
  __syncthreads();

  // ---- x . W^T, 16-column units dealt out over the wavefronts; take(unit, sums): sums[m][i] of row 16 m + 4 (lane >> 4) + i, column lane & 15
  auto product = [&](const T* W, int N, int K, const T* x, int ldx, auto take) __attribute__((always_inline)) {
    const int cps = K / 64, units = N / 16, chunks = wave < units ? ((units - 1 - wave) / kWaves + 1) * cps : 0;
    const T* wl = W + (size_t)(lane & 15) * K + (lane >> 4) * VN;
    const T* xl = x + (lane & 15) * ldx + (lane >> 4) * VN;
    vec w[3][St::n];
    int lu = wave, lc = 0;   // unit and chunk of the next request (past the end: the last one again)
    auto load = [&](vec (&to)[St::n]) {
      const T* p = wl + (size_t)lu * 16 * K + lc * 64;
#pragma unroll
      for (int s = 0; s < St::n; ++s) to[s] = *reinterpret_cast<const vec*>(p + s * 4 * VN);
      if (++lc == cps) {
        if (lu + kWaves < units) { lc = 0; lu += kWaves; }
        else lc = cps - 1;
      }
    };
    if (chunks == 0) return;
    load(w[0]);
    load(w[1]);
    load(w[2]);
    floatx4 sum[MB];
    for (int c = 0, u = wave, part = 0; c < chunks; ++c) {
      vec cur[St::n];
#pragma unroll
      for (int s = 0; s < St::n; ++s) { cur[s] = w[0][s]; w[0][s] = w[1][s]; w[1][s] = w[2][s]; }
      load(w[2]);
      floatx4 acc[MB][St::sums];   // of 64 k: short sums, added up afterwards, lose no more than the separate products' do
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < St::sums; ++i) acc[m][i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < St::n; ++s)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          St::mul(*reinterpret_cast<const vec*>(xl + m * 16 * ldx + part * 64 + s * 4 * VN), cur[s], s, acc[m]);
#pragma unroll
      for (int m = 0; m < MB; ++m) sum[m] = part == 0 ? St::total(acc[m]) : sum[m] + St::total(acc[m]);
      if (++part == cps) {
        take(u, sum);
        part = 0;
        u += kWaves;
      }
    }
  };
  const int row0 = lane >> 4 << 2, col = lane & 15;
  // y = T(x . W^T + bias), ReLU on request
  auto rows_of = [&](const T* W, const T* bias, int N, int K, const T* x, int ldx, T* y, int ldy, bool relu) __attribute__((always_inline)) {
    product(W, N, K, x, ldx, [&](int u, floatx4 (&acc)[MB]) {
      const float bv = (float)bias[u * 16 + col];
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = acc[m][i] + bv;
          if (relu) v = fmaxf(v, 0.f);
          y[(m * 16 + row0 + i) * ldy + u * 16 + col] = (T)v;
        }
    });
    __syncthreads();
  };
  // x = LayerNorm(x + (input . W^T + bias))
  auto add_norm = [&](const T* W, const T* bias, const T* g, const T* bt, int K, const T* in, int ldin, float* sums) __attribute__((always_inline)) {
    product(W, D, K, in, ldin, [&](int u, floatx4 (&acc)[MB]) {
      const float bv = (float)bias[u * 16 + col];
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) sums[(m * 16 + row0 + i) * LT + u * 16 + col] = acc[m][i] + bv;
    });
    constexpr int NC = D / 64;
    float gv[NC], bv[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) { gv[j] = (float)g[j * 64 + lane]; bv[j] = (float)bt[j * 64 + lane]; }
    __syncthreads();
    for (int r = wave; r < n; r += kWaves) {
      float v[NC], s = 0.f, q = 0.f;
#pragma unroll
      for (int j = 0; j < NC; ++j) { v[j] = (float)xs[r * LX + j * 64 + lane] + sums[r * LT + j * 64 + lane]; s += v[j]; }
      const float mean = wave_sum(s) * (1.0f / D);
#pragma unroll
      for (int j = 0; j < NC; ++j) { v[j] -= mean; q = fmaf(v[j], v[j], q); }
      const float rstd = __fdiv_rn(1.0f, __fsqrt_rn(wave_sum(q) * (1.0f / D) + a->eps));
#pragma unroll
      for (int j = 0; j < NC; ++j) xs[r * LX + j * 64 + lane] = (T)fmaf(gv[j], v[j] * rstd, bv[j]);
    }
    __syncthreads();
  };
  // a wavefront per (four rows, head), whose chains of instructions run side by side: a lane per key for the scores, then DQ lanes per value row
  auto attend = [&](auto dh) __attribute__((always_inline)) {
    constexpr int DH = decltype(dh)::value, DQ = DH / 4, GK = 64 / DQ;
    typedef T T4 __attribute__((ext_vector_type(4)));
    const int gk = lane / DQ, c4 = lane % DQ * 4;
    for (int unit = wave; unit < (n + kQ - 1) / kQ * H; unit += kWaves) {
      const int first = unit / H * kQ, h = unit % H;
      const T* key = bigT + min(lane, n - 1) * LQ + D + h * DH;
      float s[kQ], inv[kQ];
#pragma unroll
      for (int u = 0; u < kQ; ++u) {
        const T* q = bigT + min(first + u, n - 1) * LQ + h * DH;
        float sp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < DQ; ++i) {
          const T4 q4 = *reinterpret_cast<const T4*>(q + i * 4), k4 = *reinterpret_cast<const T4*>(key + i * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) sp[e] = fmaf((float)q4[e], (float)k4[e], sp[e]);
        }
        s[u] = lane < n ? (sp[0] + sp[1]) + (sp[2] + sp[3]) : -INFINITY;
      }
#pragma unroll
      for (int u = 0; u < kQ; ++u) {
        s[u] = __builtin_amdgcn_exp2f((s[u] - wave_max(s[u])) * a->qscale);   // scaled behind the difference: large scores lose nothing to it
        prob[wave][u][lane] = s[u];   // LDS keeps a wavefront's order
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < kQ; ++u) inv[u] = 1.0f / wave_sum(s[u]);
      float acc[kQ][4] = {};
      for (int j = gk; j < n; j += GK) {
        const T4 v4 = *reinterpret_cast<const T4*>(bigT + j * LQ + 2 * D + h * DH + c4);
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
          const float pj = prob[wave][u][j];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[u][e] = fmaf(pj, (float)v4[e], acc[u][e]);
        }
      }
      for_lane_bits<DQ>([&](auto bit) {
#pragma unroll
        for (int u = 0; u < kQ; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[u][e] = add_lane_xor<decltype(bit)::value>(acc[u][e]);
      });
#pragma unroll
      for (int u = 0; u < kQ; ++u)
        if (gk == 0 && first + u < n)
          *reinterpret_cast<T4*>(ctxT + (first + u) * LX + h * DH + c4) =
              T4{(T)(acc[u][0] * inv[u]), (T)(acc[u][1] * inv[u]), (T)(acc[u][2] * inv[u]), (T)(acc[u][3] * inv[u])};
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  };
  auto of = [&](const void* p, int l) { return reinterpret_cast<const T*>(reinterpret_cast<const char*>(global(p)) + (size_t)l * a->enc_stride); };
  for (int l = 0; l < a->enc_layers; ++l) {
    rows_of(of(a->Wqkv, l), of(a->bqkv, l), 3 * D, D, xs, LX, bigT, LQ, false);
    if (D == 16 * H) attend(std::integral_constant<int, 16>{});
    else attend(std::integral_constant<int, 32>{});
    add_norm(of(a->Wo, l), of(a->bo, l), of(a->ln1g, l), of(a->ln1b, l), D, ctxT, LX, bigF);
    rows_of(of(a->W1, l), of(a->b1, l), F, D, xs, LX, bigT, LF, true);
    add_norm(of(a->W2, l), of(a->b2, l), of(a->ln2g, l), of(a->ln2b, l), F, bigT, LF, ctxF);
  }
  // ---- the encoder's output, for whoever inspects it, and the decoder layers' keys and values of it
  for (int i = tid; i < n * (D / 4); i += kThreads) {
    typedef T T4 __attribute__((ext_vector_type(4)));
    const int r = i / (D / 4), c = i % (D / 4) * 4;
    *reinterpret_cast<T4*>(reinterpret_cast<T*>(global(a->memory)) + (size_t)(off + r) * D + c) = *reinterpret_cast<const T4*>(&xs[r * LX + c]);
  }
  for (int l = 0; l < a->dec_layers; ++l) {
    const T* W = reinterpret_cast<const T*>(reinterpret_cast<const char*>(global(a->Wkv)) + (size_t)l * a->dec_stride);
    const T* bias = reinterpret_cast<const T*>(reinterpret_cast<const char*>(global(a->bkv)) + (size_t)l * a->dec_stride);
    T* kv = reinterpret_cast<T*>(global(a->cross) + (size_t)l * a->cross_stride) + (size_t)off * 2 * D;
    product(W, 2 * D, D, xs, LX, [&](int u, floatx4 (&acc)[MB]) {
      const float bv = (float)bias[u * 16 + col];
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = m * 16 + row0 + i;
          if (r < n) kv[(size_t)r * 2 * D + u * 16 + col] = (T)(acc[m][i] + bv);
        }
    });
  }
}

template <typename T>
const void* encoder_kernel_of(int d, int blocks) {
#define LSQ_ENC(D_, MB_) if (d == D_ && blocks == MB_) return (const void*)small_encoder_kernel<T, D_, MB_>
  LSQ_ENC(64, 1); LSQ_ENC(64, 2); LSQ_ENC(64, 3); LSQ_ENC(128, 1); LSQ_ENC(128, 2); LSQ_ENC(128, 3);
#undef LSQ_ENC
  return nullptr;
}

}  // namespace

// One workgroup per sentence against the separate launches, encodings of 4 + 4 layers in us (every sentence of 8, 16, 32, 48 tokens):
//   d = 64, float32    1 sentence 87 / 142   97 / 144  126 / 151  163 / 187;   32  91 / 199  101 / 205  132 / 217  169 / 232
//           float16    1          59 / 128   71 / 130   95 / 127  122 / 146;   32  64 / 138   74 / 142  100 / 149  126 / 157
//   d = 128, 8 heads,
//           float32    1         188 / 153  207 / 158  283 / 165  378 / 207;   32 190 / 223  210 / 236  287 / 265  382 / 314;   200 203 / 318 ... 412 / 931
//           float16    1         116 / 124  136 / 126  182 / 128  228 / 152;   32 120 / 146  140 / 154  186 / 170  233 / 189;   200 128 / 191 ... 253 / 431
// At d = 128 one compute unit's matrix rate and its row-by-row attention are behind what the chip does with the rows of few sentences: from a batch
// of twice the longest source on it is ahead.
bool small_encoder_ahead(int d, int batch, int longest) { return longest <= kSmallEncoderRows && batch <= 256 && (d == 64 || batch >= 2 * longest); }

hipError_t launch_small_encoder(int dtype, int batch, int longest, const SmallEncoderArgs& args, hipStream_t s) {
  const int blocks = (longest + 15) / 16;
  const void* kernel = dtype == DT_F16 ? encoder_kernel_of<half_t>(args.d, blocks) : encoder_kernel_of<float>(args.d, blocks);
  if (!kernel || batch < 1 || longest > kSmallEncoderRows) return hipErrorInvalidValue;
  SmallEncoderArgs a = args;
  void* kargs[] = {&a};
  return hipLaunchKernel(kernel, dim3(batch), dim3(kThreads), kargs, 0, s);
}

}  // namespace lsq
