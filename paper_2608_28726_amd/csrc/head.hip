// The paper's verifier head on the GPU (Pro-Router, Sec. 3.1, the paragraph
// after Eq. 3; Sec. 4.2): each request's input sequence X (T tokens x 4
// features) is projected to 64 features with a sinusoidal positional
// encoding, passes two post-norm transformer encoder layers (4 heads of 16,
// feed-forward width 128, LayerNorm eps 1e-5), is mean-pooled over its
// tokens and mapped to one shipping confidence by a linear map and a sigmoid.
//
// The tokens of all requests are processed together as rows:
//  head_embed_kernel  per 16 rows: projection + encoding, and the first
//                     layer's queries, keys and values; one more workgroup
//                     lists the row blocks of the requests, the heaviest
//                     first;
//  head_layer_kernel  per block of up to 16 rows of one request, one
//                     encoder layer: attention over the request's keys,
//                     output projection, residual, LayerNorm, feed-forward,
//                     residual, LayerNorm, and the next layer's queries, keys
//                     and values (or, in the last layer, each row's product
//                     with the output map);
//  head_score_kernel  per request: the mean of its rows' products, sigmoid.
// Everything is float32 (the per-request mean in float64). The float32 matrix
// instructions run on the vector ALUs of this part, at their rate and in
// their time (a v_mfma_f32_16x16x4_f32 and an exp take 44 cycles together
// with four waves on a SIMD, 32 + 9 alone), so most products run on the
// bfloat16 matrix cores instead, without giving up float32: an operand is
// split exactly into three bfloat16 terms of 8 bits each, x = x1 + x2 + x3,
// and the six products of weight 2^-16 and more are accumulated in float32
// (the three left out sum to less than 2^-25 of |x y|, a float32 product's own
// rounding is 2^-24). Six products of 16 x 16 x 32 take 96 cycles against 256
// in float32. The weights are split once per call, activations where they
// are made; only the attention's value products stay in float32 (splitting
// the probabilities would cost what it saves).
#include "head.h"

namespace pr {

namespace {

constexpr int D = kHeadD;       // 64
constexpr int FF = kHeadFF;     // 128
constexpr int NH = kHeadHeads;  // 4
constexpr int DH = D / NH;      // 16
constexpr int QKV = 3 * D;      // 192
constexpr int kHalves = 2;                      // waves per head: each takes half of the keys
constexpr int kWaves = NH * kHalves;
constexpr int kThreads = kWaves * kWave;
constexpr float kLnEps = 1e-5f;
constexpr int kRows = 16;  // rows of a block

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));  // an operand's 8 consecutive k

// Offsets (floats) of the parameter tensors in the flat weight buffer.
constexpr int kW_in = 0;
constexpr int kB_in = kW_in + D * 4;
constexpr int kLayer0 = kB_in + D;
constexpr int kLayerSize = QKV * D + QKV + D * D + D + 2 * D + FF * D + FF + D * FF + D + 2 * D;
constexpr int kW_qkv = 0, kB_qkv = kW_qkv + QKV * D, kW_o = kB_qkv + QKV, kB_o = kW_o + D * D;
constexpr int kLn1g = kB_o + D, kLn1b = kLn1g + D, kW_1 = kLn1b + D, kB_1 = kW_1 + FF * D;
constexpr int kW_2 = kB_1 + FF, kB_2 = kW_2 + D * FF, kLn2g = kB_2 + D, kLn2b = kLn2g + D;
constexpr int kW_out = kLayer0 + kHeadLayers * kLayerSize;
constexpr int kB_out = kW_out + D;
static_assert(kLayerSize == 33472 && kB_out + 1 == kHeadWeights, "parameter layout");
static_assert(kLn2b + D == kLayerSize, "layer layout");
static_assert(kLayer0 % 4 == 0 && kLayerSize % 4 == 0 && kB_qkv % 4 == 0 && kW_o % 4 == 0 && kB_o % 4 == 0 &&
                  kLn1g % 4 == 0 && kW_1 % 4 == 0 && kB_1 % 4 == 0 && kW_2 % 4 == 0 && kB_2 % 4 == 0 &&
                  kLn2g % 4 == 0 && kW_out % 4 == 0,
              "16-byte loads of the parameters");

// Padded LDS row strides: rows of 68 floats, or of 72 or 136 bfloat16 (36 and
// 68 words), so that the 16 rows of a 16-byte fragment read fall on 16
// distinct groups of 4 banks.
constexpr int kSA = D + 4;   // 64-wide activations, float32
constexpr int kBA = D + 8;   // the same, one bfloat16 term
constexpr int kBF = FF + 8;  // 128-wide, one bfloat16 term

constexpr int kKT = 64;  // keys per attention tile

// f_i = 10000^(-2i / 64), the encoding's frequencies.
__device__ const double kFreq[D / 2] = {
    0x1.0000000000000p+0,  0x1.7ff2224115d9ap-1,  0x1.1feb33c1c381ep-1,  0x1.afd1354c40d50p-2,
    0x1.43d136248490fp-2,  0x1.e5a84719edcd2p-3,  0x1.6c310e3769f3fp-3,  0x1.111aedafb9a9dp-3,
    0x1.999999999999ap-4,  0x1.33281b6744ae1p-4,  0x1.ccab8602d2697p-5,  0x1.59742aa36710dp-5,
    0x1.030dc4ea03a72p-5,  0x1.84869f47f170fp-6,  0x1.235a71c5ee5ccp-6,  0x1.b4f7e2b2c2a95p-7,
    0x1.47ae147ae147bp-7,  0x1.eb735f0ba1168p-8,  0x1.7089380241edfp-8,  0x1.145ceee91f40bp-8,
    0x1.9e7c6e43390b7p-9,  0x1.36d219065ac0cp-9,  0x1.d22a4fa316facp-10, 0x1.5d931bc235544p-10,
    0x1.0624dd2f1a9fcp-10, 0x1.892918d61a787p-11, 0x1.26d42cce9b24cp-11, 0x1.ba2e4b0e98677p-12,
    0x1.4b96be9c2da2cp-12, 0x1.f150280a2ace0p-13, 0x1.74eea61c12623p-13, 0x1.17a8e301c4436p-13};

// Sine and cosine of a non-negative angle: formed and reduced to [-pi/4, pi/4]
// in float64 (positions reach 10^3 and more), then the Taylor polynomials of
// degree 9 and 10 (remainders below 2e-9) in float32.
__device__ __forceinline__ void sin_cos(double angle, float& sn, float& cs) {
  const double q = rint(angle * 0.63661977236758134);  // quarter turns
  const float x = static_cast<float>(fma(-q, 6.123233995736766e-17, fma(-q, 1.5707963267948966, angle)));
  const float x2 = x * x;
  float s = fmaf(x2, 1.0f / 362880.0f, -1.0f / 5040.0f);
  s = fmaf(s, x2, 1.0f / 120.0f);
  s = fmaf(s, x2, -1.0f / 6.0f);
  s = fmaf(s * x2, x, x);
  float c = fmaf(x2, -1.0f / 3628800.0f, 1.0f / 40320.0f);
  c = fmaf(c, x2, -1.0f / 720.0f);
  c = fmaf(c, x2, 1.0f / 24.0f);
  c = fmaf(c, x2, -0.5f);
  c = fmaf(c, x2, 1.0f);
  const uint32_t n = static_cast<uint32_t>(static_cast<int32_t>(q));
  const float ss = (n & 1u) ? c : s, cc = (n & 1u) ? s : c;
  sn = (n & 2u) ? -ss : ss;
  cs = ((n + 1u) & 2u) ? -cc : cc;
}

// Largest i in [lo, hi] with offsets[i] <= r (offsets non-decreasing), or lo.
__device__ __forceinline__ int32_t request_in(const int32_t* offsets, int32_t lo, int32_t hi, int64_t r) {
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if (offsets[mid] <= r) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Largest i in [0, n_req) with offsets[i] <= r, or 0: a 64-ary search by one
// wave (one memory round trip per factor of 64 requests).
__device__ __forceinline__ int32_t request_of_wave(const int32_t* offsets, int32_t n_req, int64_t r) {
  const int lane = threadIdx.x % kWave;
  int64_t lo = 0, span = n_req;  // the answer lies in [lo, lo + span)
  while (span > 1) {
    const int64_t step = (span + kWave - 1) / kWave;
    const int64_t k = lane * step;
    const int cnt = __popcll(__ballot(k < span && offsets[lo + k] <= r));
    const int64_t skip = cnt > 0 ? (cnt - 1) * step : 0;
    lo += skip;
    span = step < span - skip ? step : span - skip;
  }
  return static_cast<int32_t>(lo);
}

// The three bfloat16 terms of four floats, each rounded to nearest: every
// remainder is exact, and the third term holds what is left of 24 bits. Two
// values share a conversion, whose halves are taken back as floats.
struct Split4 {
  uint2 t[3];
};
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
}
__device__ __forceinline__ Split4 split4(f4 x) {
  Split4 s;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    s.t[p] = uint2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
    x -= f4{bf16_lo(s.t[p].x), bf16_hi(s.t[p].x), bf16_lo(s.t[p].y), bf16_hi(s.t[p].y)};
  }
  return s;
}
// The terms of four consecutive values into three planes `plane` elements apart.
__device__ __forceinline__ void store_split(__bf16* dst, int64_t plane, f4 x) {
  const Split4 s = split4(x);
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(dst + p * plane) = s.t[p];
}

// Fragments in memory are laid out in lane order: a load of a wave then reads
// one contiguous KB. (Loads that take 16 bytes of each of 16 rows keep the
// address unit busy for four times as long, and with it this whole path: 193
// instead of 160 us for 64 requests of 512 tokens, all else alike.)
//
// A split weight matrix [N][K] of the parameters starts at three times its
// float offset: for every 16 rows and 32 columns the three terms' fragments,
// each of the lanes' 8 consecutive columns, lane l those of row l % 16 from
// column 8 (l / 16). A lane's fragments of the jb-th 16 rows:
constexpr int kFrag = 8 * kWave;  // elements of a fragment
constexpr int64_t kWSplit = 3 * static_cast<int64_t>(kW_out);  // elements of all of them
template <int K>
struct Weights {
  b8 v[3][K / 32];
  __device__ __forceinline__ void load(const __bf16* W, int jb) {
    const __bf16* f = W + jb * (K / 32) * 3 * kFrag + 8 * (threadIdx.x % kWave);
#pragma unroll
    for (int b = 0; b < K / 32; ++b)
#pragma unroll
      for (int p = 0; p < 3; ++p) v[p][b] = *reinterpret_cast<const b8*>(f + (3 * b + p) * kFrag);
  }
};
// Splits the parameters i .. i + 7 (i a multiple of 8) into their place, when
// they belong to a matrix.
__device__ __forceinline__ void split_weights(const HeadArgs& a, int64_t i) {
  if (i < kLayer0 || i >= kW_out) return;
  const int64_t l0 = kLayer0 + (i - kLayer0) / kLayerSize * kLayerSize;
  const int o = static_cast<int>(i - l0);
  int base, K;
  if (o < kB_qkv) base = kW_qkv, K = D;
  else if (o >= kW_o && o < kB_o) base = kW_o, K = D;
  else if (o >= kW_1 && o < kB_1) base = kW_1, K = D;
  else if (o >= kW_2 && o < kB_2) base = kW_2, K = FF;
  else return;
  const int n = (o - base) / K, k = (o - base) % K;
  __bf16* dst = a.Ws + 3 * (l0 + base) + ((n / 16) * (K / 32) + k / 32) * 3 * kFrag + ((k % 32) / 8 * 16 + n % 16) * 8;
  const f4* src = reinterpret_cast<const f4*>(a.weights + i);
  store_split(dst, kFrag, src[0]);
  store_split(dst + 4, kFrag, src[1]);
}
static_assert(kLayer0 % 8 == 0 && kLayerSize % 8 == 0 && kB_qkv % 8 == 0 && kW_o % 8 == 0 && kW_1 % 8 == 0 &&
                  kW_2 % 8 == 0 && kW_out % 8 == 0,
              "8 columns of one row");

// The same of 16 activation rows in LDS (planes `plane` apart, row stride sa).
template <int K>
struct Rows {
  b8 v[3][K / 32];
  __device__ __forceinline__ void load(const __bf16* A, int plane, int sa) {
    const int lane = threadIdx.x % kWave;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int b = 0; b < K / 32; ++b)
        v[p][b] = *reinterpret_cast<const b8*>(A + p * plane + (lane % 16) * sa + 32 * b + 8 * (lane / 16));
  }
};

// The 16 x 16 product x y^T of two split operands, the small terms first:
// lane l receives columns (rows of y) l % 16, rows (of x) 4 (l / 16) .. + 3.
template <int K, typename X, typename Y>
__device__ __forceinline__ f4 product(const X& x, const Y& y) {
  f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int kP[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
  for (int t = 0; t < 6; ++t)
#pragma unroll
    for (int b = 0; b < K / 32; ++b)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v[kP[t][0]][b], y.v[kP[t][1]][b], acc, 0, 0, 0);
  return acc;
}

// Queries and keys are stored split, values in float32, all of them per head
// and group of 16 rows (16 k .. 16 k + 15 of all rows) in the attention's operand
// order. Of a group of Q (scaled by log2(e) / sqrt(16)) or K, term p of
// dimension d of row s is element 256 p + 128 (d / 8) + 8 s + d % 8; of a
// group of V, dimension d of row s is element 64 (s / 4) + 4 d + s % 4.
constexpr int kQK = 3 * DH * 16;  // elements of a group of Q or K
constexpr int kVG = DH * 16;      // of V
__device__ __forceinline__ int64_t group_of(const HeadArgs& a, int hd, int64_t row) {
  return hd * (a.np >> 4) + (row >> 4);
}

// Q or K of one row of head hd, a lane holding dimensions 4 (l / 16) .. + 3.
__device__ __forceinline__ void store_qk(const HeadArgs& a, __bf16* X, int hd, int64_t row, f4 x) {
  const int g = (threadIdx.x % kWave) / 16;
  store_split(X + group_of(a, hd, row) * kQK + 128 * (g / 2) + 8 * (row & 15) + 4 * (g % 2), 256, x);
}
// V of the rows row4 .. + 3 (row4 a multiple of 4) that lie in [lo, hi), a
// lane holding dimension l % 16.
__device__ __forceinline__ void store_v(const HeadArgs& a, float* Vl, int hd, int64_t row4, int64_t lo, int64_t hi,
                                        f4 x) {
  float* dst = Vl + group_of(a, hd, row4) * kVG + 16 * (row4 & 15) + 4 * (threadIdx.x % 16);
  if (row4 >= lo && row4 + 4 <= hi) {
    *reinterpret_cast<f4*>(dst) = x;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (row4 + e >= lo && row4 + e < hi) dst[e] = x[e];
  }
}
constexpr float kScale = 1.4426950408889634f / 4.0f;  // log2(e) / sqrt(DH)

// A wave's parameters for the projections of head w % 4: waves 0-3 make Q and
// K, waves 4-7 V.
struct QkvWeights {
  Weights<D> w0, w1;  // Q and K, or V and none
  f4 bq, bk;
  float bv;
  __device__ __forceinline__ void load(const __bf16* W, const float* bias) {
    const int wv = threadIdx.x / kWave, hd = wv % NH, lane = threadIdx.x % kWave;
    const float* b = bias + DH * hd;
    w0.load(W, wv < NH ? hd : 2 * NH + hd);
    if (wv < NH) w1.load(W, NH + hd);
    bq = *reinterpret_cast<const f4*>(b + 4 * (lane / 16));
    bk = *reinterpret_cast<const f4*>(b + D + 4 * (lane / 16));
    bv = b[2 * D + lane % 16];
  }
};

// The list of row blocks: for every request of 1..max_len tokens the blocks
// of 16 rows from its first row, rounded down to a multiple of 4 (rows of
// a block that are not its request's are computed and not written), ordered
// by the request's number of key tiles, most first (a counting sort over that number, clamped to kPlanBins - 1).
// The layer kernel's workgroups are dispatched in this order, so that a long
// request's blocks do not start last. One workgroup.
constexpr int kPlanBins = 1024;
struct PlanShared {
  int32_t cnt[kPlanBins];
  int32_t wsum[kWaves];
};
__device__ void plan_blocks(const HeadArgs& a, PlanShared& sh) {
  for (int b = threadIdx.x; b < kPlanBins; b += kThreads) sh.cnt[b] = 0;
  __syncthreads();
  auto blocks_of = [&](int32_t i, int32_t& lo, int32_t& hi, int& bin) -> int32_t {
    lo = a.offsets[i];
    hi = a.offsets[i + 1];
    const int64_t T = static_cast<int64_t>(hi) - lo;
    if (T < 1 || T > a.max_len || lo < 0 || hi > a.n_rows) return 0;
    const int64_t tiles = (T + kKT - 1) / kKT;
    bin = static_cast<int>(tiles < kPlanBins ? tiles : kPlanBins - 1);
    return static_cast<int32_t>((hi - (lo & ~3) + kRows - 1) / kRows);
  };
  int32_t lo, hi;
  int bin;
  for (int32_t i = threadIdx.x; i < a.n_req; i += kThreads) {
    const int32_t nb = blocks_of(i, lo, hi, bin);
    if (nb > 0) atomicAdd(&sh.cnt[bin], nb);
  }
  __syncthreads();
  {  // starting positions, largest bin first: thread j takes kPer bins from the top
    constexpr int kPer = kPlanBins / kThreads;
    const int j = threadIdx.x, lane = j % kWave, wv = j / kWave;
    int32_t c[kPer], tot = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      c[k] = sh.cnt[kPlanBins - 1 - (kPer * j + k)];
      tot += c[k];
    }
    int32_t x = tot;  // inclusive scan within the wave
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int32_t t = __shfl_up(x, d);
      if (lane >= d) x += t;
    }
    if (lane == kWave - 1) sh.wsum[wv] = x;
    __syncthreads();
    int32_t before = 0;
    for (int k = 0; k < wv; ++k) before += sh.wsum[k];
    // the count fits the list when the offsets meet their precondition
    // (non-decreasing, within the rows), and the list is never written past
    // its size in any case
    if (j == kThreads - 1) a.ctl[0] = before + x < a.cap ? before + x : a.cap;
    int32_t at = before + x - tot;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      sh.cnt[kPlanBins - 1 - (kPer * j + k)] = at;
      at += c[k];
    }
  }
  __syncthreads();
  for (int32_t i = threadIdx.x; i < a.n_req; i += kThreads) {
    const int32_t nb = blocks_of(i, lo, hi, bin);
    if (nb == 0) continue;
    const int32_t p = atomicAdd(&sh.cnt[bin], nb);
    for (int32_t b = 0; b < nb; ++b)
      if (p + b < a.cap) a.items[p + b] = HeadBlock{(lo & ~3) + static_cast<int32_t>(kRows) * b, lo, hi, i};
  }
}

}  // namespace

// Projection and positional encoding of 16 rows at a time and the first
// layer's queries, keys and values (in float32: its weights are not split
// yet). The first workgroups list the blocks and split the weights
// meanwhile; each of the others stages the 48 KB of weights once and takes
// every grid's tile of rows.
constexpr int kSplitWgs = (kW_out / 8 + kThreads - 1) / kThreads;
constexpr int kEmbedWgs = 512;  // two per CU: what their LDS allows
__global__ __launch_bounds__(kThreads) void head_embed_kernel(HeadArgs a) {
  __shared__ union {
    struct {
      __attribute__((aligned(16))) float A[kRows * kSA];
      __attribute__((aligned(16))) float W[QKV * kSA];
    } e;
    PlanShared plan;
  } sh;
  __shared__ int32_t sReq[2];
  if (blockIdx.x == 0) {
    plan_blocks(a, sh.plan);
    return;
  }
  if (blockIdx.x <= kSplitWgs) {
    split_weights(a, 8 * (static_cast<int64_t>(blockIdx.x - 1) * kThreads + threadIdx.x));
    return;
  }
  const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave, hd = wv % NH;
  const int i16 = lane % 16, g = lane / 16;
  constexpr int kWVecs = QKV * D / 4 / kThreads;
  f4 wreg[kWVecs];  // on its way to LDS
#pragma unroll
  for (int k = 0; k < kWVecs; ++k)
    wreg[k] = reinterpret_cast<const f4*>(a.weights + kLayer0 + kW_qkv)[threadIdx.x + k * kThreads];
  const float* bias = a.weights + kLayer0 + kB_qkv + DH * hd;
  const f4 bq = *reinterpret_cast<const f4*>(bias + 4 * g), bk = *reinterpret_cast<const f4*>(bias + D + 4 * g);
  const float bv = bias[2 * D + i16];
  // A thread has one feature pair (2p, 2p + 1) of one row: the sine and the
  // cosine of (t - 1) f_p.
  constexpr int kPairs = D / 2;
  static_assert(kThreads == kRows * kPairs, "one pair per thread");
  const int pair = threadIdx.x % kPairs, rr = threadIdx.x / kPairs;
  const double freq = kFreq[pair];
  const f4 w0 = *reinterpret_cast<const f4*>(a.weights + kW_in + 8 * pair);
  const f4 w1 = *reinterpret_cast<const f4*>(a.weights + kW_in + 8 * pair + 4);
  const float b0 = a.weights[kB_in + 2 * pair], b1 = a.weights[kB_in + 2 * pair + 1];
#pragma unroll
  for (int k = 0; k < kWVecs; ++k) {
    const int i = threadIdx.x + k * kThreads;
    *reinterpret_cast<f4*>(&sh.e.W[(i / (D / 4)) * kSA + (i % (D / 4)) * 4]) = wreg[k];
  }
  const int64_t tiles = (a.n_rows + kRows - 1) / kRows;
  for (int64_t tile = blockIdx.x - 1 - kSplitWgs; tile < tiles; tile += gridDim.x - 1 - kSplitWgs) {
    const int64_t r0 = tile * kRows, r = r0 + rr;
    float x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = r < a.n_rows ? a.X[r * 4 + c] : 0.0f;
    // the requests of the tile's first and last row
    if (threadIdx.x < 2 * kWave) {
      const int64_t rl = r0 + kRows <= a.n_rows ? r0 + kRows - 1 : a.n_rows - 1;
      const int32_t i = request_of_wave(a.offsets, a.n_req, threadIdx.x < kWave ? r0 : rl);
      if (threadIdx.x % kWave == 0) sReq[threadIdx.x / kWave] = i;
    }
    __syncthreads();  // also: the last tile's rows in LDS have been read
    float2 h = {0.0f, 0.0f};
    if (r < a.n_rows) {
      const int32_t req = request_in(a.offsets, sReq[0], sReq[1], r);
      h.x = b0;
      h.y = b1;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        h.x = fmaf(w0[c], x[c], h.x);
        h.y = fmaf(w1[c], x[c], h.y);
      }
      float sn, cs;
      sin_cos(static_cast<double>(r - a.offsets[req]) * freq, sn, cs);
      h.x += sn;
      h.y += cs;
    }
    *reinterpret_cast<float2*>(&sh.e.A[rr * kSA + 2 * pair]) = h;
    *reinterpret_cast<float2*>(a.H + r * D + 2 * pair) = h;
    __syncthreads();
    // k = 16 b + 4 (l / 16) + m for product m of block b (any assignment of a
    // block's 16 values of k works when both operands share it), so that a
    // lane's four values of either operand are one 16-byte read
    f4 p0 = {0.0f, 0.0f, 0.0f, 0.0f}, p1 = p0;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) {
      const int at = 16 * b + 4 * g;
      auto wfrag = [&](int j) { return *reinterpret_cast<const f4*>(&sh.e.W[(j * D + DH * hd + i16) * kSA + at]); };
      const f4 a4 = *reinterpret_cast<const f4*>(&sh.e.A[i16 * kSA + at]);
      if (wv < NH) {
        const f4 wq = wfrag(0), wk = wfrag(1);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          p0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[m], a4[m], p0, 0, 0, 0);
          p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wk[m], a4[m], p1, 0, 0, 0);
        }
      } else {  // operands the other way round: the lanes then hold four consecutive rows
        const f4 wvv = wfrag(2);
#pragma unroll
        for (int m = 0; m < 4; ++m) p0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[m], wvv[m], p0, 0, 0, 0);
      }
    }
    if (wv < NH) {
      store_qk(a, a.Q, hd, r0 + i16, (p0 + bq) * kScale);
      store_qk(a, a.K[0], hd, r0 + i16, p1 + bk);
    } else {
      store_v(a, a.V[0], hd, r0 + 4 * g, 0, a.np, p0 + bv);
    }
  }
}

// Attention state of a wave: its queries' references, its lanes' shares of
// the sums, and four output dimensions of query l % 16 per lane.
struct Attn {
  float m, l;
  f4 o;
};

// A wave's queries as operands of 32 k, each two products of 16 dimensions:
// against the keys' [k1 | k2] the operands [q1 | q1] and [q2 | q2], against
// [k1 | k3] the operand [q3 | q1].
struct Queries {
  b8 q11, q22, q31;
};

// Attention of 16 queries, one head (Kh, Vh: its first group's fragments),
// over those keys of the request [lo, hi) that lie in the tiles from first to
// below last (first a multiple of 16; first < last only where a tile holds a
// key of the request).
// Per tile of 64 keys the wave forms the transposed scores S^T = K Q^T, so that
// lane l holds the scores of query l % 16 for keys 4 (l / 16) + r, r = 0..3 of
// each group of 16; then O^T += V^T P^T with v_mfma_f32_16x16x4f32, in which
// the score registers already are the second operand (keys of a group taken
// in the order 4 (l / 16) + r) and every lane keeps the outputs of its own
// query. Keys and values come straight from memory in operand layout: a
// tile's values are asked for before its scores are formed, the next tile's
// keys as soon as they are; no LDS and no barrier, so the waves of a
// workgroup run apart.
// The softmax is online in base 2 against a reference m that moves only when
// a score exceeds it by more than kSlack (the masses stay below 2^kSlack, in
// float32 a change of exponent only). The products start from -m, so that in
// all but the first tiles the update is an exp and an add per score; the
// query's sum over its four lanes is taken once at the end. Each query's
// reference moves by its own scores alone (a wave enters the step for all its
// queries as soon as one needs it, and the others move by 0): a move by a
// fraction of an octave changes the rounding of what follows, and the result of
// a query must not depend on the queries beside it.
constexpr float kSlack = 8.0f;

__device__ __forceinline__ void attend(const __bf16* Kh, const float* Vh, int64_t first, int64_t last, int64_t lo,
                                       int64_t hi, const Queries& q, Attn& st) {
  constexpr int kSub = kKT / 16;
  const int lane = threadIdx.x % kWave;
  const int g = lane / 16;
  st.m = -INFINITY;
  st.l = 0.0f;
  st.o = f4{0.0f, 0.0f, 0.0f, 0.0f};
  if (first >= last) return;
  const __bf16* K12 = Kh + 8 * lane;                    // [k1 | k2]
  const __bf16* K13 = K12 + (lane < kWave / 2 ? 0 : 256);  // [k1 | k3]
  b8 k12[kSub], k13[kSub];
  auto load_keys = [&](int64_t t) {
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
      k12[j] = *reinterpret_cast<const b8*>(K12 + ((t >> 4) + j) * kQK);
      k13[j] = *reinterpret_cast<const b8*>(K13 + ((t >> 4) + j) * kQK);
    }
  };
  load_keys(first);
  f4 s[kSub], v[kSub];
  st.m = 0.0f;
  for (int64_t t = first; t < last; t += kKT) {
#pragma unroll
    for (int j = 0; j < kSub; ++j) v[j] = *reinterpret_cast<const f4*>(Vh + ((t >> 4) + j) * kVG + 4 * lane);
    const float nm = -st.m;
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
      s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k13[j], q.q31, f4{nm, nm, nm, nm}, 0, 0, 0);
      s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k12[j], q.q22, s[j], 0, 0, 0);
      s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k12[j], q.q11, s[j], 0, 0, 0);
    }
    if (t + kKT < last) load_keys(t + kKT);
    if (t < lo || t + kKT > hi) {
      // keys outside the request: probability 0; their values may be anything
      // (another request's NaN) and must read as 0
      const int from = static_cast<int>(lo - t) - 4 * g, in = static_cast<int>(hi - t) - 4 * g;
#pragma unroll
      for (int j = 0; j < kSub; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * j + r < from || 16 * j + r >= in) {
            v[j][r] = 0.0f;
            s[j][r] = -INFINITY;
          }
    }
    float tm = s[0][0];
#pragma unroll
    for (int j = 0; j < kSub; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) tm = fmaxf(tm, s[j][r]);
    if (t == first || __any(tm > kSlack)) {
      // the reference of a query that needs it moves to its largest score so
      // far (from 0 to the first tile's, which may lie below)
      tm = fmaxf(tm, __shfl_xor(tm, 16));
      tm = fmaxf(tm, __shfl_xor(tm, 32));
      const float d = t == first || tm > kSlack ? tm : 0.0f;
      const float corr = fast_exp2(-d);
      st.l = t == first ? 0.0f : st.l * corr;
      st.o = t == first ? f4{0.0f, 0.0f, 0.0f, 0.0f} : st.o * corr;
      st.m += d;
#pragma unroll
      for (int j = 0; j < kSub; ++j) s[j] -= d;
    }
    f4 ps = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s[j][r] = fast_exp2(s[j][r]);
      ps += s[j];
    }
    st.l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
#pragma unroll
    for (int j = 0; j < kSub; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        st.o = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j][r], s[j][r], st.o, 0, 0, 0);
  }
}

// Sum over the 16 lanes of a row of the wave, in every lane (lane moves
// within the row: an LDS exchange per step would be most of a LayerNorm's
// time).
__device__ __forceinline__ float row_sum(float v) {
  using namespace dpp;
  v += movf<kXor1, 0xf>(0.0f, v);
  v += movf<kXor2, 0xf>(0.0f, v);
  v += movf<kHalfMirror, 0xf>(0.0f, v);
  v += movf<kMirror, 0xf>(0.0f, v);
  return v;
}

// LayerNorm of a row whose 64 values are held by 16 consecutive lanes, four
// each. Biased variance, eps 1e-5.
constexpr int kTPR = D / 4;
static_assert(kTPR == 16, "a row of lanes per row of values");
__device__ __forceinline__ void layer_norm(f4& x, const f4& g, const f4& b) {
  x -= row_sum((x[0] + x[1]) + (x[2] + x[3])) * (1.0f / D);
  const float v = row_sum(fmaf(x[0], x[0], x[1] * x[1]) + fmaf(x[2], x[2], x[3] * x[3]));
  const float inv = 1.0f / sqrtf(v * (1.0f / D) + kLnEps);
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = fmaf(x[e] * inv, g[e], b[e]);
}

// One encoder layer of one block (see the top of the file), block `from` of
// the list and those after it. LAST: the rows'
// products with the output map instead of the next layer's projections.
// Eight waves: in the attention wave w is head w % 4 over half w / 4 of the
// key tiles; of the dense products waves 0-3 make those with 64 columns, 16
// each, and all eight the feed-forward's first. 110-122 registers: two
// workgroups per CU (a barrier of one is the other's work; blocks of 32 rows
// took 143, one workgroup per CU, and 104 instead of 86 us on 64 requests of
// 16 to 512 tokens).
template <bool LAST>
__global__ __launch_bounds__(kThreads) void head_layer_kernel(HeadArgs a, int layer, int32_t from) {
  constexpr int kPA = kRows * kBA, kPF = kRows * kBF;  // planes of split activations
  __shared__ __attribute__((aligned(16))) __bf16 sB[3 * kPA];     // attention output, then h1, then h2, split
  __shared__ __attribute__((aligned(16))) float sY[kRows * kSA];  // y, then h1, then z
  __shared__ union {
    __attribute__((aligned(16))) __bf16 F[3 * kPF];  // feed-forward hidden layer, split
    struct {  // the second half's attention states
      f4 o[NH][kWave];
      float m[NH][kWave], l[NH][kWave];
    } at;
  } su;
  const int32_t count = a.ctl[0];
  const int32_t block = from + static_cast<int32_t>(blockIdx.x);
  const HeadBlock it = a.items[block];
  if (block >= count) return;
  const int64_t r0 = it.r0, lo = it.lo, hi = it.hi;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int i16 = lane % 16, g = lane / 16;
  const int hd = w % NH, half = w / NH;
  const int64_t at = kLayer0 + static_cast<int64_t>(layer) * kLayerSize;
  const float* Wl = a.weights + at;
  const __bf16* Ws = a.Ws + 3 * at;
  Attn st;
  // Q and H have one buffer: in this launch the workgroups of the neighbouring
  // requests write the next layer's into their rows, and rows past the last
  // group hold whatever the workspace held. In the place of a block's rows that
  // are not its request's (computed and never written) the nearest of the
  // request's is read.
  const int64_t own = min(max(r0 + i16, lo), hi - 1);
  {
    Queries q;
    const __bf16* Q = a.Q + group_of(a, hd, own) * kQK + 128 * (g % 2) + 8 * (own & 15);
    q.q11 = *reinterpret_cast<const b8*>(Q);
    q.q22 = *reinterpret_cast<const b8*>(Q + 256);
    q.q31 = *reinterpret_cast<const b8*>(Q + (g < 2 ? 512 : 0));
    const int64_t first = lo & ~int64_t{15};
    const int64_t tiles = (hi - first + kKT - 1) / kKT;
    const int64_t mid = first + (tiles + 1) / 2 * kKT;
    const __bf16* Kh = a.K[layer] + group_of(a, hd, 0) * kQK;
    const float* Vh = a.V[layer] + group_of(a, hd, 0) * kVG;
    attend(Kh, Vh, half ? mid : first, half ? hi : (mid < hi ? mid : hi), lo, hi, q, st);
  }
  Weights<D> wo;
  f4 bo, hres;
  if (half == 0) {
    wo.load(Ws + 3 * kW_o, hd);
    bo = *reinterpret_cast<const f4*>(Wl + kB_o + 16 * hd + 4 * g);
    hres = *reinterpret_cast<const f4*>(a.H + own * D + 16 * hd + 4 * g);
  }
  const int lr = threadIdx.x / kTPR, lc = (threadIdx.x % kTPR) * 4;  // LayerNorm: row and first column
  const f4 g1 = *reinterpret_cast<const f4*>(Wl + kLn1g + lc), e1 = *reinterpret_cast<const f4*>(Wl + kLn1b + lc);
  if (half == 1) {
    su.at.o[hd][lane] = st.o;
    su.at.m[hd][lane] = st.m;
    su.at.l[hd][lane] = st.l;
  }
  __syncthreads();
  if (half == 0) {
    const float m1 = su.at.m[hd][lane];
    const float m = fmaxf(st.m, m1);
    const float c0 = fast_exp2(st.m - m), c1 = fast_exp2(m1 - m);
    float l = st.l * c0 + su.at.l[hd][lane] * c1;
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const f4 o = st.o * c0 + su.at.o[hd][lane] * c1;
    store_split(&sB[i16 * kBA + DH * hd + 4 * g], kPA, o * (1.0f / l));
  }
  Weights<D> w1;  // all eight waves: 16 columns of the hidden layer each
  w1.load(Ws + 3 * kW_1, w);
  const f4 b1 = *reinterpret_cast<const f4*>(Wl + kB_1 + 16 * w + 4 * g);
  __syncthreads();
  // y = att W_o^T + b_o + h; h1 = LN1(y)
  if (half == 0) {
    Rows<D> x;
    x.load(sB, kPA, kBA);
    *reinterpret_cast<f4*>(&sY[i16 * kSA + 16 * hd + 4 * g]) = product<D>(wo, x) + (bo + hres);
  }
  __syncthreads();
  f4 x;
  if (lr < kRows) {
    x = *reinterpret_cast<const f4*>(&sY[lr * kSA + lc]);
    layer_norm(x, g1, e1);
    *reinterpret_cast<f4*>(&sY[lr * kSA + lc]) = x;
    store_split(&sB[lr * kBA + lc], kPA, x);
  }
  Weights<FF> w2;  // issued now, used after the next product
  f4 b2;
  if (half == 0) {
    w2.load(Ws + 3 * kW_2, hd);
    b2 = *reinterpret_cast<const f4*>(Wl + kB_2 + 16 * hd + 4 * g);
  }
  __syncthreads();
  // f = relu(h1 W_1^T + b_1)
  {
    Rows<D> h1;
    h1.load(sB, kPA, kBA);
    f4 f = product<D>(w1, h1) + b1;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = fmaxf(f[e], 0.0f);
    store_split(&su.F[i16 * kBF + 16 * w + 4 * g], kPF, f);
  }
  const f4 g2 = *reinterpret_cast<const f4*>(Wl + kLn2g + lc), e2 = *reinterpret_cast<const f4*>(Wl + kLn2b + lc);
  __syncthreads();
  // z = f W_2^T + b_2 + h1; h2 = LN2(z)
  if (half == 0) {
    Rows<FF> f;
    f.load(su.F, kPF, kBF);
    f4* y = reinterpret_cast<f4*>(&sY[i16 * kSA + 16 * hd + 4 * g]);
    *y = product<FF>(w2, f) + (b2 + *y);
  }
  QkvWeights wq;
  if constexpr (!LAST) wq.load(Ws + 3 * (kLayerSize + kW_qkv), Wl + kLayerSize + kB_qkv);
  __syncthreads();
  if (lr < kRows) {
    x = *reinterpret_cast<const f4*>(&sY[lr * kSA + lc]);
    layer_norm(x, g2, e2);
  }
  if constexpr (LAST) {
    // the row's product with the output map (the mean over the rows follows)
    if (lr < kRows) {
      const f4 wout = *reinterpret_cast<const f4*>(a.weights + kW_out + lc);
      const float s = row_sum(fmaf(x[0], wout[0], x[1] * wout[1]) + fmaf(x[2], wout[2], x[3] * wout[3]));
      if (threadIdx.x % kTPR == 0 && r0 + lr >= lo && r0 + lr < hi) a.z[r0 + lr] = s;
    }
  } else {
    if (lr < kRows) {
      if (r0 + lr >= lo && r0 + lr < hi) *reinterpret_cast<f4*>(a.H + (r0 + lr) * D + lc) = x;
      store_split(&sB[lr * kBA + lc], kPA, x);
    }
    __syncthreads();
    Rows<D> h2;
    h2.load(sB, kPA, kBA);
    const int64_t row = r0 + i16;
    if (half == 0) {
      const f4 q = product<D>(wq.w0, h2) + wq.bq, k = product<D>(wq.w1, h2) + wq.bk;
      if (row >= lo && row < hi) {
        store_qk(a, a.Q, hd, row, q * kScale);
        store_qk(a, a.K[1 - layer], hd, row, k);
      }
    } else {  // operands the other way round: the lanes then hold four consecutive rows
      store_v(a, a.V[1 - layer], hd, r0 + 4 * g, lo, hi, product<D>(h2, wq.w0) + wq.bv);
    }
  }
}

// The mean of a request's row products plus the output bias, sigmoid. An
// empty request, or one longer than max_len, scores NaN. One wave per
// request.
__global__ __launch_bounds__(kWave) void head_score_kernel(HeadArgs a) {
  const int64_t req = blockIdx.x;
  const int64_t lo = a.offsets[req], hi = a.offsets[req + 1];
  const int64_t T = hi - lo;
  const bool ok = T > 0 && T <= a.max_len && lo >= 0 && hi <= a.n_rows;
  double s = 0.0;
  if (ok) {
#pragma unroll 8
    for (int64_t r = lo + threadIdx.x; r < hi; r += kWave) s += static_cast<double>(a.z[r]);
  }
  s = wave_sum_d(s);
  if (threadIdx.x == 0) {
    const float z = static_cast<float>(s / static_cast<double>(T > 0 ? T : 1)) + a.weights[kB_out];
    a.scores[req] = ok ? 1.0f / (1.0f + expf(-z)) : __uint_as_float(0x7fc00000u);
  }
}

namespace {

// Rows of the workspace's arrays: whole blocks, and a key tile from the last
// group of rows.
int64_t padded_rows(int64_t n_rows) { return (n_rows + kRows - 1) / kRows * kRows + kKT; }

}  // namespace

// The split weights; per padded row H, Q, two buffers each of K and V (a layer
// reads one while it writes the next layer's) and the row's product; then the
// list of blocks (at most one per row) and its length.
size_t head_workspace_bytes(int64_t n_rows) {
  const size_t np = static_cast<size_t>(padded_rows(n_rows));
  return kWSplit * sizeof(__bf16) + np * (3 * NH * 3 * DH * sizeof(__bf16) + (3 * D + 1) * sizeof(float)) +
         static_cast<size_t>(n_rows) * sizeof(HeadBlock) + 4 * sizeof(int32_t);
}

hipError_t launch_head(const HeadArgs& args, hipStream_t stream) {
  if (args.n_req == 0) return hipSuccess;
  HeadArgs a = args;
  static_assert(kHeadLayers == 2, "two buffers of keys and values");
  a.np = padded_rows(a.n_rows);
  a.cap = static_cast<int32_t>(a.n_rows);
  char* p = static_cast<char*>(a.ws);
  auto take = [&](size_t bytes) {
    char* at = p;
    p += bytes;
    return at;
  };
  const size_t np = static_cast<size_t>(a.np);
  static_assert(kWSplit * sizeof(__bf16) % 16 == 0, "16-byte aligned arrays");
  a.Ws = reinterpret_cast<__bf16*>(take(kWSplit * sizeof(__bf16)));
  a.Q = reinterpret_cast<__bf16*>(take(np * NH * 3 * DH * sizeof(__bf16)));
  for (int l = 0; l < kHeadLayers; ++l)
    a.K[l] = reinterpret_cast<__bf16*>(take(np * NH * 3 * DH * sizeof(__bf16)));
  a.H = reinterpret_cast<float*>(take(np * D * sizeof(float)));
  for (int l = 0; l < kHeadLayers; ++l) a.V[l] = reinterpret_cast<float*>(take(np * D * sizeof(float)));
  a.z = reinterpret_cast<float*>(take(np * sizeof(float)));
  a.items = reinterpret_cast<HeadBlock*>(take(static_cast<size_t>(a.n_rows) * sizeof(HeadBlock)));
  a.ctl = reinterpret_cast<int32_t*>(a.items + a.n_rows);
  if (a.n_rows > 0) {
    const int64_t tiles = (a.n_rows + kRows - 1) / kRows;
    // at most this many blocks: a request of T rows has at most (T + 3) / 16 + 1, and at most T
    const int64_t most = (a.n_rows + 3 * static_cast<int64_t>(a.n_req)) / kRows + a.n_req;
    const int64_t blocks = most < a.n_rows ? most : a.n_rows;
    // A launch holds fewer than 2^32 threads (more are cut off without an
    // error), so a longer list takes several.
    constexpr int64_t kMaxBlocks = (int64_t{1} << 32) / kThreads - 1;
    auto each_launch = [&](auto&& launch) {
      for (int64_t from = 0; from < blocks; from += kMaxBlocks)
        launch(static_cast<unsigned>(blocks - from < kMaxBlocks ? blocks - from : kMaxBlocks), static_cast<int32_t>(from));
    };
    head_embed_kernel<<<static_cast<unsigned>((tiles < kEmbedWgs ? tiles : kEmbedWgs) + 1 + kSplitWgs), kThreads, 0,
                        stream>>>(a);
    for (int l = 0; l + 1 < kHeadLayers; ++l)
      each_launch([&](unsigned n, int32_t from) { head_layer_kernel<false><<<n, kThreads, 0, stream>>>(a, l, from); });
    each_launch([&](unsigned n, int32_t from) {
      head_layer_kernel<true><<<n, kThreads, 0, stream>>>(a, kHeadLayers - 1, from);
    });
  }
  head_score_kernel<<<static_cast<unsigned>(a.n_req), kWave, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace pr
