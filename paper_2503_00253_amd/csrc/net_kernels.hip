// Kernels of the warm-start network (a 1-D convolutional net over the m observation rows; the
// method's extension for initial guesses of the shifted systems, Appendix E, eq. E.1).
//
// Layout: activations of a batch are (B, C, m) row-contiguous, element (b, c, x) at
// (b * C + c) * m + x.  Weights (Cout, Cin, K) row-contiguous, K odd, "same" zero padding:
//
//   y[b, o, x] = bias[o] + sum_c sum_k W[o, c, k] a[b, c, x + k - K/2].
//
// All arithmetic is FP32 (accumulation in FP32, reductions in a fixed order).
#include <algorithm>
#include <cmath>

#include "internal.hpp"

namespace infoesrf {

namespace {

constexpr int kCIC = 16;   // input channels staged per chunk
typedef float nf4 __attribute__((ext_vector_type(4)));

__device__ inline float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float z) {
  const float Phi = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
  const float phi = 0.39894228040143268f * expf(-0.5f * z * z);
  return Phi + z * phi;
}

// The correlation with FP32 FMAs.  Block: kVX positions (one a lane) x 4 CPW output channels (CPW a
// wavefront); input window and weight chunk in LDS, the weights read as wave-uniform broadcasts.  It
// does no work for channels that are not there, so it takes the layers that leave k_conv_mfma's tiles
// mostly empty (launch_conv_fwd has the rule).  A chunk's sums start at zero and are added to the total.
constexpr int kVX = 64;
template <int CPW>
__global__ __launch_bounds__(256) void k_conv_fma(const float* __restrict__ in, int Cin, const float* __restrict__ W,
                                                  const float* __restrict__ bias, int Cout, int K, int m,
                                                  float* __restrict__ pre, float* __restrict__ act, int gelu) {
  extern __shared__ float sm[];
  const int h = K / 2;
  const int WX = kVX + K - 1;
  float* win = sm;              // kCIC x WX
  float* wts = sm + kCIC * WX;  // (4 CPW) x kCIC x K
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x0 = blockIdx.x * kVX;
  const int o0 = blockIdx.y * 4 * CPW;
  const int64_t b = blockIdx.z;
  const float* inb = in + b * (int64_t)Cin * m;
  float tot[CPW];
#pragma unroll
  for (int j = 0; j < CPW; ++j) tot[j] = 0.f;
  for (int c0 = 0; c0 < Cin; c0 += kCIC) {
    const int cc = min(kCIC, Cin - c0);
    __syncthreads();
    for (int t = threadIdx.x; t < cc * WX; t += 256) {
      const int ci = t / WX, u = t % WX;
      const int x = x0 - h + u;
      win[t] = (x >= 0 && x < m) ? inb[(int64_t)(c0 + ci) * m + x] : 0.f;
    }
    for (int t = threadIdx.x; t < 4 * CPW * cc * K; t += 256) {
      const int o = t / (cc * K), u = t % (cc * K);
      wts[o * kCIC * K + u] = o0 + o < Cout ? W[((int64_t)(o0 + o) * Cin + c0) * K + u] : 0.f;
    }
    __syncthreads();
    float acc[CPW];
#pragma unroll
    for (int j = 0; j < CPW; ++j) acc[j] = 0.f;
    for (int ci = 0; ci < cc; ++ci)
      for (int k = 0; k < K; ++k) {
        const float v = win[ci * WX + lane + k];
#pragma unroll
        for (int j = 0; j < CPW; ++j) acc[j] = fmaf(wts[((wave * CPW + j) * kCIC + ci) * K + k], v, acc[j]);
      }
#pragma unroll
    for (int j = 0; j < CPW; ++j) tot[j] += acc[j];
  }
  const int x = x0 + lane;
  if (x >= m) return;
#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    const int o = o0 + wave * CPW + j;
    if (o >= Cout) continue;
    const float z = tot[j] + (bias ? bias[o] : 0.f);
    const int64_t at = (b * Cout + o) * (int64_t)m + x;
    if (pre) pre[at] = z;
    act[at] = gelu ? gelu_f(z) : z;
  }
}

// The correlation as an implicit GEMM on FP32 MFMA (v_mfma_f32_16x16x4_f32: FP32 operands and
// accumulation): output channels x positions, contracted over input channels four at a time and taps.
// Block: 64 output channels (16 a wavefront) x 32 positions.  Input channels come in chunks of 16 whose
// weights and window lie in LDS; the next chunk's values are loaded into registers while this one is
// multiplied.  LDS strides: a window row of kWinS = 80 words puts the 16 positions x 4 channels of an
// operand on 64 banks, a weight row of 16 K + 4 words the 16 outputs x 4 channels (K is odd).  32
// positions a block, so that the smallest training batches (8 members x 1024 positions) still give one
// block a CU.  The chunk held in registers bounds it: from 9 taps on (256 registers and 44 accumulation
// registers) one wavefront a SIMD is resident, which has nothing to hide its LDS reads (3 words a lane
// for 2 MFMA) and its chunk's loads behind.  8 members x 1024 positions, 64 x 64 channels, 9 taps (604
// MFLOP): 46 us with FP32 FMAs, four output channels a wavefront; 18 us so.
// FLIP: the weights are those of the layer whose input gradient this is, W (Cin, Cout, K), read as
// W'[o, c, k] = W[c, o, K - 1 - k] (the input gradient of a "same" correlation is the correlation of
// the output gradient with W').  dz (nullable): the outputs are multiplied by GELU'(dz).
constexpr int kCX = 32;    // positions per block
constexpr int kWinS = 80;  // words per window row: at least kCX + 14, 16 (mod 64)
constexpr int kMaxTaps = 15;
__host__ __device__ constexpr int conv_row(int K) { return kCIC * K + 4; }

template <int K, bool FLIP>
__global__ __launch_bounds__(256) void k_conv_mfma(const float* __restrict__ in, int Cin, const float* __restrict__ W,
                                                   const float* __restrict__ bias, int Cout, int m,
                                                   float* __restrict__ pre, float* __restrict__ act, int gelu,
                                                   const float* __restrict__ dz) {
  extern __shared__ float sm[];
  float* win = sm;                  // kCIC x kWinS
  float* wts = sm + kCIC * kWinS;   // 64 x conv_row(K)
  constexpr int h = K / 2, RS = conv_row(K), WX = kCX + K - 1;
  constexpr int NW = 64 * kCIC * K / 256, NI = (kCIC * WX + 255) / 256;  // weights, window values a thread loads
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int x0 = blockIdx.x * kCX;
  const int o0 = blockIdx.y * 64;
  const int64_t b = blockIdx.z;
  const float* inb = in + b * (int64_t)Cin * m;
  float rw[NW], ri[NI];
  auto load = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = tid + 256 * i;
      float v = 0.f;
      if (!FLIP) {
        const int o = t / (kCIC * K), u = t % (kCIC * K);
        if (o0 + o < Cout && u < (Cin - c0) * K) v = W[((int64_t)(o0 + o) * Cin + c0) * K + u];
      } else {
        const int c = t / (64 * K), u = t % (64 * K);
        if (c0 + c < Cin && u < (Cout - o0) * K) v = W[((int64_t)(c0 + c) * Cout + o0) * K + u];
      }
      rw[i] = v;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int t = tid + 256 * i, c = t / WX, u = t % WX, x = x0 - h + u;
      ri[i] = (c < kCIC && c0 + c < Cin && x >= 0 && x < m) ? inb[(int64_t)(c0 + c) * m + x] : 0.f;
    }
  };
  // a chunk's sums start at zero and are added to the total, which shortens the FP32 chains
  nf4 tot[2] = {nf4{0.f, 0.f, 0.f, 0.f}, nf4{0.f, 0.f, 0.f, 0.f}};
  load(0);
  for (int c0 = 0; c0 < Cin; c0 += kCIC) {
    __syncthreads();  // the previous chunk's reads are done
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = tid + 256 * i;
      if (!FLIP) {
        wts[(t / (kCIC * K)) * RS + t % (kCIC * K)] = rw[i];
      } else {
        const int c = t / (64 * K), u = t % (64 * K);
        wts[(u / K) * RS + c * K + K - 1 - u % K] = rw[i];
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int t = tid + 256 * i, c = t / WX;
      if (c < kCIC) win[c * kWinS + t % WX] = ri[i];
    }
    __syncthreads();
    if (c0 + kCIC < Cin) load(c0 + kCIC);
    nf4 acc[2] = {nf4{0.f, 0.f, 0.f, 0.f}, nf4{0.f, 0.f, 0.f, 0.f}};
    const int cq = min(kCIC, (Cin - c0 + 3) & ~3);
    for (int c = lq; c < cq; c += 4) {
      const float* wr = wts + (16 * wave + l16) * RS + c * K;
      const float* ir = win + c * kWinS + l16;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const float a = wr[k];
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ir[k], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ir[k + 16], acc[1], 0, 0, 0);
      }
    }
    tot[0] += acc[0];
    tot[1] += acc[1];
  }
  // D register v of lane l: output channel 4 (l / 16) + v of the wavefront's 16, position l % 16
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int x = x0 + 16 * t + l16;
    if (x >= m) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = o0 + 16 * wave + 4 * lq + v;
      if (o >= Cout) continue;
      const float z = tot[t][v] + (bias ? bias[o] : 0.f);
      const int64_t at = (b * Cout + o) * (int64_t)m + x;
      if (pre) pre[at] = z;
      act[at] = dz ? z * gelu_grad_f(dz[at]) : (gelu ? gelu_f(z) : z);
    }
  }
}

// ---- BF16 inference on MFMA (FP32 accumulation) --------------------------------------------
// The same correlation as an implicit GEMM: y[o, x] = bias[o] + sum_kd Wp[o, kd] A[kd, x] with
// kd = k Cp + c (Cp = input channels rounded up to 8, so the 8 values a lane feeds to one MFMA
// share k and are consecutive channels), A[kd, x] = a[c, x + k - K/2].  Weights are packed once
// per call to BF16 rows of KD = round_up(K Cp, 32) entries (Cout rounded up to 16 rows, zeros in
// the padding).  Activations between layers are BF16, position-major (b, x, c).
typedef __bf16 nbf8 __attribute__((ext_vector_type(8)));

__global__ void k_pack_weights_bf16(const float* __restrict__ W, int Cout, int Cin, int K, int Cp, int KD, int Opad,
                                    __hip_bfloat16* __restrict__ out) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)Opad * KD) return;
  const int o = (int)(t / KD), kd = (int)(t % KD);
  const int k = kd / Cp, c = kd % Cp;
  const float v = (o < Cout && k < K && c < Cin) ? W[((int64_t)o * Cin + c) * K + k] : 0.f;
  out[t] = __float2bfloat16(v);
}

// Block: 64 positions x 64 output channels (wavefront w: channels o0 + 16 w .. + 15, four
// 16-position tiles).  The input window (64 + K - 1 positions x Cp channels) is staged in LDS as
// BF16, rows padded by 8 channels (16 bytes) against bank conflicts.
// IN_F32: input (B, Cin, m) FP32, else (B, m, Cp) BF16.  OUT_F32: output (B, Cout, m) FP32, else
// (B, m, Cout) BF16.
template <bool IN_F32, bool OUT_F32>
__global__ __launch_bounds__(256) void k_conv_bf16(const void* __restrict__ in, int Cin, int Cp,
                                                   const __hip_bfloat16* __restrict__ Wp, int KD,
                                                   const float* __restrict__ bias, int Cout, int K, int m,
                                                   void* __restrict__ out, int gelu) {
  extern __shared__ __attribute__((aligned(16))) unsigned char nsm[];
  __hip_bfloat16* win = reinterpret_cast<__hip_bfloat16*>(nsm);
  const int h = K / 2;
  const int WX = 64 + K - 1;
  const int Cs = Cp + 8;  // LDS row stride (channels)
  const int x0 = blockIdx.x * 64;
  const int o0 = blockIdx.y * 64;
  const int64_t b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lrow = lane & 15, lk = lane >> 4;
  for (int t = tid; t < WX * Cp; t += 256) {
    const int u = t / Cp, c = t % Cp;
    const int x = x0 - h + u;
    float v = 0.f;
    if (x >= 0 && x < m && c < Cin) {
      if (IN_F32) v = static_cast<const float*>(in)[(b * Cin + c) * (int64_t)m + x];
      else v = __bfloat162float(static_cast<const __hip_bfloat16*>(in)[(b * m + x) * (int64_t)Cp + c]);
    }
    win[u * Cs + c] = __float2bfloat16(v);
  }
  __syncthreads();
  const int ob = o0 + 16 * wave;
  if (ob >= Cout) return;  // no channels for this wavefront (after the only barrier)
  nf4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = nf4{0.f, 0.f, 0.f, 0.f};
  const __hip_bfloat16* wrow = Wp + (int64_t)(ob + lrow) * KD + 8 * lk;
  for (int kd0 = 0; kd0 < KD; kd0 += 32) {
    const nbf8 a = *reinterpret_cast<const nbf8*>(wrow + kd0);
    const int kd = kd0 + 8 * lk;
    const int k = kd / Cp, c0 = kd % Cp;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      nbf8 bv;
      if (k < K) {
        bv = *reinterpret_cast<const nbf8*>(win + (16 * t + lrow + k) * Cs + c0);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) bv[i] = (__bf16)0.f;
      }
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bv, acc[t], 0, 0, 0);
    }
  }
  // D register v of lane l: channel ob + 4 (l / 16) + v, position x0 + 16 t + l % 16
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int x = x0 + 16 * t + lrow;
    if (x >= m) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = ob + 4 * lk + v;
      if (o >= Cout) continue;
      const float z = acc[t][v] + (bias ? bias[o] : 0.f);
      const float y = gelu ? gelu_f(z) : z;
      if (OUT_F32) static_cast<float*>(out)[(b * Cout + o) * (int64_t)m + x] = y;
      else static_cast<__hip_bfloat16*>(out)[(b * m + x) * (int64_t)Cout + o] = __float2bfloat16(y);
    }
  }
}

// Weight gradient of one layer: gW[o, c, k] = sum_{b, x} g[b, o, x] a[b, c, x + k - K/2] and
// gb[o] = sum_{b, x} g[b, o, x], as one product per tap on FP32 MFMA (v_mfma_f32_16x16x4_f32, FP32
// operands and accumulation): output channels x input channels, contracted over positions.  The B m
// positions come in chunks of kGX of one member; block (s, c-tile, o-group) adds the chunks s, s + nsplit,
// ... for 64 output channels (16 a wavefront) and 16 input channels, every tap in registers, and writes
// its partial sums; k_wgrad_reduce adds the nsplit partials in order in FP64.  Sums of 32 positions start
// at zero and are added to the block's, so the FP32 chains stay short.  The split fills the chip, which one
// block per (output channel, 8 input channels) did not: 64 x 64 channels, 9 taps, 8 members x 1024
// positions (604 MFLOP) 570 us before, 22 us and 5 us for the reduction now.  LDS rows are 4 (mod 8) words apart, so the
// 16 channels x 4 positions of an operand lie on 64 banks.
constexpr int kGX = 128;
constexpr int kGS = kGX + 4, kAS = kGX + 20;  // row strides of g and of the window (kGX + 14 at most)

template <int K>
__global__ __launch_bounds__(256) void k_wgrad_mfma(const float* __restrict__ a, int Cin, const float* __restrict__ g,
                                                    int Cout, int m, int64_t B, float* __restrict__ part) {
  extern __shared__ float sm[];
  float* sg = sm;                // 64 x kGS
  float* sa = sm + 64 * kGS;     // 16 x kAS
  constexpr int h = K / 2, WX = kGX + K - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int c0 = blockIdx.y * 16, o0 = blockIdx.z * 64;
  const int per = (m + kGX - 1) / kGX;          // chunks a member
  const int64_t chunks = B * per;
  const bool mine = o0 + 16 * wave < Cout;      // the wavefront has output channels
  nf4 tot[K], acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) tot[k] = acc[k] = nf4{0.f, 0.f, 0.f, 0.f};
  float sb = 0.f;
  auto flush = [&]() {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      tot[k] += acc[k];
      acc[k] = nf4{0.f, 0.f, 0.f, 0.f};
    }
  };
  for (int64_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const int64_t b = ch / per;
    const int x0 = (int)(ch % per) * kGX;
    const float* gp = g + (b * Cout + o0) * (int64_t)m;
    const float* ap = a + (b * Cin + c0) * (int64_t)m;
    __syncthreads();  // the previous chunk's reads are done
#pragma unroll 8
    for (int i = 0; i < 64 * kGX / 256; ++i) {
      const int t = tid + 256 * i, o = t / kGX, x = x0 + t % kGX;
      sg[o * kGS + t % kGX] = (o0 + o < Cout && x < m) ? gp[(int64_t)o * m + x] : 0.f;
    }
#pragma unroll 5
    for (int t = tid; t < 16 * WX; t += 256) {
      const int c = t / WX, u = t % WX, x = x0 - h + u;
      sa[c * kAS + u] = (c0 + c < Cin && x >= 0 && x < m) ? ap[(int64_t)c * m + x] : 0.f;
    }
    __syncthreads();
    if (!mine) continue;
    const float* gr = sg + (16 * wave + l16) * kGS + lq;
    const float* ar = sa + l16 * kAS + lq;
    const int nx = min(kGX, m - x0), full = nx & ~3;
    for (int x = 0; x < full; x += 4) {
      const float gv = gr[x];
      sb += gv;
#pragma unroll
      for (int k = 0; k < K; ++k)
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(gv, ar[x + k], acc[k], 0, 0, 0);
      if ((x & 28) == 28) flush();
    }
    if (full < nx) {  // the last positions: an operand past m may pair a zero g with a real activation
      const bool in = full + lq < nx;
      const float gv = gr[full];
      sb += gv;
#pragma unroll
      for (int k = 0; k < K; ++k)
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(gv, in ? ar[full + k] : 0.f, acc[k], 0, 0, 0);
    }
    flush();
  }
  if (!mine) return;
  float* pp = part + (int64_t)blockIdx.x * ((int64_t)Cout * Cin * K + Cout);
  // D register v of lane l: output channel 4 (l / 16) + v of the wavefront's 16, input channel l % 16
  const int c = c0 + l16;
  if (c < Cin) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = o0 + 16 * wave + 4 * lq + v;
      if (o >= Cout) continue;
#pragma unroll
      for (int k = 0; k < K; ++k)
        pp[((int64_t)o * Cin + c) * K + k] = tot[k][v];
    }
  }
  if (blockIdx.y == 0) {
    sb += __shfl_xor(sb, 16, 64);
    sb += __shfl_xor(sb, 32, 64);
    const int o = o0 + 16 * wave + l16;
    if (lq == 0 && o < Cout) pp[(int64_t)Cout * Cin * K + o] = sb;
  }
}

// gW and gb from the nsplit partial sums, added in order in FP64, eight loads in flight.
__global__ void k_wgrad_reduce(const float* __restrict__ part, int64_t nW, int64_t total, int nsplit,
                               float* __restrict__ gW, float* __restrict__ gb) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= total) return;
  double s = 0.0;
  int i = 0;
  for (; i + 8 <= nsplit; i += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = part[(int64_t)(i + j) * total + t];
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; i < nsplit; ++i) s += part[(int64_t)i * total + t];
  if (t < nW) gW[t] = (float)s;
  else gb[t - nW] = (float)s;
}

// mean of B values in one block (fixed order)
__global__ void k_mean(const float* __restrict__ v, int64_t B, float* __restrict__ out) {
  __shared__ float s[256];
  float a = 0.f;
  for (int64_t i = threadIdx.x; i < B; i += 256) a += v[i];
  s[threadIdx.x] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    float tot = 0.f;
    for (int i = 0; i < 256; ++i) tot += s[i];
    *out = tot / (float)B;
  }
}

// Adam (Kingma & Ba, Algorithm 1); c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ mo,
                       float* __restrict__ ve, int64_t n, float lr, float beta1, float beta2, float eps, float c1,
                       float c2) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float gi = g[t];
  const float m1 = beta1 * mo[t] + (1.f - beta1) * gi;
  const float v1 = beta2 * ve[t] + (1.f - beta2) * gi * gi;
  mo[t] = m1;
  ve[t] = v1;
  p[t] -= lr * (m1 * c1) / (sqrtf(v1 * c2) + eps);
}

// The shift head (per system (b, q) of a batch of B members x Q shifts, c_q = 1 / (1 + s_q)):
// y_{b,q} = sum_d c_q^(d+1) Y[b, d] over the trunk output Y (B, D, m).
__device__ inline float head_value(const float* __restrict__ Y, int64_t b, int D, int m, int x, float c) {
  float y = 0.f, p = c;
  for (int d = 0; d < D; ++d) {
    y = fmaf(p, Y[(b * D + d) * (int64_t)m + x], y);
    p *= c;
  }
  return y;
}

// Relative L2 loss of each system against its target T (B, Q, m): per[b Q + q] = ||y - t|| / ||t||
// and scale[b Q + q] = 1 / (||y - t|| ||t|| B Q), the factor of its gradient.  One block per system.
__global__ __launch_bounds__(256) void k_head_rel_l2(const float* __restrict__ Y, int D, const float* __restrict__ cq,
                                                     int Q, const float* __restrict__ T, int m, int64_t B,
                                                     float* __restrict__ per, float* __restrict__ scale) {
  __shared__ float sd[4], st[4];
  const int64_t sys = blockIdx.x, b = sys / Q;
  const float c = cq[sys % Q];
  float dd = 0.f, tt = 0.f;
  for (int x = threadIdx.x; x < m; x += 256) {
    const float tv = T[sys * m + x];
    const float d = head_value(Y, b, D, m, x, c) - tv;
    dd = fmaf(d, d, dd);
    tt = fmaf(tv, tv, tt);
  }
  for (int off = 32; off > 0; off >>= 1) {
    dd += __shfl_xor(dd, off, 64);
    tt += __shfl_xor(tt, off, 64);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sd[wave] = dd;
    st[wave] = tt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const float dn = sqrtf(((sd[0] + sd[1]) + sd[2]) + sd[3]);
    const float tn = sqrtf(((st[0] + st[1]) + st[2]) + st[3]);
    scale[sys] = (dn > 0.f && tn > 0.f) ? 1.0f / (dn * tn * (float)(B * Q)) : 0.f;
    per[sys] = tn > 0.f ? dn / tn : 0.f;
  }
}

// Gradient of the mean loss w.r.t. the trunk output: gY[b, d, x] = sum_q c_q^(d+1) scale_{b,q}
// (y_{b,q}[x] - T_{b,q}[x]).  One thread per (b, x).
__global__ void k_head_grad(const float* __restrict__ Y, int D, const float* __restrict__ cq, int Q,
                            const float* __restrict__ T, const float* __restrict__ scale, int m, int64_t B,
                            float* __restrict__ gY) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= B * m) return;
  const int64_t b = t / m;
  const int x = (int)(t % m);
  float g[16];
  for (int d = 0; d < D; ++d) g[d] = 0.f;
  for (int q = 0; q < Q; ++q) {
    const float c = cq[q];
    const float r = scale[b * Q + q] * (head_value(Y, b, D, m, x, c) - T[(b * Q + q) * (int64_t)m + x]);
    float p = c;
    for (int d = 0; d < D; ++d) {
      g[d] = fmaf(p, r, g[d]);
      p *= c;
    }
  }
  for (int d = 0; d < D; ++d) gY[(b * D + d) * (int64_t)m + x] = g[d];
}

}  // namespace

static unsigned nb1(int64_t n) { return (unsigned)((n + 255) / 256); }

namespace {
template <int K>
hipError_t conv_go(const float* in, int Cin, const float* W, const float* bias, int Cout, int m, int64_t B,
                   float* pre, float* act, int gelu, hipStream_t st, bool flip, const float* dz) {
  constexpr size_t lds = sizeof(float) * ((size_t)kCIC * kWinS + 64 * conv_row(K));
  const dim3 grid((unsigned)((m + kCX - 1) / kCX), (unsigned)((Cout + 63) / 64), (unsigned)B);
  auto* fn = flip ? k_conv_mfma<K, true> : k_conv_mfma<K, false>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, grid, dim3(256), lds, st, in, Cin, W, bias, Cout, m, pre, act, gelu, dz);
  return hipGetLastError();
}
// Where the forward correlation runs on the matrix cores, whose tiles are 64 output channels wide and whose
// chunks 16 input channels deep, full or not.  The FMA kernel does only the channels that are there, and
// wins once the chip is full: 640 members x 1024 positions, 9 taps: 1 -> 64 channels 519 us on the matrix
// cores and 92 with FMAs, 64 -> 4: 1122 / 235, 16 -> 16: 575 / 140, 32 -> 32: 851 / 510; 64 -> 64: 1485 /
// 1990.  Below that, one or two rounds of blocks on the matrix cores are the shorter chain (8 members, 64
// -> 64: 21 / 61; 64 -> 4: 16 / 37; 16 members, 32 -> 32 still 21 / 33).  Fewer taps leave the matrix kernel
// its registers, several wavefronts a SIMD, and its line lies lower: forwards of 320 members with 40 hidden
// channels 1780 us with MFMA and 1120 with FMAs at 9 taps, of 64 members with 130, one tap, 166 and 430.
bool conv_on_mfma(int Cin, int Cout, int K, int m, int64_t B) {
  const int64_t tiles = (Cout + 63) / 64, blocks = B * ((m + kCX - 1) / kCX) * tiles;
  if (Cin < kCIC) return false;
  const int fill = K == 1 ? 17 : (K <= 5 ? 32 : (K == 7 ? 40 : 42));  // output channels a tile has to hold
  if (Cout >= fill * tiles) return true;
  return blocks <= (K == 1 ? 2048 : (K <= 7 || Cin >= 32 ? 512 : 256));
}
}  // namespace

hipError_t launch_conv_fwd(const float* in, int Cin, const float* W, const float* bias, int Cout, int K, int m,
                           int64_t B, float* pre, float* act, int gelu, hipStream_t st, bool flip, const float* dz) {
  if (B <= 0) return hipSuccess;
  if (!in || !W || !act || K < 1 || K > kMaxTaps || (K % 2) == 0) return hipErrorInvalidValue;
  if (!flip && !dz && !conv_on_mfma(Cin, Cout, K, m, B)) {
    const unsigned gx = (unsigned)((m + kVX - 1) / kVX);
    const int cpw = Cout >= 16 ? 4 : 1;
    const size_t lds = sizeof(float) * ((size_t)kCIC * (kVX + K - 1) + 4 * cpw * kCIC * K);
    const dim3 grid(gx, (unsigned)((Cout + 4 * cpw - 1) / (4 * cpw)), (unsigned)B);
    hipLaunchKernelGGL(cpw == 4 ? k_conv_fma<4> : k_conv_fma<1>, grid, dim3(256), lds, st, in, Cin, W, bias, Cout, K, m,
                       pre, act, gelu);
    return hipGetLastError();
  }
  switch (K) {
    case 1: return conv_go<1>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 3: return conv_go<3>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 5: return conv_go<5>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 7: return conv_go<7>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 9: return conv_go<9>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 11: return conv_go<11>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    case 13: return conv_go<13>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
    default: return conv_go<15>(in, Cin, W, bias, Cout, m, B, pre, act, gelu, st, flip, dz);
  }
}

int bf16_cp(int Cin) { return (Cin + 7) / 8 * 8; }
int bf16_kd(int Cin, int K) { return (K * bf16_cp(Cin) + 31) / 32 * 32; }
int bf16_opad(int Cout) { return (Cout + 15) / 16 * 16; }

hipError_t launch_pack_weights_bf16(const float* W, int Cout, int Cin, int K, __hip_bfloat16* out, hipStream_t st) {
  const int Cp = bf16_cp(Cin), KD = bf16_kd(Cin, K), Op = bf16_opad(Cout);
  const int64_t cnt = (int64_t)Op * KD;
  hipLaunchKernelGGL(k_pack_weights_bf16, dim3(nb1(cnt)), dim3(256), 0, st, W, Cout, Cin, K, Cp, KD, Op, out);
  return hipGetLastError();
}

hipError_t launch_conv_bf16(const void* in, bool in_f32, int Cin, const __hip_bfloat16* Wp, const float* bias, int Cout,
                            int K, int m, int64_t B, void* out, bool out_f32, int gelu, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  if (!in || !Wp || !out || K < 1 || K > 15 || (K % 2) == 0 || Cin > 64 || Cout > 64) return hipErrorInvalidValue;

  if (!in_f32 && bf16_cp(Cin) != Cin) return hipErrorInvalidValue;  // BF16 inputs carry Cp channels
  const int Cp = bf16_cp(Cin), KD = bf16_kd(Cin, K);
  const size_t smem = sizeof(__hip_bfloat16) * (size_t)(64 + K - 1) * (Cp + 8);
  const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((Cout + 63) / 64), (unsigned)B);
#define IE_CB(I, O)                                                                                             \
  hipLaunchKernelGGL((k_conv_bf16<I, O>), grid, dim3(256), smem, st, in, Cin, Cp, Wp, KD, bias, Cout, K, m, out, \
                     gelu)
  if (in_f32 && out_f32) IE_CB(true, true);
  else if (in_f32) IE_CB(true, false);
  else if (out_f32) IE_CB(false, true);
  else IE_CB(false, false);
#undef IE_CB
  return hipGetLastError();
}

// Enough blocks (1024) for the chip; at most 64 partials, which the reduction reads in ~ 5 us, and no
// more than there are chunks.
int wgrad_splits(int Cin, int Cout, int m, int64_t B) {
  const int64_t tiles = (int64_t)((Cin + 15) / 16) * ((Cout + 63) / 64);
  const int64_t chunks = B * ((m + kGX - 1) / kGX);
  return (int)std::max<int64_t>(1, std::min<int64_t>({chunks, 64, 1024 / tiles}));
}
int64_t wgrad_part_floats(int Cin, int Cout, int K, int m, int64_t B) {
  return (int64_t)wgrad_splits(Cin, Cout, m, B) * ((int64_t)Cout * Cin * K + Cout);
}

hipError_t launch_conv_wgrad(const float* a, int Cin, const float* g, int Cout, int K, int m, int64_t B, float* gW,
                             float* gb, float* part, hipStream_t st) {
  if (!part || K < 1 || K > kMaxTaps || (K % 2) == 0) return hipErrorInvalidValue;
  const int ns = wgrad_splits(Cin, Cout, m, B);
  const dim3 grid((unsigned)ns, (unsigned)((Cin + 15) / 16), (unsigned)((Cout + 63) / 64));
  constexpr size_t lds = sizeof(float) * (64 * kGS + 16 * kAS);
#define IE_WG(KK) \
  case KK: hipLaunchKernelGGL(k_wgrad_mfma<KK>, grid, dim3(256), lds, st, a, Cin, g, Cout, m, B, part); break
  switch (K) {
    IE_WG(1);
    IE_WG(3);
    IE_WG(5);
    IE_WG(7);
    IE_WG(9);
    IE_WG(11);
    IE_WG(13);
    IE_WG(15);
  }
#undef IE_WG
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t nW = (int64_t)Cout * Cin * K, total = nW + Cout;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(nb1(total)), dim3(256), 0, st, part, nW, total, ns, gW, gb);
  return hipGetLastError();
}

hipError_t launch_head_loss_grad(const float* Y, int D, const float* cq, int Q, const float* T, int m, int64_t B,
                                 float* per, float* scale, float* mean, float* gY, hipStream_t st) {
  if (D < 1 || D > 16 || Q < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_head_rel_l2, dim3((unsigned)(B * Q)), dim3(256), 0, st, Y, D, cq, Q, T, m, B, per, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mean, dim3(1), dim3(256), 0, st, per, B * Q, mean);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_head_grad, dim3(nb1(B * m)), dim3(256), 0, st, Y, D, cq, Q, T, scale, m, B, gY);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* mo, float* ve, int64_t n, float lr, int64_t t,
                       hipStream_t st) {
  const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
  const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)t)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)t)));
  hipLaunchKernelGGL(k_adam, dim3(nb1(n)), dim3(256), 0, st, p, g, mo, ve, n, lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace infoesrf
