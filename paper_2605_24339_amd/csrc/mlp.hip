// Per-vertex MLP for the learned warm start: 9 -> 128 -> 128 -> 128 -> 3,
// SiLU activations, inputs padded to 16 features and outputs to 16.
// Dense layers run on the matrix cores: v_mfma_f32_32x32x16_bf16 with bf16
// operands (converted from the float32 tensors while staging tiles in LDS)
// and float32 accumulation; bias and SiLU are fused into the GEMM epilogue.
// Weight gradients (a reduction over the batch) use split-K partials summed
// in a fixed order, so training is deterministic.
//
// Parameter layout (float32, contiguous):
//   W1 [16][128], b1 [128], W2 [128][128], b2 [128], W3 [128][128], b3 [128],
//   W4 [128][16], b4 [16]
// Saved activations for the backward pass ("act", float32, [B][768]):
//   Z1 | H1 | Z2 | H2 | Z3 | H3, 128 columns each, row-major per row block.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "../../include/gmcp_mlp.h"
#include "common.h"

// Scratch of gmcp_mlp_mse_noalloc (the per-block partial losses), in static
// device memory: every GPU the library runs on holds its own copy until the
// process ends.  Host code must not pass this name to a kernel (on the host
// it is only a stand-in for the symbol): it uses the device address that
// hipGetSymbolAddress returns for each device.
constexpr int64_t kMseScratch = int64_t(1) << 20;  // floats, 4 MiB per GPU
static __device__ __align__(256) float scratch[kMseScratch];

namespace {

using gmcp::kWave;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // four floats of a caller's array, at any float

constexpr int IN = 16, HID = 128, OUT = 16;
constexpr int64_t OFF_W1 = 0, OFF_B1 = OFF_W1 + IN * HID, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
                  OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID * HID, OFF_W4 = OFF_B3 + HID,
                  OFF_B4 = OFF_W4 + HID * OUT, N_PARAMS = OFF_B4 + OUT;
constexpr int ACT = 6 * HID;  // saved activations per row

// 1 + exp(-z), at most 2^126: beyond (z < -87) silu and its derivative are
// below 1e-35 either way, and the reciprocal stays a normal number
__device__ inline float one_exp(float z) {
  return 1.0f + __builtin_amdgcn_exp2f(fminf(z * -1.44269504f, 126.0f));
}
// z / d and 1 / d for such a d >= 1 from the hardware reciprocal and one
// correction step (errors within an ulp, as measured against the division:
// the IEEE sequence scales for exponents that d cannot have and took most of
// the activation's instructions)
__device__ inline float div_one(float z, float d) {
  const float r = __builtin_amdgcn_rcpf(d), q = z * r;
  return __builtin_fmaf(__builtin_fmaf(-d, q, z), r, q);
}
__device__ inline float silu(float z) { return div_one(z, one_exp(z)); }
__device__ inline float silu_grad(float z) {
  const float s = div_one(1.0f, one_exp(z));
  return s * (1.0f + z * (1.0f - s));
}

// C = op(A) op(B), op(A) is M x K, op(B) is K x N (gmcp_gemm_bf16).
// A(m,k) = transA ? A[k*lda + m] : A[m*lda + k]; B(k,n) likewise.
// Block tile 64 x 64 (four waves of 32 x 32), K step 32 (two MFMAs).
__global__ __launch_bounds__(256) void k_gemm(const float *__restrict__ A, int lda, int transA,
                                               const float *__restrict__ B, int ldb, int transB, int M, int N, int K,
                                               float *__restrict__ C, int ldc) {
  __shared__ __bf16 As[64][32 + 8];
  __shared__ __bf16 Bs[32][64 + 8];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  f32x16 acc = {};
  for (int k0 = 0; k0 < K; k0 += 32) {
    for (int e = tid; e < 64 * 32; e += 256) {
      int r = e >> 5, kk = e & 31, m = m0 + r, k = k0 + kk;
      float v = (m < M && k < K) ? (transA ? A[(int64_t)k * lda + m] : A[(int64_t)m * lda + k]) : 0.0f;
      As[r][kk] = (__bf16)v;
    }
    for (int e = tid; e < 32 * 64; e += 256) {
      int kk = e >> 6, cc = e & 63, k = k0 + kk, n = n0 + cc;
      float v = (k < K && n < N) ? (transB ? B[(int64_t)n * ldb + k] : B[(int64_t)k * ldb + n]) : 0.0f;
      Bs[kk][cc] = (__bf16)v;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 a, b;
      const int kq = h * 16 + 8 * (lane >> 5);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a[j] = As[wm * 32 + (lane & 31)][kq + j];
        b[j] = Bs[kq + j][wn * 32 + (lane & 31)];
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
  }
  const int n = n0 + wn * 32 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
    if (m >= M || n >= N) continue;
    C[(int64_t)m * ldc + n] = acc[r];
  }
}

// out[i] = sum_s part[s][i], 64 outputs per block of 1024 threads: thread
// group g (of 16) adds the partials s = g, g + 16, ... in that order, then
// the 16 group sums are added in group order (a fixed order, so runs agree
// bitwise; sixteen short chains of loads instead of one long one)
constexpr int kRedGroups = 16;
__global__ __launch_bounds__(kWave *kRedGroups) void k_reduce_split(const float *__restrict__ part, int S, int64_t n,
                                                                     float *__restrict__ out) {
  __shared__ float red[kRedGroups][kWave];
  const int e = threadIdx.x & (kWave - 1), g = threadIdx.x / kWave;
  const int64_t i = (int64_t)blockIdx.x * kWave + e;
  float s = 0.0f;
  if (i < n)
    for (int z = g; z < S; z += kRedGroups) s += part[(int64_t)z * n + i];
  red[g][e] = s;
  __syncthreads();
  if (g == 0 && i < n) {
    float t = 0.0f;
    for (int k = 0; k < kRedGroups; ++k) t += red[k][e];
    out[i] = t;
  }
}

// dY = 2 (Y - T) / (B n_out) on the first n_out columns, 0 on the padding;
// loss partials per block
__global__ void k_mse(const float *__restrict__ Y, const float *__restrict__ T, int64_t B, int n_out,
                      float *__restrict__ dY, float *__restrict__ part) {
  __shared__ float s[256];
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float l = 0.0f;
  if (i < B * OUT) {
    int c = (int)(i % OUT);
    float d = c < n_out ? Y[i] - T[i] : 0.0f;
    dY[i] = c < n_out ? 2.0f * d / (float)(B * n_out) : 0.0f;
    l = d * d / (float)(B * n_out);
  }
  s[threadIdx.x] = l;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

__global__ void k_sum(const float *__restrict__ part, int64_t n, float *out) {
  __shared__ float s[256];
  float v = 0.0f;
  for (int64_t j = threadIdx.x; j < n; j += 256) v += part[j];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = s[0];
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = g[i];
  float mi = b1 * m[i] + (1.0f - b1) * gi;
  float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------- fused forward
// The whole network for 32 rows per wave, activations in registers.  Each
// layer is computed transposed, out^T (features x rows) = W^T (features x
// k) . in^T (k x rows), on v_mfma_f32_32x32x16_bf16, so the accumulator of
// a 32-feature output tile holds, in lane l, row (l & 31) and features
// (r >> 2) * 8 + 4 (l >> 5) + (r & 3) of its register r.  Those registers
// are exactly the B operand of the next layer's k-steps if the k slots are
// taken in that order: slot j of lane half h in k-step s stands for input
// feature 16 s + (j >> 2) * 8 + 4 h + (j & 3).  The weights are staged once
// per block into LDS as bf16 A fragments in the same slot order (64 lanes x
// 8 values, one 16-byte read per lane and MFMA), so the activations never
// leave the registers between layers.
constexpr int kFrag = kWave * 8;                     // bf16 per A fragment
constexpr int kFragL1 = 4, kFragL2 = 32, kFragL3 = 32, kFragL4 = 8;  // 32-feature tiles x k-steps
constexpr int kFragAll = kFragL1 + kFragL2 + kFragL3 + kFragL4;      // 76 fragments, 76 KB
// waves per block: one block of 16 fills a compute unit for inference (the
// weights are staged once per unit); saving the activations needs more
// registers and is bound by its 3 KB of stores per row
constexpr int fwd_waves(bool save) { return save ? 8 : 16; }
constexpr size_t kFwdLds = (size_t)kFragAll * kFrag * sizeof(__bf16) + (3 * HID + OUT) * sizeof(float);

// The activations bound it: 384 SiLU per row, each two transcendental
// instructions (16 cycles a wave) and about eight plain ones; the matrix
// products of a tile take a quarter of that and overlap other waves'
// activations.  The tiles of a layer are unrolled, so the next layer's
// operands are named registers.  262144 rows: 46 us, 420 TFLOP/s (103 us with
// the IEEE division, rolled tiles whose operands were placed by selects, and
// two blocks per unit staging the weights).  65536 rows with the activations
// saved: 60 us, 3.4 TB/s of stores (88 us).
template <bool SAVE>
__global__ __launch_bounds__(kWave *fwd_waves(SAVE)) __attribute__((amdgpu_waves_per_eu(SAVE ? 2 : 4))) void k_mlp_fwd(
    const float *__restrict__ P, const float *__restrict__ x, int64_t B, float *__restrict__ y,
    float *__restrict__ act) {
  extern __shared__ __align__(16) unsigned char smem[];
  bf16x8 *frag = reinterpret_cast<bf16x8 *>(smem);  // [kFragAll][64 lanes]
  float *sb = reinterpret_cast<float *>(smem + (size_t)kFragAll * kFrag * sizeof(__bf16));  // b1 | b2 | b3 | b4
  constexpr int kThreadsF = kWave * fwd_waves(SAVE);
  for (int i = threadIdx.x; i < 3 * HID + OUT; i += kThreadsF)
    sb[i] = P[i < HID ? OFF_B1 + i : (i < 2 * HID ? OFF_B2 + i - HID : (i < 3 * HID ? OFF_B3 + i - 2 * HID
                                                                                 : OFF_B4 + i - 3 * HID))];
  // stage: fragment f of layer L = (tile t, k-step s), lane l, slot j holds
  // W_L[k = 16 s + (j >> 2) * 8 + 4 (l >> 5) + (j & 3)][n = 32 t + (l & 31)]
  // (0 beyond N): eight loads per lane, each of two runs of 32 columns, and
  // one 16-byte write.  kBatch fragments are in flight per wave (one pass of
  // this latency chain is what a small batch takes).
  constexpr int kLanes = kFragAll * kWave, kBatch = 5;
  for (int e0 = threadIdx.x; e0 < kLanes; e0 += kBatch * kThreadsF) {
    float v[kBatch][8];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int f = (e0 + u * kThreadsF) / kWave, l = threadIdx.x % kWave;
      int ff, S, N;
      int64_t off;
      if (f < kFragL1) { ff = f; S = 1; N = HID; off = OFF_W1; }
      else if (f < kFragL1 + kFragL2) { ff = f - kFragL1; S = 8; N = HID; off = OFF_W2; }
      else if (f < kFragL1 + kFragL2 + kFragL3) { ff = f - kFragL1 - kFragL2; S = 8; N = HID; off = OFF_W3; }
      else { ff = f - kFragL1 - kFragL2 - kFragL3; S = 8; N = OUT; off = OFF_W4; }
      const int n = 32 * (ff / S) + (l & 31), k0 = 16 * (ff % S) + 4 * (l >> 5);
      const bool on = f < kFragAll && n < N;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[u][j] = on ? P[off + (int64_t)(k0 + (j >> 2) * 8 + (j & 3)) * N + n] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int e = e0 + u * kThreadsF;
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (__bf16)v[u][j];
      if (e < kLanes) frag[e] = o;
    }
  }
  __syncthreads();
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int h = lane >> 5;
  const int64_t tiles = (B + 31) / 32;
  // neighbouring tiles go to different blocks: a batch of few tiles spreads
  // over the compute units
  for (int64_t tile = (int64_t)w * gridDim.x + blockIdx.x; tile < tiles;
       tile += (int64_t)gridDim.x * fwd_waves(SAVE)) {
    // the weights are read from LDS for every tile: kept in registers across
    // tiles (they do not change) they would spill
    asm volatile("" ::: "memory");
    const int64_t row = tile * 32 + (lane & 31);
    const bool live = row < B;
    // layer 1 input: x features {4h..4h+3, 8+4h..8+4h+3} of the lane's row
    bf16x8 bin;
    {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
      if (live) {
        a = *reinterpret_cast<const float4 *>(x + row * IN + 4 * h);
        c = *reinterpret_cast<const float4 *>(x + row * IN + 8 + 4 * h);
      }
      bin[0] = (__bf16)a.x; bin[1] = (__bf16)a.y; bin[2] = (__bf16)a.z; bin[3] = (__bf16)a.w;
      bin[4] = (__bf16)c.x; bin[5] = (__bf16)c.y; bin[6] = (__bf16)c.z; bin[7] = (__bf16)c.w;
    }
    // bias + SiLU on the accumulator of output tile t, optional save of Z and
    // H; the 16 values are the bf16 operands of k-steps 2t (lo) and 2t + 1
    // (hi) of the next layer
    auto epilogue = [&](const f32x16 &acc, int t, const float *bias, int save_off, bf16x8 &lo, bf16x8 &hi) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // four groups of four consecutive features
        const int f0 = 32 * t + q * 8 + 4 * h;
        const float4 bv = *reinterpret_cast<const float4 *>(bias + f0);
        const float z[4] = {acc[4 * q] + bv.x, acc[4 * q + 1] + bv.y, acc[4 * q + 2] + bv.z, acc[4 * q + 3] + bv.w};
        float hv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          hv[i] = silu(z[i]);
          if (q < 2) lo[4 * q + i] = (__bf16)hv[i];
          else hi[4 * (q - 2) + i] = (__bf16)hv[i];
        }
        if (SAVE && live) {
          *reinterpret_cast<float4 *>(act + row * ACT + save_off + f0) = make_float4(z[0], z[1], z[2], z[3]);
          *reinterpret_cast<float4 *>(act + row * ACT + save_off + HID + f0) =
              make_float4(hv[0], hv[1], hv[2], hv[3]);
        }
      }
    };
    bf16x8 h1[8], h2[8];
    // layer 1: K = 16, one k-step
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x16 zero = {};
      const f32x16 a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[t * kWave + lane], bin, zero, 0, 0, 0);
      epilogue(a, t, sb, 0, h1[2 * t], h1[2 * t + 1]);
    }
    // layers 2 and 3: K = 128, eight k-steps per output tile
    auto layer = [&](int fbase, const bf16x8 *in, bf16x8 *out, const float *bias, int save_off) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        f32x16 a = {};
#pragma unroll
        for (int sk = 0; sk < 8; ++sk)
          a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[(fbase + t * 8 + sk) * kWave + lane], in[sk], a, 0, 0, 0);
        epilogue(a, t, bias, save_off, out[2 * t], out[2 * t + 1]);
      }
    };
    layer(kFragL1, h1, h2, sb + HID, 2 * HID);
    layer(kFragL1 + kFragL2, h2, h1, sb + 2 * HID, 4 * HID);
    // layer 4: one 32-feature tile, the first 16 are the outputs
    {
      const int fbase = kFragL1 + kFragL2 + kFragL3;
      f32x16 a = {};
#pragma unroll
      for (int sk = 0; sk < 8; ++sk)
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[(fbase + sk) * kWave + lane], h1[sk], a, 0, 0, 0);
      if (live) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int f0 = q * 8 + 4 * h;
          const float *b4 = sb + 3 * HID;
          *reinterpret_cast<float4 *>(y + row * OUT + f0) =
              make_float4(a[4 * q] + b4[f0], a[4 * q + 1] + b4[f0 + 1], a[4 * q + 2] + b4[f0 + 2],
                          a[4 * q + 3] + b4[f0 + 3]);
        }
      }
    }
  }
}

// --------------------------------------------------------------- fused backward
// Gradients of all parameters in one pass over the batch, 256 rows per block
// at a time.  Each of the 16 waves takes 16 rows through the chain
//   dZ3 = (dY W4^T) silu'(Z3),  dZ2 = (dZ3 W3^T) silu'(Z2),  dZ1 likewise,
// transposed as in the forward pass (features x rows, here on
// v_mfma_f32_16x16x32_bf16: lane l holds row l & 15 and features 4 (l >> 4) ..
// + 3 of a 16-feature tile), so that a layer's dZ is the next product's
// operand in registers when the k slots follow that order (W staged once per
// block as bf16 A fragments).  A layer's dZ also goes to LDS in bf16,
// feature-major (two rows per word, neighbouring lanes exchange), where the
// block's waves read it as the operand of dW = H^T dZ: each wave owns one
// 32 x 32 tile of the gradient and reads H's columns from memory with
// coalesced loads.  The gradients stay in accumulators over all of the
// block's rows; one partial per block is written and k_reduce_split adds
// them in block order.  Bias gradients are sums of the float dZ over the
// lanes (rows of 16 with DPP), then over the waves in order.
//
// Bound by latency: 201 MB of activations (41 us at the copy rate) and about
// 25 us of SiLU derivatives and products pass through phases that the block
// takes together.  65536 rows: 75 us and 13 us for the partials' sum;
// one GEMM per product with 64 x 64 tiles staged through scalar LDS writes,
// float dZ in memory between them, split partials for each weight and
// column-sum launches took 560 us.  Eight waves of 32 rows (250 registers)
// took 220 us and loads behind per-lane conditions 240 us; the activations
// are loaded four tiles at a time because eight spill.
constexpr int kBwdWaves = 16;
constexpr int kBwdRows = 16 * kBwdWaves;
constexpr int kBwdBlocks = 256;                       // partials at most: a block per compute unit
constexpr int kBwdL4 = 8, kBwdL = 32;                 // fragments: W4 8 tiles x 1 k-step, W3 and W2 8 x 4
constexpr int kBwdFrags = kBwdL4 + 2 * kBwdL;
constexpr int kTPitch = kBwdRows + 8;                 // bf16 per feature (a pitch of 4 words modulo the banks)
constexpr size_t kBwdW = (size_t)kBwdFrags * kFrag * sizeof(__bf16), kBwdT = (size_t)HID * kTPitch * sizeof(__bf16);
constexpr size_t kBwdLds = kBwdW + kBwdT + sizeof(float) * kBwdWaves * (HID + OUT);

// v plus the lane CTRL names (within rows of 16)
template <int CTRL>
__device__ inline float add_lane(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf,
                                                                   false));
}
// sum over the lane's row of 16, in every lane
__device__ inline float row16_sum(float v) {
  v = add_lane<0xB1>(v);   // 1 lane apart
  v = add_lane<0x4E>(v);   // 2
  v = add_lane<0x141>(v);  // mirror of 8
  return add_lane<0x140>(v);  // mirror of 16
}

__global__ __launch_bounds__(kWave *kBwdWaves) void k_mlp_bwd(const float *__restrict__ P,
                                                              const float *__restrict__ x,
                                                              const float *__restrict__ act,
                                                              const float *__restrict__ dy, int64_t B,
                                                              float *__restrict__ part) {
  extern __shared__ __align__(16) unsigned char smem[];
  bf16x8 *frag = reinterpret_cast<bf16x8 *>(smem);                 // [kBwdFrags][64]
  __bf16 *T = reinterpret_cast<__bf16 *>(smem + kBwdW);            // [128 features][kTPitch rows]
  float *red = reinterpret_cast<float *>(smem + kBwdW + kBwdT);    // [waves][128], bias sums of a layer
  float *red4 = red + kBwdWaves * HID;                             // [waves][16], of the output layer
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int g16 = lane >> 4, r16 = lane & 15, h = lane >> 5, r32 = lane & 31;
  // stage: fragment (layer, tile t, k-step s), lane l, slot j holds
  // W[16 t + (l & 15)][32 s + 16 (j >> 2) + 4 (l >> 4) + (j & 3)]
  for (int e = threadIdx.x; e < kBwdFrags * kWave; e += kWave * kBwdWaves) {
    const int f = e / kWave;
    const int S = f < kBwdL4 ? 1 : 4, N = f < kBwdL4 ? OUT : HID, ff = f < kBwdL4 ? f : (f - kBwdL4) % kBwdL;
    const float *src = P + (f < kBwdL4 ? OFF_W4 : (f < kBwdL4 + kBwdL ? OFF_W3 : OFF_W2)) +
                       (16 * (ff / S) + r16) * N + 32 * (ff % S) + 4 * g16;
    f32x4 a = *reinterpret_cast<const f32x4u *>(src), c = {};
    if (N == HID) c = *reinterpret_cast<const f32x4u *>(src + 16);
    bf16x8 v;
    v[0] = (__bf16)a.x; v[1] = (__bf16)a.y; v[2] = (__bf16)a.z; v[3] = (__bf16)a.w;
    v[4] = (__bf16)c.x; v[5] = (__bf16)c.y; v[6] = (__bf16)c.z; v[7] = (__bf16)c.w;
    frag[e] = v;
  }
  const int ft = w >> 2, nt = w & 3;        // the wave's tile of dW3 and dW2: inputs 32 ft.., outputs 32 nt..
  f32x16 g3 = {}, g2 = {};
  const int xt = w & 7, xk = w >> 3;        // and of dW4 and dW1: 16 inputs / outputs 16 xt.., half xk of the rows
  f32x4 g4 = {}, g1 = {};
  float b1 = 0.0f, b2 = 0.0f, b3 = 0.0f, b4 = 0.0f;  // bias gradients of feature threadIdx.x
  __syncthreads();
  for (int64_t row0 = (int64_t)blockIdx.x * kBwdRows; row0 < B; row0 += (int64_t)gridDim.x * kBwdRows) {
    // Rows beyond the batch read the last row: their dY is set to 0, so their
    // dZ and their share of every sum are 0.  (Loads behind a per-lane
    // condition were waited for one by one.)
    const int64_t row = row0 + 16 * w + r16, rowc = row < B ? row : B - 1;
    const int last = (int)(B - 1 - row0 < kBwdRows - 1 ? B - 1 - row0 : kBwdRows - 1);
    // rows r .. r + 7 of a column of X [B][ld] as an MFMA operand
    auto rows8 = [&](const float *X, int ld, int r) {
      const float *p = X + row0 * ld;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[min(r + j, last) * ld];
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (__bf16)v[j];
      return o;
    };
    auto dy_op = [&](int r) {  // rows8 of dY, 0 beyond the batch
      bf16x8 o = rows8(dy + r16, OUT, r);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (r + j > last) o[j] = (__bf16)0.0f;
      return o;
    };
    f32x4 z[4];
    auto load_z = [&](int z_off) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        z[t] = *reinterpret_cast<const f32x4u *>(act + rowc * ACT + z_off + 16 * t + 4 * g16);
    };
    // dZ^T of a layer: the products of S k-steps times silu'(Z), to `out`
    // (operands of the next layer), T and red
    auto chain = [&](int fbase, int S, const bf16x8 *in, bf16x8 *out, int z_off) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (t == 0) load_z(z_off);
        if (t == 4) load_z(z_off + 64);
        f32x4 a = {};
#pragma unroll
        for (int sk = 0; sk < S; ++sk)
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag[(fbase + t * S + sk) * kWave + lane], in[sk], a, 0, 0, 0);
        float sum[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = a[i] * silu_grad(z[t & 3][i]);
          out[t >> 1][4 * (t & 1) + i] = (__bf16)v;
          sum[i] = row16_sum(v);
        }
        if (r16 == 0)
          *reinterpret_cast<float4 *>(red + w * HID + 16 * t + 4 * g16) = make_float4(sum[0], sum[1], sum[2], sum[3]);
        // features f, f + 1 of rows r, r + 1: the even lane writes f, the odd one f + 1
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const uint32_t mine = __builtin_bit_cast(uint4, out[t >> 1])[2 * (t & 1) + k];
          const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xf, 0xf, false);
          const uint32_t two = (lane & 1) ? (other >> 16) | (mine & 0xffff0000u) : (mine & 0xffffu) | (other << 16);
          *reinterpret_cast<uint32_t *>(T + (16 * t + 4 * g16 + 2 * k + (lane & 1)) * kTPitch + 16 * w + (r16 & ~1)) = two;
        }
      }
    };
    auto wgrad = [&](int h_off, f32x16 &g) {
      const float *X = act + h_off + 32 * ft + r32;
      const __bf16 *D = T + (32 * nt + r32) * kTPitch + 8 * h;
#pragma unroll 4
      for (int ks = 0; ks < kBwdRows / 16; ++ks)
        g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows8(X, ACT, 16 * ks + 8 * h),
                                                    *reinterpret_cast<const bf16x8 *>(D + 16 * ks), g, 0, 0, 0);
    };
    auto bias = [&](float &b) {  // waves in order
      if (threadIdx.x < HID)
        for (int k = 0; k < kBwdWaves; ++k) b += red[k * HID + threadIdx.x];
    };
    // output layer: dY as the first operand (the k-step's second half is zero), db4
    bf16x8 d0[4], d1[4];
    {
      f32x4 v = *reinterpret_cast<const f32x4u *>(dy + rowc * OUT + 4 * g16);
      if (row >= B) v = f32x4{};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        d0[0][j] = (__bf16)v[j];
        d0[0][4 + j] = (__bf16)0.0f;
        const float sum = row16_sum(v[j]);
        if (r16 == 0) red4[w * OUT + 4 * g16 + j] = sum;
      }
    }
    chain(0, 1, d0, d1, 4 * HID);
    __syncthreads();
    if (threadIdx.x < OUT)
      for (int k = 0; k < kBwdWaves; ++k) b4 += red4[k * OUT + threadIdx.x];
    bias(b3);
    // dW4 = H3^T dY: 16 x 16 tiles, half of the rows per wave
#pragma unroll 2
    for (int ks = 0; ks < kBwdRows / 64; ++ks) {
      const int r = (kBwdRows / 2) * xk + 32 * ks + 8 * g16;
      g4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rows8(act + 5 * HID + 16 * xt + r16, ACT, r),
                                                   dy_op(r), g4, 0, 0, 0);
    }
    wgrad(3 * HID, g3);
    __syncthreads();
    chain(kBwdL4, 4, d1, d0, 2 * HID);
    __syncthreads();
    bias(b2);
    wgrad(HID, g2);
    __syncthreads();
    chain(kBwdL4 + kBwdL, 4, d0, d1, 0);
    __syncthreads();
    bias(b1);
    // dW1 = x^T dZ1
#pragma unroll 2
    for (int ks = 0; ks < kBwdRows / 64; ++ks) {
      const int r = (kBwdRows / 2) * xk + 32 * ks + 8 * g16;
      g1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          rows8(x + r16, IN, r), *reinterpret_cast<const bf16x8 *>(T + (16 * xt + r16) * kTPitch + r), g1, 0, 0, 0);
    }
    __syncthreads();
  }
  // the block's partial gradient; register r of a 32 x 32 tile is row
  // (r >> 2) * 8 + 4 h + (r & 3), of a 16 x 16 tile row 4 (l >> 4) + r
  float *out = part + (int64_t)blockIdx.x * N_PARAMS;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int at = (32 * ft + (r >> 2) * 8 + 4 * h + (r & 3)) * HID + 32 * nt + r32;
    out[OFF_W3 + at] = g3[r];
    out[OFF_W2 + at] = g2[r];
  }
  // dW4 and dW1: the second half of the rows through LDS, added to the first
  float *half = reinterpret_cast<float *>(T);
  static_assert(kBwdT >= sizeof(float) * 8 * kWave * 8, "the second halves fit");
  if (xk == 1)
    for (int r = 0; r < 4; ++r) {
      half[(r * 8 + xt) * kWave + lane] = g4[r];
      half[((4 + r) * 8 + xt) * kWave + lane] = g1[r];
    }
  __syncthreads();
  if (xk == 0)
    for (int r = 0; r < 4; ++r) {
      const int m = 4 * g16 + r;
      out[OFF_W4 + (16 * xt + m) * OUT + r16] = g4[r] + half[(r * 8 + xt) * kWave + lane];
      out[OFF_W1 + m * HID + 16 * xt + r16] = g1[r] + half[((4 + r) * 8 + xt) * kWave + lane];
    }
  if (threadIdx.x < HID) {
    out[OFF_B1 + threadIdx.x] = b1;
    out[OFF_B2 + threadIdx.x] = b2;
    out[OFF_B3 + threadIdx.x] = b3;
  }
  if (threadIdx.x < OUT) out[OFF_B4 + threadIdx.x] = b4;
}

inline unsigned nb(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_address(hipStream_t s, float **out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return GMCP_E_HIP;
  if (s) {
    hipDevice_t sd = 0;
    if (hipStreamGetDevice(s, &sd) != hipSuccess) return GMCP_E_HIP;
    if ((int)sd != dev) return GMCP_E_ARG;  // the stream must belong to the current device
  }
  if (dev < 0 || dev >= kMaxDevices) return GMCP_E_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GMCP_E_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = (float *)g_scratch_ptr[dev];
  return GMCP_OK;
}

// blocks of the backward pass, one partial gradient each
unsigned bwd_blocks(int64_t B) { return (unsigned)std::min<int64_t>(kBwdBlocks, (B + kBwdRows - 1) / kBwdRows); }

}  // namespace

extern "C" {

int64_t gmcp_mlp_param_count(void) { return N_PARAMS; }

size_t gmcp_mlp_work_bytes(int64_t B) { return B > 0 ? sizeof(float) * (size_t)bwd_blocks(B) * N_PARAMS : 0; }

int gmcp_mlp_forward(const float *params, const float *x, int64_t B, float *y, float *act, void *stream) {
  if (!params || !x || !y || B <= 0 || B > (int64_t(1) << 30)) return GMCP_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  // one fused launch: every wave runs the whole network on 32 rows at a
  // time; a block per compute unit at most, which stages the weights once
  static int n_cu[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GMCP_E_HIP;
  if (n_cu[dev] == 0 && (hipDeviceGetAttribute(&n_cu[dev], hipDeviceAttributeMultiprocessorCount, dev) !=
                             hipSuccess || n_cu[dev] < 1))
    n_cu[dev] = 256;
  const int64_t tiles = (B + 31) / 32;
  const unsigned grid = (unsigned)std::min<int64_t>(tiles, n_cu[dev]);
  const size_t lds = kFwdLds;
  if (act)
    hipLaunchKernelGGL(k_mlp_fwd<true>, dim3(grid), dim3(kWave * fwd_waves(true)), lds, s, params, x, B, y, act);
  else
    hipLaunchKernelGGL(k_mlp_fwd<false>, dim3(grid), dim3(kWave * fwd_waves(false)), lds, s, params, x, B, y, act);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_mlp_backward(const float *params, const float *x, const float *act, const float *dy, int64_t B, float *grad,
                      void *work, size_t work_bytes, void *stream) {
  if (!params || !x || !act || !dy || !grad || !work || B <= 0 || B > (int64_t(1) << 30)) return GMCP_E_ARG;
  if (work_bytes < gmcp_mlp_work_bytes(B)) return GMCP_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  const unsigned blocks = bwd_blocks(B);
  float *part = (float *)work;
  hipLaunchKernelGGL(k_mlp_bwd, dim3(blocks), dim3(kWave * kBwdWaves), kBwdLds, s, params, x, act, dy, B, part);
  hipLaunchKernelGGL(k_reduce_split, dim3(nb(N_PARAMS, kWave)), dim3(kWave * kRedGroups), 0, s, part, (int)blocks,
                     N_PARAMS, grad);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_mlp_mse(const float *y, const float *t, int64_t B, int n_out, float *loss, float *dy, void *work,
                 size_t work_bytes, void *stream) {
  if (!y || !t || !loss || !dy || !work || B <= 0 || n_out < 1 || n_out > OUT) return GMCP_E_ARG;
  int64_t blocks = (B * OUT + 255) / 256;
  if (work_bytes < sizeof(float) * (size_t)blocks) return GMCP_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_mse, dim3((unsigned)blocks), dim3(256), 0, s, y, t, B, n_out, dy, (float *)work);
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, (const float *)work, blocks, loss);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int64_t gmcp_mlp_mse_noalloc_max_rows(void) { return kMseScratch * 256 / OUT; }

int gmcp_mlp_mse_noalloc(const float *y, const float *t, int64_t B, int n_out, float *loss, float *dy,
                         void *stream) {
  if (!y || !t || !loss || !dy || B <= 0 || n_out < 1 || n_out > OUT) return GMCP_E_ARG;
  if (B > gmcp_mlp_mse_noalloc_max_rows()) return GMCP_E_ARG;
  const int64_t blocks = (B * OUT + 255) / 256;  // <= kMseScratch partials
  hipStream_t s = (hipStream_t)stream;
  float *part = nullptr;
  const int rc = scratch_address(s, &part);
  if (rc != GMCP_OK) return rc;
  // k_mse writes every partial it reads back, so nothing needs clearing
  hipLaunchKernelGGL(k_mse, dim3((unsigned)blocks), dim3(256), 0, s, y, t, B, n_out, dy, part);
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, (const float *)part, blocks, loss);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_mlp_adam(float *params, const float *grad, float *m, float *v, int64_t n, float lr, float beta1, float beta2,
                  float eps, int step, void *stream) {
  if (!params || !grad || !m || !v || n <= 0 || step < 1) return GMCP_E_ARG;
  float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(nb(n)), dim3(256), 0, (hipStream_t)stream, params, grad, m, v, n, lr, beta1, beta2,
                     eps, c1, c2);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_gemm_bf16(const float *A, int lda, int transA, const float *B, int ldb, int transB, int M, int N, int K,
                   float *C, int ldc, void *stream) {
  if (!A || !B || !C || M <= 0 || N <= 0 || K <= 0) return GMCP_E_ARG;
  hipLaunchKernelGGL(k_gemm, dim3((unsigned)((N + 63) / 64), (unsigned)((M + 63) / 64)), dim3(256), 0,
                     (hipStream_t)stream, A, lda, transA, B, ldb, transB, M, N, K, C, ldc);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

}  // extern "C"
