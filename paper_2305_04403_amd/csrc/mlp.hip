// Fourier-feature MLP for the learned control variate, on the gfx950 matrix
// cores: forward, backward (mean-squared error), deterministic gradient
// reduction and Adam.  Architecture fixed at compile time: 16 frequencies
// (32 features), 4 hidden layers of 128 with SiLU, scalar output.
//
// Matrix products use v_mfma_f32_16x16x32_bf16: bfloat16 operands, binary32
// accumulation.  Rounding to bfloat16 happens at: the features, each hidden
// activation, each weight matrix (a bfloat16 copy refreshed by Adam) and each
// pre-activation gradient that enters a product; biases, accumulators, the
// output layer and all element-wise math stay in binary32.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/wob.h"

namespace {

constexpr int KF = 16;        // Fourier frequencies
constexpr int F0 = 2 * KF;    // features
constexpr int HD = 128;       // hidden width
constexpr int NL = 4;         // hidden layers
constexpr int TR = 64;        // rows per workgroup
constexpr int NT = 512;       // threads per workgroup of the forward pass (8 wavefronts)
constexpr int GT = 1024;      // threads per workgroup of the backward pass (16 wavefronts)
constexpr int kFwdGrid = 512;  // forward-pass workgroups (256 CUs x the 2 resident on each)

// parameter offsets (floats): W_l [out][in] then b_l, layers 0..NL (NL = output)
constexpr int in_of(int l) { return l == 0 ? F0 : HD; }
constexpr int out_of(int l) { return l == NL ? 1 : HD; }
constexpr int offW(int l) { return l == 0 ? 0 : offW(l - 1) + out_of(l - 1) * in_of(l - 1) + out_of(l - 1); }
constexpr int offB(int l) { return offW(l) + out_of(l) * in_of(l); }
constexpr int NP = offB(NL) + 1;
static_assert(NP == 53889, "parameter count");
constexpr int NPP = (NP + 3) / 4 * 4;  // floats per partial gradient (16-byte aligned)

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

struct Net {
  int dim;
  float* p;       // binary32 master parameters
  float* m;       // Adam first moment
  float* v;       // Adam second moment
  __bf16* wq;     // bfloat16 copy, [out][in] per layer (bias slots unused)
  __bf16* wt;     // bfloat16 transposed copy, [in][out] per layer
  float* fourier; // KF x dim
};

// SiLU with the hardware reciprocal (1 ulp; the result is rounded to bfloat16
// or multiplies a bfloat16-rounded gradient, so an IEEE division buys nothing)
__device__ __forceinline__ float sigmoid_(float s) { return __builtin_amdgcn_rcpf(1.f + __expf(-s)); }
// The activation that is rounded to bfloat16: s / (1 + e^-s) correctly
// rounded to binary32 wherever that decides the bfloat16 rounding.  The fast
// binary32 evaluation (hardware exp2 of s log2 e, hardware reciprocal) is
// within (|s| + 3) ulp of the exact value (the product s log2 e carries |s| u
// of absolute error into the exponent); its bfloat16 rounding can differ from
// that of the exact value only when it lies that close to a bfloat16 rounding
// boundary (low half-word 0x8000), and there the value is recomputed in
// binary64 and rounded once to binary32.  The rounded activation then departs
// from exact arithmetic only through the accumulation of s.
__device__ __forceinline__ float silu_rounded(float s) {
  const float h = s * sigmoid_(s);
  const int lo = (int)(__float_as_uint(h) & 0xffffu);
  const float win = 8.f + 2.f * fabsf(s);  // ulps, twice the error bound
  if (fabsf((float)(lo - 0x8000)) <= win) {
    const double d = (double)s;
    return (float)(d / (1.0 + exp(-d)));
  }
  return h;
}
__device__ __forceinline__ float silu_grad(float s) {
  const float sg = sigmoid_(s);
  return sg * (1.f + s * (1.f - sg));
}

// MFMA 16x16x32 operand fragments.  Lane l holds rows/cols (l % 16) and the
// eight k values 8 (l / 16) .. +7; the accumulator holds rows 4 (l / 16) + v.
__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The forward pass alone: two activation buffers (layer l writes buffer l % 2)
// whose rows are padded by 8 elements, so that the 16 rows of an operand
// fragment start 16 bytes apart and spread over the LDS banks.  About 40 KiB.
constexpr int LDA0 = F0 + 8, LDH = HD + 8, LDT = TR + 8;
struct FwdSmem {
  __bf16 a0[TR * LDA0];
  __bf16 act[2][TR * LDH];
  float w5[HD];  // the output layer's weights (their bfloat16 values)
  float bias[NL][HD];
};

// The backward pass.  The weight gradients contract over the rows, so what enters
// them lies transposed too ([column][row], rows of LDT): every operand
// fragment of either product is 16 contiguous bytes.  `row` holds the
// activations in turn and then the gradients dq, `dqt` dq transposed: two buffers
// each, so that a layer needs one barrier.  About 140 KiB.
struct GradSmem {
  __bf16 row[2][TR * LDH];
  __bf16 a0[TR * LDA0];
  __bf16 a0t[F0 * LDT];
  __bf16 at[NL - 1][HD * LDT];
  __bf16 dqt[2][HD * LDT];
  float outp[HD / 16][TR];  // the output layer's partial sums per column block
  float half[3][HD];        // column sums of rows 32 .. 63 (two layers in turn, the output layer)
  float g5[TR];
};

// The Fourier features of rows r0 .. r0 + 63 into a0 (row stride lda; rows
// past n are zero), by T threads; transposed to a0t as well when it is not null.
template <int T>
__device__ void features_tile(const Net& net, const float* y, int64_t n, int64_t r0, __bf16* a0, int lda,
                              __bf16* a0t = nullptr) {
#pragma unroll 1  // the binary64 sine beside a kernel's weights: two at once do not fit its registers
  for (int idx = threadIdx.x; idx < TR * KF; idx += T) {
    const int r = idx / KF, k = idx % KF;
    const int64_t row = r0 + r;
    float sv = 0.f, cv = 0.f;
    if (row < n) {
      // B y in binary64 (each product of two binary32 values is exact), the
      // period taken out exactly, sin and cos of 2 pi (B y) in binary64: the
      // features are then the binary32 roundings of the exact values except
      // within ~1e-16 of a rounding boundary
      double arg = 0.0;
      for (int d = 0; d < net.dim; ++d) arg += (double)net.fourier[k * net.dim + d] * (double)y[row * net.dim + d];
      const double r = arg - rint(arg);  // exact (Sterbenz), in [-1/2, 1/2]
      double sd, cd;
      sincospi(2.0 * r, &sd, &cd);
      sv = (float)sd;
      cv = (float)cd;
    }
    a0[r * lda + k] = (__bf16)sv;
    a0[r * lda + KF + k] = (__bf16)cv;
    if (a0t) {
      a0t[k * LDT + r] = (__bf16)sv;
      a0t[(KF + k) * LDT + r] = (__bf16)cv;
    }
  }
}

// Forward pass, weight-stationary: wavefront w computes output columns
// 16 w .. 16 w + 15 of every hidden layer, and holds those columns of the first
// layers' bfloat16 weights in registers as MFMA operand fragments (9 fragments,
// 36 registers), loaded once per workgroup; the workgroups then take 64-row
// tiles in turn.  The last hidden layer's fragments are loaded for each tile: with
// them the kernel's 128 registers, four wavefronts per SIMD, spill.  Per layer
// and tile a wavefront reads the four row blocks' activation fragments from LDS
// and issues four MFMAs per 32-wide k step.  Bound by the activations'
// arithmetic (18 lane operations each): 1,048,576 rows 398 us, and 200,992
// rows 84 against 97 us with four wavefronts of 32 columns and all weights in
// registers, two per SIMD.  The accumulation order of each output (k ascending
// in steps of 32), the bias, the activation and its rounding are those of the
// backward pass's forward tile.
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) mlp_forward_kernel(Net net, const float* y,
                                                                                        int64_t n, float* out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  FwdSmem& sm = *reinterpret_cast<FwdSmem*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kq = 8 * (lane >> 4);  // the lane's eight k values within a 32-wide step
  // weight fragments: B[k][o] = W[o][k], o = 16 wave + lane % 16
  const int col = 16 * wave + (lane & 15);
  const bf16x8 w0 = *(const bf16x8*)(net.wq + offW(0) + col * F0 + kq);
  bf16x8 wh[NL - 2][HD / 32];
#pragma unroll
  for (int l = 1; l < NL - 1; ++l)
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) wh[l - 1][ks] = *(const bf16x8*)(net.wq + offW(l) + col * HD + 32 * ks + kq);
  if (tid < HD) sm.w5[tid] = (float)net.wq[offW(NL) + tid];
  static_assert(NT == NL * HD, "a bias per thread");
  sm.bias[tid / HD][tid % HD] = net.p[offB(tid / HD) + tid % HD];
  const float b5 = net.p[offB(NL)];
  const int64_t n_tiles = (n + TR - 1) / TR;
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int64_t r0 = t * TR;
    features_tile<NT>(net, y, n, r0, sm.a0, LDA0);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const __bf16* A = l == 0 ? sm.a0 : sm.act[(l - 1) & 1];
      const int lda = l == 0 ? LDA0 : LDH;
      __bf16* O = sm.act[l & 1];
      floatx4 acc[4];
      bf16x8 wl[HD / 32];
      if (l == NL - 1) {
        const __bf16* W = net.wq;
#ifdef __HIP_DEVICE_COMPILE__
        asm volatile("" : "+s"(W));  // loaded for each tile, not kept across them
#endif
#pragma unroll
        for (int ks = 0; ks < HD / 32; ++ks) wl[ks] = *(const bf16x8*)(W + offW(NL - 1) + col * HD + 32 * ks + kq);
      }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) acc[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < in_of(l) / 32; ++ks)
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
          const bf16x8 af = *(const bf16x8*)(A + (16 * rb + (lane & 15)) * lda + 32 * ks + kq);
          acc[rb] = mfma(af, l == 0 ? w0 : l == NL - 1 ? wl[ks] : wh[l == 0 || l == NL - 1 ? 0 : l - 1][ks], acc[rb]);
        }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * rb + 4 * (lane >> 4) + v;
          O[r * LDH + col] = (__bf16)silu_rounded(acc[rb][v] + sm.bias[l][col]);
        }
      __syncthreads();
    }
    // output layer: 4 lanes per row, 32 terms each in order, then two butterfly
    // steps, with the weights from LDS
    if (tid < 4 * TR) {
      const int r = tid >> 2, part = tid & 3;
      const __bf16* h4 = sm.act[(NL - 1) & 1] + r * LDH;
      float acc = 0.f;
      for (int i = part * 32; i < part * 32 + 32; ++i) acc += sm.w5[i] * (float)h4[i];
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      if (part == 0 && r0 + r < n) out[r0 + r] = acc + b5;
    }
    __syncthreads();  // the next tile's features and layers overwrite a0 and act
  }
}

// Target transform t -> (t - shift) inv_scale, clamped to [-clip, clip] when clip > 0.
struct TargetMap {
  int on;
  float shift, inv_scale, clip;
};

// Loss and gradient of one tile: writes the tile's partial gradient (NP floats)
// and partial loss (sum of squared errors).  scale = 1 / (rows in the batch).
//
// A chain of small products with a barrier after each: latency bounds it, so the
// tile has all 16 wavefronts of a CU.  Wavefront w takes columns 16 (w % 8) .. + 15 and
// rows 32 (w / 8) .. + 31 of every 64 x 128 array, forward and backward alike, so
// the pre-activations and the binary32 gradients of a lane's eight elements per
// layer stay in its registers; its weights are loaded ahead of the layer that
// needs them.  16,384 rows (256 tiles): 94 us with four wavefronts,
// 16-bit reads of the transposed operands and the pre-activations in memory.  All
// launches: the gradient 122 -> 45 us, with a separate Adam step 133 -> 47, the
// training step, whose sum takes the Adam step along, 126 -> 48.
__global__ void __launch_bounds__(GT) mlp_grad_kernel(Net net, const float* y, const float* target,
                                                      TargetMap tm, int64_t n, float scale,
                                                      float* part_grad, float* part_loss) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  GradSmem& sm = *reinterpret_cast<GradSmem*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, lc = lane & 15, lg = lane >> 4, kq = 8 * lg;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), cb = wave & 7, rh = wave >> 3;
  const int col = 16 * cb + lc;
  const int64_t r0 = (int64_t)blockIdx.x * TR;
  float* G = part_grad + (int64_t)blockIdx.x * NPP;
  // weight fragments: B[k][o] = W[o][k], o = col
  const bf16x8 w0 = *(const bf16x8*)(net.wq + offW(0) + col * F0 + kq);
  bf16x8 wh[NL - 1][HD / 32];
#pragma unroll
  for (int l = 1; l < NL; ++l)
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) wh[l - 1][ks] = *(const bf16x8*)(net.wq + offW(l) + col * HD + 32 * ks + kq);
  float bias[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) bias[l] = net.p[offB(l) + col];
  const float w5 = (float)net.wq[offW(NL) + col];
  features_tile<GT>(net, y, n, r0, sm.a0, LDA0, sm.a0t);
  __syncthreads();

  // element (j, v) of the lane: row 32 rh + 16 j + 4 lg + v, column col
  const int rj[2] = {32 * rh + 4 * lg, 32 * rh + 16 + 4 * lg};
  float s[NL][2][4], h4[2][4];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const __bf16* A = l == 0 ? sm.a0 : sm.row[(l - 1) & 1];
    const int lda = l == 0 ? LDA0 : LDH;
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < in_of(l) / 32; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 af = *(const bf16x8*)(A + (32 * rh + 16 * j + lc) * lda + 32 * ks + kq);
        acc[j] = mfma(af, l == 0 ? w0 : wh[l == 0 ? 0 : l - 1][ks], acc[j]);
      }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x4 h;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[l][j][v] = acc[j][v] + bias[l];
        h[v] = (__bf16)silu_rounded(s[l][j][v]);
        if (l < NL - 1) sm.row[l & 1][(rj[j] + v) * LDH + col] = h[v];
        else h4[j][v] = (float)h[v];
      }
      if (l < NL - 1) *(bf16x4*)(sm.at[l < NL - 1 ? l : 0] + col * LDT + rj[j]) = h;
    }
    if (l < NL - 1) __syncthreads();
  }

  // output layer f = W5 . h4 + b5: 16 columns by butterfly, the column blocks in order
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float f = w5 * h4[j][v];
#pragma unroll
      for (int off = 1; off < 16; off *= 2) f += __shfl_xor(f, off, 64);
      if (lc == 0) sm.outp[cb][rj[j] + v] = f;
    }
  __syncthreads();
  if (wave == 0) {
    float f = 0.f;
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) f += sm.outp[c][lane];
    f += net.p[offB(NL)];
    float e = 0.f;
    if (r0 + lane < n) {
      float tv = target[r0 + lane];
      // a non-finite target (a boundary point whose every path was non-finite)
      // has no weight in the loss: e = 0 (clamping would turn NaN into -clip)
      if (isfinite(tv)) {
        if (tm.on) {
          tv = (tv - tm.shift) * tm.inv_scale;
          if (tm.clip > 0.f) tv = fminf(fmaxf(tv, -tm.clip), tm.clip);
        }
        e = f - tv;
      }
    }
    const float g = 2.f * e * scale;
    sm.g5[lane] = g;
    float se = e * e, sg = g;  // the tile's loss and db5
#pragma unroll
    for (int off = 1; off < 64; off *= 2) {
      se += __shfl_xor(se, off, 64);
      sg += __shfl_xor(sg, off, 64);
    }
    if (lane == 0) {
      part_loss[blockIdx.x] = se;
      G[offB(NL)] = sg;
    }
  }
  __syncthreads();

  // dW5[i] = sum_r g5 h4[r][i]; ds of the last hidden layer: g5 W5 silu'(s4)
  float ds[2][4], t5 = 0.f;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float g = sm.g5[rj[j] + v];
      t5 += g * h4[j][v];
      ds[j][v] = g * w5 * silu_grad(s[NL - 1][j][v]);
    }
  t5 += __shfl_xor(t5, 16, 64);
  t5 += __shfl_xor(t5, 32, 64);
  if (rh == 1 && lg == 0) sm.half[2][col] = t5;

#pragma unroll
  for (int l = NL - 1; l >= 0; --l) {
    const int K = in_of(l);  // input width of layer l
    // dh's weights: B[o][i] = W[o][i], i = col, from the transposed copy
    bf16x8 wt[HD / 32];
    if (l > 0) {
#pragma unroll
      for (int ks = 0; ks < HD / 32; ++ks) wt[ks] = *(const bf16x8*)(net.wt + offW(l) + col * HD + 32 * ks + kq);
    }
    // bfloat16 copy of ds for the products; bias gradient from binary32 ds
    __bf16* const dq = sm.row[l & 1];
    __bf16* const dqt = sm.dqt[l & 1];
    float tb = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x4 q;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        q[v] = (__bf16)ds[j][v];
        if (l > 0) dq[(rj[j] + v) * LDH + col] = q[v];
        tb += ds[j][v];
      }
      *(bf16x4*)(dqt + col * LDT + rj[j]) = q;
    }
    tb += __shfl_xor(tb, 16, 64);
    tb += __shfl_xor(tb, 32, 64);
    if (rh == 1 && lg == 0) sm.half[l & 1][col] = tb;
    __syncthreads();
    if (rh == 0 && lg == 0) {
      G[offB(l) + col] = tb + sm.half[l & 1][col];
      if (l == NL - 1) G[offW(NL) + col] = t5 + sm.half[2][col];
    }
    // dW_l[o][i] = sum_r a_{l-1}[r][i] dq[r][o]: the lane holds four consecutive
    // i of one o; this wavefront's o are 16 cb .. + 15, its i half of the K
    {
      const __bf16* AT = l == 0 ? sm.a0t : sm.at[l == 0 ? 0 : l - 1];
      bf16x8 bf[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) bf[ks] = *(const bf16x8*)(dqt + col * LDT + 32 * ks + kq);
#pragma unroll
      for (int t = 0; t < K / 32; ++t) {
        const int ib = rh * (K / 32) + t;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          acc = mfma(*(const bf16x8*)(AT + (16 * ib + lc) * LDT + 32 * ks + kq), bf[ks], acc);
        *(floatx4*)(G + offW(l) + col * K + 16 * ib + 4 * lg) = acc;
      }
    }
    if (l == 0) break;
    // dh_{l-1}[r][i] = sum_o dq[r][o] W_l[o][i]: (TR x HD) x (HD x HD)
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j] = mfma(*(const bf16x8*)(dq + (32 * rh + 16 * j + lc) * LDH + 32 * ks + kq), wt[ks], acc[j]);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) ds[j][v] = acc[j][v] * silu_grad(s[l == 0 ? 0 : l - 1][j][v]);
  }
}

// Adam on the binary32 master copy, then the bfloat16 copies for the products.
struct AdamStep {
  float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ void adam_param(const Net& net, int p, float g, const AdamStep& a) {
  const float m = a.b1 * net.m[p] + (1.f - a.b1) * g;
  const float v = a.b2 * net.v[p] + (1.f - a.b2) * g * g;
  net.m[p] = m;
  net.v[p] = v;
  const float w = net.p[p] - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
  net.p[p] = w;
  // bfloat16 copies
  int l = 0;
  while (l < NL && p >= offW(l + 1)) ++l;
  const int q = p - offW(l);
  const int K = in_of(l), O = out_of(l);
  if (q < O * K) {
    const int o = q / K, i = q % K;
    net.wq[p] = (__bf16)w;
    net.wt[offW(l) + i * O + o] = (__bf16)w;
  }
}

// grad[p] = the sum of the tiles' partial gradients, loss = sum part_loss * scale
// (in the last workgroup), and with ADAM the parameters' step.  A workgroup takes 64
// parameters: wavefront w adds tiles w, w + 16, ... in order, then the first adds the
// 16 sums in order, so the gradient is deterministic.  Bound by reading the
// partial gradients once (55 MB for 256 tiles; two passes over slices of 32
// tiles, the loss summed by one thread and Adam apart took 12 + 18 + 5 us).
template <bool ADAM>
__global__ void __launch_bounds__(1024) reduce_grad_kernel(Net net, const float* part, int n_tiles, float* grad,
                                                           const float* part_loss, float* loss, float scale,
                                                           AdamStep adam) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == gridDim.x - 1) {
    if (wave != 0 || !loss) return;
    float acc = 0.f;
    for (int t = lane; t < n_tiles; t += 64) acc += part_loss[t];
    for (int off = 1; off < 64; off *= 2) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) *loss = acc * scale;
    return;
  }
  const int p = blockIdx.x * 64 + lane;
  float acc = 0.f;
  if (p < NP) {
#pragma unroll 8
    for (int t = wave; t < n_tiles; t += 16) acc += part[(int64_t)t * NPP + p];
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave != 0 || p >= NP) return;
  for (int w = 1; w < 16; ++w) acc += red[w][lane];
  grad[p] = acc;
  if constexpr (ADAM) adam_param(net, p, acc, adam);
}

__global__ void adam_kernel(Net net, const float* grad, AdamStep adam) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NP) adam_param(net, p, grad[p], adam);
}

__global__ void refresh_bf16_kernel(Net net) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= NP) return;
  int l = 0;
  while (l < NL && p >= offW(l + 1)) ++l;
  const int q = p - offW(l);
  const int K = in_of(l), O = out_of(l);
  if (q < O * K) {
    const int o = q / K, i = q % K;
    net.wq[p] = (__bf16)net.p[p];
    net.wt[offW(l) + i * O + o] = (__bf16)net.p[p];
  }
}

}  // namespace

struct wob_mlp_s {
  Net net{};
  int64_t max_batch = 0;
  int n_tiles_max = 0;
  float* part = nullptr;      // n_tiles_max x NPP
  float* part_loss = nullptr; // n_tiles_max
  float* grad = nullptr;      // NP
};

namespace {

void mlp_destroy(wob_mlp_s* h) {
  if (!h) return;
  void* ptrs[] = {h->net.p, h->net.m, h->net.v, h->net.wq, h->net.wt, h->net.fourier,
                  h->part, h->part_loss, h->grad};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  delete h;
}

wob_status refresh(wob_mlp_s* h, hipStream_t st) {
  hipLaunchKernelGGL(refresh_bf16_kernel, dim3((NP + 255) / 256), dim3(256), 0, st, h->net);
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

}  // namespace

extern "C" {

int64_t wob_mlp_n_params(void) { return NP; }

wob_status wob_mlp_create(int32_t dim, const float* fourier, const float* params, int64_t max_batch,
                          wob_mlp* out) {
  if (!out) return WOB_E_ARG;
  *out = nullptr;
  if ((dim != 2 && dim != 3) || !fourier || !params || max_batch < 0) return WOB_E_ARG;
  for (int i = 0; i < KF * dim; ++i)
    if (!std::isfinite(fourier[i])) return WOB_E_ARG;
  for (int i = 0; i < NP; ++i)
    if (!std::isfinite(params[i])) return WOB_E_ARG;
  // the backward pass keeps every activation of its 64 rows in LDS (> 64 KiB)
  if (hipFuncSetAttribute((const void*)mlp_forward_kernel,
                          hipFuncAttributeMaxDynamicSharedMemorySize, sizeof(FwdSmem)) != hipSuccess ||
      hipFuncSetAttribute((const void*)mlp_grad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          sizeof(GradSmem)) != hipSuccess)
    return WOB_E_DEVICE;
  wob_mlp_s* h = new (std::nothrow) wob_mlp_s();
  if (!h) return WOB_E_ALLOC;
  h->net.dim = dim;
  h->max_batch = max_batch;
  h->n_tiles_max = (int)((max_batch + TR - 1) / TR);
  bool ok = hipMalloc((void**)&h->net.p, NP * 4) == hipSuccess &&
            hipMalloc((void**)&h->net.m, NP * 4) == hipSuccess &&
            hipMalloc((void**)&h->net.v, NP * 4) == hipSuccess &&
            hipMalloc((void**)&h->net.wq, NP * 2) == hipSuccess &&
            hipMalloc((void**)&h->net.wt, NP * 2) == hipSuccess &&
            hipMalloc((void**)&h->net.fourier, KF * dim * 4) == hipSuccess &&
            hipMalloc((void**)&h->grad, NP * 4) == hipSuccess;
  if (ok && h->n_tiles_max > 0)
    ok = hipMalloc((void**)&h->part, (size_t)h->n_tiles_max * NPP * 4) == hipSuccess &&
         hipMalloc((void**)&h->part_loss, (size_t)h->n_tiles_max * 4) == hipSuccess;
  if (!ok) {
    mlp_destroy(h);
    return WOB_E_ALLOC;
  }
  std::vector<float> zeros(NP, 0.f);
  ok = hipMemcpy(h->net.p, params, NP * 4, hipMemcpyHostToDevice) == hipSuccess &&
       hipMemcpy(h->net.m, zeros.data(), NP * 4, hipMemcpyHostToDevice) == hipSuccess &&
       hipMemcpy(h->net.v, zeros.data(), NP * 4, hipMemcpyHostToDevice) == hipSuccess &&
       hipMemcpy(h->net.fourier, fourier, KF * dim * 4, hipMemcpyHostToDevice) == hipSuccess &&
       refresh(h, nullptr) == WOB_OK && hipDeviceSynchronize() == hipSuccess;
  if (!ok) {
    mlp_destroy(h);
    return WOB_E_DEVICE;
  }
  *out = h;
  return WOB_OK;
}

void wob_mlp_free(wob_mlp h) { mlp_destroy(h); }

wob_status wob_mlp_get_params(wob_mlp h, float* params) {
  if (!h || !params) return WOB_E_ARG;
  return hipMemcpy(params, h->net.p, NP * 4, hipMemcpyDeviceToHost) == hipSuccess ? WOB_OK
                                                                                  : WOB_E_DEVICE;
}

wob_status wob_mlp_set_params(wob_mlp h, const float* params) {
  if (!h || !params) return WOB_E_ARG;
  std::vector<float> zeros(NP, 0.f);
  if (hipMemcpy(h->net.p, params, NP * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(h->net.m, zeros.data(), NP * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(h->net.v, zeros.data(), NP * 4, hipMemcpyHostToDevice) != hipSuccess)
    return WOB_E_DEVICE;
  if (refresh(h, nullptr) != WOB_OK || hipDeviceSynchronize() != hipSuccess) return WOB_E_DEVICE;
  return WOB_OK;
}

wob_status wob_mlp_get_moments(wob_mlp h, float* m, float* v) {
  if (!h || !m || !v) return WOB_E_ARG;
  return hipMemcpy(m, h->net.m, NP * 4, hipMemcpyDeviceToHost) == hipSuccess &&
                 hipMemcpy(v, h->net.v, NP * 4, hipMemcpyDeviceToHost) == hipSuccess
             ? WOB_OK
             : WOB_E_DEVICE;
}

wob_status wob_mlp_set_moments(wob_mlp h, const float* m, const float* v) {
  if (!h || !m || !v) return WOB_E_ARG;
  if (hipMemcpy(h->net.m, m, NP * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(h->net.v, v, NP * 4, hipMemcpyHostToDevice) != hipSuccess || hipDeviceSynchronize() != hipSuccess)
    return WOB_E_DEVICE;
  return WOB_OK;
}

wob_status wob_mlp_forward(wob_mlp h, const float* y, int64_t n, float* out, void* stream) {
  if (!h || n < 0 || (n > 0 && (!y || !out))) return WOB_E_ARG;
  if (n == 0) return WOB_OK;
  const int64_t tiles = (n + TR - 1) / TR;
  // persistent workgroups, their weight fragments loaded once (two resident per CU)
  const int64_t grid = tiles < kFwdGrid ? tiles : kFwdGrid;
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((unsigned)grid), dim3(NT), sizeof(FwdSmem),
                     (hipStream_t)stream, h->net, y, n, out);
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

}  // extern "C"

namespace {

AdamStep adam_step(int64_t step, float lr, float b1, float b2, float eps) {
  return AdamStep{lr, b1, b2, eps, 1.f - std::pow(b1, (float)step), 1.f - std::pow(b2, (float)step)};
}
bool valid_adam(int64_t step, float lr, float b1, float b2, float eps) {
  return step >= 1 && lr > 0.f && std::isfinite(lr) && b1 >= 0.f && b1 < 1.f && b2 >= 0.f && b2 < 1.f && eps > 0.f;
}

// The gradient into `grad`, and with `adam` the step that it gives.
wob_status backward(wob_mlp h, const float* y, const float* target, const wob_target_map* tmap, int64_t n,
                    float* grad, float* loss, const AdamStep* adam, hipStream_t st) {
  if (!h || n <= 0 || n > h->max_batch || !y || !target || !grad) return WOB_E_ARG;
  TargetMap tm{0, 0.f, 1.f, 0.f};
  if (tmap) {
    if (!std::isfinite(tmap->shift) || !(tmap->scale > 0.f) || !std::isfinite(tmap->scale) ||
        !(tmap->clip >= 0.f))
      return WOB_E_ARG;
    tm = TargetMap{1, tmap->shift, 1.f / tmap->scale, tmap->clip};
  }
  const int tiles = (int)((n + TR - 1) / TR);
  const float scale = 1.f / (float)n;
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(tiles), dim3(GT), sizeof(GradSmem), st, h->net, y, target, tm, n, scale,
                     h->part, h->part_loss);
  const dim3 grid((NP + 63) / 64 + 1), block(1024);
  if (adam)
    hipLaunchKernelGGL(reduce_grad_kernel<true>, grid, block, 0, st, h->net, h->part, tiles, grad, h->part_loss,
                       loss, scale, *adam);
  else
    hipLaunchKernelGGL(reduce_grad_kernel<false>, grid, block, 0, st, h->net, h->part, tiles, grad, h->part_loss,
                       loss, scale, AdamStep{});
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

}  // namespace

extern "C" {

wob_status wob_mlp_backward(wob_mlp h, const float* y, const float* target,
                            const wob_target_map* tmap, int64_t n, float* grad, float* loss,
                            void* stream) {
  return backward(h, y, target, tmap, n, grad, loss, nullptr, (hipStream_t)stream);
}

wob_status wob_mlp_adam_step(wob_mlp h, const float* grad, int64_t step, float lr, float b1, float b2,
                             float eps, void* stream) {
  if (!h || !grad || !valid_adam(step, lr, b1, b2, eps)) return WOB_E_ARG;
  hipLaunchKernelGGL(adam_kernel, dim3((NP + 255) / 256), dim3(256), 0, (hipStream_t)stream, h->net,
                     grad, adam_step(step, lr, b1, b2, eps));
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

wob_status wob_mlp_train_step(wob_mlp h, const float* y, const float* target,
                              const wob_target_map* tmap, int64_t n, int64_t step, float lr,
                              float* loss, void* stream) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  if (!valid_adam(step, lr, b1, b2, eps)) {
    // the gradient and the loss of the refused step are left as ever
    const wob_status s = wob_mlp_backward(h, y, target, tmap, n, h ? h->grad : nullptr, loss, stream);
    return s != WOB_OK ? s : WOB_E_ARG;
  }
  const AdamStep adam = adam_step(step, lr, b1, b2, eps);
  return backward(h, y, target, tmap, n, h ? h->grad : nullptr, loss, &adam, (hipStream_t)stream);
}

}  // extern "C"
