// The learned warm start of the entropy filter's search: a 16-64-64-1 tanh MLP in
// FP32 (inference, backward pass, Adam), written as plain HIP kernels.
//
//   x_s = (x - mean) / std;  h1 = tanh(W1 x_s + b1);  h2 = tanh(W2 h1 + b2);  y = w3.h2 + b3
//   loss = mean over the batch of (y - t)^2
// Flat parameters (5,313): W1[64][16] b1[64] W2[64][64] b2[64] w3[64] b3[1].
// Gradients are reduced over the batch in a fixed order (deterministic).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace frmi {

constexpr int MLP_IN = 16, MLP_H = 64;
constexpr int MLP_OW1 = 0, MLP_OB1 = MLP_OW1 + MLP_H * MLP_IN, MLP_OW2 = MLP_OB1 + MLP_H,
              MLP_OB2 = MLP_OW2 + MLP_H * MLP_H, MLP_OW3 = MLP_OB2 + MLP_H, MLP_OB3 = MLP_OW3 + MLP_H,
              MLP_NP = MLP_OB3 + 1;

// Stage parameters and input scaling into LDS.
__device__ __forceinline__ void mlp_stage(const float* __restrict__ w, const float* __restrict__ scale, float* W,
                                          float* sc) {
  for (int i = threadIdx.x; i < MLP_NP; i += blockDim.x) W[i] = w[i];
  for (int i = threadIdx.x; i < 2 * MLP_IN; i += blockDim.x) sc[i] = scale[i];
  __syncthreads();
}

__device__ __forceinline__ float mlp_eval(const float* W, const float* sc, const float* x, float* h1, float* h2) {
  float xs[MLP_IN];
#pragma unroll
  for (int k = 0; k < MLP_IN; ++k) xs[k] = (x[k] - sc[k]) / sc[MLP_IN + k];
  for (int i = 0; i < MLP_H; ++i) {
    float a = W[MLP_OB1 + i];
#pragma unroll
    for (int k = 0; k < MLP_IN; ++k) a += W[MLP_OW1 + i * MLP_IN + k] * xs[k];
    h1[i] = tanhf(a);
  }
  float y = W[MLP_OB3];
  for (int j = 0; j < MLP_H; ++j) {
    float a = W[MLP_OB2 + j];
    for (int i = 0; i < MLP_H; ++i) a += W[MLP_OW2 + j * MLP_H + i] * h1[i];
    const float t = tanhf(a);
    if (h2) h2[j] = t;
    y += W[MLP_OW3 + j] * t;
  }
  return y;
}

// Inference for rows with flag != 0 (flag may be null: all rows).  With n_bits > 0
// the output is the predicted dyadic index k^ = 2^(n_bits y) instead of y.
__global__ void __launch_bounds__(256) mlp_forward(const float* __restrict__ w, const float* __restrict__ scale,
                                                   const float* __restrict__ x, const int32_t* __restrict__ flag,
                                                   int64_t n, int n_bits, float* __restrict__ y) {
  __shared__ float W[MLP_NP];
  __shared__ float sc[2 * MLP_IN];
  mlp_stage(w, scale, W, sc);
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n || (flag && flag[r] == 0)) return;
  float h1[MLP_H];
  const float out = mlp_eval(W, sc, x + r * MLP_IN, h1, nullptr);
  y[r] = n_bits > 0 ? exp2f((float)n_bits * out) : out;
}

// Per-sample forward and backward quantities of one batch (rows idx[0..B)).
// Scratch per sample s: xs[16] | h1[64] | h2[64] | d1[64] | d2[64] | dy
constexpr int MLP_SS = MLP_IN + 4 * MLP_H + 1;
constexpr int MLP_FB_WAVES = 4;            // samples per block of mlp_fwd_bwd

// One wave per sample, lane j = hidden unit j: every dot product is the sequential sum the
// single-thread form takes (same terms, same order), so the values are those of
// mlp_eval.  The weights sit in LDS twice, W2 as stored (rows read by the backward pass:
// consecutive lanes, consecutive words) and transposed in rows of 65 (W2^T and W1^T for the
// forward pass: neither the transposing stores nor the reads conflict; in rows of 64 every
// store of a wave fell on one bank).  All global loads of a thread (16 bytes each for the
// weights) are issued first.  An Adam step of batch 256: 21.1 -> 16.2 us.
__global__ void __launch_bounds__(64 * MLP_FB_WAVES) mlp_fwd_bwd(const float* __restrict__ w,
                                                                 const float* __restrict__ scale,
                                                                 const float* __restrict__ x,
                                                                 const float* __restrict__ t,
                                                                 const int32_t* __restrict__ idx, int B,
                                                                 float* __restrict__ scratch,
                                                                 float* __restrict__ sqerr) {
  constexpr int LD = MLP_H + 1, NT = 64 * MLP_FB_WAVES, N2 = MLP_H * MLP_H / 4 / NT;
  static_assert(MLP_H * MLP_IN == 4 * NT && MLP_H * MLP_H % (4 * NT) == 0 && MLP_OW2 % 4 == 0, "16-byte loads");
  __shared__ __align__(16) float W2[MLP_H * MLP_H];
  __shared__ float W2T[MLP_H * LD], W1T[MLP_IN * LD];
  __shared__ float BV[3 * MLP_H + 1];       // b1 | b2 | w3 | b3
  __shared__ float sc[2 * MLP_IN];
  __shared__ float H[MLP_FB_WAVES][3][MLP_H];   // per wave: h1 | h2 | d2
  // every wave passes the barriers below; a wave past the batch computes nothing
  const int tid = threadIdx.x, wv = tid / 64, j = tid % 64;
  const int s = blockIdx.x * MLP_FB_WAVES + wv;
  const bool valid = s < B;
  const int64_t row = valid ? (idx ? idx[s] : s) : 0;
  const float4* w4 = reinterpret_cast<const float4*>(w);
  float4 q2[N2];
#pragma unroll
  for (int k = 0; k < N2; ++k) q2[k] = w4[MLP_OW2 / 4 + tid + k * NT];
  const float4 q1 = w4[MLP_OW1 / 4 + tid];
  const float bv = w[tid < MLP_H ? MLP_OB1 + tid : (tid < 3 * MLP_H ? MLP_OB2 + (tid - MLP_H) % MLP_H +
                                                    (tid < 2 * MLP_H ? 0 : MLP_OW3 - MLP_OB2) : MLP_OB3)];
  const float tgt = t[row];
  float xs[MLP_IN];
#pragma unroll
  for (int k = 0; k < MLP_IN; ++k) xs[k] = x[row * MLP_IN + k];
  if (tid < 2 * MLP_IN) sc[tid] = scale[tid];
  if (tid <= 3 * MLP_H) BV[tid] = bv;
#pragma unroll
  for (int k = 0; k < N2; ++k) {
    const int i = 4 * (tid + k * NT);
    *reinterpret_cast<float4*>(&W2[i]) = q2[k];
    const float v[4] = {q2[k].x, q2[k].y, q2[k].z, q2[k].w};
#pragma unroll
    for (int c = 0; c < 4; ++c) W2T[((i + c) % MLP_H) * LD + (i + c) / MLP_H] = v[c];
  }
  {
    const int i = 4 * tid;
    const float v[4] = {q1.x, q1.y, q1.z, q1.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) W1T[((i + c) % MLP_IN) * LD + (i + c) / MLP_IN] = v[c];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < MLP_IN; ++k) xs[k] = (xs[k] - sc[k]) / sc[MLP_IN + k];
  float a = BV[j];
#pragma unroll
  for (int k = 0; k < MLP_IN; ++k) a += W1T[k * LD + j] * xs[k];
  const float h1 = tanhf(a);
  H[wv][0][j] = h1;
  __syncthreads();
  a = BV[MLP_H + j];
  for (int i = 0; i < MLP_H; ++i) a += W2T[i * LD + j] * H[wv][0][i];
  const float h2 = tanhf(a);
  H[wv][1][j] = h2;
  __syncthreads();
  float y = BV[3 * MLP_H];
  for (int i = 0; i < MLP_H; ++i) y += BV[2 * MLP_H + i] * H[wv][1][i];
  const float r = y - (valid ? tgt : 0.0f);
  const float dy = 2.0f * r / (float)B;
  const float d2 = dy * BV[2 * MLP_H + j] * (1.0f - h2 * h2);
  H[wv][2][j] = d2;
  __syncthreads();
  a = 0;
  for (int i = 0; i < MLP_H; ++i) a += H[wv][2][i] * W2[i * MLP_H + j];
  const float d1 = a * (1.0f - h1 * h1);
  if (!valid) return;
  float* S = scratch + (int64_t)s * MLP_SS;
  if (j < MLP_IN) S[j] = xs[j];
  S[MLP_IN + j] = h1;
  S[MLP_IN + MLP_H + j] = h2;
  S[MLP_IN + 2 * MLP_H + j] = d1;
  S[MLP_IN + 3 * MLP_H + j] = d2;
  if (j == 0) {
    S[MLP_SS - 1] = dy;
    sqerr[s] = r * r;
  }
}

// One Adam step of a parameter (c1 = 1 - b1^t, c2 = 1 - b2^t of the step count t).
struct AdamArgs {
  float *w, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};

// Gradient of every parameter: a fixed-order sum over the batch.  Each parameter's term is
// a product of two per-sample quantities (or one of them alone: biases, b3), so a thread
// takes their two offsets within a sample's scratch once and walks the batch with them.
// A block takes 64 parameters, its 8 waves an eighth of the batch each (their sums are added
// in wave order): one thread per parameter walked 256 samples in 32 rounds of loads.  With
// ADAM the block then updates its parameters (grad may be null).  Bound by load latency and
// launches: an Adam step of batch 256 took 34.3 us in three kernels with one thread per
// parameter, 21.1 us here (batch 500: 54 -> 31).
constexpr int MLP_GR_P = 64, MLP_GR_Q = 8, MLP_GR_NT = MLP_GR_P * MLP_GR_Q;
template <bool ADAM>
__global__ void __launch_bounds__(MLP_GR_NT) mlp_grad_reduce(const float* __restrict__ scratch, int B,
                                                             const float* __restrict__ sqerr, float* __restrict__ grad,
                                                             float* __restrict__ loss, AdamArgs A) {
  __shared__ float part[MLP_GR_Q][MLP_GR_P];
  const int lane = threadIdx.x % MLP_GR_P, q = threadIdx.x / MLP_GR_P;
  const int p = blockIdx.x * MLP_GR_P + lane;
  float w0 = 0, m0 = 0, v0 = 0;
  if constexpr (ADAM) {
    if (q == 0 && p < MLP_NP) {
      w0 = A.w[p];
      m0 = A.m[p];
      v0 = A.v[p];
    }
  }
  constexpr int XS = 0, H1 = MLP_IN, H2 = H1 + MLP_H, D1 = H2 + MLP_H, D2 = D1 + MLP_H, DY = MLP_SS - 1;
  int oa = DY, ob = -1;            // term = S[oa] * S[ob] (S[oa] alone when ob < 0)
  if (p < MLP_OB1) { oa = D1 + (p - MLP_OW1) / MLP_IN; ob = XS + (p - MLP_OW1) % MLP_IN; }
  else if (p < MLP_OW2) oa = D1 + (p - MLP_OB1);
  else if (p < MLP_OB2) { oa = D2 + (p - MLP_OW2) / MLP_H; ob = H1 + (p - MLP_OW2) % MLP_H; }
  else if (p < MLP_OW3) oa = D2 + (p - MLP_OB2);
  else if (p < MLP_OB3) { oa = DY; ob = H2 + (p - MLP_OW3); }
  const int per = (B + MLP_GR_Q - 1) / MLP_GR_Q, s0 = min(q * per, B), s1 = min(s0 + per, B);
  float a = 0;
  if (p == MLP_NP) {               // the loss
    for (int s = s0; s < s1; ++s) a += sqerr[s];
  } else if (p < MLP_NP && ob >= 0) {
    const float* Ap = scratch + oa;
    const float* Bp = scratch + ob;
#pragma unroll 16
    for (int s = s0; s < s1; ++s) a += Ap[(int64_t)s * MLP_SS] * Bp[(int64_t)s * MLP_SS];
  } else if (p < MLP_NP) {
    const float* Ap = scratch + oa;
#pragma unroll 16
    for (int s = s0; s < s1; ++s) a += Ap[(int64_t)s * MLP_SS];
  }
  part[q][lane] = a;
  __syncthreads();
  if (q != 0 || p > MLP_NP) return;
#pragma unroll
  for (int k = 1; k < MLP_GR_Q; ++k) a += part[k][lane];
  if (p == MLP_NP) {
    *loss = a / (float)B;
    return;
  }
  if (grad) grad[p] = a;
  if constexpr (ADAM) {
    const float mi = A.b1 * m0 + (1.0f - A.b1) * a;
    const float vi = A.b2 * v0 + (1.0f - A.b2) * a * a;
    A.m[p] = mi;
    A.v[p] = vi;
    A.w[p] = w0 - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
  }
}

}  // namespace frmi
