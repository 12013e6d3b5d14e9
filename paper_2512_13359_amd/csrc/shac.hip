// SHAC (short-horizon actor-critic; the differentiable-simulation learner of paper Sec.
// III-A3) on the paper's own task: the actor objective of one window of h control steps,
//   L = -(1 / (N h)) sum_i [ sum_{t<h} gamma^t r_t^i + gamma^h V(o(s_h^i)) ],
// and its gradient with respect to the policy parameters, by reverse-mode differentiation
// through the reward, the observation, RK4 + Fossen and the policy network.
//
// Kernels, in launch order:
//   k_frags        the bf16 weights of each network rearranged into the MFMA A fragments
//                  that the window kernel reads (W1, W2, W3 and their transposes)
//   k_window<mode> one workgroup of four waves per 16 environments, the whole window in one
//                  launch.  Every wave steps the physics of all 16 environments, four lanes
//                  per environment (shac_quad.hpp), so each wave has the observations, actions
//                  and adjoints it needs without an exchange; the networks are split by hidden
//                  feature, wave w owning features 64 w .. 64 w + 63 of both hidden layers (its
//                  64 rows of W2, then of W2^T, in LDS; its small weights in registers).  At
//                  workgroup barriers the waves exchange through LDS only hidden layer 1 and
//                  the output partials (two barriers per forward step), q(dz2) and the
//                  input-gradient partials (two per reverse step).  Forward sweep: policy on
//                  MFMA, RK4 of the paper task, reward, and what the reverse sweep needs (every
//                  RK4 stage's input, the observation with the factors of its derivative, the
//                  action and its moving average, every wave's hidden-2 activations); terminal
//                  value and its input gradient; the environment update (reset where the
//                  window ends the episode); reverse sweep: per step, the state adjoint
//                  through RK4 from the stored stage inputs, the clip, the policy's input
//                  gradient (backward on MFMA from the stored hidden-2 activations), and one
//                  observation adjoint that takes the policy's and the reward's cotangents
//                  together.  Bound by the instruction stream of one wave per SIMD (at 4096
//                  environments every CU holds one workgroup): with the physics in one-lane
//                  form, every lane row a copy, and the RK4 stages re-integrated in the
//                  reverse sweep, a 32-step window took 693 us in all; with four lanes per
//                  environment 457 us; with the small weight gradients summed here, in place
//                  of a kernel that read 200 MB of their operands back, 398 us; with the action
//                  noise drawn once for the four waves 382 us.  Those sums' 48 accumulators are
//                  live through both sweeps: the policy modes spill 30 registers (68 and 84 bytes
//                  of scratch per lane; none before).  Each wave adds its features' dW1, dW3 and
//                  bias gradients up in registers and stores the bf16 operands of dW2 (q(h1),
//                  q(dz2)) as "half fragments"
//   k_dw2          (PPO update) dW2 = sum q(dz2) q(h1)^T over all N h samples
//   k_reduce       (PPO update) fixed-order sums of the partials -> packed gradient
//   k_finalize     loss statistics, gradient norm, clipping factor
//
// MFMA layout as in mlp_mfma.hpp (v_mfma_f32_16x16x32_bf16, lane l = 16 g + r, K slot
// (g, j) = feature 16 (j / 4) + 4 g + j % 4 of a 32-wide K step).  In the window kernel
// the N dimension is the workgroup's 16 environments (one N-tile), M the output features.
// A half fragment (8 bytes, lane (g, r)) holds feature r of a 16-feature tile for
// samples 4g .. 4g + 3 of a 16-sample tile; sample tile (t, workgroup) = t G + workgroup,
// G = workgroups.
#include <cmath>

#include "auv_internal.hpp"
#include "mlp_mfma.hpp"
#include "shac_quad.hpp"

namespace auv {
namespace shac {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
constexpr int EPG = 16;                  // environments per workgroup (one MFMA N-tile)
constexpr int WAVES = 4;                 // waves per workgroup; wave w owns hidden features 64 w ..
constexpr int WF = 32;                   // W2 (or W2^T) fragments of one wave: 4 M-tiles x 8 K steps
constexpr int MAX_H = 64;                // window length bound
constexpr int MAX_S = 4;                 // RK4 substeps per control step bound
constexpr int MODE_EXTERNAL = 0, MODE_MEAN = 2, MODE_SAMPLE = 3;

// Fragment arrays of one network, in 64-lane fragments of 16 bytes per lane.
constexpr int F_W1 = 0;                  // [16 M-tiles] W1, K = the 32 (padded) inputs
constexpr int F_W2 = F_W1 + 16;          // [16 M-tiles][8 K steps] W2
constexpr int F_W3 = F_W2 + 128;         // [8 K steps] W3 (M = 16 output rows)
constexpr int F_W3T = F_W3 + 8;          // [16 M-tiles] W3^T (K = the output rows)
constexpr int F_W2T = F_W3T + 16;        // [16 M-tiles][8 K steps] W2^T
constexpr int F_W1T = F_W2T + 128;       // [2 M-tiles][8 K steps] W1^T (M = the 32 inputs)
constexpr int F_END = F_W1T + 16;

struct NetF {
  const bf16x8* f;   // fragments (F_END x 64)
  const float* b;    // b1[256] b2[256] b3[n_out]
  int n_out;
};

struct WinArgs {
  int steps, want_grad, has_val;
  uint32_t step0;                      // Philox counter word of the first action
  float inv_nh;                        // 1 / (N h)
  float gamma;
  NetF pol, val;
  const float* log_std;
  // per lane of the four-lane layout, [..][group][lane]: rec [h][substeps][4 RK4 stages] (q, v,
  // omega, and p in the first, 1 / |q| in the last), obk [h] (dpb, rotation vector, sk, kn), aa [h]
  // (action components c and 3 + c before clipping, their moving averages before the step)
  f32x4 *rec, *obk, *aa;
  float *J, *Jr, *vl;
  f32x4* h2s;                          // policy hidden-2 activations [h][G][wave][M-tile][lane]
  u32x2 *h1_half, *dz2_half;
  int groups;                          // groups of 16 environments
  const float* ext;
  float *o_obs, *o_act, *o_reward, *o_done, *o_gact, *o_vlast, *o_gs0;
};

struct Lds {
  bf16x8 W[WAVES][WF][64];    // per wave: its W2 fragments (forward sweep), then its W2^T ones (reverse)
  __bf16 X[WAVES][EPG][16];   // per wave: layer-1 inputs of the 16 environments (12 used, the rest zero)
  __bf16 G[WAVES][EPG][8];    // per wave: q(dL/dy)
  float Y[2][WAVES][EPG][8];  // output partials of each wave (two buffers, alternate steps)
  bf16x8 DZ[8][64];           // a B operand of all 256 hidden features (K step s: 32 s ..): hidden 1
                              // (forward), q(dz2) (reverse)
  float GX[WAVES][EPG][16];   // input-gradient partials of each wave (inputs 0..15)
  float pw[MAX_H + 1];        // gamma^t
  float2 NZ[2][4][64];        // [step group t / 4, alternate][step][physics lane] action noise
};
static_assert(sizeof(Lds) <= 160 * 1024, "window kernel LDS exceeds a CU's 160 KB");

// Hidden-2 activations (fp32) of one wave and step, kept by the forward for the backward:
// [M-tile m][lane], features 64 w + 16 m + 4 g + i of environment r, 4 KB.
constexpr int H2_F4 = 4 * 64;

// ------------------------------------------------------------------ fragments ---------
// blockIdx.y selects the network: 0 the policy (w, n_out, out), 1 the value net (w1, n_out1,
// out1), so that both are rearranged in one launch.
__global__ __launch_bounds__(256) void k_frags(const uint16_t* __restrict__ w0, int n_out0, bf16x8* __restrict__ out0,
                                               const uint16_t* __restrict__ w1, int n_out1, bf16x8* __restrict__ out1) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= F_END * 64) return;
  const uint16_t* w = blockIdx.y ? w1 : w0;
  const int n_out = blockIdx.y ? n_out1 : n_out0;
  bf16x8* out = blockIdx.y ? out1 : out0;
  const int f = e >> 6, lane = e & 63, g = lane >> 4, r = lane & 15;
  const uint16_t* W1 = w;
  const uint16_t* W2 = w + HID * 23;
  const uint16_t* W3 = W2 + HID * HID;
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = kslot(g, j);
    uint16_t bits = 0;
    if (f < F_W2) {
      const int mt = f - F_W1;
      bits = k < 23 ? W1[(16 * mt + r) * 23 + k] : 0;
    } else if (f < F_W3) {
      const int mt = (f - F_W2) >> 3, ks = (f - F_W2) & 7;
      bits = W2[(16 * mt + r) * HID + 32 * ks + k];
    } else if (f < F_W3T) {
      const int ks = f - F_W3;
      bits = r < n_out ? W3[r * HID + 32 * ks + k] : 0;
    } else if (f < F_W2T) {
      const int mt = f - F_W3T;
      bits = k < n_out ? W3[k * HID + 16 * mt + r] : 0;
    } else if (f < F_W1T) {
      const int mt = (f - F_W2T) >> 3, ks = (f - F_W2T) & 7;
      bits = W2[(32 * ks + k) * HID + 16 * mt + r];
    } else {
      const int mt = (f - F_W1T) >> 3, ks = (f - F_W1T) & 7;
      const int in = 16 * mt + r;
      bits = in < 23 ? W1[(32 * ks + k) * 23 + in] : 0;
    }
    v[j] = bf16_of_bits(bits);
  }
  out[e] = v;
}

// ------------------------------------------------------------------ network pieces ----
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }

// biases rows r0 .. r0 + 3, times 2 log2 e (the argument scaling of tanh_bias)
__device__ __forceinline__ f32x4 bias_k(const float* b, int r0) {
  const f32x4 v = *reinterpret_cast<const f32x4*>(b + r0);
  return v * TWO_LOG2E;
}

__device__ __forceinline__ bf16x8 pack8(const f32x4& a, const f32x4& b) {
  bf16x8 f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[i] = (__bf16)a[i];
    f[4 + i] = (__bf16)b[i];
  }
  return f;
}

__device__ __forceinline__ bf16x8 join2(u32x2 a, u32x2 b) {
  return __builtin_bit_cast(bf16x8, (uint32_t __attribute__((ext_vector_type(4)))){a.x, a.y, b.x, b.y});
}

__device__ __forceinline__ bf16x8 fr(const NetF& N, int idx, int lane) { return N.f[idx * 64 + lane]; }

// Exchange between the lanes of one wave through LDS: the LDS operations of a wave complete
// in the order they are issued, so this needs only that the compiler keep the accesses in
// program order (a wavefront-scope fence and wave barrier).
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exchange between the waves of the workgroup: every wave's LDS writes before the barrier are
// seen by every wave after it.  The fences cover LDS only, so the barrier does not wait for
// the waves' outstanding global stores.
__device__ __forceinline__ void wg_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The small weights of wave w's features, loaded once per sweep so that the loops issue no
// weight loads: for the forward, its W1 rows (M-tiles 4w .. 4w + 3), their layer-1 and
// layer-2 biases (times 2 log2 e; lane (g, r): rows 16 m + 4 g .. + 3) and its two K steps of
// W3; for the backward, its W3^T M-tiles, its W1 rows and layer-1 biases, and its two K steps
// of W1^T (M-tile 0: inputs 0..15).
struct OwnF {
  bf16x8 w1[4], w3[2];
  f32x4 b1[4], b2[4];
};
struct OwnB {
  bf16x8 w3t[4], w1[4], w1t[2];
  f32x4 b1[4];
};

__device__ __forceinline__ OwnF own_fwd(const NetF& N, int w, int lane) {
  const int g = lane >> 4;
  OwnF o;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    o.w1[m] = fr(N, F_W1 + 4 * w + m, lane);
    o.b1[m] = bias_k(N.b, 64 * w + 16 * m + 4 * g);
    o.b2[m] = bias_k(N.b + HID, 64 * w + 16 * m + 4 * g);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) o.w3[j] = fr(N, F_W3 + 2 * w + j, lane);
  return o;
}

__device__ __forceinline__ OwnB own_bwd(const NetF& N, int w, int lane) {
  const int g = lane >> 4;
  OwnB o;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    o.w3t[m] = fr(N, F_W3T + 4 * w + m, lane);
    o.w1[m] = fr(N, F_W1 + 4 * w + m, lane);
    o.b1[m] = bias_k(N.b, 64 * w + 16 * m + 4 * g);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) o.w1t[j] = fr(N, F_W1T + 2 * w + j, lane);
  return o;
}

// Wave w's part of the forward pass.  Layer 1 of its 64 features goes to the other waves
// through S.DZ (the K steps 2w, 2w + 1 of layer 2's B operand); then its hidden-2
// activations h2[m] (fp32 after tanh; lane (g, r): features 64 w + 16 m + 4 g + i of
// environment r) and, returned, its partial of the outputs over those 64 features (lane
// (g, r): rows 4 g .. 4 g + 3).  w2: the wave's 32 W2 fragments [M-tile m][K step s] (in
// LDS, or the network's array in global memory).
__device__ __forceinline__ f32x4 mlp_forward(const OwnF& O, const bf16x8* w2, const bf16x8& X, int w, int lane,
                                             Lds& S, f32x4 h2[4]) {
#pragma unroll
  for (int j = 0; j < 2; ++j)
    S.DZ[2 * w + j][lane] = act_frag(mfma(O.w1[2 * j], X, zero4()), mfma(O.w1[2 * j + 1], X, zero4()),
                                     O.b1[2 * j], O.b1[2 * j + 1]);
  wg_sync();
  bf16x8 H1[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) H1[s] = S.DZ[s][lane];
  f32x4 z[4] = {zero4(), zero4(), zero4(), zero4()};
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int m = 0; m < 4; ++m) z[m] = mfma(w2[(8 * m + s) * 64 + lane], H1[s], z[m]);
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) h2[m][i] = tanh_bias(z[m][i], O.b2[m][i]);
  const f32x4 y = mfma(O.w3[0], pack8(h2[0], h2[1]), zero4());
  return mfma(O.w3[1], pack8(h2[2], h2[3]), y);
}

// The 0/1 selection operand: as B with a feature-major pair as A (lane (g, r): features
// 16 (j / 4) + 4 g + j % 4 of sample r) it gives lane (g, r) feature 16 hf + r at samples
// 4 g .. 4 g + 3, the half-fragment layout (exact: one nonzero product per output).
__device__ __forceinline__ bf16x8 select_frag(int g, int r, int hf) {
  bf16x8 f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = (__bf16)((g == (r >> 2) && j == 4 * hf + (r & 3)) ? 1.0f : 0.0f);
  return f;
}

__device__ __forceinline__ u32x2 pack4(const f32x4& v) {
  bf16x4 q;
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = (__bf16)v[i];
  return __builtin_bit_cast(u32x2, q);
}

__device__ __forceinline__ bf16x8 low_half(u32x2 a) { return join2(a, u32x2{0u, 0u}); }

// A wave's sums over its workgroup's samples of the small weight gradients of its 64 features
// (M-tiles m; lane (g, r): rows 16 m + 4 g + i): dW1 (column r: input r, column ONES: db1), the
// same product with q(dz2) (only its column ONES, db2, is used) and dW3^T (column r: output r);
// and db3 (lane (g, r): output r over samples 4 g .. + 3 of every tile).
constexpr int ONES = 12;   // the first padding input of the 12-input policy, set to 1 in the products' q(x)
struct SmallGrads {
  f32x4 w1[4], z2[4], w3[4];
  float b3;
};

// Where the reverse sweep writes the operands of dW2 of one step, and its small sums.
struct HalfOut {
  u32x2 *h1, *dz2;
  size_t tile;       // the workgroup's sample tile of this step
  bool on;           // a gradient is wanted
  bf16x8 sel[2];     // select_frag
};

// Wave w's part of the backward pass from q(dL/dy) (GY, B operand with K = the output rows),
// the layer-1 operand X and the wave's hidden-2 activations h2: dz2 of its features, given
// to the other waves through LDS; dz1 = (W2^T q(dz2)) (1 - h1^2) of its hidden-1 features
// (h1 recomputed from X); its partial of the input gradient W1^T q(dz1), and the sum of the
// four waves' partials in wave order, gxo (inputs c, 3 + c, 6 + c, 9 + c of environment lane / 4,
// c = min(lane mod 4, 2)).  With
// H.on it also stores q(dz2) and q(h1) of its features as half fragments and adds the
// step's share of the small weight gradients.  w2t: the wave's 32 W2^T
// fragments [M-tile m][K step s].
__device__ __forceinline__ void mlp_backward(const OwnB& O, const bf16x8* w2t, const bf16x8& X, const bf16x8& GY,
                                             const f32x4 h2[4], int w, int lane, Lds& S, const HalfOut& H,
                                             SmallGrads& sums, float gxo[4]) {
  const int g = lane >> 4, r = lane & 15;
  // hidden 2 (this wave's features): dz2 = (W3^T q(gy)) (1 - h2^2)
  f32x4 d[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    d[m] = mfma(O.w3t[m], GY, zero4());
#pragma unroll
    for (int i = 0; i < 4; ++i) d[m][i] *= 1.0f - h2[m][i] * h2[m][i];
  }
  const bf16x8 pd[2] = {pack8(d[0], d[1]), pack8(d[2], d[3])};
  S.DZ[2 * w][lane] = pd[0];
  S.DZ[2 * w + 1][lane] = pd[1];
  bf16x8 xh;
  if (H.on) {
    const bf16x4 one = {(__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f};
    u32x2 xq = pack4(mfma(X, H.sel[0], zero4()));
    if (r == ONES) xq = __builtin_bit_cast(u32x2, one);
    xh = low_half(xq);
    const f32x4 gyv = mfma(GY, H.sel[0], zero4());   // exact: bf16 values
    const bf16x8 gyh = low_half(pack4(gyv));
    sums.b3 += (gyv[0] + gyv[1]) + (gyv[2] + gyv[3]);
    const bf16x8 ph[2] = {pack8(h2[0], h2[1]), pack8(h2[2], h2[3])};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bf16x8 h2h = low_half(pack4(mfma(ph[m >> 1], H.sel[m & 1], zero4())));
      sums.w3[m] = mfma(h2h, gyh, sums.w3[m]);
      const u32x2 dh = pack4(mfma(pd[m >> 1], H.sel[m & 1], zero4()));
      H.dz2[(H.tile * 16 + 4 * w + m) * 64 + lane] = dh;
      sums.z2[m] = mfma(low_half(dh), xh, sums.z2[m]);
    }
  }
  wg_sync();
  // hidden 1 (this wave's features): dz1 = (W2^T q(dz2)) (1 - h1^2), h1 recomputed
  bf16x8 dz[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) dz[s] = S.DZ[s][lane];
  f32x4 e[4] = {zero4(), zero4(), zero4(), zero4()};
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int m = 0; m < 4; ++m) e[m] = mfma(w2t[(8 * m + s) * 64 + lane], dz[s], e[m]);
  f32x4 k[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const f32x4 y = mfma(O.w1[m], X, zero4());
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      k[m][i] = tanh_bias(y[i], O.b1[m][i]);
      e[m][i] *= 1.0f - k[m][i] * k[m][i];
    }
  }
  // input gradient: the partial over this wave's hidden-1 features (M-tile 0: inputs 0..15)
  const bf16x8 pe[2] = {pack8(e[0], e[1]), pack8(e[2], e[3])};
  const f32x4 gx = mfma(O.w1t[1], pe[1], mfma(O.w1t[0], pe[0], zero4()));
  *reinterpret_cast<f32x4*>(&S.GX[w][r][4 * g]) = gx;
  if (H.on) {
    const bf16x8 pk[2] = {pack8(k[0], k[1]), pack8(k[2], k[3])};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      H.h1[(H.tile * 16 + 4 * w + m) * 64 + lane] = pack4(mfma(pk[m >> 1], H.sel[m & 1], zero4()));
      const bf16x8 eh = low_half(pack4(mfma(pe[m >> 1], H.sel[m & 1], zero4())));
      sums.w1[m] = mfma(eh, xh, sums.w1[m]);
    }
  }
  wg_sync();
  const int slot = lane >> 2, c = min(lane & 3, 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float s = S.GX[0][slot][3 * j + c];
#pragma unroll
    for (int v = 1; v < WAVES; ++v) s += S.GX[v][slot][3 * j + c];
    gxo[j] = s;
  }
}

// The wave's 32 fragments of a network's array, starting at fragment `first`, into its LDS slice.
__device__ __forceinline__ void fill_w(Lds& S, const NetF& N, int first, int w, int lane) {
  lds_sync();   // earlier readers of the slice (this wave) are done
#pragma unroll 8
  for (int f = 0; f < WF; ++f) S.W[w][f][lane] = N.f[(first + f) * 64 + lane];
  lds_sync();
}

// ---------------------------------------------------------- lane <-> fragment moves ----
// The 12 inputs (bf16) of the wave's 16 environments into its S.X, lanes c < 3 of each quad
// writing inputs c, 3 + c, 6 + c, 9 + c (the others were zeroed at the start).
__device__ __forceinline__ void put_inputs(Lds& S, int w, int lane, float dpb, float rv, float v, float om) {
  const int slot = lane >> 2, c = lane & 3;
  if (c == 3) return;
  __bf16* x = &S.X[w][slot][c];
  x[0] = (__bf16)dpb;
  x[3] = (__bf16)rv;
  x[6] = (__bf16)v;
  x[9] = (__bf16)om;
}

__device__ __forceinline__ bf16x8 input_frag(const Lds& S, int w, int lane) {
  const int g = lane >> 4, r = lane & 15;
  return join2(*reinterpret_cast<const u32x2*>(&S.X[w][r][4 * g]), u32x2{0u, 0u});
}

// q(dL/dy) of the wave's 16 environments into its S.G: lanes c < 3 of each quad write rows c and
// 3 + c (rows 6, 7 were zeroed at the start).
__device__ __forceinline__ void put_gy(Lds& S, int w, int lane, float g0, float g1) {
  const int slot = lane >> 2, c = lane & 3;
  if (c == 3) return;
  S.G[w][slot][c] = (__bf16)g0;
  S.G[w][slot][3 + c] = (__bf16)g1;
}

__device__ __forceinline__ bf16x8 gy_frag(const Lds& S, int w, int lane) {
  const int g = lane >> 4, r = lane & 15;
  const u32x2 lo = g < 2 ? *reinterpret_cast<const u32x2*>(&S.G[w][r][4 * g]) : u32x2{0u, 0u};
  return join2(lo, u32x2{0u, 0u});
}

// Output row j of environment r: the waves' partials summed in wave order.
__device__ __forceinline__ float out_sum(const Lds& S, int b, int r, int j) {
  float s = S.Y[b][0][r][j];
#pragma unroll
  for (int v = 1; v < WAVES; ++v) s += S.Y[b][v][r][j];
  return s;
}

// ------------------------------------------------------------------ environment --------
// This lane's model constants (component c of each triple, zero in lane 3): no current, weight
// gamma W (gamma in parameter row 13), buoyancy centre at the centre of gravity.
__device__ __forceinline__ qadj::QM<float> model_of(const VehArgs& V, const Params& P, const quad::QK& Q) {
  Model S;
  make_model(V, P, S);
  auto at = [&](const float* x) { return quad::pick(Q, x[0], x[1], x[2], 0.0f); };
  qadj::QM<float> M;
  M.Ml = at(S.Mlin);
  M.iMl = at(S.iMlin);
  M.Ma = at(S.Mang);
  M.iMa = at(S.iMang);
  M.A1 = at(S.A1);
  M.DLi = at(S.DL) * M.iMl;
  M.DQi = at(S.DQ) * M.iMl;
  M.BmWi = __builtin_fmaf(-P.amp[0], V.W, V.B) * M.iMl;
  M.DLa = at(S.DL + 3);
  M.DQa = at(S.DQ + 3);
  qadj::derive(M);
  return M;
}

// Noise of the sampled actions c and 3 + c at one step: the Box-Muller pair of words
// (2c, 2c + 1) of counter (global id, step, 2, block); zero in lane 3.
__device__ __forceinline__ void paper_noise(const EnvArgs& E, uint32_t gid, uint32_t step, int c, float& e0, float& e1) {
  const U4 b = philox(U4{gid, step, 2u, (uint32_t)(c >> 1)}, E.key0, E.key1);
  const uint32_t w0 = (c & 1) ? b.z : b.x, w1 = (c & 1) ? b.w : b.y;
  const float rad = sqrtf(-2.0f * logf(u01_open0(w0)));
  float sn, cs;
  sincos_turns(u01(w1), &sn, &cs);
  e0 = c < 3 ? rad * cs : 0.0f;
  e1 = c < 3 ? rad * sn : 0.0f;
}

// ------------------------------------------------------------------ window kernel ------
template <int MODE>
__global__ __launch_bounds__(64 * WAVES, 1) void k_window(EnvArgs E, VehArgs V, WinArgs A, GradParts P_) {
  __shared__ Lds S;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;      // lane of the MFMA layouts
  const int slot = lane >> 2, c = lane & 3;    // lane of the four-lane physics
  const quad::QK Q = quad::make_qk(lane);
  const qadj::LaneK<float> K{Q.m3, 1.0f - Q.m3, Q.e1, Q.e2, Q.d2};
  const int N = E.n;
  const size_t Nz = (size_t)N;
  const int h = A.steps;
  if (threadIdx.x <= MAX_H) S.pw[threadIdx.x] = powf(A.gamma, (float)threadIdx.x);
  for (int k = threadIdx.x; k < WAVES * EPG * 16; k += 64 * WAVES) (&S.X[0][0][0])[k] = (__bf16)0.0f;
  for (int k = threadIdx.x; k < WAVES * EPG * 8; k += 64 * WAVES) (&S.G[0][0][0])[k] = (__bf16)0.0f;
  SmallGrads sums;
#pragma unroll
  for (int m = 0; m < 4; ++m) sums.w1[m] = sums.z2[m] = sums.w3[m] = zero4();
  sums.b3 = 0.0f;
  HalfOut H{A.h1_half, A.dz2_half, 0, MODE != MODE_EXTERNAL && A.want_grad,
            {select_frag(g, r, 0), select_frag(g, r, 1)}};
  float gls0 = 0.0f, gls1 = 0.0f;   // d log sigma of actions c and 3 + c
  const size_t G = (size_t)A.groups;

  // one group of 16 environments after another (a workgroup's LDS fills its CU, so groups past
  // the CUs would run in turn anyway; the small gradients' sums stay in registers)
#pragma unroll 1
  for (int grp = blockIdx.x; grp < A.groups; grp += gridDim.x) {
  const int i = grp * EPG + slot;
  const bool valid = i < N;
  const int ic = valid ? i : N - 1;            // idle slots step a copy of the last environment
  const uint32_t gid = E.env_offset + (uint32_t)i;
  // the networks as this group reads them: loads not hoisted out of the loop over groups, where
  // both sweeps' weights would be live at once
  NetF pol = A.pol, val = A.val;
  asm volatile("" : "+s"(pol.f), "+s"(pol.b), "+s"(val.f), "+s"(val.b));
  // wave 0 writes the state's results, wave 1 the recorded observations, wave 2 the actions and
  // their gradients, wave 3 rewards and done flags (every wave holds all of them)
  const bool w_obs = w == 1 && valid && A.o_obs, w_act = w == 2 && valid && A.o_act;
  const bool w_gact = w == 2 && valid && A.o_gact, w_rew = w == 3 && valid && c == 0;

  wg_sync();   // LDS set up, or the group before done with it

  // environment of this quad: row k of a 3-vector in lanes c < 3, zero in lane 3
  auto row3 = [&](const float* p, int k) { return c < 3 ? p[(size_t)(k + min(c, 2)) * Nz + ic] : 0.0f; };
  float p = row3(E.state, 0);
  qadj::QX<float> x{E.state[(size_t)(c < 3 ? 4 + c : 3) * Nz + ic], row3(E.state, 7), row3(E.state, 10)};
  Params P;
  load_params(E.params, N, ic, P);
  const qadj::QM<float> M = model_of(V, P, Q);
  const float pg = quad::pick(Q, P.pg[0], P.pg[1], P.pg[2], 0.0f);
  const float qg = quad::pick(Q, P.qg[1], P.qg[2], P.qg[3], P.qg[0]);
  const int ep = E.ep_step[ic];
  const uint32_t episode = E.episode[ic];
  float ab0 = row3(E.obs, 12), ab1 = row3(E.obs, 15);
  const bool ends = ep + h == E.H;
  const TaskArgs& tk = E.tk;
  const float dc = quad::pick(Q, tk.d_pos[0], tk.d_pos[1], tk.d_pos[2], 0.0f);
  float sig0 = 0.0f, sig1 = 0.0f, b30 = 0.0f, b31 = 0.0f;
  if (c < 3) {
    if (MODE == MODE_SAMPLE) {
      sig0 = expf(A.log_std[c]);
      sig1 = expf(A.log_std[3 + c]);
    }
    if (MODE != MODE_EXTERNAL) {
      b30 = pol.b[2 * HID + c];
      b31 = pol.b[2 * HID + 3 + c];
    }
  }
  // where this workgroup's lanes keep the forward sweep's records
  const size_t at0 = (size_t)grp * 64 + lane;
  auto rec_at = [&](int t, int s, int stage) { return A.rec + (((size_t)t * E.substeps + s) * 4 + stage) * G * 64 + at0; };
  auto row_at = [&](f32x4* a, int t) { return a + (size_t)t * G * 64 + at0; };
  // Action noise, four steps at a time: wave w draws that of step t - t % 4 + w for every wave (each
  // drawing all of it for itself, a Philox block and a Box-Muller pair per step and sweep, 4096
  // environments x 32 steps with the actor's step took 390 us, so 384).  Read after the step's next barrier.
  auto deal_noise = [&](int t) {
    float e0, e1;
    paper_noise(E, gid, A.step0 + (uint32_t)((t & ~3) + w), c, e0, e1);
    S.NZ[(t >> 2) & 1][w][lane] = float2{e0, e1};
  };
  auto noise_at = [&](int t) { return S.NZ[(t >> 2) & 1][t & 3][lane]; };
  auto h2_at = [&](int t) { return A.h2s + (((size_t)t * G + grp) * WAVES + w) * H2_F4 + lane; };

  // ---------------------------------------------------------------- forward sweep
  OwnF of{};
  if (MODE != MODE_EXTERNAL) {
    fill_w(S, pol, F_W2 + WF * w, w, lane);
    of = own_fwd(pol, w, lane);
  }
  float Jr = 0.0f;
  qadj::QObsK<float> o = qadj::observe(K, p, x.q, pg, qg);
  for (int t = 0; t < h; ++t) {
    float a0, a1;
    if (MODE == MODE_EXTERNAL) {
      a0 = c < 3 ? A.ext[((size_t)c * h + t) * Nz + ic] : 0.0f;
      a1 = c < 3 ? A.ext[((size_t)(3 + c) * h + t) * Nz + ic] : 0.0f;
    } else {
      lds_sync();
      put_inputs(S, w, lane, o.dpb, o.rv, x.v, x.w);
      lds_sync();
      const bf16x8 X = input_frag(S, w, lane);
      f32x4 h2[4];
      const f32x4 y = mlp_forward(of, &S.W[w][0][0], X, w, lane, S, h2);
      f32x4* hs = h2_at(t);
#pragma unroll
      for (int m = 0; m < 4; ++m) hs[m * 64] = h2[m];
      const int b = t & 1;
      if (g < 2) *reinterpret_cast<f32x4*>(&S.Y[b][w][r][4 * g]) = y;
      if (MODE == MODE_SAMPLE && (t & 3) == 0) deal_noise(t);
      wg_sync();
      a0 = c < 3 ? out_sum(S, b, slot, min(c, 2)) + b30 : 0.0f;
      a1 = c < 3 ? out_sum(S, b, slot, 3 + min(c, 2)) + b31 : 0.0f;
      if (MODE == MODE_SAMPLE) {
        const float2 e = noise_at(t);
        a0 = __builtin_fmaf(sig0, e.x, a0);
        a1 = __builtin_fmaf(sig1, e.y, a1);
      }
    }
    if (w == 0) {
      *row_at(A.aa, t) = f32x4{a0, a1, ab0, ab1};
    } else if (w == 1) {
      *row_at(A.obk, t) = f32x4{o.dpb, o.rv, o.sk, o.kn};
    }
    const size_t at = (size_t)t * Nz + i, rs = (size_t)h * Nz;
    if (w_obs) {
      if (c < 3) {
        A.o_obs[c * rs + at] = o.dpb;
        A.o_obs[(3 + c) * rs + at] = o.rv;
        A.o_obs[(6 + c) * rs + at] = x.v;
        A.o_obs[(9 + c) * rs + at] = x.w;
      }
#pragma unroll
      for (int k = 12; k < 24; k += 4)
        if (k + c < 23) A.o_obs[(k + c) * rs + at] = 0.0f;
    }
    if (w_act) {
      if (c < 3) {
        A.o_act[c * rs + at] = a0;
        A.o_act[(3 + c) * rs + at] = a1;
      } else {
        A.o_act[6 * rs + at] = 0.0f;
        A.o_act[7 * rs + at] = 0.0f;
      }
    }
    const float u0 = fminf(fmaxf(a0, -1.0f), 1.0f), u1 = fminf(fmaxf(a1, -1.0f), 1.0f);
    const float tfi = tk.f_max * u0 * M.iMl, tm = tk.tau_max * u1;
    for (int s = 0; s < E.substeps; ++s) {
      qadj::QX<float> st[4];
      float inv;
      const float p0 = p;
      qadj::substep(K, M, tfi, tm, E.h, p, x, st, inv);
      // wave w stores stage w's input
      auto mine = [&](float s0, float s1, float s2, float s3) { return w == 0 ? s0 : (w == 1 ? s1 : (w == 2 ? s2 : s3)); };
      *rec_at(t, s, w) = f32x4{mine(st[0].q, st[1].q, st[2].q, st[3].q), mine(st[0].v, st[1].v, st[2].v, st[3].v),
                               mine(st[0].w, st[1].w, st[2].w, st[3].w), w == 0 ? p0 : inv};
    }
    o = qadj::observe(K, p, x.q, pg, qg);
    const quad::QObs ob{o.dpb, o.rv, 0.0f};
    const float rw = quad::paper_reward(tk, dc, ob, x.w, u0, u1, ab0, ab1);
    ab0 = __builtin_fmaf(tk.beta, ab0, (1.0f - tk.beta) * u0);
    ab1 = __builtin_fmaf(tk.beta, ab1, (1.0f - tk.beta) * u1);
    Jr = __builtin_fmaf(S.pw[t], rw, Jr);
    if (w_rew) {
      if (A.o_reward) A.o_reward[at] = rw;
      if (A.o_done) A.o_done[at] = (t == h - 1 && ends) ? 1.0f : 0.0f;
    }
  }
  __syncthreads();   // the waves' records are read by every wave in the reverse sweep

  // ------------------------------------------------ terminal value, its input gradient
  float go[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // cotangents of dpb, rotation vector, v, omega
  float vlast = 0.0f;
  if (A.has_val) {
    lds_sync();
    put_inputs(S, w, lane, o.dpb, o.rv, x.v, x.w);
    put_gy(S, w, lane, (valid && c == 0) ? -S.pw[h] * A.inv_nh : 0.0f, 0.0f);
    lds_sync();
    const bf16x8 X = input_frag(S, w, lane), GY = gy_frag(S, w, lane);
    f32x4 h2[4];
    const f32x4 y = mlp_forward(own_fwd(val, w, lane), val.f + (size_t)(F_W2 + WF * w) * 64, X, w, lane, S, h2);
    const int b = h & 1;
    if (g < 2) *reinterpret_cast<f32x4*>(&S.Y[b][w][r][4 * g]) = y;
    wg_sync();
    vlast = out_sum(S, b, slot, 0) + val.b[2 * HID];
    HalfOut off = H;
    off.on = false;
    mlp_backward(own_bwd(val, w, lane), val.f + (size_t)(F_W2T + WF * w) * 64, X, GY, h2, w, lane, S, off, sums, go);
  }

  // ------------------------------------------- environment update (reset at the episode end)
  if (w == 0 && valid) {
    quad::QEnv X;
    X.p = p;
    X.q = x.q;
    X.v = x.v;
    X.om = x.w;
    X.u0 = ab0;
    X.u1 = ab1;
    X.ep = ep + h;
    X.episode = episode;
    X.ob = quad::QObs{o.dpb, o.rv, 0.0f};
    // non-finite components of the window's end state, before any reset
    report_status(E.status, quad::nonfinite_quad(c, X), 0u);
    if (ends) {
      quad::QModel Mn;
      quad::QRef Fn;
      quad::QRefCols rc;
      float prn, qrn, dist;
      quad::new_episode<true>(V, E, Q, gid, i, true, X, Mn, Fn, prn, qrn, rc, dist);
    }
    quad::store_state(E.state, Nz, (size_t)i, c, X);
    if (c < 3) {
      E.obs[c * Nz + i] = X.ob.dpb;
      E.obs[(3 + c) * Nz + i] = X.ob.c0;
      E.obs[(6 + c) * Nz + i] = X.v;
      E.obs[(9 + c) * Nz + i] = X.om;
      E.obs[(12 + c) * Nz + i] = X.u0;
      E.obs[(15 + c) * Nz + i] = X.u1;
    }
    if (c == 0) {
      E.ep_step[i] = X.ep;
      E.episode[i] = X.episode;
      if (A.o_vlast) A.o_vlast[i] = vlast;
    }
  }

  // ---------------------------------------------------------------- reverse sweep
  OwnB ob{};
  if (MODE != MODE_EXTERNAL) {
    fill_w(S, pol, F_W2T + WF * w, w, lane);
    ob = own_bwd(pol, w, lane);
  }
  float lp = 0.0f;
  qadj::QX<float> l{0.0f, 0.0f, 0.0f};
  // Cotangents of the observation at one point of the trajectory, the network's in go, those of
  // the reward r_t that it enters added (weight -gamma^t / (N h)), through the observation.
  auto through_obs = [&](int t, float cr, const qadj::QObsK<float>& ok, float pp, const qadj::QX<float>& xx) {
    if (t >= 0) {
      go[0] -= 2.0f * cr * tk.w_pos * dc * dc * ok.dpb;
      go[1] -= 2.0f * cr * tk.w_att * ok.rv;
      go[3] -= 2.0f * cr * tk.w_vel * xx.w;
    }
    go[0] *= K.m3;
    go[1] *= K.m3;
    qadj::observe_vjp(K, pp, xx.q, pg, qg, ok.sk, ok.kn, go[0], go[1], lp, l.q);
    l.v += K.m3 * go[2];
    l.w += K.m3 * go[3];
  };
  float cr = valid ? -S.pw[h - 1] * A.inv_nh : 0.0f;   // weight of the reward r_t being taken backward
  through_obs(h - 1, cr, o, p, x);
  float qn = x.q;                                        // the quaternion at the end of the substep
  float la0 = 0.0f, la1 = 0.0f;
  f32x4 rs[4];                                           // the substep's stage records, loaded one substep ahead
#pragma unroll
  for (int k = 0; k < 4; ++k) rs[k] = *rec_at(h - 1, E.substeps - 1, k);
  for (int t = h - 1; t >= 0; --t) {
    f32x4 h2[4];
    if (MODE != MODE_EXTERNAL) {   // issued first: the loads complete during the state adjoint
      const f32x4* hs = h2_at(t);
#pragma unroll
      for (int m = 0; m < 4; ++m) h2[m] = hs[m * 64];
    }
    const f32x4 aa = *row_at(A.aa, t), okv = *row_at(A.obk, t);
    const float u0 = fminf(fmaxf(aa.x, -1.0f), 1.0f), u1 = fminf(fmaxf(aa.y, -1.0f), 1.0f);
    // RK4 substeps in reverse; one copy of the adjoint in the loop keeps the code within the
    // instruction cache
    float gtf = 0.0f, gtm = 0.0f, pt = 0.0f;
    qadj::QX<float> x0{};
#pragma unroll 1
    for (int s = E.substeps - 1; s >= 0; --s) {
      f32x4 nx[4];
      const int tn = s > 0 ? t : max(t - 1, 0), sn = s > 0 ? s - 1 : (t > 0 ? E.substeps - 1 : 0);
#pragma unroll
      for (int k = 0; k < 4; ++k) nx[k] = *rec_at(tn, sn, k);
      qadj::QX<float> st[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) st[k] = qadj::QX<float>{rs[k].x, rs[k].y, rs[k].z};
      qadj::substep_vjp(K, M, E.h, st, rs[3].w, qn, lp, l, gtf, gtm);
      qn = st[0].q;
      x0 = st[0];
      pt = rs[0].w;
#pragma unroll
      for (int k = 0; k < 4; ++k) rs[k] = nx[k];
    }
    // reward terms of the action and abar_{t+1} = beta abar_t + (1 - beta) u_t
    const float m0 = 2.0f * cr * tk.w_mavg * (u0 - aa.z), m1 = 2.0f * cr * tk.w_mavg * (u1 - aa.w);
    const float gu0 = (1.0f - tk.beta) * la0 - m0 + tk.f_max * gtf;
    const float gu1 = (1.0f - tk.beta) * la1 - m1 - 2.0f * cr * tk.w_act * u1 + tk.tau_max * gtm;
    la0 = __builtin_fmaf(tk.beta, la0, m0);
    la1 = __builtin_fmaf(tk.beta, la1, m1);
    // clip: the derivative passes on [-1, 1]
    const float ga0 = (c < 3 && aa.x >= -1.0f && aa.x <= 1.0f) ? gu0 : 0.0f;
    const float ga1 = (c < 3 && aa.y >= -1.0f && aa.y <= 1.0f) ? gu1 : 0.0f;
    if (w_gact) {
      const size_t at = (size_t)t * Nz + i, rs_ = (size_t)h * Nz;
      if (c < 3) {
        A.o_gact[c * rs_ + at] = ga0;
        A.o_gact[(3 + c) * rs_ + at] = ga1;
      } else {
        A.o_gact[6 * rs_ + at] = 0.0f;
        A.o_gact[7 * rs_ + at] = 0.0f;
      }
    }
    go[0] = go[1] = go[2] = go[3] = 0.0f;
    const qadj::QObsK<float> ok{okv.x, okv.y, okv.z, okv.w};
    if (MODE != MODE_EXTERNAL) {
      if (MODE == MODE_SAMPLE && ((t & 3) == 3 || t == h - 1)) deal_noise(t);
      // the policy's input gradient at o_t = o(s_t)
      lds_sync();
      put_inputs(S, w, lane, ok.dpb, ok.rv, x0.v, x0.w);
      put_gy(S, w, lane, ga0, ga1);
      lds_sync();
      const bf16x8 X = input_frag(S, w, lane), GY = gy_frag(S, w, lane);
      H.tile = (size_t)t * G + grp;
      mlp_backward(ob, &S.W[w][0][0], X, GY, h2, w, lane, S, H, sums, go);
      if (MODE == MODE_SAMPLE) {   // after the exchanges of the backward pass
        const float2 e = noise_at(t);
        gls0 = __builtin_fmaf(ga0 * sig0, e.x, gls0);
        gls1 = __builtin_fmaf(ga1 * sig1, e.y, gls1);
      }
    }
    cr = (valid && t > 0) ? -S.pw[t > 0 ? t - 1 : 0] * A.inv_nh : 0.0f;
    through_obs(t - 1, cr, ok, pt, x0);
  }
  if (w == 0 && valid && A.o_gs0) {
    if (c < 3) {
      A.o_gs0[c * Nz + i] = lp;
      A.o_gs0[(7 + c) * Nz + i] = l.v;
      A.o_gs0[(10 + c) * Nz + i] = l.w;
    }
    A.o_gs0[(size_t)(c < 3 ? 4 + c : 3) * Nz + i] = l.q;
  }
  if (w == 0 && c == 0) {
    A.J[i] = valid ? __builtin_fmaf(S.pw[h], vlast, Jr) : 0.0f;
    A.Jr[i] = valid ? Jr : 0.0f;
    A.vl[i] = valid ? vlast : 0.0f;
  }
  }

  // ------------------------------------------------ this workgroup's small gradient sums
  if (MODE == MODE_EXTERNAL || !A.want_grad) return;
  const size_t wg = blockIdx.x;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (r < ACT) *reinterpret_cast<f32x4*>(&P_.part_w3[(wg * ACT + r) * HID + 64 * w + 16 * m + 4 * g]) = sums.w3[m];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t f = wg * HID + 64 * w + 16 * m + 4 * g + q;
      P_.part_w1[f * 32 + r] = r < ONES ? sums.w1[m][q] : 0.0f;
      P_.part_w1[f * 32 + 16 + r] = 0.0f;   // inputs 12.. of the paper task are zero
      if (r == ONES) {
        P_.part_b1[f] = sums.w1[m][q];
        P_.part_b2[f] = sums.z2[m][q];
      }
    }
  }
  if (w == 0) {
    float b3 = sums.b3;   // over the lane rows g, in a fixed order
    b3 += __shfl_xor(b3, 16);
    b3 += __shfl_xor(b3, 32);
    if (g == 0) P_.part_b3[wg * 16 + r] = b3;
    float d0 = gls0, d1 = gls1;   // over the wave's 16 environments
#pragma unroll
    for (int o = 4; o < 64; o *= 2) {
      d0 += __shfl_xor(d0, o);
      d1 += __shfl_xor(d1, o);
    }
    if (slot == 0) {
      P_.part_ls[wg * 16 + (c < 3 ? c : 6)] = c < 3 ? d0 : 0.0f;
      P_.part_ls[wg * 16 + (c < 3 ? 3 + c : 7)] = c < 3 ? d1 : 0.0f;
    }
  }
}

// ------------------------------------------------------------------ statistics ---------
// stats: [0] loss, [1] mean over envs of sum_t gamma^t r_t, [2] mean V(o_h), [5] |grad|^2,
// [7] clipping factor min(1, c / (|grad| + 1e-6)) (1 without clipping or without gradient).
// One workgroup of four waves; every sum in a fixed order (thread-strided with four loads in
// flight, then over each wave, then the waves' sums in wave order).
__global__ __launch_bounds__(256) void k_finalize(const float* __restrict__ J, const float* __restrict__ Jr,
                                                  const float* __restrict__ vl, int N, float inv_nh,
                                                  const float* __restrict__ ss, int nss, float max_norm,
                                                  float* __restrict__ stats) {
  __shared__ float part[4][4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  float sj = 0.0f, sr = 0.0f, sv = 0.0f, sg = 0.0f;
#pragma unroll 4
  for (int k = tid; k < N; k += 256) {
    sj += J[k];
    sr += Jr[k];
    sv += vl[k];
  }
#pragma unroll 4
  for (int k = tid; k < nss; k += 256) sg += ss[k];
  const float v[4] = {wave_sum(sj), wave_sum(sr), wave_sum(sv), wave_sum(sg)};
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) part[wv][j] = v[j];
  __syncthreads();
  if (tid == 0) {
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = ((part[0][j] + part[1][j]) + part[2][j]) + part[3][j];
    sj = t[0];
    sr = t[1];
    sv = t[2];
    sg = t[3];
    stats[0] = -sj * inv_nh;
    stats[1] = sr / (float)N;
    stats[2] = sv / (float)N;
    stats[3] = 0.0f;
    stats[4] = 0.0f;
    stats[5] = sg;
    stats[6] = 0.0f;
    stats[7] = (max_norm > 0.0f && nss > 0) ? fminf(1.0f, max_norm / (sqrtf(sg) + 1e-6f)) : 1.0f;
  }
}

__global__ __launch_bounds__(256) void k_zero(uint32_t* __restrict__ p, size_t n) {
  for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) p[k] = 0u;
}

// ------------------------------------------------------------------ workspace ----------
inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr int WORK_PARTS = 17;
constexpr int MAX_GROUPS = 256;

struct Shape {
  int NG, Np, tiles, tiles_p, steps, GW, G3;
};

inline Shape shape_of(int N, int h, int cus) {
  Shape s;
  s.NG = (N + EPG - 1) / EPG;
  s.Np = EPG * s.NG;
  s.tiles = h * s.NG;
  s.tiles_p = (s.tiles + 7) / 8 * 8;     // whole rounds of the dW2 loop (4 steps of 2 tiles)
  s.steps = s.tiles_p / 2;
  s.GW = std::min({MAX_GROUPS, s.NG, cus});   // workgroups of the window
  s.G3 = std::max(1, std::min({MAX_GROUPS, s.steps / 4, cus}));
  return s;
}

inline size_t work_layout(int N, int h, size_t off[WORK_PARTS]) {
  const Shape s = shape_of(N, h, MAX_GROUPS);
  const size_t Np = s.Np, tp = s.tiles_p, G = MAX_GROUPS, half = tp * 64 * 8;
  const size_t sizes[WORK_PARTS] = {
      2 * (size_t)F_END * 64 * 16,          // 0 fragments of the policy and the value net
      (size_t)h * (Np / EPG) * 64 * 16,   // 1 observations with their derivative factors
      (size_t)h * (Np / EPG) * 64 * 16,     // 2 actions and action averages
      Np * 4, Np * 4, Np * 4,               // 3 J, 4 Jr, 5 V(o_h)
      half * 16, half * 16,                 // 6 h1, 7 dz2
      G * HID * 32 * 4, G * HID * 4,        // 8 part_w1, 9 part_b1
      G * ACT * HID * 4, G * HID * 4,       // 10 part_w3, 11 part_b2
      G * 16 * 4 + G * 16 * 4,              // 12 part_b3 + part_ls
      G * HID * HID * 4,                    // 13 part_w2
      4096 * 4,                             // 14 per-block sums of squares
      (size_t)h * (Np / EPG) * WAVES * H2_F4 * 16,   // 15 policy hidden-2 activations
      (size_t)h * MAX_S * 4 * (Np / EPG) * 64 * 16};   // 16 RK4 stage inputs
  size_t o = 0;
  for (int k = 0; k < WORK_PARTS; ++k) {
    off[k] = o;
    o += a256(sizes[k]);
  }
  return o;
}

}  // namespace shac
}  // namespace auv

// ------------------------------------------------------------------ C interface ----
using namespace auv;

extern "C" {

int64_t auv_shac_work_bytes(int32_t n_envs, int32_t h) {
  if (n_envs < 1 || n_envs > (1 << 22) || h < 1 || h > shac::MAX_H) return -1;
  size_t off[shac::WORK_PARTS];
  return (int64_t)shac::work_layout(n_envs, h, off);
}

int auv_shac_window(auv_env* env, const auv_shac_config* cfg, const auv_mlp* policy, const auv_mlp* value,
                    const auv_shac_buffers* out, float* grad_policy, float* stats, void* work, void* stream) {
  using namespace shac;
  if (!env || !cfg || !stats || !work) return set_error(AUV_EINVAL, "auv_shac_window: NULL handle, config, stats or work");
  const int N = env->cfg.n_envs, h = cfg->h, H = env->cfg.episode_len, mode = cfg->mode;
  if (env->E.task != TASK_PAPER) return set_error(AUV_EINVAL, "auv_shac_window: needs the paper task (auv_set_task)");
  if (env->cfg.flags & AUV_F_STAGGER) return set_error(AUV_EINVAL, "auv_shac_window: staggered episodes are not supported");
  if (env->cfg.substeps > MAX_S) return set_error(AUV_EINVAL, "auv_shac_window: at most %d substeps", MAX_S);
  if (N > (1 << 22)) return set_error(AUV_EINVAL, "auv_shac_window: at most 2^22 environments");
  if (h < 1 || h > MAX_H || h > H) return set_error(AUV_EINVAL, "auv_shac_window: h must be in [1, min(64, H)], got %d", h);
  if (env->global_step % H + h > H)
    return set_error(AUV_EINVAL, "auv_shac_window: the window would cross an episode end (step %lld of %d, h %d)",
                     (long long)(env->global_step % H), H, h);
  if (mode != AUV_ACT_EXTERNAL && mode != AUV_ACT_POLICY_MEAN && mode != AUV_ACT_POLICY_SAMPLE)
    return set_error(AUV_EINVAL, "auv_shac_window: mode must be external, policy mean or policy sample");
  if (!(cfg->gamma > 0.0f && cfg->gamma <= 1.0f) || !std::isfinite(cfg->max_grad_norm))
    return set_error(AUV_EINVAL, "auv_shac_window: gamma must be in (0, 1], max_grad_norm finite");
  const bool ext = mode == AUV_ACT_EXTERNAL;
  if (ext && (!out || !out->actions)) return set_error(AUV_EINVAL, "auv_shac_window: external mode reads out->actions");
  if (ext && grad_policy) return set_error(AUV_EINVAL, "auv_shac_window: no policy gradient in external mode");
  if (!ext) {
    if (!policy || !policy->w || !policy->b || policy->n_out != ACT)
      return set_error(AUV_EINVAL, "auv_shac_window: policy modes need a 23-256-256-8 policy");
    if (mode == AUV_ACT_POLICY_SAMPLE && !policy->log_std)
      return set_error(AUV_EINVAL, "auv_shac_window: policy sample mode needs log_std");
  }
  if (value && (!value->w || !value->b || value->n_out != 1))
    return set_error(AUV_EINVAL, "auv_shac_window: the value net must be 23-256-256-1");
  const void* ptrs[] = {work, stats, grad_policy, policy ? policy->w : nullptr, policy ? policy->b : nullptr,
                        value ? value->w : nullptr, value ? value->b : nullptr};
  for (const void* p : ptrs)
    if (p && !aligned16(p)) return set_error(AUV_EINVAL, "auv_shac_window: pointers must be 16-byte aligned");
  if (out) {
    const void* o[] = {out->actions, out->obs, out->act, out->reward, out->done, out->grad_act, out->value_last,
                       out->grad_state0};
    for (const void* p : o)
      if (p && !aligned16(p)) return set_error(AUV_EINVAL, "auv_shac_window: output buffers must be 16-byte aligned");
  }

  hipStream_t s = (hipStream_t)stream;
  const Shape sh = shape_of(N, h, compute_units());
  size_t off[WORK_PARTS];
  work_layout(N, h, off);
  char* base = (char*)work;
  auto at = [&](int k) { return (void*)(base + off[k]); };
  bf16x8* frags = (bf16x8*)at(0);
  const int fb = (F_END * 64 + 255) / 256;
  // both networks' fragments in one launch (grid y: the networks given, the policy first)
  {
    const uint16_t* wn[2] = {nullptr, nullptr};
    int no[2] = {0, 0};
    bf16x8* dst[2] = {nullptr, nullptr};
    int nn = 0;
    if (!ext) wn[nn] = policy->w, no[nn] = ACT, dst[nn++] = frags;
    if (value) wn[nn] = value->w, no[nn] = 1, dst[nn++] = frags + F_END * 64;
    if (nn > 0)
      hipLaunchKernelGGL(k_frags, dim3(fb, nn), dim3(256), 0, s, wn[0], no[0], dst[0], wn[1], no[1], dst[1]);
  }

  WinArgs A{};
  A.steps = h;
  A.want_grad = grad_policy ? 1 : 0;
  A.has_val = value ? 1 : 0;
  A.step0 = (uint32_t)(env->global_step & 0xffffffffu);
  A.inv_nh = (float)(1.0 / ((double)N * (double)h));
  A.gamma = cfg->gamma;
  A.pol = NetF{frags, ext ? nullptr : policy->b, ACT};
  A.val = NetF{frags + F_END * 64, value ? value->b : nullptr, 1};
  A.log_std = (!ext && policy->log_std) ? policy->log_std : nullptr;
  A.obk = (f32x4*)at(1);
  A.aa = (f32x4*)at(2);
  A.J = (float*)at(3);
  A.Jr = (float*)at(4);
  A.vl = (float*)at(5);
  A.h1_half = (u32x2*)at(6);
  A.dz2_half = (u32x2*)at(7);
  A.h2s = (f32x4*)at(15);
  A.rec = (f32x4*)at(16);
  A.groups = sh.NG;
  if (out) {
    A.ext = out->actions;
    A.o_obs = out->obs;
    A.o_act = out->act;
    A.o_reward = out->reward;
    A.o_done = out->done;
    A.o_gact = out->grad_act;
    A.o_vlast = out->value_last;
    A.o_gs0 = out->grad_state0;
  }
  GradParts P;
  P.part_w1 = (float*)at(8);
  P.part_b1 = (float*)at(9);
  P.part_w3 = (float*)at(10);
  P.part_b2 = (float*)at(11);
  P.part_b3 = (float*)at(12);
  P.part_ls = P.part_b3 + MAX_GROUPS * 16;
  P.part_w2 = (float*)at(13);
  const dim3 wgrid(sh.GW), wblock(64 * WAVES);
  if (mode == AUV_ACT_EXTERNAL)
    hipLaunchKernelGGL(k_window<MODE_EXTERNAL>, wgrid, wblock, 0, s, env->E, env->veh, A, P);
  else if (mode == AUV_ACT_POLICY_MEAN)
    hipLaunchKernelGGL(k_window<MODE_MEAN>, wgrid, wblock, 0, s, env->E, env->veh, A, P);
  else
    hipLaunchKernelGGL(k_window<MODE_SAMPLE>, wgrid, wblock, 0, s, env->E, env->veh, A, P);

  const int rb = grad_reduce_blocks(ACT);
  float* ss = (float*)at(14);
  if (grad_policy) {
    // padding sample tiles (beyond the window's) hold zeros and so add nothing
    if (sh.tiles_p > sh.tiles) {
      const size_t pad = (size_t)(sh.tiles_p - sh.tiles) * 16 * 64 * 2;   // u32
      for (u32x2* half : {A.h1_half, A.dz2_half})
        hipLaunchKernelGGL(k_zero, dim3(64), dim3(256), 0, s, (uint32_t*)(half + (size_t)sh.tiles * 16 * 64), pad);
    }
    if (int rc = launch_dw2(A.dz2_half, A.h1_half, sh.steps, sh.G3, P.part_w2, s)) return rc;
    if (int rc = launch_grad_reduce(P, ACT, 6, sh.GW, sh.GW, sh.G3, grad_policy, ss, s)) return rc;
  }
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, A.J, A.Jr, A.vl, N, A.inv_nh, ss, grad_policy ? rb : 0,
                     cfg->max_grad_norm, stats);
  const int rc = check_launch("auv_shac_window");
  if (rc == AUV_OK) env->global_step += h;
  return rc;
}

}  // extern "C"
