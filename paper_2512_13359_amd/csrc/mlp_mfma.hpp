// bf16 MFMA building blocks of the MLP 23 -> 256 -> 256 -> n_out (tanh hidden, linear
// output): operand types, the K-slot order, the MFMA call and the activation.
//
// Formulation: Z^T = W H^T, so MFMA rows (M) are output features, columns (N) are
// environments and the contraction (K) runs over input features.  v_mfma_f32_16x16x32_bf16
// lane l = 16 g + r holds A[m = r][k-slot (g, j)], B[k-slot (g, j)][n = r] for j = 0..7,
// and D[m = 4 g + i][n = r] for i = 0..3.
//
// Within a 32-wide K tile, slot (g, j) holds feature 16 (j / 4) + 4 g + (j % 4).  With that
// order a lane's four D values of two consecutive 16-row M-tiles are exactly its eight B
// values of the next layer's K tile made of those 32 features, so a hidden layer's output
// becomes the next layer's operand without any lane exchange (act_frag).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace auv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int HID = 256;
constexpr int NOUT_PAD = 8;   // output rows kept (policy 8, value 1)

__device__ __forceinline__ int kslot(int g, int j) { return 16 * (j >> 2) + 4 * g + (j & 3); }

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ __bf16 bf16_of_bits(uint16_t b) { return __builtin_bit_cast(__bf16, b); }

constexpr float TWO_LOG2E = 2.88539008177792681f;   // 2 log2(e)

// tanh(d + b) = 1 - 2 / (1 + 2^{(d + b) 2 log2 e}) with bk = b * 2 log2 e folded into
// one fma; saturates correctly at both ends (2^x -> inf gives 1, -> 0 gives -1).
// Absolute error a few 1e-7.
__device__ __forceinline__ float tanh_bias(float d, float bk) {
  const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(d, TWO_LOG2E, bk));
  return __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + e), 1.0f);
}

// tanh(D + bias) of two consecutive M-tiles -> the eight-value K-tile fragment of the next
// layer's B operand (bf16, round to nearest even).
__device__ __forceinline__ bf16x8 act_frag(const f32x4& d0, const f32x4& d1, const f32x4& b0, const f32x4& b1) {
  bf16x8 f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[i] = (__bf16)tanh_bias(d0[i], b0[i]);
    f[4 + i] = (__bf16)tanh_bias(d1[i], b1[i]);
  }
  return f;
}

// A workgroup's copy of W1 and W2 (row-major in memory) into LDS as MFMA A fragments: lane (g, r) of
// fragment (M-tile mt, K tile kt) holds row 16 mt + r, inputs 32 kt + kslot(g, j), W2's at slot(lane)
// of its fragment.  load() issues every load, store() writes LDS, so that a kernel can issue its
// other loads in between and wait for memory once.  W2 is read in 16-byte pieces of a row; the
// piece of row 16 mt + r at columns 32 kt + o .. + 7 (o = 0, 8, 16, 24) is the half o / 16 (K slots
// 4 (o / 16) .. + 3) of lanes 16 g + r and 16 (g + 1) + r, g = (o % 16) / 4.  A wave's load takes 128
// bytes of each of eight rows: its stores then meet on a bank at most four at a time (with two whole
// rows per load sixteen at a time, 3 us of every launch that stages the weights).  W1's rows have 23
// inputs: lane (g, r) reads inputs 4 g .. + 3 and 16 + 4 g .. + 3 of its row as 8 bytes each, not
// aligned, those past the row masked (the last row's reach into W2, which follows).  A load in
// which every lane reads another row goes through the L1 at one lane per cycle, so their number is
// what counts: two per fragment, not eight.
template <int WAVES>
struct StageWeights {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  static constexpr int P2 = HID * HID / 8 / (64 * WAVES), P1 = 16 / WAVES;
  u32x4 v2[P2];
  uint2 v1[P1][2];

  __device__ __forceinline__ static int row(int q, int wave, int lane) { return 8 * ((q * WAVES + wave) >> 2) + (lane >> 3); }
  __device__ __forceinline__ static int col(int q, int wave, int lane) {
    return 64 * ((q * WAVES + wave) & 3) + 8 * (lane & 7);
  }
  __device__ __forceinline__ void load(const uint16_t* __restrict__ w1, const uint16_t* __restrict__ w2, int wave,
                                       int lane) {
#pragma unroll
    for (int q = 0; q < P2; ++q)
      v2[q] = *reinterpret_cast<const u32x4*>(w2 + row(q, wave, lane) * HID + col(q, wave, lane));
#pragma unroll
    for (int q = 0; q < P1; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        __builtin_memcpy(&v1[q][h], w1 + (16 * (q * WAVES + wave) + (lane & 15)) * 23 + min(kslot(lane >> 4, 4 * h), 20), 8);
  }
  template <class Slot>
  __device__ __forceinline__ void store(bf16x8 (*w1)[64], bf16x8 (*w2)[8][64], int wave, int lane, Slot slot) const {
#pragma unroll
    for (int q = 0; q < P2; ++q) {
      const int rw = row(q, wave, lane), c = col(q, wave, lane), o = c & 31, g0 = (o & 15) >> 2, rr = rw & 15;
      char* frag = reinterpret_cast<char*>(&w2[rw >> 4][c >> 5][0]) + 8 * (o >> 4);
      *reinterpret_cast<uint2*>(frag + 16 * slot(16 * g0 + rr)) = uint2{v2[q].x, v2[q].y};
      *reinterpret_cast<uint2*>(frag + 16 * slot(16 * (g0 + 1) + rr)) = uint2{v2[q].z, v2[q].w};
    }
#pragma unroll
    for (int q = 0; q < P1; ++q) {
      const uint32_t d[4] = {v1[q][0].x, v1[q][0].y, v1[q][1].x, v1[q][1].y};
      bf16x8 v;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = bf16_of_bits(kslot(lane >> 4, j) < 23 ? (uint16_t)(d[j >> 1] >> (16 * (j & 1))) : (uint16_t)0);
      w1[q * WAVES + wave][lane] = v;
    }
  }
};

}  // namespace auv
