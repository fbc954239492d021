// Look-ahead recurrences (inference, bf16 operands, K >= 64, E >= 4): the tiles
// that their prep kernel writes.
//
// The chunk recurrence of Eq. joint-chunk has a serial chain per chunk:
// W_c = sum_e diag(a_e) K_c S_c, then U_c = Tu (V - W_c), then the state
// update that W_{c+1} waits for.  With the update line put into W_{c+1},
//   W_{c+1} = sum_e diag(a_{c+1,e} gamma^C_{c,e}) K_{c+1} S_{c,e} + G_{c+1} U_c,
//   G_{c+1} = (K_{c+1} K_c^T) o sum_e a_{c+1,e} c_{c,e}^T        (C x C),
// the state contraction uses the state one chunk back, so it runs beside the
// update instead of after it, and only the two C x C products G U and Tu X
// remain on the chain.
#pragma once
#include "tla_common.hpp"
#include "tla_internal.hpp"

namespace tla {

// Operand tiles of one chunk.  M and Tu (lower block-triangular) and G are
// kept as bf16 (hi, lo) pairs of 32-deep A operands, 1 KiB each: lane (g, n) of
// operand (rt, p) holds row 16 rt + n at columns 32 p + 4 g + j (elements
// 0..3) and 32 p + 16 + 4 g + j (elements 4..7), the order in which two
// accumulator tiles make a 32-deep B operand.  K^T is
// [K][C] with row R holding key la_key(R) and the 16-byte pieces of a row in
// the order of SwzTile, so that a plain copy fills the shared tile.
template <int KD, int C>
struct LaOps {
  static constexpr int NT = C / 16, NP = NT / 2;
  static constexpr int NTRI = NP * (NP + 1);  // operands of a lower-triangular matrix
  static constexpr int FR = 512;              // elements of one operand part
  static __host__ __device__ constexpr int tri(int rt, int p) {
    return (rt >> 1) * ((rt >> 1) + 1) + (rt & 1) * ((rt >> 1) + 1) + p;
  }
  static __host__ __device__ constexpr int full(int rt, int p) { return rt * NP + p; }
  static constexpr size_t M = 0, Tu = (size_t)NTRI * 2 * FR, G = 2 * Tu;
  static constexpr size_t Kt = G + (size_t)NT * NP * 2 * FR;
  static constexpr size_t STRIDE = Kt + (size_t)KD * C;
};

// Key order of the state tiles.  Row m of a 32-row accumulator tile lies in
// register 4 (m / 8) + m % 4 of lane half (m / 4) % 2; it holds the key that
// makes a lane's registers 0..7 and 8..15 eight consecutive keys each, the
// 16-deep operands of the state contractions.
__host__ __device__ constexpr int la_key(int R) {
  return (R & ~31) | (R & 16) | ((R & 4) << 1) | ((R & 8) >> 1) | (R & 3);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 x;
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = 0.f;
  return x;
}
__device__ __forceinline__ f32x16 mma_32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma_16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 join8(bf16x4 a, bf16x4 b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
// registers 8 k .. 8 k + 7 of an accumulator tile as a bf16 operand
__device__ __forceinline__ bf16x8 half_op(const f32x16& x, int k) {
  return join8(cvt_frag<bf16_t>(f32x4{x[8 * k], x[8 * k + 1], x[8 * k + 2], x[8 * k + 3]}),
               cvt_frag<bf16_t>(f32x4{x[8 * k + 4], x[8 * k + 5], x[8 * k + 6], x[8 * k + 7]}));
}
// One 1 KiB piece of a linear copy into shared memory (off = 16 lane).
__device__ __forceinline__ void dma_kib(void* dst, const void* src, uint32_t off) {
  lds_dma<16>(uniform_ptr(src), off, lds_addr(dst));
}

}  // namespace tla
