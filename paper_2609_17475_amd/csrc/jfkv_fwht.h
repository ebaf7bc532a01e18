// Walsh-Hadamard transform of 256-element vectors in registers, shared by the
// TQ4 encoder, reconstruction and decode kernels.
//
// A wave transforms four vectors at a time, one per row of 16 lanes.  The lane
// of chunk c (0..15) holds elements 8c .. 8c + 7 and 128 + 8c .. 128 + 8c + 7
// (two 16-byte loads; 16 lanes read 256 contiguous bytes each time).  Of the
// eight butterfly stages of the Walsh-Hadamard transform, those on element
// index bits 0, 1, 2 and 7 stay in the lane and those on bits 3..6 (the bits of
// c) exchange with another lane of the row.  Lane r of the row holds the chunk
// c with r = c0 * 1 ^ c1 * 2 ^ c2 * 7 ^ c3 * 15, so that the four exchanges are
// the lane permutations a DPP operand can make by itself (pairs swapped, quad
// halves swapped, half row and row mirrored), and a stage is one instruction
// per element: f = e + sg * partner(e) with sg = -1 in the lanes whose bit is
// set, which there is minus the butterfly's output.  A pair of lanes differs
// only in the bit of its own stage, so the signs left by earlier stages agree
// in it and multiply to one sign per lane, which the final scaling takes out.
// (One lane per four elements, 64 lanes per vector, needed six exchanges of
// every element, four of them through the LDS unit.)  The additions and their
// order are those of the textbook in-place transform, stage by stage.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace jfkv {

// The lane that differs in bit K of the chunk number (see above).
template <int K>
__device__ __forceinline__ float partner(float v) {
  constexpr int kCtrl[4] = {0xB1, 0x4E, 0x141, 0x140};  // quad_perm 1,0,3,2; 2,3,0,1; half, row mirror
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kCtrl[K],
                                                            0xF, 0xF, true));
}

// Chunk held by lane r of a row, and the signs of the four exchanges.
struct RowLane {
  int chunk;
  float sg[4], sign;  // sign: their product
  __device__ __forceinline__ explicit RowLane(int r) {
    const int r0 = r & 1, r1 = (r >> 1) & 1, r2 = (r >> 2) & 1, r3 = r >> 3;
    const int c[4] = {r0 ^ r2, r1 ^ r2, r2 ^ r3, r3};
    chunk = c[0] + 2 * c[1] + 4 * c[2] + 8 * c[3];
    sign = 1.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      sg[k] = c[k] ? -1.0f : 1.0f;
      sign *= sg[k];
    }
  }
};

// The four exchanging stages (element index bits 3..6): one instruction per
// element and stage.  Written out, since the compiler makes each a move with
// the permutation and an fma; a DPP operand may not be read within two wait
// states of being written, which the s_nop (before the first stage) and the
// sixteen instructions of a stage (between stages) provide.  Every lane of the
// wave is active here.
__device__ __forceinline__ void exchange_stages(float (&e)[2][8], const RowLane& rl) {
#define JF_X(R, S, C) "v_fmac_f32_dpp %" #R ", %" #R ", %" #S " " C " row_mask:0xf bank_mask:0xf\n\t"
#define JF_STAGE(S, C)                                                                          \
  JF_X(0, S, C) JF_X(1, S, C) JF_X(2, S, C) JF_X(3, S, C) JF_X(4, S, C) JF_X(5, S, C)           \
  JF_X(6, S, C) JF_X(7, S, C) JF_X(8, S, C) JF_X(9, S, C) JF_X(10, S, C) JF_X(11, S, C)         \
  JF_X(12, S, C) JF_X(13, S, C) JF_X(14, S, C) JF_X(15, S, C)
  asm("s_nop 1\n\t" JF_STAGE(16, "quad_perm:[1,0,3,2]") JF_STAGE(17, "quad_perm:[2,3,0,1]")
      JF_STAGE(18, "row_half_mirror") JF_STAGE(19, "row_mirror")
      : "+&v"(e[0][0]), "+&v"(e[0][1]), "+&v"(e[0][2]), "+&v"(e[0][3]), "+&v"(e[0][4]), "+&v"(e[0][5]),
        "+&v"(e[0][6]), "+&v"(e[0][7]), "+&v"(e[1][0]), "+&v"(e[1][1]), "+&v"(e[1][2]), "+&v"(e[1][3]),
        "+&v"(e[1][4]), "+&v"(e[1][5]), "+&v"(e[1][6]), "+&v"(e[1][7])
      : "v"(rl.sg[0]), "v"(rl.sg[1]), "v"(rl.sg[2]), "v"(rl.sg[3]));
#undef JF_STAGE
#undef JF_X
}

// Stages 1..7 of the transform (stage 0, on neighbouring elements, is the
// caller's); leaves rl.sign times the result.
__device__ __forceinline__ void fwht_from1(float (&e)[2][8], const RowLane& rl) {
#pragma unroll
  for (int m = 2; m <= 4; m *= 2)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (!(i & m)) {
          const float u = e[h][i], v = e[h][i + m];
          e[h][i] = u + v;
          e[h][i + m] = u - v;
        }
  exchange_stages(e, rl);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float u = e[0][i], v = e[1][i];
    e[0][i] = u + v;
    e[1][i] = u - v;
  }
}

}  // namespace jfkv
