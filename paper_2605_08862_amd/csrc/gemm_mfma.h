// Operands of the projection GEMMs and the LM head on the f16 MFMA (bf16 models).
//
// Precision.  Weights are bf16 values; activations handed from one operator to the next are kept
// in float16 (11 significant bits) and the products run on the f16 MFMA with float32 accumulation.
// With bf16 (8-bit) activation operands the full-vocabulary logits of a 28-layer decoder drift by
// ~9e-2 from the exact forward; with 11-bit operands they stay near 1e-2.  bf16 weight values
// convert to float16 exactly for 6.1e-5 <= |w| <= 65504 (below that the absolute error is < 6e-8).
//
// Weights are re-packed once (at context creation) into MFMA operand order: for each (32-row tile, 64-wide K tile) a
// 4 KiB block [s = 0..3][lane = 0..63][8 halves], blocks of one row tile consecutive along K.  A row tile is a purely
// sequential stream of 1 KiB pieces (32 rows x 16 of K).  The contraction index inside a K tile is permuted: piece s of
// lane group g (lane / 32) holds k = 32 g + 8 s + j.  Activations have the same order of k (act_index).  A 16 x 16 x 32 product reads 16 rows of two
// consecutive pieces (frag_lane): lane groups 0 .. 3 of 16 lanes have the k of group 0 and 1 of piece s, then of piece s + 1, for both operands alike.
// The products are mfma(W, X): the accumulator holds C^T tiles (rows = weight rows, lane % 16 = activation row), so that a lane has four consecutive
// columns of a row and a reduction over the columns of a tile takes the four lanes of a row together.  Main loops: gemm_dma.h, skinny.hip.
#pragma once
#include "common.h"

typedef _Float16 f16;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // of a caller's array: aligned to its elements only
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;                    // K tile (elements)
constexpr int kWBlock = 32 * kBK;          // elements of one packed (row tile, K tile) block

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// The GEMM loops multiply 16 x 16 x 32: the same rate and the same operand bytes as 32 x 32 x 16, but half of the accumulator bytes per product.
// Under a power limit that is speed: MFMA loops on random operands, every CU busy, 1.64 -> 1.95 PFLOP/s from registers, 1.48 -> 1.69 with fragments
// read from LDS.
// (A function of its own: the host pass does not accept the builtin inside templates.)
__device__ __forceinline__ f32x4 mfma_f16(u32x4 a, u32x4 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(b), c, 0, 0, 0); }

// A fragment of that product is 16 rows of a 32-row tile x two consecutive 1 KiB pieces: byte offset of this lane (row lane % 16, the
// eight k of group lane / 16), and from the tile's first 16 rows to its last 16.
__device__ __forceinline__ int frag_lane() { const int lane = threadIdx.x & 63; return (lane >> 5) * 1024 + ((lane >> 4) & 1) * 512 + (lane & 15) * 16; }
constexpr int kWHalf = 256;
// Accumulator acc[a][b][e] of C^T: activation row 16 a + acc_col, weight row 16 b + acc_row + e.
__device__ __forceinline__ int acc_row(int lane) { return 4 * (lane >> 4); }
__device__ __forceinline__ int acc_col(int lane) { return lane & 15; }
