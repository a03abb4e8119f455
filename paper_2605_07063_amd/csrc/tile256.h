// Main loop of a 256 x 256 output tile on bf16 MFMA (gfx950), shared by the
// kernels whose operands are row panels streamed through LDS.
//
// Four waves (one per SIMD) hold a 128 x 128 fp32 accumulator each, in the
// AGPRs; two 64 KB stages of a 64-column step (A and B panels of 256 rows x
// 128 bytes) are filled by buffer->LDS DMA.  A wave reads 16 fragments per
// 64 products; with eight waves of 128 x 64 it would read 12 per 32, and the
// LDS reads plus the DMA writes would take as long as the products.
#pragma once

#include "common.h"

namespace dr {

constexpr int kTileRows = 256;                        // rows of either panel
constexpr int kTileStepCols = 64;                     // bf16 columns per step (128-byte rows)
constexpr int kTilePanel = kTileRows * kTileStepCols * 2;
constexpr int kTileStage = 2 * kTilePanel;            // A, then B
constexpr int kTileRing = 2 * kTileStage;

__device__ __forceinline__ void tile256_clear(f32x4 (&acc)[8][8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      // the zeros are in place before the products: the compiler does not
      // see the MFMAs inside the asm, so it would not space a register write
      // and the product that reads it apart
      asm volatile("" : "+a"(acc[i][j]));
    }
}

// The last products' results are read next: wait states after an MFMA that the
// compiler does not see inside the asm.  Every accumulator then passes through
// an asm, so that no read of it can be scheduled before the wait.
__device__ __forceinline__ void tile256_settle(f32x4 (&acc)[8][8]) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// acc[i][j] (i over A's 16-row blocks of this wave, j over B's) += the
// products of nk steps.  dma1(t, st, q), q = 0..15: one DMA of step t into
// stage st (zeros for t >= nk).  rd1(fa, fb, stage, kh, q): fragment read q
// of 32-column half kh (q even A block q / 2, q odd B block q / 2).  Each
// product is an in-place asm MFMA on its accumulator, so every accumulator
// stays where it is (the compiler's own MFMA form moves them between register
// files at this size); volatile asm also keeps the written order: each
// fragment read and DMA issue sits between MFMAs.
//
// Per step t (stage t & 1): the first half's products with the second half's
// fragment reads between them; one barrier (step t + 1 landed everywhere,
// every wave done with stage t & 1); then the second half's products with
// the DMA of step t + 2 into stage t & 1 and the reads of step t + 1's first
// half between them.  On return two steps of zeros may still be in flight to
// the ring.
template <class Dma, class Rd>
__device__ __forceinline__ void tile256_loop(unsigned char* lds, int nk, Dma&& dma1, Rd&& rd1, f32x4 (&acc)[8][8]) {
  auto mma = [&](int i, int j, const u32x4* fa, const u32x4* fb) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fa[i]), "v"(fb[j]));
  };
  u32x4 fa0[8], fb0[8], fa1[8], fb1[8];
#pragma unroll
  for (int q = 0; q < 16; ++q) dma1(0, 0, q);
  DR_WAIT_VM(0);
  DR_LDS_SYNC();
#pragma unroll
  for (int q = 0; q < 16; ++q) dma1(1, 1, q);
#pragma unroll
  for (int q = 0; q < 16; ++q) rd1(fa0, fb0, lds, 0, q);
  for (int t = 0; t < nk; ++t) {
    const unsigned char* sa = lds + (t & 1) * kTileStage;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      rd1(fa1, fb1, sa, 1, q);
#pragma unroll
      for (int m = 4 * q; m < 4 * q + 4; ++m) mma(m & 7, m >> 3, fa0, fb0);
    }
    DR_WAIT_VM(0);
    DR_LDS_SYNC();
    const unsigned char* sn = lds + ((t + 1) & 1) * kTileStage;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      dma1(t + 2, t & 1, q);
      rd1(fa0, fb0, sn, 0, q);
#pragma unroll
      for (int m = 4 * q; m < 4 * q + 4; ++m) mma(m & 7, m >> 3, fa1, fb1);
    }
  }
  tile256_settle(acc);
}

}  // namespace dr
