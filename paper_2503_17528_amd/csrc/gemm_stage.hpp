// Operand stages of the FP64 MFMA products: pieces of 16 bytes moved from global
// memory straight into LDS, their placement there, and the barrier between
// stages.
#pragma once
#include "bta_device.hpp"

namespace bta {

// ---------------------------------------------------------------- direct-to-LDS tile body
// The same product with operands moved from global memory straight into LDS
// (global_load_lds_dwordx4: each lane moves one 16-byte piece, the pieces of a
// wave instruction land contiguously), two LDS stages of BK = 16, one barrier
// per stage and no register staging.  Piece placement within a stage:
//   k-contiguous operand (N): slot m*8 + (p ^ swzN(m)) holds k = 2p, 2p+1 of row m;
//   m-contiguous operand (T): slot k*(TM/2) + (q ^ swzT(k)) holds m = 2q, 2q+1 of row k.
// Both swizzles make the MFMA operand reads (16-byte reads of rows m for N,
// 8-byte reads of 16 consecutive m for T) free of LDS bank conflicts.
// Requirements (checked on the host by dl_ok): 16-byte aligned operand bases,
// even leading dimensions and batch strides, even K, and even M (N) for a
// transposed A (B), so that no piece straddles the edge of an operand.
__device__ __forceinline__ int swzN(int m) { return (m ^ (m >> 3)) & 7; }
__device__ __forceinline__ int swzT(int k) { return ((k >> 2) & 1) << 3; }

__device__ __forceinline__ void load_piece_lds(const double* src, double* lds_wave) {
  __builtin_amdgcn_global_load_lds(static_cast<const void*>(src),
                                   (__attribute__((address_space(3))) void*)(lds_wave), 16, 0, 0);
}

// The same pieces with every address one lane offset past a scalar row base
// (no per-piece pointer registers: the 64 x 64 kernels fit four waves a SIMD
// instead of two).  BYTES 16: a piece per lane.  BYTES 4: four lanes a piece,
// from operands at any 8-byte alignment (odd leading dimensions, where a
// 16-byte load would need every row on a 16-byte line).  Wave w of the operand
// fills slots SPI NI w .. SPI NI (w + 1) - 1, SPI per instruction; the rows of
// an instruction are wave-uniform but for the lane's part, and the swizzle is
// an xor of the lane's offset with a constant.
// SC1: device-coherent loads (operands that the same kernel produces).
template <int TR, int NI, int BYTES, bool SC1 = false>
__device__ __forceinline__ void stage_pieces(const double* base, int64_t ld, int trans, int r0, int rext, int k, int kext,
                                             double* dst, int w, int lane) {
  constexpr int LPP = 16 / BYTES, SPI = 64 / LPP;
  const int slot = lane / LPP;
  const unsigned part = BYTES * (unsigned)(lane % LPP);
  double* const d0 = dst + w * NI * SPI * 2;
  const bool full = rext >= TR && kext >= 16;
  auto load = [&](const char* src, int i) {
    auto* const to = (__attribute__((address_space(3))) void*)(d0 + 2 * SPI * i);
    if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds(src, to, 16, 0, SC1 ? 16 : 0);
    else __builtin_amdgcn_global_load_lds(src, to, 4, 0, SC1 ? 16 : 0);
  };
  const char* const zero = reinterpret_cast<const char*>(k_zero_pair);
  if (!trans) {
    // rows m = mw + RPI i + h, piece (slot % 8) ^ swzN(m)
    constexpr int RPI = SPI / 8;
    const int h = slot >> 3, mw = RPI * NI * w;
    const unsigned x0 = 16u * ((slot & 7) ^ h ^ swzN(mw)) + part, hoff = h * (unsigned)(8 * ld);
    const char* row = reinterpret_cast<const char*>(base + (int64_t)(r0 + mw) * ld + k);
    if (full) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        load(row + (hoff + (x0 ^ (16u * swzN(RPI * i)))), i);
        row += 8 * RPI * ld;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const unsigned x = x0 ^ (16u * swzN(RPI * i));
        load(mw + RPI * i + h < rext && (int)(x >> 3) < kext ? row + (hoff + x) : zero, i);
        row += 8 * RPI * ld;
      }
    }
  } else {
    // k rows kk = kw + SPI i / PR + h, piece (SPI i + slot) % PR ^ swzT(kk)
    constexpr int PR = TR / 2, RPI = SPI > PR ? SPI / PR : 1, IPR = SPI > PR ? 1 : PR / SPI;
    const int h = slot / PR, kw = w * (NI * SPI / PR);
    const unsigned x0 = 16u * (slot % PR) + part, hoff = h * (unsigned)(8 * ld);
    const char* row = reinterpret_cast<const char*>(base + (int64_t)(k + kw) * ld + r0);
    if (full) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        load(row + (hoff + (x0 ^ (16u * swzT(kw + i * SPI / PR))) + 16u * (i % IPR * SPI)), i);
        if (i % IPR == IPR - 1) row += 8 * RPI * ld;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int kk = kw + i * SPI / PR;
        const unsigned x = (x0 ^ (16u * swzT(kk))) + 16u * (i % IPR * SPI);
        load(kk + h < kext && (int)(x >> 3) < rext ? row + (hoff + x) : zero, i);
        if (i % IPR == IPR - 1) row += 8 * RPI * ld;
      }
    }
  }
}

// Operand values of one stage for MFMA blocks i = 0..W-1 at rows r0 + 16 i + lane%16,
// v[i][s] = X(row, 4*(lane/16) + s).
template <int TR, int W>
__device__ __forceinline__ void stage_read(double (&v)[W][4], const double* st, int trans, int r0, int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int m = r0 + 16 * i + (lane & 15);
    if (!trans) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const d2v x = *reinterpret_cast<const d2v*>(st + 2 * (m * 8 + ((2 * g + h) ^ swzN(m))));
        v[i][2 * h] = x[0];
        v[i][2 * h + 1] = x[1];
      }
    } else {
      constexpr int PR = TR / 2;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 4 * g + s;
        v[i][s] = st[2 * (k * PR + ((m >> 1) ^ swzT(k))) + (m & 1)];
      }
    }
  }
}

// Wait until at most N of this thread's vector memory loads are outstanding and
// its LDS reads are done, then meet the workgroup at a barrier; the statement's
// memory clobber keeps the compiler from moving LDS accesses or direct-to-LDS
// loads across it.  Every stage's barrier is this one: __syncthreads() may
// leave direct-to-LDS loads outstanding (the compiler waits for them before the
// wave's own reads only, and the barrier is what tells the other waves), and
// where it does wait, it waits for the newer stages' loads too.
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

}  // namespace bta
