// Layouts and products shared by the embedding-net kernels (force path and
// parameter gradients).
#pragma once

#include "dp_device.h"

namespace dpse {

// Returns 0 in a register the optimiser cannot see through; added to LDS
// indices inside the neighbour-tile loop it keeps fragment loads in the loop.
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+v"(z));
  return z;
}

// per-net vector block: W1s[32] | b1s[32] | b2s[64] | b3s[128] | b3f[128]
constexpr int kV_W1 = 0, kV_B1 = 32, kV_B2 = 64, kV_B3S = 128, kV_B3F = 256, kVecPerNet = 384;

template <int W>
__device__ __forceinline__ int slot2_of_feat(int f) {  // f in [0, 2W)
  return (f / W) * 32 + (f % W);
}
template <int W>
__device__ __forceinline__ int feat3_of_slot(int p) {  // -1 for padding slots
  const int q = p & 63;
  if ((q & 31) >= W) return -1;
  return (p >> 6) * 2 * W + (q >> 5) * W + (q & 31);
}

// FP64 k-step (t, v) covers slots 16t + 4v + {0..3}; with w = 25 the slot
// groups 28..31 (mod 32) hold only padding, so those k-steps are skipped and
// the activations of those slots (tanh(0) = 0) are not evaluated.
//
// The FP64 kernels use a denser layout of the width-2w layer for w = 25
// (the mixed kernels, whose k-steps are 32 wide, keep the plain one).  Each
// half of the layer ends in a k-step (slots 24..27, 56..59) holding a
// single feature; both halves' last features (24 and 49) go to slots 24 and
// 25, and slots 26 and 27 hold copies of them, so that slots 56..59 are
// padding and their k-steps drop out.  A copy is computed like a feature
// (its layer-1 slot partner, slots 25..27 of layer 1, holds a copy of
// feature 24 of layer 1) but has no outgoing weights: the layer above
// reads only the original, and a copy reaches the output only through the
// identity skip.  That skip pairs layer-3 slot 64 zo + q with layer-2 slot
// q, so slots 24..27 of the first layer-3 half hold features 24, 49, 74
// and 99 (whose skip partners are 24, 49, 24, 49), and slots 24..27 of the
// second half are padding.  Gradients flow through the copies like
// through any other unit.
template <int W>
constexpr bool kDense2 = (W == 25);
template <int W>
__device__ __forceinline__ constexpr bool kpad(int t, int v) {  // layer-1 slots
  return W <= 28 && (t & 1) && v == 3;
}
template <int W>
__device__ __forceinline__ constexpr bool kpad2(int t, int v) {  // layer-2 slots, FP64 layout
  return kpad<W>(t, v) || (kDense2<W> && t == 3 && v == 2);
}
template <int W>
__device__ __forceinline__ constexpr bool kpad3(int zo, int t, int v) {  // layer-3 slots 64 zo + 16 t + 4 v + g
  return kpad2<W>(t, v) || (kDense2<W> && zo == 1 && t == 1 && v == 2);
}
// elements of a 16-slot tile before its padding (padding is always last)
template <int W>
__device__ __forceinline__ constexpr int nv1(int t) {
  return 4 - kpad<W>(t, 3);
}
template <int W>
__device__ __forceinline__ constexpr int nv2(int t) {
  return 4 - kpad2<W>(t, 3) - kpad2<W>(t, 2);
}
template <int W>
__device__ __forceinline__ constexpr int nv3(int zo, int t) {
  return 4 - kpad3<W>(zo, t, 3) - kpad3<W>(zo, t, 2);
}
// Compact numbering of the FP64 kernels' elements (four slots each, padding
// ones left out; the elements of full tiles first), shared with the blocks the
// host lays out: of a product's operand, the m elements of a full tile as
// [k element][64] in lane order, a single m element as [k element][16], row i
// and sub-k kk at i + 4 kk (lane offset lo4); k values one after another, so
// that one LDS instruction reads two of them.
template <int W>
struct EmbLay {
  static constexpr int n1 = nv1<W>(0) + nv1<W>(1);
  static constexpr int n2 = nv2<W>(0) + nv2<W>(1) + nv2<W>(2) + nv2<W>(3);
  static constexpr int n3 = n2 + nv3<W>(1, 0) + nv3<W>(1, 1) + nv3<W>(1, 2) + nv3<W>(1, 3);
  static constexpr int F2 = 16 * n1 * n2, F3n = 16 * n2 * W, F3t = 16 * n2 * n3, B3 = F3t, B2 = F2;
  // first element of tile t in layers 2 and 3 (layer 3: t = 4 zo + tile)
  static __device__ __forceinline__ constexpr int e2(int t) {
    int before = 0, full = 0;
    for (int u = 0; u < 4; ++u) {
      full += nv2<W>(u) == 4;
      if (u < t && (nv2<W>(u) == 4) == (nv2<W>(t) == 4)) before += nv2<W>(u);
    }
    return before + (nv2<W>(t) == 4 ? 0 : 4 * full);
  }
  static __device__ __forceinline__ constexpr int e3(int t) {
    int before = 0, full = 0;
    for (int u = 0; u < 8; ++u) {
      full += nv3<W>(u >> 2, u & 3) == 4;
      if (u < t && (nv3<W>(u >> 2, u & 3) == 4) == (nv3<W>(t >> 2, t & 3) == 4)) before += nv3<W>(u >> 2, u & 3);
    }
    return before + (nv3<W>(t >> 2, t & 3) == 4 ? 0 : 4 * full);
  }
  // compact column of slot p
  static __device__ __forceinline__ int col2(int p) {
    const int t = p >> 4;
    return 4 * (t == 0 ? e2(0) : t == 1 ? e2(1) : t == 2 ? e2(2) : e2(3)) + (p & 15);
  }
  static __device__ __forceinline__ int col3(int p) {  // -1 for padding slots
    const int t = p >> 4;
    int e = 0, n = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (t == u) {
        e = e3(u);
        n = nv3<W>(u >> 2, u & 3);
      }
    return (p & 15) < 4 * n ? 4 * e + (p & 15) : -1;
  }
};

// What bounds the FP64 kernels is the FP64 pipe: matrix and vector FP64
// instructions do not overlap on a SIMD (16x16x4 64 cycles, 4x4x4 16, a vector
// operation 4), and a third wave per SIMD (12-wave work-groups) changed
// nothing (forward 460 -> 461 us).  So the work itself was cut: products whose
// tile holds three or fewer elements as 4x4x4 ones, and a tanh of 16 FP64
// operations (tanh_lut).  water12k: forward 518 -> 460 us (577 -> 513 with the
// activation store), backward 887 -> 782 us (583 -> 522 with the store).

// z += A B for the nv elements of a tile that hold slots and k element k of
// nk, blk at the tile's first element (e0 16 nk from the operand's start); nv
// is a constant once the loops are unrolled.  A 16x16x4 product takes 64
// cycles whatever its rows hold, a 4x4x4 one 16 per element.
__device__ __forceinline__ d4 mfma_f64_el(int nv, const double* blk, int nk, int k, int lane, int lo4, double b, d4 z) {
  if (nv == 4) return mfma_f64(blk[64 * k + lane], b, z);
#pragma unroll
  for (int e = 0; e < nv; ++e) z[e] = mfma4_f64(blk[16 * (e * nk + k) + lo4], b, z[e]);
  return z;
}

template <int W>
__device__ __forceinline__ int slot2d_of_feat(int f) {  // f in [0, 2W), FP64 layout
  if (kDense2<W> && f == 2 * W - 1) return W;
  return slot2_of_feat<W>(f);
}
template <int W>
__device__ __forceinline__ int feat3d_of_slot(int p) {  // FP64 layout; -1 for padding slots
  if constexpr (kDense2<W>) {
    const int q = p & 63;
    if (q >= W - 1 && q < W + 3) return p < 64 ? (W - 1) + W * (q - (W - 1)) : -1;
    if (q >= 32 + W - 1) return -1;
  }
  return feat3_of_slot<W>(p);
}

}  // namespace dpse
