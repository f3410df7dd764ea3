// FP32 complex products on the 16x16x32 FP16 MFMA with FP32 accumulation: both
// factors as unevaluated sums of two FP16 numbers (Markidis et al., IPDPSW
// 2018; Ootomo and Yokota, IJHPCA 2022).
//
// Panels hold c x for the FP32 value x, c a power of two (and a product of two
// of them is multiplied by 1 / c); c x is split into hi = fp16(c x) and
// lo = fp16(c x - hi) (round to nearest even; the difference is exact), and a
// real product is taken as A_hi B_hi + A_hi B_lo + A_lo B_hi.  Each factor keeps 22 bits and a sign of
// lo, the dropped A_lo B_lo is of relative size 2^-22 with random sign, and
// K = 32 terms are summed per instruction, so that an accumulator is rounded
// once per 32 terms and product instead of once per 4: against FP64 the error of
// a d = 64 complex product of unitaries is below that of the FP32 MFMA's.
// An FP32 MFMA step of K = 32 takes 8 x 32 cycles per SIMD, the three FP16
// ones 3 x 16, which moves the d = 64 kernels from the matrix cores' rate to
// that of HBM.
//
// FP16's range (normal 2^-14 ... 2^16) is met by the scale: every factor of
// the unitary path is bounded by a small constant (propagator products by 1,
// U - I by 2, A / 2^s by 1, the target is normalised by a power of two, and
// the Frechet block's entries stay below a few times the target's), so that
// with c = 2^12 nothing overflows, and what falls below FP16's subnormals is
// below 2^-37 of that bound.  General generators, whose products have no
// such bound, take the FP32 MFMA kernels.
//
// The operand layouts are those of the split-BF16 products: register panels
// stay FP32 in the accumulator layout (rows 16 rb + 4g + r); for K step t the
// B operand of lane (g, c16) is the 8 values of row blocks 2t and 2t + 1 it
// holds, K index 8g + j standing for matrix row 32t + 16 (j / 4) + 4g + j % 4;
// the left factor is staged in LDS as four planes (re hi, re lo, im hi,
// im lo), row stride D + 8, with the columns of each 32-column block permuted
// by phys() so that those 8 K values of a row are one 16-byte read.
#pragma once

#include "qoc_bf16.hpp"

namespace qoc {

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));

constexpr float kF16Scale = 4096.0f;  // c
constexpr float kF16Inv = 1.0f / kF16Scale;

// Two scaled values at once; element 0 sits in the low 16 bits of the packed
// results.  (The opaque factor 1 keeps x - hi one v_fma_mix_f32, which reads
// hi as FP16, instead of a conversion and a subtraction.)
__device__ __forceinline__ void f16_split2(float x0, float x1, unsigned& hi, unsigned& lo) {
  const f2v v = {x0, x1};
  const h2v h = __builtin_convertvector(v, h2v);
  float one = 1.0f;
  asm("" : "+v"(one));
  const f2v r = {fmaf(x0, one, -(float)h[0]), fmaf(x1, one, -(float)h[1])};
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector(r, h2v));
}

template <int D>
struct F16Ops {
  using Tp = float;
  static constexpr int SB = D + 8;     // row stride in FP16 elements
  static constexpr int PLANE = D * SB;  // elements per plane
  static constexpr int BYTES = 4 * PLANE * 2;
  static_assert(D % 32 == 0, "K steps of 32");

  __device__ static __forceinline__ int phys(int c) { return Bf3Ops<D>::phys(c); }
  __device__ static __forceinline__ unsigned short* plane(void* lds, int i) {
    return static_cast<unsigned short*>(lds) + i * PLANE;
  }
  __device__ static __forceinline__ const unsigned short* plane(const void* lds, int i) {
    return static_cast<const unsigned short*>(lds) + i * PLANE;
  }

  __device__ static __forceinline__ void store(void* lds, const Panel<float, D>& P, const Lane& L) {
    const int pc = phys(16 * L.w + L.c16);
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        unsigned rh, rl, ih, il;
        f16_split2(P.re[rb][r], P.re[rb][r + 1], rh, rl);
        f16_split2(P.im[rb][r], P.im[rb][r + 1], ih, il);
        const int o0 = (16 * rb + 4 * L.g + r) * SB + pc, o1 = o0 + SB;
        plane(lds, 0)[o0] = (unsigned short)rh;
        plane(lds, 0)[o1] = (unsigned short)(rh >> 16);
        plane(lds, 1)[o0] = (unsigned short)rl;
        plane(lds, 1)[o1] = (unsigned short)(rl >> 16);
        plane(lds, 2)[o0] = (unsigned short)ih;
        plane(lds, 2)[o1] = (unsigned short)(ih >> 16);
        plane(lds, 3)[o0] = (unsigned short)il;
        plane(lds, 3)[o1] = (unsigned short)(il >> 16);
      }
  }

  // The conjugate transpose (SR = 1, SI = -1), or its negative (SR = -1,
  // SI = 1): the four rows of a row block are contiguous after phys(), so each
  // plane takes one 8-byte write instead of four 2-byte ones.
  template <bool NEG>
  __device__ static __forceinline__ void store_t(void* lds, const Panel<float, D>& P, const Lane& L) {
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb) {
      const int off = (16 * L.w + L.c16) * SB + phys(16 * rb + 4 * L.g);
      u2v rh, rl, ih, il;
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        unsigned h, l;
        f16_split2(P.re[rb][r], P.re[rb][r + 1], h, l);
        rh[r / 2] = NEG ? h ^ 0x80008000u : h;
        rl[r / 2] = NEG ? l ^ 0x80008000u : l;
        f16_split2(P.im[rb][r], P.im[rb][r + 1], h, l);
        ih[r / 2] = NEG ? h : h ^ 0x80008000u;
        il[r / 2] = NEG ? l : l ^ 0x80008000u;
      }
      *reinterpret_cast<u2v*>(plane(lds, 0) + off) = rh;
      *reinterpret_cast<u2v*>(plane(lds, 1) + off) = rl;
      *reinterpret_cast<u2v*>(plane(lds, 2) + off) = ih;
      *reinterpret_cast<u2v*>(plane(lds, 3) + off) = il;
    }
  }
  __device__ static __forceinline__ void store_ct(void* lds, const Panel<float, D>& P, const Lane& L) {
    store_t<false>(lds, P, L);
  }
  __device__ static __forceinline__ void store_nct(void* lds, const Panel<float, D>& P, const Lane& L) {
    store_t<true>(lds, P, L);
  }

  // The right factor of one wavefront, split: K step t's values of its 16 columns.
  struct Frag {
    h8v rh[D / 32], rl[D / 32], ih[D / 32], il[D / 32];
  };

  __device__ static __forceinline__ void frag(Frag& F, const Panel<float, D>& P) {
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
      u4v rh, rl, ih, il;
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) {
        const int rb = 2 * t + (jp >> 1), r = 2 * (jp & 1);
        unsigned h, l;
        f16_split2(P.re[rb][r], P.re[rb][r + 1], h, l);
        rh[jp] = h;
        rl[jp] = l;
        f16_split2(P.im[rb][r], P.im[rb][r + 1], h, l);
        ih[jp] = h;
        il[jp] = l;
      }
      F.rh[t] = __builtin_bit_cast(h8v, rh);
      F.rl[t] = __builtin_bit_cast(h8v, rl);
      F.ih[t] = __builtin_bit_cast(h8v, ih);
      F.il[t] = __builtin_bit_cast(h8v, il);
    }
  }

  // The conjugate transpose of the stored matrix, or its negative, as a right
  // factor: column 16 w + c16 is a row of the matrix, whose K values phys()
  // has put together, so the split values are read as they are.
  template <bool NEG>
  __device__ static __forceinline__ void frag_t(Frag& F, const void* lds, const Lane& L) {
    const int off = (16 * L.w + L.c16) * SB + 8 * L.g;
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
      F.rh[t] = *reinterpret_cast<const h8v*>(plane(lds, 0) + off + 32 * t);
      F.rl[t] = *reinterpret_cast<const h8v*>(plane(lds, 1) + off + 32 * t);
      F.ih[t] = *reinterpret_cast<const h8v*>(plane(lds, 2) + off + 32 * t);
      F.il[t] = *reinterpret_cast<const h8v*>(plane(lds, 3) + off + 32 * t);
      if (NEG) {
        F.rh[t] = neg(F.rh[t]);
        F.rl[t] = neg(F.rl[t]);
      } else {
        F.ih[t] = neg(F.ih[t]);
        F.il[t] = neg(F.il[t]);
      }
    }
  }
  __device__ static __forceinline__ void frag_ct(Frag& F, const void* lds, const Lane& L) { frag_t<false>(F, lds, L); }
  __device__ static __forceinline__ void frag_nct(Frag& F, const void* lds, const Lane& L) { frag_t<true>(F, lds, L); }

  __device__ static __forceinline__ h8v neg(h8v x) {
    u4v u = __builtin_bit_cast(u4v, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] ^= 0x80008000u;
    return __builtin_bit_cast(h8v, u);
  }

  __device__ static __forceinline__ f4 mfma(h8v a, h8v b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }

  // acc (+)= A B with A the LDS matrix.  Per K step and row block 4 x 16-byte reads and 12 MFMAs, the
  // smallest terms first.
  __device__ static __forceinline__ void gemm(Panel<float, D>& acc, const void* lds, const Frag& B,
                                                   const Lane& L, bool zero_acc) {
    constexpr int RB = D / 16;
    constexpr int KT = D / 32;
    __builtin_amdgcn_sched_barrier(0);
    if (zero_acc) panel_zero(acc);
    const int base = L.c16 * SB + 8 * L.g;
    h8v a[2][4];
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) a[0][pl] = *reinterpret_cast<const h8v*>(plane(lds, pl) + base);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const h8v brh = B.rh[t], brl = B.rl[t], bih = B.ih[t], bil = B.il[t];
      const h8v nih = neg(bih), nil = neg(bil);
#pragma unroll
      for (int mb = 0; mb < RB; ++mb) {
        const int st = t * RB + mb, cur = st & 1;
        if (st + 1 < KT * RB) {
          const int off = base + 16 * ((st + 1) % RB) * SB + 32 * ((st + 1) / RB);
#pragma unroll
          for (int pl = 0; pl < 4; ++pl) a[cur ^ 1][pl] = *reinterpret_cast<const h8v*>(plane(lds, pl) + off);
        }
        const h8v arh = a[cur][0], arl = a[cur][1], aih = a[cur][2], ail = a[cur][3];
        f4 re = acc.re[mb], im = acc.im[mb];
        re = mfma(arh, brl, re);
        im = mfma(arh, bil, im);
        re = mfma(arl, brh, re);
        im = mfma(arl, bih, im);
        re = mfma(aih, nil, re);
        im = mfma(aih, brl, im);
        re = mfma(ail, nih, re);
        im = mfma(ail, brh, im);
        re = mfma(arh, brh, re);
        im = mfma(arh, bih, im);
        re = mfma(aih, nih, re);
        im = mfma(aih, brh, im);
        acc.re[mb] = re;
        acc.im[mb] = im;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  __device__ static __forceinline__ void gemm(Panel<float, D>& acc, const void* lds, const Panel<float, D>& P,
                                                     const Lane& L, bool zero_acc) {
    Frag B;
    frag(B, P);
    gemm(acc, lds, B, L, zero_acc);
  }
};

}  // namespace qoc
