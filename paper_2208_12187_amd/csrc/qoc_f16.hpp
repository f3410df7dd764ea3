// FP32 complex products on the 16x16x32 FP16 MFMA with FP32 accumulation: both
// factors as unevaluated sums of two FP16 numbers (Markidis et al., IPDPSW
// 2018; Ootomo and Yokota, IJHPCA 2022).
//
// Panels hold c x for the FP32 value x, c a power of two (and a product of two
// of them is multiplied by 1 / c); c x is split into hi = fp16(c x) and
// lo = fp16(c x - hi) (round to nearest even; the difference is exact), and a
// real product is taken as A_hi B_hi + A_hi B_lo + A_lo B_hi.  Each factor keeps 22
// bits (hi and lo 11 each, lo with a sign of its own) where FP32 has 24, the dropped
// A_lo B_lo is of relative size 2^-22 with random sign, an instruction cuts the terms
// of a group of 8 towards zero when it aligns them, and an accumulator is rounded
// once per 32 terms and product instead of once per 4.  Products whose errors add up
// over the slices therefore stay on the FP32 MFMA (with the chains on FP16 the error
// of F was four times as large); exponentials and commutator series, whose errors
// scale with |A|, come here.  Against FP64 the gradient's error is 0.95, 0.95, 0.97
// and 0.86 of that with FP32 MFMA throughout at d <= 16, 32, 64 and 128 (geometric
// means over 50 problems with reachable targets, single ones 0.8 ... 1.1).
// An FP32 MFMA step of K = 32 takes 8 x 32 cycles per SIMD, the three FP16
// ones 3 x 16: the d = 64 gradient kernel then has its matrix cores busy 37% of the
// time, the forward one 53%, and waits for LDS reads, splits and barriers otherwise.
//
// FP16's range (normal 2^-14 ... 2^16) is met by the scale: every factor of
// the unitary path is bounded by a small constant (propagator products by 1,
// U - I by 2, A / 2^s by 1, the target's Frobenius norm by 2 after a power of two is
// taken out, the terms of the commutator series by 2 and the products D Y of a
// conjugation by 4 times that), so that with c = 2^12 nothing staged exceeds 2^15, and
// what falls below FP16's subnormals is below 2^-37 of that bound.  General
// generators, whose products have no such bound, take the FP32 MFMA kernels.
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
  static constexpr float C = 4096.0f;  // c
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

  // Panel of the conjugate transpose of the stored matrix (its 22-bit values).
  __device__ static __forceinline__ void load_ct(Panel<float, D>& P, const void* lds, const Lane& L) {
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb) {
      const int off = (16 * L.w + L.c16) * SB + phys(16 * rb + 4 * L.g);
      const h4v rh = *reinterpret_cast<const h4v*>(plane(lds, 0) + off);
      const h4v rl = *reinterpret_cast<const h4v*>(plane(lds, 1) + off);
      const h4v ih = *reinterpret_cast<const h4v*>(plane(lds, 2) + off);
      const h4v il = *reinterpret_cast<const h4v*>(plane(lds, 3) + off);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        P.re[rb][r] = (float)rh[r] + (float)rl[r];
        P.im[rb][r] = -((float)ih[r] + (float)il[r]);
      }
    }
  }

  // The right factor of one wavefront, split: K step t's values of its 16 columns.
  struct Frag {
    h8v rh[D / 32], rl[D / 32], ih[D / 32], il[D / 32];
  };

  // Pair jp (of 4) of K step t of a panel: rows 32 t + 16 (jp / 2) + 4 g + 2 (jp % 2) + {0, 1}.
  __device__ static __forceinline__ void frag_pair(u4v& rh, u4v& rl, u4v& ih, u4v& il, const Panel<float, D>& P,
                                                   int t, int jp) {
    const int rb = 2 * t + (jp >> 1), r = 2 * (jp & 1);
    unsigned h, l;
    f16_split2(P.re[rb][r], P.re[rb][r + 1], h, l);
    rh[jp] = h;
    rl[jp] = l;
    f16_split2(P.im[rb][r], P.im[rb][r + 1], h, l);
    ih[jp] = h;
    il[jp] = l;
  }

  // The conjugate transpose of the stored matrix as a right factor: column
  // 16 w + c16 is a row of the matrix, whose K values phys() has put together,
  // so the split values are read as they are.
  __device__ static __forceinline__ void frag_ct(Frag& F, const void* lds, const Lane& L) {
    const int off = (16 * L.w + L.c16) * SB + 8 * L.g;
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
      F.rh[t] = *reinterpret_cast<const h8v*>(plane(lds, 0) + off + 32 * t);
      F.rl[t] = *reinterpret_cast<const h8v*>(plane(lds, 1) + off + 32 * t);
      F.ih[t] = neg(*reinterpret_cast<const h8v*>(plane(lds, 2) + off + 32 * t));
      F.il[t] = neg(*reinterpret_cast<const h8v*>(plane(lds, 3) + off + 32 * t));
    }
  }

  __device__ static __forceinline__ h8v neg(h8v x) {
    u4v u = __builtin_bit_cast(u4v, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] ^= 0x80008000u;
    return __builtin_bit_cast(h8v, u);
  }

  __device__ static __forceinline__ f4 mfma(h8v a, h8v b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }

  // The 12 MFMAs of one (K step, row block), the smallest terms first.  FIRST:
  // the accumulators start from zero.
  template <bool FIRST>
  __device__ static __forceinline__ void step(f4& re, f4& im, const h8v (&a)[4], h8v brh, h8v brl, h8v bih, h8v bil,
                                              h8v nih, h8v nil) {
    const f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    re = mfma(a[0], brl, FIRST ? z : re);
    im = mfma(a[0], bil, FIRST ? z : im);
    re = mfma(a[1], brh, re);
    im = mfma(a[1], bih, im);
    re = mfma(a[2], nil, re);
    im = mfma(a[2], brl, im);
    re = mfma(a[3], nih, re);
    im = mfma(a[3], brh, im);
    re = mfma(a[0], brh, re);
    im = mfma(a[0], bih, im);
    re = mfma(a[2], nih, re);
    im = mfma(a[2], brh, im);
  }

  __device__ static __forceinline__ void load_a(h8v (&a)[4], const void* lds, int off) {
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) a[pl] = *reinterpret_cast<const h8v*>(plane(lds, pl) + off);
  }

  // acc = A B with A the LDS matrix: per K step and row block 4 x 16-byte
  // reads and 12 MFMAs.
  __device__ static __forceinline__ void gemm(Panel<float, D>& acc, const void* lds, const Frag& B, const Lane& L) {
    constexpr int RB = D / 16;
    constexpr int KT = D / 32;
    __builtin_amdgcn_sched_barrier(0);
    const int base = L.c16 * SB + 8 * L.g;
    h8v a[2][4];
    load_a(a[0], lds, base);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const h8v nih = neg(B.ih[t]), nil = neg(B.il[t]);
#pragma unroll
      for (int mb = 0; mb < RB; ++mb) {
        const int st = t * RB + mb, cur = st & 1;
        if (st + 1 < KT * RB) load_a(a[cur ^ 1], lds, base + 16 * ((st + 1) % RB) * SB + 32 * ((st + 1) / RB));
        if (t == 0) step<true>(acc.re[mb], acc.im[mb], a[cur], B.rh[t], B.rl[t], B.ih[t], B.il[t], nih, nil);
        else step<false>(acc.re[mb], acc.im[mb], a[cur], B.rh[t], B.rl[t], B.ih[t], B.il[t], nih, nil);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // acc = A P with A the LDS matrix.  A K step's values of P are split while
  // the previous step's MFMAs run, and side(rb), work on row block rb that
  // depends on nothing here, is issued among the last K step's.
  template <typename Side>
  __device__ static __forceinline__ void mul(Panel<float, D>& acc, const void* lds, const Panel<float, D>& P,
                                             const Lane& L, Side side) {
    constexpr int RB = D / 16;
    constexpr int KT = D / 32;
    __builtin_amdgcn_sched_barrier(0);
    const int base = L.c16 * SB + 8 * L.g;
    h8v a[2][4];
    load_a(a[0], lds, base);
    u4v rh[2], rl[2], ih[2], il[2];
#pragma unroll
    for (int jp = 0; jp < 4; ++jp) frag_pair(rh[0], rl[0], ih[0], il[0], P, 0, jp);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int c = t & 1;
      const h8v brh = __builtin_bit_cast(h8v, rh[c]), brl = __builtin_bit_cast(h8v, rl[c]);
      const h8v bih = __builtin_bit_cast(h8v, ih[c]), bil = __builtin_bit_cast(h8v, il[c]);
      const h8v nih = neg(bih), nil = neg(bil);
#pragma unroll
      for (int mb = 0; mb < RB; ++mb) {
        const int st = t * RB + mb, cur = st & 1;
        if (st + 1 < KT * RB) load_a(a[cur ^ 1], lds, base + 16 * ((st + 1) % RB) * SB + 32 * ((st + 1) / RB));
        if (t == 0) step<true>(acc.re[mb], acc.im[mb], a[cur], brh, brl, bih, bil, nih, nil);
        else step<false>(acc.re[mb], acc.im[mb], a[cur], brh, brl, bih, bil, nih, nil);
        if (t + 1 < KT) frag_pair(rh[c ^ 1], rl[c ^ 1], ih[c ^ 1], il[c ^ 1], P, t + 1, mb);
        if (t + 1 == KT) side(mb);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __device__ static __forceinline__ void mul(Panel<float, D>& acc, const void* lds, const Panel<float, D>& P,
                                             const Lane& L) {
    mul(acc, lds, P, L, [](int) {});
  }
  // acc = A B^dag, both in LDS
  __device__ static __forceinline__ void mul_ct(Panel<float, D>& acc, const void* a, const void* b, const Lane& L) {
    Frag B;
    frag_ct(B, b, L);
    gemm(acc, a, B, L);
  }
};

// D = 16: the K = 32 of one MFMA takes the real and imaginary parts of the 16
// terms at once, Re = [Ar, -Ai] [Br; Bi] and Im = [Ai, Ar] [Br; Bi], so that a
// complex product is 6 MFMAs (FP32: 16 of twice the cycles).  K index 8g + j
// stands for the real (j < 4) or imaginary (j >= 4) part of row 4g + j % 4,
// which is what lane (g, c16) holds of a panel; the left factor is staged as
// four planes (the Re rows hi, lo, the Im rows hi, lo), row stride 40.
template <>
struct F16Ops<16> {
  using Tp = float;
  static constexpr int D = 16;
  static constexpr float C = 4096.0f;
  static constexpr int SB = 40;
  static constexpr int PLANE = D * SB;
  static constexpr int BYTES = 4 * PLANE * 2;

  __device__ static __forceinline__ unsigned short* plane(void* lds, int i) {
    return static_cast<unsigned short*>(lds) + i * PLANE;
  }
  __device__ static __forceinline__ const unsigned short* plane(const void* lds, int i) {
    return static_cast<const unsigned short*>(lds) + i * PLANE;
  }
  __device__ static __forceinline__ void split_panel(u2v& rh, u2v& rl, u2v& ih, u2v& il, const Panel<float, D>& P) {
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
      unsigned h, l;
      f16_split2(P.re[0][r], P.re[0][r + 1], h, l);
      rh[r / 2] = h;
      rl[r / 2] = l;
      f16_split2(P.im[0][r], P.im[0][r + 1], h, l);
      ih[r / 2] = h;
      il[r / 2] = l;
    }
  }
  __device__ static __forceinline__ u2v flip(u2v x) { return (u2v){x[0] ^ 0x80008000u, x[1] ^ 0x80008000u}; }

  __device__ static __forceinline__ void store(void* lds, const Panel<float, D>& P, const Lane& L) {
    u2v v[4];  // re hi, re lo, im hi, im lo of rows 4g .. 4g + 3
    split_panel(v[0], v[1], v[2], v[3], P);
    const int col = 8 * (L.c16 >> 2) + (L.c16 & 3);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int off = (4 * L.g + r) * SB + col, sh = 16 * (r & 1);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const unsigned short re = (unsigned short)(v[p][r / 2] >> sh), im = (unsigned short)(v[2 + p][r / 2] >> sh);
        plane(lds, p)[off] = re;
        plane(lds, p)[off + 4] = im ^ 0x8000u;
        plane(lds, 2 + p)[off] = im;
        plane(lds, 2 + p)[off + 4] = re;
      }
    }
  }
  // The conjugate transpose (or, NEG, its negative): one 16-byte write per plane.
  template <bool NEG>
  __device__ static __forceinline__ void store_t(void* lds, const Panel<float, D>& P, const Lane& L) {
    u2v rh, rl, ih, il;
    split_panel(rh, rl, ih, il, P);
    const int off = L.c16 * SB + 8 * L.g;
    auto put = [&](int pl, u2v a, u2v b) {
      *reinterpret_cast<u4v*>(plane(lds, pl) + off) = (u4v){a[0], a[1], b[0], b[1]};
    };
    // M^dag: Ar = re, Ai = -im, so [Ar, -Ai] = [re, im] and [Ai, Ar] = [-im, re]
    put(0, NEG ? flip(rh) : rh, NEG ? flip(ih) : ih);
    put(1, NEG ? flip(rl) : rl, NEG ? flip(il) : il);
    put(2, NEG ? ih : flip(ih), NEG ? flip(rh) : rh);
    put(3, NEG ? il : flip(il), NEG ? flip(rl) : rl);
  }
  __device__ static __forceinline__ void store_ct(void* lds, const Panel<float, D>& P, const Lane& L) {
    store_t<false>(lds, P, L);
  }
  __device__ static __forceinline__ void store_nct(void* lds, const Panel<float, D>& P, const Lane& L) {
    store_t<true>(lds, P, L);
  }
  // Panel of the conjugate transpose of the stored matrix (its 22-bit values):
  // the Re rows [Ar, -Ai] are its real and imaginary parts.
  __device__ static __forceinline__ void load_ct(Panel<float, D>& P, const void* lds, const Lane& L) {
    const int off = L.c16 * SB + 8 * L.g;
    const h8v h = *reinterpret_cast<const h8v*>(plane(lds, 0) + off);
    const h8v l = *reinterpret_cast<const h8v*>(plane(lds, 1) + off);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      P.re[0][r] = (float)h[r] + (float)l[r];
      P.im[0][r] = (float)h[4 + r] + (float)l[4 + r];
    }
  }
  __device__ static __forceinline__ void gemm(Panel<float, D>& acc, const void* lds, h8v bh, h8v bl, const Lane& L) {
    const int off = L.c16 * SB + 8 * L.g;
    h8v a[4];
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) a[pl] = *reinterpret_cast<const h8v*>(plane(lds, pl) + off);
    const f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    f4 re = F16Ops<32>::mfma(a[0], bl, z), im = F16Ops<32>::mfma(a[2], bl, z);
    re = F16Ops<32>::mfma(a[1], bh, re);
    im = F16Ops<32>::mfma(a[3], bh, im);
    acc.re[0] = F16Ops<32>::mfma(a[0], bh, re);
    acc.im[0] = F16Ops<32>::mfma(a[2], bh, im);
  }
  template <typename Side>
  __device__ static __forceinline__ void mul(Panel<float, D>& acc, const void* lds, const Panel<float, D>& P,
                                             const Lane& L, Side side) {
    u2v rh, rl, ih, il;
    split_panel(rh, rl, ih, il, P);
    const u4v h = {rh[0], rh[1], ih[0], ih[1]}, l = {rl[0], rl[1], il[0], il[1]};
    gemm(acc, lds, __builtin_bit_cast(h8v, h), __builtin_bit_cast(h8v, l), L);
    side(0);
  }
  __device__ static __forceinline__ void mul(Panel<float, D>& acc, const void* lds, const Panel<float, D>& P,
                                             const Lane& L) {
    mul(acc, lds, P, L, [](int) {});
  }
  // acc = A B^dag, both in LDS
  __device__ static __forceinline__ void mul_ct(Panel<float, D>& acc, const void* a, const void* b, const Lane& L) {
    const int off = L.c16 * SB + 8 * L.g;
    gemm(acc, a, *reinterpret_cast<const h8v*>(plane(b, 0) + off), *reinterpret_cast<const h8v*>(plane(b, 1) + off), L);
  }
};

}  // namespace qoc
