// Hermitian path at d = 128 in FP32: the segments of the d <= 64 path (see
// qoc_kernels.hip) with one workgroup of eight wavefronts per segment.
//
// One FP32 matrix as split FP16 planes is 136 KB, so that the LDS holds the one
// left factor and an exchange buffer, and a wavefront's 256 registers hold
// three panels (its 16 columns, 64 registers each) and the product's operands.
// The commutator series is therefore summed by Horner's rule, which keeps Y,
// the running sum R and the product:
//   R <- Y + [A, R] / n  for n = m, ..., 2 (from R = Y) gives Z,
//   and n = 1 gives the next slice's Y:  sum_n C_n / n! = Y + [A, Z].
// [A, R] = A R + (A R)^dag takes the transposed blocks of the other wavefronts'
// panels, which go through the exchange buffer in four rounds: in round j
// wavefront w meets the two of pair (w / 2) ^ j.  So that the registers of a
// round are the same in every wavefront, panel index i of wavefront w stands
// for row block i ^ (w & 6).
//
// A slice takes m products of 12288 MFMA cycles per SIMD (5.1 us) and nothing
// per order from memory.  Measured at m = 14 controls, N = 1000, eight problems:
// gradient 2.38 ms (8 us per product with its exchange, 0.3 ms in all, and the
// splitting; assembly 0.29, traces 0.1), forward 1.84 ms (the FP32 chain product
// 0.57).  The block form took X^2, S, W and three products per two orders with
// its chain state in global scratch (6.96 ms), a scan each way (2.0) and 2.28 for
// the exponentials.
//
// Included by qoc_kernels.hip.
#pragma once

struct S128 {
  static constexpr int NT = 512;
  static constexpr float C = 4096.0f, CI = 1.0f / 4096.0f, CI2 = CI * CI;
  static constexpr int PLANE = 128 * 256;        // bytes of a plane
  static constexpr int PLANES = 4 * PLANE;
  static constexpr int XBLK = 2 * 256;           // floats of an exchanged 16 x 16 block
  static constexpr int BYTES = PLANES + 16 * XBLK * 4;  // all of the 160 KB
  static constexpr int SD = 132;                 // row stride of a planar FP32 matrix
};
static_assert(2 * 128 * S128::SD * 4 <= S128::BYTES, "FP32 matrix");
static_assert(S128::BYTES <= 160 * 1024, "LDS");

using Panel128 = Panel<float, 128>;

// The wavefront's index as a scalar; the row block of panel index i.
__device__ __forceinline__ int wave128() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
__device__ __forceinline__ int px_rb(int i) { return i ^ (wave128() & 6); }

// A plane of the left factor: rows of 256 bytes, K step T's 16 bytes of lane
// group g (8 values: rows 4g ... of row blocks 2T and 2T + 1 of the right factor)
// at unit (4 T + g) ^ (row % 16), which spreads the 16 rows that a read takes at
// once over all banks whichever lanes are served together.
__device__ __forceinline__ int px_unit(int row16, int T, int g) { return 16 * ((4 * T + g) ^ row16); }

// This wavefront's panel of a PF matrix in the permuted order.
__device__ __forceinline__ void px_load(Panel128& P, const float* M, const Lane& L) {
  const int w = wave128();
#pragma unroll
  for (int i = 0; i < 8; ++i) pf_rb_load<float>(P.re[i], P.im[i], M, w, px_rb(i), L.lane);
}
__device__ __forceinline__ void px_store(float* M, const Panel128& P, const Lane& L) {
  const int w = wave128();
#pragma unroll
  for (int i = 0; i < 8; ++i) pf_rb_store<float>(M, P.re[i], P.im[i], w, px_rb(i), L.lane);
}
__device__ __forceinline__ void px_add_identity(f4& re, int i, const Lane& L, float a) {  // to index i
  if (i > 1) return;  // the diagonal block is index w % 2
  const float x = (wave128() & 1) == i ? a : 0.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (4 * L.g + r == L.c16) re[r] += x;
}

// ---------------------------------------------------------------- left factors

// The planes of C M from the panel of M: M = -M^dag (SGN = -1) or M = M^dag
// (SGN = 1), one 8-byte write per plane and row block.
template <int SGN>
__device__ __forceinline__ void px_stage_sym(void* lds, const Panel128& P, const Lane& L) {
  unsigned char* p = static_cast<unsigned char*>(lds) + (16 * L.w + L.c16) * 256;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    unsigned char* q = p + px_unit(L.c16, px_rb(i) >> 1, L.g) + 8 * (i & 1);
    u2v v[4];
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
      unsigned h, l;
      f16_split2(S128::C * P.re[i][r], S128::C * P.re[i][r + 1], h, l);
      v[0][r / 2] = SGN < 0 ? h ^ 0x80008000u : h;
      v[1][r / 2] = SGN < 0 ? l ^ 0x80008000u : l;
      f16_split2(S128::C * P.im[i][r], S128::C * P.im[i][r + 1], h, l);
      v[2][r / 2] = SGN < 0 ? h : h ^ 0x80008000u;
      v[3][r / 2] = SGN < 0 ? l : l ^ 0x80008000u;
    }
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) *reinterpret_cast<u2v*>(q + pl * S128::PLANE) = v[pl];
    if (i & 1) __builtin_amdgcn_sched_barrier(0);
  }
}

// The planes of C M, f(i, re, im) giving index i of the panel of C M.
template <typename Fn>
__device__ __forceinline__ void px_stage(void* lds, const Lane& L, Fn f) {
  unsigned char* p = static_cast<unsigned char*>(lds) + 8 * (L.w & 1) + 2 * (L.c16 & 3);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    f4 re, im;
    f(i, re, im);
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
      unsigned v[4];
      f16_split2(re[r], re[r + 1], v[0], v[1]);
      f16_split2(im[r], im[r + 1], v[2], v[3]);
      const int row = 4 * L.g + r, o = 16 * px_rb(i) * 256;
      const int o0 = o + row * 256 + px_unit(row, L.w >> 1, L.c16 >> 2);
      const int o1 = o + (row + 1) * 256 + px_unit(row + 1, L.w >> 1, L.c16 >> 2);
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) {
        *reinterpret_cast<unsigned short*>(p + pl * S128::PLANE + o0) = (unsigned short)v[pl];
        *reinterpret_cast<unsigned short*>(p + pl * S128::PLANE + o1) = (unsigned short)(v[pl] >> 16);
      }
    }
    if (i & 1) __builtin_amdgcn_sched_barrier(0);
  }
}

// ---------------------------------------------------------------- products

// A right factor, split: K step t holds panel indices 2t and 2t + 1, row blocks
// 2T and 2T + 1 with T = t ^ (w / 2).
struct Frag128 {
  u4v rh[4], rl[4], ih[4], il[4];
};

// Indices 2t and 2t + 1 from their values times C.
__device__ __forceinline__ void frag_put(Frag128& F, int t, const f4 (&a)[2], const f4 (&b)[2]) {
#pragma unroll
  for (int jp = 0; jp < 4; ++jp) {
    const int h = jp >> 1, r = 2 * (jp & 1);
    unsigned x, y;
    f16_split2(a[h][r], a[h][r + 1], x, y);
    F.rh[t][jp] = x;
    F.rl[t][jp] = y;
    f16_split2(b[h][r], b[h][r + 1], x, y);
    F.ih[t][jp] = x;
    F.il[t][jp] = y;
  }
}

// f(i, re, im): index i of the panel, times C.
template <typename Fn>
__device__ __forceinline__ void frag_from(Frag128& F, Fn f) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f4 re[2], im[2];
    f(2 * t, re[0], im[0]);
    f(2 * t + 1, re[1], im[1]);
    frag_put(F, t, re, im);
    __builtin_amdgcn_sched_barrier(0);
  }
}
__device__ __forceinline__ void frag_panel(Frag128& F, const Panel128& P, float c) {
  frag_from(F, [&](int i, f4& re, f4& im) {
    re = (c * S128::C) * P.re[i];
    im = (c * S128::C) * P.im[i];
  });
}

// acc = C^2 M B, M in LDS: per K step and row block 4 x 16-byte reads and 12 MFMAs.
__device__ __forceinline__ void px_mul(Panel128& acc, const void* lds, const Frag128& B, const Lane& L) {
  using O = F16Ops<32>;
  const unsigned char* p = static_cast<const unsigned char*>(lds);
  const int w = wave128(), own = L.c16 * 256 + 16 * (L.g ^ L.c16);
  auto load = [&](h8v (&a)[4], int st) {
    const int off = (own ^ (64 * ((st >> 3) ^ (w >> 1)))) + 4096 * ((st & 7) ^ (w & 6));
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) a[pl] = *reinterpret_cast<const h8v*>(p + pl * S128::PLANE + off);
  };
  __builtin_amdgcn_sched_barrier(0);
  h8v a[2][4];
  load(a[0], 0);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const h8v brh = __builtin_bit_cast(h8v, B.rh[t]), brl = __builtin_bit_cast(h8v, B.rl[t]);
    const h8v bih = __builtin_bit_cast(h8v, B.ih[t]), bil = __builtin_bit_cast(h8v, B.il[t]);
    const h8v nih = O::neg(bih), nil = O::neg(bil);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int st = 8 * t + i, cur = st & 1;
      if (st + 1 < 32) load(a[cur ^ 1], st + 1);
      if (t == 0) O::step<true>(acc.re[i], acc.im[i], a[cur], brh, brl, bih, bil, nih, nil);
      else O::step<false>(acc.re[i], acc.im[i], a[cur], brh, brl, bih, bil, nih, nil);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// f(i, tr, ti) receives index i of the panel of P^dag.  Starts with no barrier
// (the buffer's last use was an exchange) and ends with one.  A block's column c
// is stored at position 4 (c % 4) + c / 4, its four row groups in an order that
// spreads writes and reads over the banks.
template <typename Fn>
__device__ __forceinline__ void px_exchange(const Panel128& P, float* xb, const Lane& L, Fn f) {
  const int w = wave128();
  float* own = xb + 2 * w * S128::XBLK + 16 * (4 * (L.c16 & 3) + (L.c16 >> 2)) + 4 * (L.g ^ (L.c16 & 3));
  const float* oth = xb + (w & 1) * S128::XBLK + 16 * L.g + (L.c16 & 3);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // row block of wavefront 2 ((w / 2) ^ j) + h
      *reinterpret_cast<f4*>(own + h * S128::XBLK) = P.re[2 * j + h];
      *reinterpret_cast<f4*>(own + h * S128::XBLK + 256) = P.im[2 * j + h];
    }
    __syncthreads();
    f4 tr[2], ti[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* o = oth + 2 * (2 * ((w >> 1) ^ j) + h) * S128::XBLK;
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // column 4 g + r, row c16
        const int off = 64 * r + 4 * ((L.c16 >> 2) ^ r);
        tr[h][r] = o[off];
        ti[h][r] = -o[256 + off];
      }
    }
    __syncthreads();
    f(2 * j, tr[0], ti[0]);
    f(2 * j + 1, tr[1], ti[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ---------------------------------------------------------------- assembly

// X = -i c H_k (the sums of assemble()), H_k read back by rows: X = -X^dag.
// Starts and ends with a barrier.
__device__ __forceinline__ void px_assemble(Panel128& X, float* pl, const ProbDesc& P, int k, double c, bool mono,
                                            const Lane& L) {
  constexpr int D = 128, NT = S128::NT, NV = 8, SD = S128::SD;
  const float* H = reinterpret_cast<const float*>(P.Hint);
  float* pi = pl + D * SD;
  const int e0 = 4 * threadIdx.x;
  f4 hr[NV], hi[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    hr[v] = Prec<float>::gld4(H + e0 + 4 * NT * v);
    hi[v] = Prec<float>::gld4(H + D * D + e0 + 4 * NT * v);
  }
  if (!mono) {
    for (int j = 0; j < P.m; ++j) {
      const float uj = (float)gp(P.u)[(size_t)j * P.N + k];
      const float* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const f4 a = Prec<float>::gld4(Hj + 4 * NT * v), b = Prec<float>::gld4(Hj + D * D + 4 * NT * v);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          hr[v][r] = fmaf(uj, a[r], hr[v][r]);
          hi[v][r] = fmaf(uj, b[r], hi[v][r]);
        }
      }
    }
  }
  __syncthreads();  // the left factor's last readers are done
  {
    const int off = (threadIdx.x >> 5) * SD + 4 * (threadIdx.x & 31);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      Prec<float>::st4(pl + off + 16 * v * SD, hr[v]);
      Prec<float>::st4(pi + off + 16 * v * SD, hi[v]);
    }
  }
  __syncthreads();
  if (mono) {
    // the thread of row a adds the row's entry of each control in turn, four
    // controls' entries loaded together
    if ((int)threadIdx.x < D) {
      const int a = threadIdx.x;
      const float* mv = reinterpret_cast<const float*>(P.mval);
      int off = -1;
      float sr = 0, si = 0;
      for (int j0 = 0; j0 < P.m; j0 += 4) {
        int col[4];
        float vr[4], vi[4], uj[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = min(j0 + i, P.m - 1);
          const size_t idx = (size_t)j * D + a;
          col[i] = gp(P.mcol)[idx];
          vr[i] = gp(mv)[2 * idx];
          vi[i] = gp(mv)[2 * idx + 1];
          uj[i] = (float)gp(P.u)[(size_t)j * P.N + k];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (j0 + i < P.m) {
            const int o = a * SD + col[i];
            if (o != off) {
              if (off >= 0) {
                pl[off] = sr;
                pi[off] = si;
              }
              off = o;
              sr = pl[o];
              si = pi[o];
            }
            sr = fmaf(uj[i], vr[i], sr);
            si = fmaf(uj[i], vi[i], si);
          }
        }
      }
      pl[off] = sr;
      pi[off] = si;
    }
    __syncthreads();
  }
  // c in two numbers (as in assemble_panel)
  const float f = (float)c, fl = (float)(c - (double)f);
  const int w = wave128();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int off = (16 * L.w + L.c16) * SD + 16 * px_rb(i) + 4 * L.g;
    const f4 a = Prec<float>::ld4(pl + off), b = Prec<float>::ld4(pi + off);
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // H[row][col] = conj(H[col][row])
      X.re[i][r] = -fmaf(f, b[r], fl * b[r]);
      X.im[i][r] = -fmaf(f, a[r], fl * a[r]);
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------- exponential

// X <- exp(A) - I from the panel X = A / 2^s, whose planes are staged (and are
// replaced): Paterson-Stockmeyer with A2 = X X as the step, so that only X, the
// running C and the product are held,
//   p(X) - I = X + A2 C,  C = sum_{n=2..q} X^(n-2) / n!,  C <- D_t + A2 C,
//   D_t = I / (2t+2)! + X / (2t+3)!,
// expm_products(q) products, then s squarings.  (The degree-8 form in three
// products holds four panels: through global scratch it took 120 us per slice
// and compute unit.)
__device__ __forceinline__ void px_taylor(Panel128& X, void* lds, int s, int q, const Lane& L) {
  constexpr float C = S128::C, CI = S128::CI, CI2 = S128::CI2;
  const int n = expm_products(q), top = (q - 2) / 2;
  const bool even = (q & 1) == 0;
  Frag128 F;
  Panel128 acc;
#pragma unroll 1
  for (int i = 0; i < n + s; ++i) {  // one instance of the product: registers and instruction cache
    const bool square = i >= n;
    if (square) {
      __syncthreads();
      px_stage(lds, L, [&](int b, f4& re, f4& im) {
        re = C * X.re[b];
        im = C * X.im[b];
      });
    }
    if (square || i == 0) {
      frag_panel(F, X, 1.0f);
      __syncthreads();
    }
    px_mul(acc, lds, F, L);
    if (square || i == n - 1) {
      const float x = square ? 2.0f : 1.0f, f = !square && q == 2 ? 0.5f * CI2 : CI2;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        X.re[b] = x * X.re[b] + f * acc.re[b];
        X.im[b] = x * X.im[b] + f * acc.im[b];
      }
    } else {
      // C = I / (q-2)! + X / (q-1)! + A2 / q! or I / (q-1)! + X / q!, then D_t + A2 C
      float c0, c1, c2;
      if (i == 0) {
        panel_scale(acc, CI2);
        __syncthreads();
        px_stage_sym<1>(lds, acc, L);  // A2 = A2^dag
        __syncthreads();
        c0 = (float)inv_factorial(even ? q - 2 : q - 1);
        c1 = (float)inv_factorial(even ? q - 1 : q);
        c2 = even ? C * (float)inv_factorial(q) : 0.0f;
      } else {
        const int t = (even ? top - 1 : top) - i;
        c0 = (float)inv_factorial(2 * t + 2);
        c1 = (float)inv_factorial(2 * t + 3);
        c2 = CI;
      }
      frag_from(F, [&](int b, f4& re, f4& im) {
        re = (C * c1) * X.re[b] + c2 * acc.re[b];
        im = (C * c1) * X.im[b] + c2 * acc.im[b];
        px_add_identity(re, b, L, C * c0);
      });
    }
  }
}

// ---------------------------------------------------------------- forward

// S <- S + R S in FP32, R and S as panels; the planar R goes through lds.
// Starts with a barrier.
__device__ __forceinline__ void px_chain(Panel128& S, const Panel128& R, float* pl, const Lane& L) {
  constexpr int SD = S128::SD;
  float* pi = pl + 128 * SD;
  const int w = wave128();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int off = (16 * px_rb(i) + 4 * L.g + r) * SD + 16 * L.w + L.c16;
      pl[off] = R.re[i][r];
      pi[off] = R.im[i][r];
    }
  __syncthreads();
  // three real products: T1 = Rr Sr, T2 = Ri Si, T3 = (Rr + Ri)(Sr + Si)
  f4 t1[8], t2[8], t3[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) t1[i] = t2[i] = t3[i] = (f4){0, 0, 0, 0};
  const int base = L.c16 * SD + 4 * L.g;
  auto load = [&](f4& a, f4& b, int st) {
    const int off = base + 16 * px_rb(st & 7) * SD + 16 * px_rb(st >> 3);
    a = Prec<float>::ld4(pl + off);
    b = Prec<float>::ld4(pi + off);
  };
  f4 ar[2], ai[2];
  load(ar[0], ai[0], 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int st = 0; st < 64; ++st) {
    const int kb = st >> 3, mb = st & 7, cur = st & 1;
    if (st + 1 < 64) load(ar[cur ^ 1], ai[cur ^ 1], st + 1);
    const f4 as = ar[cur] + ai[cur], bs = S.re[kb] + S.im[kb];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      t1[mb] = Prec<float>::mfma(ar[cur][r], S.re[kb][r], t1[mb]);
      t2[mb] = Prec<float>::mfma(ai[cur][r], S.im[kb][r], t2[mb]);
      t3[mb] = Prec<float>::mfma(as[r], bs[r], t3[mb]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    S.re[i] += t1[i] - t2[i];
    S.im[i] += t3[i] - t1[i] - t2[i];
  }
}

// One item's region of the scratch; parts of an item have their own.
__device__ __forceinline__ float* slot_part(void* scratch, int i) {
  return static_cast<float*>(scratch) +
         ((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * kScratchMats + i) * K128<float>::ELEMS;
}

// The totals U_{kb-1} ... U_{ka} of the segments less I, into xprev at the
// segment's first slice: the exponential's products on the FP16 matrix cores, the
// chain's, whose errors add up over the N slices, in FP32.
__global__ __launch_bounds__(512) void k_seg_fwd128(Work W, void* scratch) {
  __shared__ __align__(16) unsigned char lds[2 * 128 * S128::SD * 4];
  Lane L;
  float* SS = slot_part(scratch, 0);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    const SegItem g = seg_split(item, W.rg, I, W.descs);
    if (g.ka < g.kb) {
      const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
      const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
      for (int k = g.ka; k < g.kb; ++k) {
        int s, q, qb;
        unpack_sq(gp(P.sq)[k], s, q, qb);
        Panel128 R;
        px_assemble(R, reinterpret_cast<float*>(lds), P, k, ldexp(P.dt, -s), mono, L);
        px_stage_sym<-1>(lds, R, L);
        __syncthreads();
        px_taylor(R, lds, s, q, L);
        Panel128 S;
        if (k == g.ka) {
          S = R;
          px_add_identity(S.re[0], 0, L, 1.0f);
          px_add_identity(S.re[1], 1, L, 1.0f);
        } else {
          px_load(S, SS, L);  // own panel
          px_chain(S, R, reinterpret_cast<float*>(lds), L);
        }
        if (k + 1 < g.kb) {
          px_store(SS, S, L);
        } else {
          px_add_identity(S.re[0], 0, L, -1.0f);
          px_add_identity(S.re[1], 1, L, -1.0f);
          px_store(pf_mat<float, 128>(P.xprev, g.ka - W.rg.kbase), S, L);
        }
      }
    }
    __syncthreads();
  }
}

// Per chunk: the prefixes at its segment starts less I (into bloc at the
// segment's first slice) and the chunk total, re-unitarised where asked for.
__global__ __launch_bounds__(512) void k_seg_join128(Work W, void* scratch) {
  __shared__ __align__(16) float lds[K128<float>::LDS_ELEMS];
  __shared__ double red[8];
  Lane L;
  float* S0 = slot_part(scratch, 0);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int k1 = min(P.N, (c + 1) * P.L), h = seg_len(P.L, P.SM);
    Panel128 S;
    panel_load(S, pf_mat<float, 128>(P.xprev, c * P.L - W.rg.kbase), L);
    for (int k = c * P.L + h; k < k1; k += h) {  // S <- S + (T - I) S, as in k_seg_join
      panel_store(pf_mat<float, 128>(P.bloc, k - W.rg.kbase), S, L);
      panel_add_identity(S, L, 1.0f);
      panel_store(S0, S, L);
      gemm128<float, false>(S, lds, pf_mat<float, 128>(P.xprev, k - W.rg.kbase), S0, L, true);
      panel_axpy_pf(S, 1.0f, S0, L);
      panel_add_identity(S, L, -1.0f);
    }
    panel_add_identity(S, L, 1.0f);
    if (!W.rg.recompute) {
      panel_store(pf_mat<float, 128>(P.tf, c), S, L);
      if (P.reun_tol >= 0)
        reunitarise128(P, pf_mat<float, 128>(P.tf, c), pf_mat<float, 128>(P.cf, c), lds, red, L);
    }
    __syncthreads();
  }
}

// Per chunk, after the carry: Y at its start, as k_seg_y.
__global__ __launch_bounds__(512) void k_seg_y128(Work W, void* scratch) {
  __shared__ __align__(16) float lds[K128<float>::LDS_ELEMS];
  Lane L;
  float* S0 = slot_part(scratch, 0);
  float* S1 = slot_part(scratch, 1);
  float* S2 = slot_part(scratch, 2);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int g = c / P.CG;
    Panel128 a;
    gemm128<float, false>(a, lds, pf_mat<float, 128>(P.cf, c), grp_mat128<float>(P, 2, g), L, true);
    panel_store(S1, a, L);  // cf[c]
    gemm128<float, false>(a, lds, pf_mat<float, 128>(P.cb, c), grp_mat128<float>(P, 3, g), L, true);
    panel_store(S2, a, L);  // cb[c]
    transpose128<float>(S0, lds, S1, L);
    gemm128<float, false>(a, lds, S2, S0, L, true);
    panel_store(S1, a, L);  // cb cf^dag
    gemm128<float, true>(a, lds, pf_mat<float, 128>(P.tf, c), S1, L, true);  // N
    const bool raw = (P.flags & RUN_RAWDG) != 0;
    double wr = 1.0, wi = 0.0;
    if (!raw) {
      const double gr = gp(P.g)[0], gi = gp(P.g)[1], n = sqrt(gr * gr + gi * gi);
      if (n > 0) {
        wr = gr / n;
        wi = gi / n;
      }
    }
#pragma unroll
    for (int rb = 0; rb < 8; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double ar = (double)a.re[rb][r], ai = (double)a.im[rb][r];
        a.re[rb][r] = (float)(wr * ar - wi * ai);
        a.im[rb][r] = (float)(wr * ai + wi * ar);
      }
    panel_store(S0, a, L);
    transpose128<float>(S2, lds, S0, L);  // (w N)^dag
    for (int part = raw ? 1 : 0; part >= 0; --part) {
      float* out = pf_mat<float, 128>(part ? P.cb : P.mc, c);
#pragma unroll
      for (int rb = 0; rb < 8; ++rb) {
        f4 br, bi, yr, yi;
        pf_rb_load<float>(br, bi, S2, L.w, rb, L.lane);
        if (part) {
          yr = 0.5f * (a.re[rb] + br);
          yi = 0.5f * (a.im[rb] + bi);
        } else {
          yr = 0.5f * (a.im[rb] - bi);
          yi = 0.5f * (br - a.re[rb]);
        }
        pf_rb_store<float>(out, yr, yi, L.w, rb, L.lane);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- gradient

// V <- f U V U^dag = f (V + G + G^dag + D G^dag) for Hermitian V, G = D V,
// D = U - I a PF matrix (complete at the first barrier).
__device__ __forceinline__ void px_conjugate(Panel128& V, float f, unsigned char* lds, float* xb, const float* Dm,
                                             const Lane& L) {
  constexpr float CI = S128::CI, CI2 = S128::CI2;
  Frag128 F;
  Panel128 G;
  __syncthreads();
  {
    const int w = wave128();
    px_stage(lds, L, [&](int i, f4& re, f4& im) {
      pf_rb_load<float>(re, im, Dm, w, px_rb(i), L.lane);
      re = S128::C * re;
      im = S128::C * im;
    });
  }
  frag_panel(F, V, 1.0f);
  __syncthreads();
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    px_mul(G, lds, F, L);
    if (h == 0) {
      f4 pr[2], pq[2];
      px_exchange(G, xb, L, [&](int i, const f4& tr, const f4& ti) {
        V.re[i] += CI2 * (G.re[i] + tr);
        V.im[i] += CI2 * (G.im[i] + ti);
        pr[i & 1] = CI * tr;
        pq[i & 1] = CI * ti;
        if (i & 1) frag_put(F, i >> 1, pr, pq);
      });
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        V.re[i] = f * (V.re[i] + CI2 * G.re[i]);
        V.im[i] = f * (V.im[i] + CI2 * G.im[i]);
      }
    }
  }
}

// t_j = Tr(Hc[j] Z) of slice k, Z a PF matrix (complete after the last barrier).
// Row-table controls: thread t takes row t % 128 of controls t / 128 + 4 i, 16
// controls at a time; others: the wavefront's panel of Z against the rows of
// Hc[j], four controls at a time.  red: 64 doubles.
__device__ __forceinline__ void px_epilogue(const ProbDesc& P, int k, int part, const float* Z, double* red, bool mono,
                                            const Lane& L) {
  constexpr int D = 128;
  if (mono) {
    const int a = threadIdx.x & 127, jj = threadIdx.x >> 7;
    const int zoff = 4 * (a >> 4) + (a & 3), lane = 16 * ((a & 15) >> 2);
    const float* mv = reinterpret_cast<const float*>(P.mval);
    for (int j0 = 0, grp = 0; j0 < P.m; j0 += 16, ++grp) {
      double v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = j0 + jj + 4 * i;
        v[i] = 0;
        if (j < P.m) {
          const size_t e = (size_t)j * D + a;
          const int col = gp(P.mcol)[e];
          const double x = (double)gp(mv)[2 * e], y = (double)gp(mv)[2 * e + 1];
          const double zr = (double)gp(Z)[pf_index<float, D>(col >> 4, 0, zoff, lane + (col & 15))];
          const double zi = (double)gp(Z)[pf_index<float, D>(col >> 4, 1, zoff, lane + (col & 15))];
          v[i] = zr * x + zi * y;  // Re(conj(z) h)
        }
      }
      const double t = wave_sum_many<4>(v, L.lane);
      double* rg = red + (grp & 1) * 32;
      if ((L.lane & 15) == 0) rg[2 * (4 * (L.lane >> 4) + jj) + (L.w & 1)] = t;
      __syncthreads();
      if (threadIdx.x < 16 && j0 + (int)threadIdx.x < P.m)
        seg_grad_put(P, j0 + threadIdx.x, k, part, rg[2 * threadIdx.x] + rg[2 * threadIdx.x + 1]);
    }
    return;
  }
  const int w = wave128();
  for (int j0 = 0, grp = 0; j0 < P.m; j0 += 4, ++grp) {
    double v[4] = {0, 0, 0, 0};
#pragma unroll
    for (int rb = 0; rb < 8; ++rb) {
      f4 zr, zi;
      pf_rb_load<float>(zr, zi, Z, w, rb, L.lane);
      const int e = (16 * w + L.c16) * D + 16 * rb + 4 * L.g;  // Hc[j][col][rows]
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const float* Hj = reinterpret_cast<const float*>(P.Hint) + (size_t)(min(j0 + jj, P.m - 1) + 1) * 2 * D * D + e;
        const f4 hr = Prec<float>::gld4(Hj), hi = Prec<float>::gld4(Hj + D * D);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          v[jj] += (double)zr[r] * (double)hr[r] - (double)zi[r] * (double)hi[r];
      }
    }
    const double t = wave_sum_many<4>(v, L.lane);
    double* rg = red + (grp & 1) * 32;
    if ((L.lane & 15) == 0) rg[8 * (L.lane >> 4) + L.w] = t;
    __syncthreads();
    if (threadIdx.x < 4 && j0 + (int)threadIdx.x < P.m) {
      double s = 0;
      for (int x = 0; x < 8; ++x) s += rg[8 * threadIdx.x + x];
      seg_grad_put(P, j0 + threadIdx.x, k, part, s);
    }
  }
}

// The gradient of the slices [ka, kb) of segment sg of chunk c.  SQ: slices
// with s > 0 among them.
template <bool SQ>
__device__ __forceinline__ void px_grad(const ProbDesc& P, int c, int sg, int ka, int kb, int kbase, int part, bool mono,
                                        unsigned char* lds, void* scratch, const Lane& L) {
  constexpr float C = S128::C;
  float* xb = reinterpret_cast<float*>(lds + S128::PLANES);
  float* SZ = slot_part(scratch, 0);
  Panel128 Y;
  px_load(Y, pf_mat<float, 128>(part ? P.cb : P.mc, c), L);
  if (sg > 0) px_conjugate(Y, 1.0f, lds, xb, pf_mat<float, 128>(P.bloc, ka - kbase), L);
  for (int k = ka; k < kb; ++k) {
    const int sqk = gp(P.sq)[k];
    int s, q, qb;
    unpack_sq(sqk, s, q, qb);
    const int m = plan_order(sqk);
    {
      Panel128 X;
      px_assemble(X, reinterpret_cast<float*>(lds), P, k, ldexp(P.dt, -s), mono, L);
      px_stage_sym<-1>(lds, X, L);
      if (SQ && s > 0) {
        px_store(slot_part(scratch, 1), X, L);
        px_store(slot_part(scratch, 2), Y, L);
      }
    }
    Frag128 F;
    frag_panel(F, Y, 1.0f);
    __syncthreads();
    for (int n = max(m, 2); n >= 1; --n) {
      Panel128 R;
      px_mul(R, lds, F, L);
      const float ck = S128::CI2 * (1.0f / n);
      f4 pr[2], pq[2];
      if (n > 1) {
        px_exchange(R, xb, L, [&](int i, const f4& tr, const f4& ti) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            pr[i & 1][r] = fmaf(ck, R.re[i][r] + tr[r], Y.re[i][r]);
            pq[i & 1][r] = fmaf(ck, R.im[i][r] + ti[r], Y.im[i][r]);
          }
          if (n == 2) pf_rb_store<float>(SZ, pr[i & 1], pq[i & 1], wave128(), px_rb(i), L.lane);
          pr[i & 1] = C * pr[i & 1];
          pq[i & 1] = C * pq[i & 1];
          if (i & 1) frag_put(F, i >> 1, pr, pq);
        });
        if (SQ && n == 2 && s > 0) break;  // Y waits for the whole slice's propagator
      } else {
        px_exchange(R, xb, L, [&](int i, const f4& tr, const f4& ti) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Y.re[i][r] = fmaf(ck, R.re[i][r] + tr[r], Y.re[i][r]);
            Y.im[i][r] = fmaf(ck, R.im[i][r] + ti[r], Y.im[i][r]);
          }
        });
      }
    }
    if constexpr (SQ) {
      if (s > 0) {
        // Z <- (Z + U Z U^dag) / 2, U <- U U, s times from U = exp(A / 2^s)
        float* SX = slot_part(scratch, 1);
        float* SD = slot_part(scratch, 3);
        Panel128 X;
        px_load(X, SX, L);
        __syncthreads();
        px_stage_sym<-1>(lds, X, L);
        __syncthreads();
        px_taylor(X, lds, 0, q, L);
        px_store(SD, X, L);
        for (int j = 0; j < s; ++j) {
          Panel128 Z;
          px_load(Z, SZ, L);
          px_conjugate(Z, 0.5f, lds, xb, SD, L);
          {
            const int w = wave128();
#pragma unroll
            for (int i = 0; i < 8; ++i) {  // (an own panel)
              f4 re, im;
              pf_rb_load<float>(re, im, SZ, w, px_rb(i), L.lane);
              Z.re[i] += 0.5f * re;
              Z.im[i] += 0.5f * im;
            }
          }
          px_store(SZ, Z, L);
          px_load(X, SD, L);  // D <- 2 D + D D, whose planes are staged
          Frag128 G;
          Panel128 R;
          frag_panel(G, X, 1.0f);
          px_mul(R, lds, G, L);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            X.re[i] = 2.0f * X.re[i] + S128::CI2 * R.re[i];
            X.im[i] = 2.0f * X.im[i] + S128::CI2 * R.im[i];
          }
          px_store(SD, X, L);
        }
        px_load(Y, slot_part(scratch, 2), L);
        px_conjugate(Y, 1.0f, lds, xb, SD, L);
      }
    }
    px_epilogue(P, k, part, SZ, reinterpret_cast<double*>(xb), mono, L);
  }
}

// One workgroup per segment, and the problems without any s > 0.
__global__ __launch_bounds__(512) void k_seg_grad128(Work W, void* scratch) {
  __shared__ __align__(16) unsigned char lds[S128::BYTES];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    const SegItem g = seg_split(item, W.rg, I, W.descs);
    if (g.ka < g.kb) {
      const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
      const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
      if (gp(P.squared)[0] == 0)
        px_grad<false>(P, g.c, g.s, g.ka, g.kb, W.rg.kbase, blockIdx.y, mono, lds, scratch, L);
    }
    __syncthreads();
  }
}

// The segments of the problems with squared slices, as k_seg_grad_sq.
__global__ __launch_bounds__(512) void k_seg_grad_sq128(Work W, void* scratch) {
  __shared__ __align__(16) unsigned char lds[S128::BYTES];
  Lane L;
  const Items I(W);
  if (I.nprob == 0 || gp(W.descs[I.desc(0)].squared)[1] == 0) return;
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    const SegItem g = seg_split(item, W.rg, I, W.descs);
    if (g.ka >= g.kb || gp(W.descs[I.desc(g.p)].squared)[0] == 0) continue;
    const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
    const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
    px_grad<true>(P, g.c, g.s, g.ka, g.kb, W.rg.kbase, blockIdx.y, mono, lds, scratch, L);
    __syncthreads();
  }
}
