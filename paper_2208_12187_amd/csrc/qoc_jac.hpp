// The Jacobian dX_N / du of one problem, all d^2 entries of every (control,
// slice), Hermitian path at d <= 64: with X_N = S_k U_k P_{k-1} and U_k unitary,
//   dX_N / du[j][k] = X_N P_{k-1}^dag Phi_k(j) P_{k-1},
//   Phi_k(j) = -i dt sum_n (-1)^n ad_A^n(Hc[j]) / (n + 1)!,
// the commutator series of one Hermitian matrix (one product per order), two
// products more and no costate.  One workgroup takes a segment and kJacGroup of
// the controls; it forms P at the segment's start from the carry and the joins
// and carries it on with the slice's exponential.  Slices with s > 0 take the
// series on A / 2^s and double it s times, Phi <- (Phi + U^dag Phi U) / 2 with U the
// propagator of the part covered so far: two products per control and doubling.
//
// At d = 16, m = 8, N = 1000 in FP64: 130 us, the latency of dependent products in
// about two wavefronts per SIMD, and 16 us for k_jac_out.  (The d^2 rows as a batch
// of d^2 copies of the problem, each with its own forward pass and the block form
// of its adjoint: 4.17 ms.)
//
// Included by qoc_kernels.hip.
#pragma once

constexpr int kJacGroup = 2;  // controls per workgroup: 2000 wavefronts at the size above

template <typename T, int D>
__global__ __launch_bounds__(4 * D) void k_jac(Work W, T* out) {
  using Ops = StdOps<T, D>;
  __shared__ __align__(16) unsigned char la[Ops::BYTES];
  __shared__ __align__(16) unsigned char lb[Ops::BYTES];
  __shared__ SegTab<T, D> tab;
  T* pt = reinterpret_cast<T*>(lb);  // planar
  Lane L;
  const Items I(W);
  const SegItem g = seg_split(blockIdx.x, W.rg, I, W.descs);
  if (g.ka >= g.kb) return;
  const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
  const int j0 = blockIdx.y * kJacGroup, j1 = min(P.m, j0 + kJacGroup);
  const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
  const SegTab<T, D>* tb = seg_tab_load<T, D>(tab, P, g.ka, g.kb, mono) ? &tab : nullptr;
  Panel<T, D> X, R, Pk, Q;  // Pk = P_{k-1}
  panel_load(X, pf_mat<T, D>(P.cf, g.c), L);
  panel_load(R, grp_mat<T, D>(P, 2, g.c / P.CG), L);
  Ops::store(la, X, L);
  __syncthreads();
  Ops::gemm(Pk, la, R, L, true);
  if (g.s > 0) {
    panel_load(X, pf_mat<T, D>(P.bloc, g.ka - W.rg.kbase), L);
    Ops::store(lb, X, L);
    __syncthreads();
    Ops::gemm(X, lb, Pk, L, true);
    panel_fma(Pk, (T)1, X);
  }
  const size_t mat = 2 * (size_t)D * D;
  for (int k = g.ka; k < g.kb; ++k) {
    const int sqk = gp(P.sq)[k];
    int s, q, qb;
    unpack_sq(sqk, s, q, qb);
    const int m = plan_order(sqk);
    // Q = X_N P_{k-1}^dag
    __syncthreads();
    Ops::store(lb, Pk, L);
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rb + Prec<T>::rowmap(r, L.g), col = 16 * L.w + L.c16;
        const bool in = row < P.d && col < P.d;
        const double* x = P.XN + 2 * ((size_t)row * P.d + col);
        X.re[rb][r] = in ? (T)gp(x)[0] : (T)0;
        X.im[rb][r] = in ? (T)gp(x)[1] : (T)0;
      }
    Ops::store(la, X, L);
    __syncthreads();
    Ops::load_ct(R, lb, L);
    Ops::gemm(Q, la, R, L, true);
    assemble_panel<T, D>(X, lb, P, k, ldexp(P.dt, -s), mono, tb, k - g.ka, L);
    Ops::store_nct(la, X, L);  // A = -A^dag (assemble_panel ends with a barrier after Q's reads)
    __syncthreads();
    T* o = out + ((size_t)j0 * P.N + k) * mat;
    const size_t oj = (size_t)P.N * mat;  // to the next control's matrix
    // dX_N / du[j][k] = -i dt Q Phi P from Phi in Z
    auto put = [&](T* dst, const Panel<T, D>& Z) {
      Panel<T, D> C;
      __syncthreads();
      Ops::store(lb, Z, L);
      __syncthreads();
      Ops::gemm(R, lb, Pk, L, true);
      __syncthreads();
      Ops::store(lb, Q, L);
      __syncthreads();
      Ops::gemm(C, lb, R, L, true);
      const T f = (T)P.dt;
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const T re = C.re[rb][r];
          C.re[rb][r] = f * C.im[rb][r];
          C.im[rb][r] = -f * re;
        }
      panel_store(dst, C, L);
    };
    for (int j = j0; j < j1; ++j) {
      const T* H = reinterpret_cast<const T*>(P.Hint) + (j + 1) * mat;
      Panel<T, D> C, Z;
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int e = (16 * rb + Prec<T>::rowmap(r, L.g)) * D + 16 * L.w + L.c16;
          C.re[rb][r] = gp(H)[e];
          C.im[rb][r] = gp(H)[D * D + e];
        }
      Z = C;
      for (int n = 1; n <= m; ++n) {  // C <- -[A, C] / n, Z <- Z + C / (n + 1)
        Ops::mul(R, la, C, L);
        __syncthreads();
        panel_to_lds_ct(pt, R, L);
        __syncthreads();
        panel_from_lds(C, pt, L);
        const T ck = (T)(-1.0 / n), zk = (T)(1.0 / (n + 1));
#pragma unroll
        for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            C.re[rb][r] = (C.re[rb][r] + R.re[rb][r]) * ck;
            C.im[rb][r] = (C.im[rb][r] + R.im[rb][r]) * ck;
            Z.re[rb][r] = fma(zk, C.re[rb][r], Z.re[rb][r]);
            Z.im[rb][r] = fma(zk, C.im[rb][r], Z.im[rb][r]);
          }
      }
      if (s == 0) put(o + (j - j0) * oj, Z);
      else panel_store(o + (j - j0) * oj, Z, L);  // (own panel: read back by this wavefront)
    }
    __syncthreads();
    if (s == 0) {
      taylor_delta<T, D, Ops>(R, X, la, 0, q, L);
      __syncthreads();
      Ops::store(la, R, L);
      __syncthreads();
    } else {
      // R = U^dag - I from -A / 2^s = (A / 2^s)^dag, the left factor of the doublings
      // and of its own squaring
      Ops::store_ct(la, X, L);
      panel_scale(X, (T)-1);
      __syncthreads();
      taylor_delta<T, D, Ops>(R, X, la, 0, q, L);
      for (int i = 0; i < s; ++i) {
        __syncthreads();
        Ops::store(la, R, L);
        __syncthreads();
        for (int j = j0; j < j1; ++j) {
          panel_load(X, o + (j - j0) * oj, L);
          conjugate_by<T, D, Ops>(X, (T)0.5, la, lb, L);
          panel_store(o + (j - j0) * oj, X, L);
        }
        Ops::mul(X, la, R, L);
        panel_scale(R, (T)2);
        panel_fma(R, (T)1, X);
      }
      __syncthreads();
      Ops::store_ct(la, R, L);  // U - I, published by put's barriers
      for (int j = j0; j < j1; ++j) {
        panel_load(X, o + (j - j0) * oj, L);
        put(o + (j - j0) * oj, X);
      }
    }
    Ops::gemm(R, la, Pk, L, true);
    panel_fma(Pk, (T)1, R);
  }
}

// J[part d^2 + a d + b][j N + k] from the stored matrices of (j, k): 64 columns by
// 64 stored elements through LDS, so that both sides are coalesced.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_jac_out(const T* in, double* J, size_t ld, int d, int cols) {
  __shared__ T t[64][65];
  const int c0 = blockIdx.x * 64, e0 = blockIdx.y * 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int i = w; i < 64; i += 4)
    if (c0 + i < cols) t[i][lane] = gp(in)[(size_t)(c0 + i) * 2 * D * D + e0 + lane];
  __syncthreads();
  for (int i = w; i < 64; i += 4) {
    // the inverse of pf_index
    constexpr int G = 16 / sizeof(T);
    const int e = e0 + i;
    const int x = e / (64 * G), ln = e / G % 64, reg = x % (D / 4 / G) * G + e % G;
    const int part = x / (D / 4 / G) % 2, pw = x / (D / 4 / G) / 2;
    const int row = 16 * (reg >> 2) + Prec<T>::rowmap(reg & 3, ln >> 4), col = 16 * pw + (ln & 15);
    if (row < d && col < d && c0 + lane < cols)
      J[((size_t)part * d * d + (size_t)row * d + col) * ld + c0 + lane] = (double)t[lane][i];
  }
}

template <typename T, int D>
static void jacobian_le64(const Launch& L, int d, int m, int N, void* mats, double* J, size_t ld) {
  const Range rg = {0, N, 0, L.uniformP, 0, 0};
  const Work segs = {L.descs, 1, L.uniformP * seg_count(L.chunk, seg_max(D, L.chunk, sizeof(T) == 8)), nullptr, rg, nullptr};
  T* out = static_cast<T*>(mats);
  hipLaunchKernelGGL((k_jac<T, D>), dim3(segs.total, (m + kJacGroup - 1) / kJacGroup), dim3(4 * D), 0, L.stream, segs,
                     out);
  hipLaunchKernelGGL((k_jac_out<T, D>), dim3((unsigned)(((size_t)m * N + 63) / 64), 2 * D * D / 64), dim3(256), 0,
                     L.stream, out, J, ld, d, m * N);
}

hipError_t launch_jacobian(int precision, int D, const Launch& L, int d, int m, int N, void* mats, double* J,
                           size_t ld) {
  if (precision == 0) {
    switch (D) {
      case 16: jacobian_le64<double, 16>(L, d, m, N, mats, J, ld); break;
      case 32: jacobian_le64<double, 32>(L, d, m, N, mats, J, ld); break;
      case 64: jacobian_le64<double, 64>(L, d, m, N, mats, J, ld); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (D) {
      case 16: jacobian_le64<float, 16>(L, d, m, N, mats, J, ld); break;
      case 32: jacobian_le64<float, 32>(L, d, m, N, mats, J, ld); break;
      case 64: jacobian_le64<float, 64>(L, d, m, N, mats, J, ld); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}
