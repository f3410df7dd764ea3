// GRAPE hot path on gfx950: slice propagators by scaling-and-squaring Taylor
// series, chunked forward/backward propagator scans, fidelity in FP64 and the
// exact gradient through the block-triangular Frechet derivative.
//
// Notation (slice k = 0..N-1, slice 0 acts first; hbar = 1):
//   A_k = -i dt H_k,  H_k = H0 + sum_j u[j][k] Hc[j],  U_k = exp(A_k)
//   X_N = U_{N-1} ... U_0,  g = Tr(V^dag X_N),  F = |g|^2 / d^2
//   P_k = U_k ... U_0 (P_{-1} = I),  Q_k = U_{k+1}^dag ... U_{N-1}^dag V
//   W_k = Q_k P_{k-1}^dag
// GRAPE gradient (Khaneja et al. 2005), taken exactly: with L(A, E) the
// Frechet derivative of exp at A in direction E,
//   dg/du[j][k] = <W_k, L(A_k, -i dt Hc[j])>,   <X, Y> = Tr(X^dag Y).
// The adjoint identity <W, L(A, E)> = <L(A^dag, W), E> (L(A, E) is the
// integral of e^{sA} E e^{(1-s)A} over s in [0, 1]) turns the m derivatives
// of a slice into one: Z_k = L(A_k^dag, W_k) and
//   dF/du[j][k] = (2 dt / d^2) Im(conj(g) Tr(Z_k^dag Hc[j])).
// Z_k is the top-right block of exp([[A^dag, W], [0, A^dag]]) (Van Loan 1978;
// Goodwin and Kuprov 2015), evaluated with the same scaling and squaring as
// the propagator.  Everything runs in "delta form": the Taylor sum keeps
// T(X) - I and a squaring maps D to 2D + D^2, so that rounding errors scale
// with |A| rather than with |U| = 1.
#include <type_traits>

#include "qoc_device.hpp"
#include "qoc_internal.hpp"
#include "qoc_plan.hpp"
#include "qoc_bf16.hpp"
#include "qoc_f16.hpp"

namespace qoc {

// ---------------------------------------------------------------- work items

__device__ __forceinline__ int locate(const int* start, int n, int item) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (gp(start)[mid] <= item) lo = mid; else hi = mid;
  }
  return lo;
}

// Map a flat work item to (problem, slice or chunk index).  Uniform launches
// (count > 0) cover indices [lo, lo + count) of every problem; otherwise the
// items of problem p are [start[p], start[p + 1]).
__device__ __forceinline__ void split_item(int item, int lo, int count, const int* start, int n, int& p, int& k) {
  if (count > 0) {
    p = item / count;
    k = lo + (item - p * count);
  } else {
    p = locate(start, n, item);
    k = item - gp(start)[p];
  }
}

// The item counts of a launch (see Work).
struct Items {
  int nprob, total;
  const int* start;
  const int* slot;  // descriptor index of each problem (engine launches), else identity
  __device__ __forceinline__ explicit Items(const Work& W) {
    if (W.dyn) {
      nprob = gp(W.dyn)[0];
      total = gp(W.dyn)[1];
      start = W.dyn + 2;
      slot = W.dyn + 3 + nprob;
    } else {
      nprob = W.nprob;
      total = W.total;
      start = W.start;
      slot = nullptr;
    }
  }
  __device__ __forceinline__ int desc(int p) const { return slot ? gp(slot)[p] : p; }
};

template <typename T, int D>
__device__ __forceinline__ T* pf_mat(void* base, int i) {
  return reinterpret_cast<T*>(base) + (size_t)i * Mat<T, D>::ELEMS;
}

// ---------------------------------------------------------------- prep

// The flags that every control of the problem has: bit 0, a usable row table
// (at most one nonzero per row, dense kernels not forced); bit 1, the table is
// also a bijection from rows to columns (minv holds its inverse).  (All the
// flags are loaded together.)
__device__ __forceinline__ int controls_flags(const ProbDesc& P) {
  int all = 3;
#pragma unroll 4
  for (int j = 0; j < P.m; ++j) all &= gp(P.mok)[j];
  return all;
}

// Bit 24 of a slice's packed plan: the FP32 adjoint may sample its last step
// there (s = 0 and permutation controls), so that the adjoint's two instances
// split the slices with the one load of the plan.
constexpr int kPlanSampled = 1 << 24;
// Bit 25: every control has a usable row table (controls_flags), so that a
// slice's workgroup does not walk the m flags, one dependent load each.
constexpr int kPlanMono = 1 << 25;

// Convert the caller's complex128 matrices to the compute precision: H0 and
// Hc[j] to planar D x D (zero padded), V to PF; also the FP64 one-norms
// (largest column sum of moduli) of H0 and Hc[j].  With general generators
// (RUN_GENERAL) the caller's G is stored as H = i G, so that every kernel's
// A = -i dt H is dt G, and the norm is the larger of the one- and
// infinity-norms: the adjoint works with A^dag, whose one-norm is A's
// infinity-norm.
// The same pass over a control builds its row table: for each row a, the
// column and value (in precision T, as the dense copy holds it) of its nonzero,
// and whether every row has at most one.  Such controls (Pauli strings, for
// instance) are then assembled and paired with Z_k entry by entry.  The table
// is written even when the control does not qualify; mok[j] says whether it may
// be used (bit 0), whether its columns are a bijection (bit 1; then
// minv[j][col_j(a)] = a; empty rows count at their own column, with a zero
// entry) and whether control j - 1 puts its entries at the same columns, as X_i
// and Y_i do (bit 2).
//
// A wavefront reads whole rows (64 / D of them at once, or half a row at a time
// at D = 128), so that a matrix takes D^2 / 256 coalesced loads per thread with
// no dependence between rows: latency-bound, one round trip deep (one thread
// per row or column walked D dependent steps: one problem of d = 64, m = 12 took
// 46 us, now 15; eight of d = 128, m = 14 take 86).
template <typename T, int D>
__device__ __forceinline__ void prep_one(const ProbDesc& P, int mat, double* colmax) {
  const int d = P.d, m = P.m;
  if (mat == 0 && threadIdx.x == 0) {
    P.diag[1] = 0.0;
    P.diag[2] = 0.0;
    P.squared[0] = P.squared[1] = 0;
  }
  if (mat <= m) {
    constexpr int LPR = D < 64 ? D : 64;  // lanes per row
    constexpr int CPL = D / LPR;          // columns per lane
    constexpr int RPW = 64 / LPR;         // rows per wavefront and step
    constexpr int STEPS = D / (4 * RPW);
    __shared__ int hits[D];               // rows whose entry lies in each column
    __shared__ double csum[4][D];         // column sums by wavefront
    const bool gen = (P.flags & RUN_GENERAL) != 0;
    const bool ctl = mat > 0;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = lane / LPR, lc = lane % LPR;
    const double* src = mat == 0 ? P.H0z : P.Hcz + (size_t)(mat - 1) * 2 * d * d;
    const double* prev = mat > 1 ? src - 2 * (size_t)d * d : nullptr;
    T* dst = reinterpret_cast<T*>(P.Hint) + (size_t)mat * 2 * D * D;
    if ((int)threadIdx.x < D) hits[threadIdx.x] = 0;
    __syncthreads();
    double cs[CPL];
    double rmax = 0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) cs[q] = 0;
    int multi = 0, same = 1;
    const unsigned long long rowmask = (LPR == 64 ? ~0ull : ((1ull << LPR) - 1) << (lr * LPR));
#pragma unroll 4
    for (int st = 0; st < STEPS; ++st) {
      const int row = (st * 4 + w) * RPW + lr;
      unsigned long long nz[CPL], pz[CPL];
      T tr[CPL], ti[CPL];
      double rs = 0;
#pragma unroll
      for (int q = 0; q < CPL; ++q) {
        const int col = lc + q * LPR;
        double re = 0, im = 0, pr = 0, pi = 0;
        if (row < d && col < d) {
          const d2 v = *(const QOC_GLOBAL d2*)(src + 2 * ((size_t)row * d + col));
          re = v.x;
          im = v.y;
          if (prev) {
            const d2 u = *(const QOC_GLOBAL d2*)(prev + 2 * ((size_t)row * d + col));
            pr = u.x;
            pi = u.y;
          }
        }
        const double a = sqrt(fma(re, re, im * im));
        cs[q] += a;
        rs += a;
        if (gen) {  // i (re + i im)
          const double t = re;
          re = -im;
          im = t;
        }
        tr[q] = (T)re;
        ti[q] = (T)im;
        gp(dst)[row * D + col] = tr[q];
        gp(dst)[D * D + row * D + col] = ti[q];
        nz[q] = __ballot(tr[q] != (T)0 || ti[q] != (T)0) & rowmask;
        pz[q] = __ballot((T)pr != (T)0 || (T)pi != (T)0) & rowmask;  // (as its own table has them)
      }
      if (gen) {  // row sums, for the infinity norm
#pragma unroll
        for (int o = 1; o < LPR; o <<= 1) rs += __shfl_xor(rs, o, 64);
        rmax = fmax(rmax, rs);
      }
      if (ctl) {
        int cnt = 0, col = row, pc = row, own = -1;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          cnt += __popcll(nz[q]);
          if (nz[q]) col = 63 - __clzll(nz[q]) - lr * LPR + q * LPR;  // the last one
          if (pz[q]) pc = 63 - __clzll(pz[q]) - lr * LPR + q * LPR;
        }
        multi |= cnt > 1;
        if (row < d) same &= pc == col;
#pragma unroll
        for (int q = 0; q < CPL; ++q)
          if (lc + q * LPR == col) own = q;
        if (own >= 0) {  // the lane of the row's entry (its own column in an empty row)
          const size_t idx = (size_t)(mat - 1) * D + row;
          T vr = tr[0], vi = ti[0];
          if (CPL > 1 && own > 0) {
            vr = tr[CPL - 1];
            vi = ti[CPL - 1];
          }
          gp(P.mcol)[idx] = col;
          gp(reinterpret_cast<T*>(P.mval))[2 * idx] = vr;
          gp(reinterpret_cast<T*>(P.mval))[2 * idx + 1] = vi;
          atomicAdd(&hits[col], 1);
          if (P.minv) gp(P.minv)[(size_t)(mat - 1) * D + col] = row;
        }
      }
    }
    // column sums: lanes of one column within the wavefront, then the wavefronts
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
#pragma unroll
      for (int o = LPR; o < 64; o <<= 1) cs[q] += __shfl_xor(cs[q], o, 64);
      if (lr == 0) csum[w][lc + q * LPR] = cs[q];
    }
    const int any = __syncthreads_or(multi);
    const int a = threadIdx.x;
    double mx = gen ? rmax : 0.0;
    if (a < D) mx = fmax(mx, (csum[0][a] + csum[1][a]) + (csum[2][a] + csum[3][a]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) colmax[w] = mx;
    const int bij = __syncthreads_and(a >= D || hits[a] == 1);
    const int all_same = __syncthreads_and(same) && mat > 1;
    if (threadIdx.x == 0) {
      P.norms[mat] = fmax(fmax(colmax[0], colmax[1]), fmax(colmax[2], colmax[3]));
      if (ctl)
        gp(P.mok)[mat - 1] =
            (!any && !(P.flags & CTRL_DENSE)) ? (1 | (bij && P.minv ? 2 : 0) | (all_same ? 4 : 0)) : 0;
    }
    __syncthreads();
  } else if (P.Vz != nullptr && P.Vint != nullptr) {
    // V / 2^e with 2^e <= |V|_F < 2^(e+1): no entry of the costates exceeds 2,
    // whatever the target, as the FP16 split of their products assumes.  The
    // gradient is linear in V and takes the exact factor back (grad_put).
    double f2 = 0;
    for (int e = threadIdx.x; e < 2 * d * d; e += 256) f2 = fma(P.Vz[e], P.Vz[e], f2);
    f2 = wave_sum(f2);
    if ((threadIdx.x & 63) == 0) colmax[threadIdx.x >> 6] = f2;
    __syncthreads();
    const double nf = sqrt((colmax[0] + colmax[1]) + (colmax[2] + colmax[3]));
    int ex = 1;
    if (nf > 0 && nf < 1e300) (void)frexp(nf, &ex);
    const double dn = ldexp(1.0, 1 - ex);
    if (threadIdx.x == 0) *P.vscale = ldexp(1.0, ex - 1);
    T* dst = reinterpret_cast<T*>(P.Vint);
    for (int e = threadIdx.x; e < D * D; e += 256) {
      int row = e / D, col = e % D;
      double re = 0, im = 0;
      if (row < d && col < d) {
        re = dn * P.Vz[2 * (row * d + col)];
        im = dn * P.Vz[2 * (row * d + col) + 1];
      }
      int w = col >> 4, c16 = col & 15, rb = row >> 4, rr = row & 15;
      int r, g;
      if (sizeof(T) == 4) { g = rr >> 2; r = rr & 3; } else { r = rr >> 2; g = rr & 3; }
      int lane = 16 * g + c16, reg = 4 * rb + r;
      dst[pf_index<T, D>(w, 0, reg, lane)] = (T)re;
      dst[pf_index<T, D>(w, 1, reg, lane)] = (T)im;
    }
    __syncthreads();  // the norm has been read: a persistent workgroup's next item may be another V
  }
}

// Items: (problem, matrix index 0..m+1) with index m+1 standing for V; 256
// threads per item.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_prep(Work W) {
  __shared__ double colmax[256];
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, mat;
    split_item(item, 0, W.rg.s_n, I.start, I.nprob, p, mat);
    prep_one<T, D>(W.descs[I.desc(p)], mat, colmax);
  }
}

// ---------------------------------------------------------------- plan

// Per slice: theta = dt (|H0|_1 + sum_j |u[j][k]| |Hc[j]|_1) in FP64, then the
// scaling exponent and Taylor degrees of choose_plan().
// flags: PlanFlags.
__global__ __launch_bounds__(256) void k_plan(Work W, double ur, int flags) {
  const Items I(W);
  for (int item = blockIdx.x * 256 + threadIdx.x; item < I.total; item += gridDim.x * 256) {
    int p, k;
    split_item(item, W.rg.s_lo, W.rg.s_n, I.start, I.nprob, p, k);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    double th = gp(P.norms)[0];
#pragma unroll 4
    for (int j = 0; j < P.m; ++j) th = fma(fabs(gp(P.u)[(size_t)j * P.N + k]), gp(P.norms)[j + 1], th);
    th *= P.dt;
    const SlicePlan pl = choose_plan(th, ur, flags);
    const int cf = controls_flags(P);
    if (pl.s > 0) {  // (every writer writes the same)
      gp(P.squared)[0] = 1;
      gp(W.descs[I.desc(0)].squared)[1] = 1;
    }
    P.sq[k] = pack_plan(pl) | (pl.s == 0 && (cf & 2) ? kPlanSampled : 0) | ((cf & 1) ? kPlanMono : 0);
  }
}

// ---------------------------------------------------------------- assembly

// The planar LDS layout of panel_to_lds (StdOps), which assemble's scatter
// form writes and reads directly.
template <typename T, int D, typename Ops>
constexpr bool kStdLds = std::is_same<Ops, StdOps<T, D>>::value;

// lds <- sgn * (-i) * c * H_k  (sgn = +1: A_k / 2^s with c = dt / 2^s;
// sgn = -1: A_k^dag / 2^s).  H_k = H0 + sum_j u[j][k] Hc[j] in precision T.
template <typename T, int D, typename Ops, int G = 1>
__device__ __forceinline__ void assemble(void* lds, const ProbDesc& P, int k, double c, double sgn, T* hk,
                                         bool mono, bool ct = false) {
  // The matrix is read as D^2/4 chunks of four consecutive row elements;
  // thread t owns chunks t, t + 4D, t + 8D, ... (D/16 of them), so that the
  // lanes of one 16-byte load read consecutive chunks.  The loads of G
  // controls are in flight together; indices past the last control are
  // clamped to it and weighted by zero, which leaves every sum unchanged.
  // Chunks are written to LDS four columns at a time.  When hk is not null,
  // H_k itself is also written there (planar, row-major) for the adjoint.
  // With mono (every control has at most one nonzero per row) each chunk
  // takes its row's entry of each control from the row tables instead: the
  // same products, minus those with structural zeros.
  using v4 = typename Prec<T>::v4;
  constexpr int NV = D / 16;
  constexpr int NT = 4 * D;
  const T* H = reinterpret_cast<const T*>(P.Hint);
  const int e0 = 4 * threadIdx.x;
  v4 hr[NV], hi[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    hr[v] = Prec<T>::gld4(H + e0 + 4 * NT * v);
    hi[v] = Prec<T>::gld4(H + D * D + e0 + 4 * NT * v);
  }
  const size_t tab_bytes = (size_t)P.m * D * (sizeof(int) + 2 * sizeof(T)) + (size_t)P.m * sizeof(T);
  if (mono && D >= 32 && !ct && kStdLds<T, D, Ops>) {
    // Scatter form (D >= 32, where the expm is the only row-table caller):
    // H0 goes to LDS unscaled; thread a < D then adds u_j Hc[j][a][col_j(a)]
    // to entry (a, col_j(a)) of its own row for j = 0 ... m - 1 (the dense
    // sum's nonzero terms in its order, so H_k is the same); every thread
    // then reads its chunks back.  O(m D) work instead of every thread
    // scanning every control for its chunks.
    T* pl = static_cast<T*>(lds);
    T* pi = pl + D * Mat<T, D>::SD;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int e = e0 + 4 * NT * v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int off = lds_off<T, D>(e / D, e % D + i);
        pl[off] = hr[v][i];
        pi[off] = hi[v][i];
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < D) {
      const int a = threadIdx.x;
      const T* mv = reinterpret_cast<const T*>(P.mval);
      for (int j = 0; j < P.m; ++j) {
        const size_t idx = (size_t)j * D + a;
        const T uj = (T)gp(P.u)[(size_t)j * P.N + k];
        const int off = lds_off<T, D>(a, gp(P.mcol)[idx]);
        pl[off] = fma(uj, gp(mv)[2 * idx], pl[off]);
        pi[off] = fma(uj, gp(mv)[2 * idx + 1], pi[off]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int e = e0 + 4 * NT * v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int off = lds_off<T, D>(e / D, e % D + i);
        hr[v][i] = pl[off];
        hi[v][i] = pi[off];
      }
    }
  } else if (mono && tab_bytes <= (size_t)Ops::BYTES) {
    // The problem's row tables and the slice's amplitudes go through LDS (the
    // left-factor space, written below only after a barrier): one round trip
    // of coalesced loads instead of one per group of controls.
    const int mD = P.m * D;
    int* lc = static_cast<int*>(lds);
    T* lv = reinterpret_cast<T*>(lc + mD);
    T* lu = lv + 2 * mD;
    const T* mv = reinterpret_cast<const T*>(P.mval);
#pragma unroll 4
    for (int i = threadIdx.x; i < mD; i += NT) {
      lc[i] = gp(P.mcol)[i];
      lv[2 * i] = gp(mv)[2 * i];
      lv[2 * i + 1] = gp(mv)[2 * i + 1];
    }
    for (int j = threadIdx.x; j < P.m; j += NT) lu[j] = (T)gp(P.u)[(size_t)j * P.N + k];
    __syncthreads();
    for (int j = 0; j < P.m; ++j) {
      const T uj = lu[j];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = e0 + 4 * NT * v;
        const int idx = j * D + e / D, c0 = e % D;
        const int col = lc[idx];
        const T vr = lv[2 * idx], vi = lv[2 * idx + 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const T w = col == c0 + i ? uj : (T)0;
          hr[v][i] += w * vr;
          hi[v][i] += w * vi;
        }
      }
    }
    __syncthreads();  // the tables are read; the LDS takes the left factor next
  } else if (mono) {
    constexpr int GM = 4;  // controls whose table entries are loaded together
    const T* mv = reinterpret_cast<const T*>(P.mval);
    for (int j0 = 0; j0 < P.m; j0 += GM) {
      int col[GM][NV];
      T vr[GM][NV], vi[GM][NV], uw[GM];
#pragma unroll
      for (int jj = 0; jj < GM; ++jj) {
        const int j = min(j0 + jj, P.m - 1);
        uw[jj] = j0 + jj < P.m ? (T)gp(P.u)[(size_t)j * P.N + k] : (T)0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const size_t idx = (size_t)j * D + (e0 + 4 * NT * v) / D;
          col[jj][v] = gp(P.mcol)[idx];
          vr[jj][v] = gp(mv)[2 * idx];
          vi[jj][v] = gp(mv)[2 * idx + 1];
        }
      }
#pragma unroll
      for (int jj = 0; jj < GM; ++jj)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const int c0 = (e0 + 4 * NT * v) % D;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const T w = col[jj][v] == c0 + i ? uw[jj] : (T)0;
            hr[v][i] += w * vr[jj][v];
            hi[v][i] += w * vi[jj][v];
          }
        }
    }
  } else
  for (int j0 = 0; j0 < P.m; j0 += G) {
    v4 ar[G][NV], ai[G][NV];
    T uw[G];
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      const int j = min(j0 + jj, P.m - 1);
      uw[jj] = j0 + jj < P.m ? (T)gp(P.u)[(size_t)j * P.N + k] : (T)0;
      const T* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        ar[jj][v] = Prec<T>::gld4(Hj + 4 * NT * v);
        ai[jj][v] = Prec<T>::gld4(Hj + D * D + 4 * NT * v);
      }
    }
#pragma unroll
    for (int jj = 0; jj < G; ++jj)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        hr[v] += uw[jj] * ar[jj][v];
        hi[v] += uw[jj] * ai[jj][v];
      }
  }
  const T f = (T)(sgn * c);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int e = e0 + 4 * NT * v;
    if (ct) {
      // (-i (-f) H)^dag = -i f H^dag (see ham_put): element (col, row) is
      // -i f conj(H[row][col]) = -f hi - i f hr
#pragma unroll
      for (int i = 0; i < 4; ++i) Ops::put(lds, e % D + i, e / D, -f * hi[v][i], -f * hr[v][i]);
    } else {
      Ops::put4(lds, e / D, e % D, f * hi[v], -f * hr[v]);  // -i f (hr + i hi)
    }
    if (hk) {
      Prec<T>::gst4(hk + e, hr[v]);
      Prec<T>::gst4(hk + D * D + e, hi[v]);
    }
  }
}

// The slice's H_k as stored by k_expm: ham_load issues the loads of this
// thread's chunks (the same chunks as assemble), ham_put writes them to LDS,
// scaled, as assemble() writes its result.
template <typename T, int D>
struct HamRegs {
  typename Prec<T>::v4 hr[D / 16], hi[D / 16];
};

template <typename T, int D>
__device__ __forceinline__ void ham_load(HamRegs<T, D>& H, const T* hk) {
  constexpr int NT = 4 * D;
  const int e0 = 4 * threadIdx.x;
#pragma unroll
  for (int v = 0; v < D / 16; ++v) {
    H.hr[v] = Prec<T>::gld4(hk + e0 + 4 * NT * v);
    H.hi[v] = Prec<T>::gld4(hk + D * D + e0 + 4 * NT * v);
  }
}

// ct: write (-i (-sgn) c H_k)^dag instead of -i sgn c H_k.  The two agree
// when H_k is Hermitian; for general generators the adjoint's call
// (sgn = -1) then gets (-i c H_k)^dag = A_k^dag / 2^s.
template <typename T, int D, typename Ops>
__device__ __forceinline__ void ham_put(void* lds, const HamRegs<T, D>& H, double c, double sgn, bool ct = false) {
  constexpr int NT = 4 * D;
  const int e0 = 4 * threadIdx.x;
  const T f = (T)(sgn * c);
#pragma unroll
  for (int v = 0; v < D / 16; ++v) {
    const int e = e0 + 4 * NT * v;
    if (ct) {
#pragma unroll
      for (int i = 0; i < 4; ++i) Ops::put(lds, e % D + i, e / D, -f * H.hi[v][i], -f * H.hr[v][i]);
    } else {
      Ops::put4(lds, e / D, e % D, f * H.hi[v], -f * H.hr[v]);
    }
  }
}

__device__ __forceinline__ void unpack_sq(int sq, int& s, int& q, int& qb) {
  s = sq & 255;
  q = (sq >> 8) & 255;
  qb = (sq >> 16) & 255;
}

// ---------------------------------------------------------------- epilogues

// S = X_N (panel): write X_N if requested, then g = Tr(V^dag X_N) and
// F = |g|^2 / d^2 with FP64 accumulation.  red: 2 * D/16 doubles of LDS.
template <typename T, int D>
__device__ __forceinline__ void fidelity_epilogue(const ProbDesc& P, const Panel<T, D>& S, const Lane& L,
                                                  double* red) {
  constexpr int NW = D / 16;
  const int d = P.d;
  if (P.XN) {
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int row = 16 * rb + Prec<T>::rowmap(r, L.g), col = 16 * L.w + L.c16;
        if (row < d && col < d) {
          P.XN[2 * (row * d + col)] = (double)S.re[rb][r];
          P.XN[2 * (row * d + col) + 1] = (double)S.im[rb][r];
        }
      }
  }
  if (P.Vz) {
    double gr = 0, gi = 0;
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int row = 16 * rb + Prec<T>::rowmap(r, L.g), col = 16 * L.w + L.c16;
        if (row < d && col < d) {
          double vr = P.Vz[2 * (row * d + col)], vi = P.Vz[2 * (row * d + col) + 1];
          double xr = (double)S.re[rb][r], xi = (double)S.im[rb][r];
          gr += vr * xr + vi * xi;  // conj(v) x
          gi += vr * xi - vi * xr;
        }
      }
    gr = wave_sum(gr);
    gi = wave_sum(gi);
    __syncthreads();
    if (L.lane == 0) { red[2 * L.w] = gr; red[2 * L.w + 1] = gi; }
    __syncthreads();
    if (threadIdx.x == 0) {
      double a = 0, b = 0;
      for (int w = 0; w < NW; ++w) { a += red[2 * w]; b += red[2 * w + 1]; }
      P.g[0] = a;
      P.g[1] = b;
      *P.F = (a * a + b * b) / ((double)d * d);
    }
  }
}

// G = S^dag S (panel): diag[0] = |G - I|_F over the d x d block, FP64 accumulation.
template <typename T, int D>
__device__ __forceinline__ void residual_epilogue(const ProbDesc& P, const Panel<T, D>& G, const Lane& L,
                                                  double* red) {
  constexpr int NW = D / 16;
  const int d = P.d;
  double e2 = 0;
#pragma unroll
  for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int row = 16 * rb + Prec<T>::rowmap(r, L.g), col = 16 * L.w + L.c16;
      if (row < d && col < d) {
        double xr = (double)G.re[rb][r] - (row == col ? 1.0 : 0.0), xi = (double)G.im[rb][r];
        e2 += xr * xr + xi * xi;
      }
    }
  e2 = wave_sum(e2);
  __syncthreads();
  if (L.lane == 0) red[L.w] = e2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0;
    for (int w = 0; w < NW; ++w) a += red[w];
    P.diag[0] = sqrt(a);
  }
}

// Gradient from Z = Z_k: T_j = Tr(Z^dag Hc[j]) with FP64 accumulation and
// grad[j][k] = (2 dt / d^2) Im(conj(g) T_j).  Controls are taken in groups
// (kEpiGroup, or kEpiDense for the FP32 dense controls): every lane forms
// its partial sums for the whole group, one multi-value wavefront reduction
// combines them, one barrier publishes the per-wavefront totals and one
// thread per control adds those up.  Control indices past the last one are
// clamped to it, so every load stays in bounds, and their sums are
// discarded.  red: 2 x 2 G x (threads / 64) doubles of LDS for groups of G
// (double-buffered by group).
constexpr int kEpiGroup = 4;
// Controls reduced together by the FP32 dense-control epilogue.
constexpr int kEpiDense = 8;

// Stores the gradient entry (j, k) from T_j = a + i b.
__device__ __forceinline__ void grad_put(const ProbDesc& P, int j, int k, double a, double b) {
  const double dt = P.dt * gp(P.vscale)[0];  // Z_k is that of the normalised target
  if (P.flags & RUN_RAWDG) {
    // dg/du[j][k] = -i dt Tr(Z_k^dag Hc[j]), complex interleaved
    const size_t o = 2 * ((size_t)j * P.N + k);
    gp(P.grad)[o] = dt * b;
    gp(P.grad)[o + 1] = -dt * a;
  } else {
    const double pref = 2.0 * dt / ((double)P.d * P.d);
    gp(P.grad)[(size_t)j * P.N + k] = pref * (gp(P.g)[0] * b - gp(P.g)[1] * a);
  }
}

template <int NWAVES, int G = kEpiGroup>
__device__ __forceinline__ void epilogue_publish(const ProbDesc& P, int k, int j0, int grp, double (&v)[2 * G],
                                                 const Lane& L, double* red) {
  constexpr int V = 2 * G;
  constexpr int SH = 6 - __builtin_ctz(V);
  const int nj = min(G, P.m - j0);
  const double t = wave_sum_many<V>(v, L.lane);
  double* rg = red + (grp & 1) * V * NWAVES;
  if ((L.lane & ((1 << SH) - 1)) == 0) rg[(L.lane >> SH) * NWAVES + L.w] = t;
  __syncthreads();
  if ((int)threadIdx.x < nj) {
    const int jj = threadIdx.x;
    double a = 0, b = 0;
    for (int w = 0; w < NWAVES; ++w) {
      a += rg[(2 * jj) * NWAVES + w];
      b += rg[(2 * jj + 1) * NWAVES + w];
    }
    grad_put(P, j0 + jj, k, a, b);
  }
}

// D <= 64: Z goes through LDS (the caller's left-factor space, free once every
// wavefront has finished its products), so that thread t owns the chunks of
// four consecutive row elements t, t + 4D, t + 8D, ... and reads each
// control's matching chunks with 16-byte loads, consecutive across lanes.
// With mono (every control has at most one nonzero per row), Tr(Z^dag Hc[j])
// is the sum over rows a of conj(Z[a][col_j(a)]) val_j(a): thread t takes row
// t % D of control j0 + t / D of each group of four controls.
template <typename T, int D>
__device__ __forceinline__ void gradient_epilogue(const ProbDesc& P, int k, const Panel<T, D>& Z, const Lane& L,
                                                  void* lds, double* red, bool mono) {
  using v4 = typename Prec<T>::v4;
  constexpr int NV = D / 16;
  constexpr int EPT = 4 * NV;
  constexpr int NT = 4 * D;
  constexpr int SD = Mat<T, D>::SD;
  static_assert(NT == kEpiGroup * D, "one (control, row) pair per thread");
  T* zl = static_cast<T*>(lds);
  __syncthreads();  // every wavefront is done with the left factors
  panel_to_lds(zl, Z, L);
  __syncthreads();
  if (mono) {
    // The D threads of lane group jj = t / D (aligned inside one wavefront)
    // take row a = t % D of controls jj, jj + 4, jj + 8, jj + 12 of each
    // pass of 16, so that one control's sum stays inside one lane group: one
    // multi-value group reduction per pass and no barrier.
    constexpr int CPT = 4;
    constexpr int V = 2 * CPT;
    constexpr int GV = D / V;  // lanes per reduced value
    const int a = threadIdx.x % D, jj = threadIdx.x / D;
    const T* mv = reinterpret_cast<const T*>(P.mval);
    for (int j0 = 0; j0 < P.m; j0 += kEpiGroup * CPT) {
      double v[V];
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const int j = j0 + jj + kEpiGroup * i;
        double tr = 0, ti = 0;
        if (j < P.m) {
          const size_t idx = (size_t)j * D + a;
          const int off = lds_off<T, D>(a, gp(P.mcol)[idx]);
          const double zr = (double)zl[off], zi = (double)zl[D * SD + off];
          const double x = (double)gp(mv)[2 * idx], y = (double)gp(mv)[2 * idx + 1];
          tr = zr * x + zi * y;  // conj(z) h
          ti = zr * y - zi * x;
        }
        v[2 * i] = tr;
        v[2 * i + 1] = ti;
      }
      const double t = group_sum_many<V, D>(v, L.lane);
      const double t1 = __shfl_xor(t, GV, 64);  // the other half of the complex sum
      const int vi = a / GV;
      if (a % GV == 0 && (vi & 1) == 0) {
        const int j = j0 + jj + kEpiGroup * (vi >> 1);
        if (j < P.m) grad_put(P, j, k, t, t1);
      }
    }
    return;
  }
  const int e0 = 4 * threadIdx.x;
  double zr[EPT], zi[EPT];
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = e0 + 4 * NT * q;
      const int off = lds_off<T, D>(e / D, e % D + i);
      zr[4 * q + i] = (double)zl[off];
      zi[4 * q + i] = (double)zl[D * SD + off];
    }
  // FP32 keeps the sums of kEpiDense controls together for one multi-value
  // reduction and one barrier; FP64 (whose values take twice the registers)
  // publishes every kEpiGroup controls.  LG controls' row segments are
  // loaded together.
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int JG = F32 ? kEpiDense : kEpiGroup;
  constexpr int LG = 2;
  const T* H = reinterpret_cast<const T*>(P.Hint);
  for (int j0 = 0, grp = 0; j0 < P.m; j0 += JG, ++grp) {
    double v[2 * JG];
#pragma unroll
    for (int jb = 0; jb < JG; jb += LG) {
      double tr[LG], ti[LG];
#pragma unroll
      for (int jj = 0; jj < LG; ++jj) tr[jj] = ti[jj] = 0.0;
      if (!F32 || j0 + jb < P.m) {  // (FP32 groups: nothing to load past the last control)
        v4 hr[LG][NV], hi[LG][NV];
#pragma unroll
        for (int jj = 0; jj < LG; ++jj) {
          const int j = min(j0 + jb + jj, P.m - 1);
          const T* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
#pragma unroll
          for (int q = 0; q < NV; ++q) {
            hr[jj][q] = Prec<T>::gld4(Hj + 4 * NT * q);
            hi[jj][q] = Prec<T>::gld4(Hj + D * D + 4 * NT * q);
          }
        }
#pragma unroll
        for (int jj = 0; jj < LG; ++jj)
#pragma unroll
          for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double a = zr[4 * q + i], b = zi[4 * q + i];
              const double x = (double)hr[jj][q][i], y = (double)hi[jj][q][i];
              tr[jj] += a * x + b * y;  // conj(z) h
              ti[jj] += a * y - b * x;
            }
      }
#pragma unroll
      for (int jj = 0; jj < LG; ++jj) {
        v[2 * (jb + jj)] = tr[jj];
        v[2 * (jb + jj) + 1] = ti[jj];
      }
    }
    epilogue_publish<D / 16, JG>(P, k, j0, grp, v, L, red);
  }
}

// ---------------------------------------------------------------- slice propagators

// Delta_k = U_k - I for every slice: one workgroup per slice, D/16 wavefronts.
// Horner in delta form: R_q = I + X/q, R_i = I + X R_{i+1} / i, Delta = X R_2
// (X = A_k / 2^s), then s squarings Delta <- 2 Delta + Delta^2.
// (Paterson-Stockmeyer in X^2, which would form X^2 as a product, needs the
// same two products at q = 3 but held 40 more VGPRs at d = 64, a workgroup
// per CU less, and was 0.4 ms slower on the d = 64 batch of 32.)
// The expm and scan kernels take the three-product form (Ops::gemm3) at
// D >= 32 with a floor of two waves per SIMD, which keeps the extra registers
// of that form from lowering their occupancy.
template <int D>
constexpr int kMinWaves = D >= 32 ? 2 : 1;

// The slice Hamiltonians are kept for the adjoint at D >= 32.  At D = 16 the
// adjoint re-assembles H_k from the (L2-resident) controls, which costs less
// than writing and reading it back through HBM.
template <int D>
constexpr bool kKeepH = D >= 32;

// The expm's products take their steps in pairs (cgemm3m) in FP32; in FP64
// the extra fragment registers would add to its spills.
template <typename T>
constexpr int kExpmPairs = sizeof(T) == 4 ? 2 : 1;
// The FP32 d = 64 expm (one slice per workgroup) takes a floor of four waves
// per SIMD: it needs 130 VGPRs otherwise, and at 128 (two spilled) four
// workgroups share a CU instead of three (expm 1.88 -> 1.80 ms on the d = 64
// batch of 32).
template <typename T, int D>
constexpr int kExpmWaves = (sizeof(T) == 4 && D == 64) ? 4 : kMinWaves<D>;

template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kExpmWaves<T, D>)))
void k_expm(Work W) {
  __shared__ __align__(16) unsigned char lds[Ops::BYTES];
  Lane L;
  const Items I(W);
  if ((int)blockIdx.x >= I.total) return;  // (one item per workgroup)
  int p, k;
  split_item((int)blockIdx.x, W.rg.s_lo, W.rg.s_n, I.start, I.nprob, p, k);
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  int s, q, qb;
  const int sqk = gp(P.sq)[k];
  unpack_sq(sqk, s, q, qb);
  T* hk = (kKeepH<D> && (P.flags & RUN_GRAD)) ? pf_mat<T, D>(P.hk, k - W.rg.kbase) : nullptr;
  assemble<T, D, Ops>(lds, P, k, ldexp(P.dt, -s), 1.0, hk, (sqk & kPlanMono) != 0);
  __syncthreads();
  Panel<T, D> R, acc;
  Ops::load(R, lds, L);
  if (q >= 2) {
    panel_scale(R, (T)(1.0 / q));
    panel_add_identity(R, L, (T)1);
    for (int i = q - 1; i >= 1; --i) {
      Ops::template gemm3<kExpmPairs<T>>(acc, lds, R, L, true);
      R = acc;
      if (i >= 2) {
        panel_scale(R, (T)(1.0 / i));
        panel_add_identity(R, L, (T)1);
      }
    }
  }
  for (int j = 0; j < s; ++j) {
    __syncthreads();
    Ops::store(lds, R, L);
    __syncthreads();
    Ops::template gemm3<kExpmPairs<T>>(acc, lds, R, L, true);
    panel_axpby(R, (T)1, acc, (T)2);
  }
  panel_store(pf_mat<T, D>(P.delta, k - W.rg.kbase), R, L);
}

// ---------------------------------------------------------------- re-unitarisation

// Check of a chunk product S (FP32 panel) in FP64: r = |S^dag S - I|_F over
// the d x d block, recorded as the largest residual of the problem.  When
// r > tol, one Newton-Schulz polar step S <- S (3I - S^dag S) / 2 (Higham
// 1986) moves S back towards the unitary group; the steps are counted.  The
// FP32 panel is moved into the FP64 register layout (and back) through LDS,
// which must hold one FP64 matrix.
template <int D>
__device__ __forceinline__ void reunitarise(const ProbDesc& P, Panel<float, D>& S, void* lds_raw, double* red,
                                            const Lane& L) {
  constexpr int NW = D / 16;
  double* M = static_cast<double*>(lds_raw);
  double* Mi = M + D * Mat<double, D>::SD;
  const int d = P.d;
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int off = lds_off<double, D>(16 * rb + Prec<float>::rowmap(r, L.g), 16 * L.w + L.c16);
      M[off] = (double)S.re[rb][r];
      Mi[off] = (double)S.im[rb][r];
    }
  __syncthreads();
  Panel<double, D> Sd, G;
  panel_from_lds(Sd, M, L);
  __syncthreads();
  panel_to_lds_ct(M, Sd, L);
  __syncthreads();
  cgemm(G, M, Sd, L, true);  // G = S^dag S
  double e2 = 0;
#pragma unroll
  for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * rb + Prec<double>::rowmap(r, L.g), col = 16 * L.w + L.c16;
      if (row < d && col < d) {
        const double xr = G.re[rb][r] - (row == col ? 1.0 : 0.0), xi = G.im[rb][r];
        e2 += xr * xr + xi * xi;
      }
    }
  e2 = wave_sum(e2);
  if (L.lane == 0) red[L.w] = e2;
  __syncthreads();
  double tot = 0;
  for (int w = 0; w < NW; ++w) tot += red[w];
  const double res = sqrt(tot);
  if (threadIdx.x == 0)
    atomicMax(reinterpret_cast<unsigned long long*>(&P.diag[1]), (unsigned long long)__double_as_longlong(res));
  if (res > P.reun_tol) {
    // T = 3I - G, S <- S T / 2
    panel_scale(G, -1.0);
    panel_add_identity(G, L, 3.0);
    __syncthreads();
    panel_to_lds(M, Sd, L);
    __syncthreads();
    Panel<double, D> Sn;
    cgemm(Sn, M, G, L, true);
    panel_scale(Sn, 0.5);
    __syncthreads();
    panel_to_lds(M, Sn, L);
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int off = lds_off<double, D>(16 * rb + Prec<float>::rowmap(r, L.g), 16 * L.w + L.c16);
        S.re[rb][r] = (float)M[off];
        S.im[rb][r] = (float)Mi[off];
      }
    if (threadIdx.x == 0) atomicAdd(reinterpret_cast<unsigned long long*>(&P.diag[2]), 1ull);
  }
  __syncthreads();
}

// ---------------------------------------------------------------- chunked scans

// One workgroup per chunk.  Forward pass (bwd = 0): running product
// S = U_k ... U_{k0}; stores xprev[k] = S before slice k and the chunk total
// tf[c].  Backward pass (bwd = 1, after the carry): S starts from
// mc[c] = cb[c] cf[c]^dag and becomes U_k^dag ... U_{k1-1}^dag mc[c]; stores
// bloc[k] = S before slice k is applied, so that the adjoint's
// W_k = bloc[k] xprev[k]^dag takes one product.  (The backward chunk total
// that the carry needs is tf[c]^dag.)  Each step is S <- S + Delta S (or
// Delta^dag S) with Delta staged in LDS (the next Delta is loaded into
// registers during a step).  The LDS buffer is double (no barrier before it
// is refilled) except in FP32 at D = 64, where one buffer and a barrier let
// three workgroups share a CU instead of two (measured on the d = 64 batch
// of 32: backward scans 1.00 -> 0.94 ms; FP64, held to one workgroup per CU
// by its registers, lost a third with one buffer).
template <typename T, int D>
constexpr int kScanBufs = (sizeof(T) == 4 && D == 64) ? 1 : 2;

template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kMinWaves<D>)))
void k_scan_local(Work W, int dir) {
  __shared__ __align__(16) unsigned char lds[kScanBufs<T, D>][Ops::BYTES];
  const int bwd = dir < 0 ? (int)blockIdx.y : dir;  // dir < 0: both passes, one per blockIdx.y
  Lane L;
  const Items I(W);
  if ((int)blockIdx.x >= I.total) return;  // (one item per workgroup)
  int p, c;
  split_item((int)blockIdx.x, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  const int k0 = c * P.L;
  const int k1 = min(P.N, k0 + P.L);
  Panel<T, D> S, nxt, acc;
  if (bwd) panel_load(S, pf_mat<T, D>(P.mc, c), L); else panel_identity(S, L);
  const int n = k1 - k0;
  int k = bwd ? k1 - 1 : k0;
  panel_load(nxt, pf_mat<T, D>(P.delta, k - W.rg.kbase), L);
  for (int i = 0; i < n; ++i) {
    void* buf = lds[i % kScanBufs<T, D>];
    if (kScanBufs<T, D> == 1 && i > 0) __syncthreads();  // every wavefront is done with the previous factor
    if (bwd) Ops::store_ct(buf, nxt, L); else Ops::store(buf, nxt, L);
    const int kn = bwd ? k - 1 : k + 1;
    // the store of S before the prefetch of the next Delta, so that the wait
    // for the prefetch at the next step covers nothing issued after it
    panel_store(pf_mat<T, D>(bwd ? P.bloc : P.xprev, k - W.rg.kbase), S, L);
    if (i + 1 < n) panel_load(nxt, pf_mat<T, D>(P.delta, kn - W.rg.kbase), L);
    __syncthreads();
    Ops::gemm3(acc, buf, S, L, true);
    panel_axpby(S, (T)1, acc, (T)1);
    k = kn;
  }
  if (!bwd && !W.rg.recompute) panel_store(pf_mat<T, D>(P.tf, c), S, L);  // (k_reun follows in FP32)
}

// The re-unitarisation of the forward chunk totals tf[c] (FP32, problems with
// reun_tol >= 0), after the forward scans: one workgroup per chunk runs
// reunitarise() on the stored total.  A kernel of its own, so that the scan
// keeps the registers and LDS of its chain alone: inside it, the check's
// FP64 registers and its FP64 matrix in LDS cost the scan a workgroup per CU.
template <int D, bool PERSIST>
__global__ __launch_bounds__(4 * D) void k_reun(Work W) {
  __shared__ __align__(16) double lds[Mat<double, D>::LDS_ELEMS];
  __shared__ double red[D / 16];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    if (P.reun_tol >= 0) {  // uniform over the workgroup
      Panel<float, D> S;
      panel_load(S, pf_mat<float, D>(P.tf, c), L);
      reunitarise<D>(P, S, lds, red, L);
      panel_store(pf_mat<float, D>(P.tf, c), S, L);
    }
    if constexpr (!PERSIST) break;  // one item per workgroup: a single-trip loop
    __syncthreads();
  }
}

// The carry over the chunk totals, in groups of CG chunks (carry_groups):
//   k_carry_grp: one workgroup per (group, direction), a serial chain over the
//     group's chunk totals that stores the carry from the group start into
//     each chunk (forward cf_loc[c] = tf[c-1] ... tf[g0] into cf, backward
//     cb_loc[c] = tf[c+1]^dag ... tf[g1-1]^dag into cb) and the group total;
//   k_carry_top: one workgroup per (problem, direction), a serial chain over
//     the group totals that stores the carry into each group (forward from I,
//     ending with X_N, its fidelity and unitarity residual; backward from V);
//   k_mc: mc[c] = cb[c] cf[c]^dag with cf[c] = cf_loc[c] gcf[g] and
//     cb[c] = cb_loc[c] gcb[g].
// The chains are serial and each runs as one workgroup, so they take the
// three-product form at D >= 32 regardless of its registers.

// n steps of S <- A_i S, storing S before each step to out[i] (i < nstore).
// A_i is the PF matrix src[i] (stride step) or, with ct, its conjugate
// transpose.  Double-buffered LDS; the next factor is loaded during a step.
template <typename T, int D, typename Ops>
__device__ __forceinline__ void carry_chain(Panel<T, D>& S, const T* src, int step, int n, bool ct, T* out,
                                            int ostep, int nstore, unsigned char (*lds)[Ops::BYTES], const Lane& L) {
  constexpr int EL = Mat<T, D>::ELEMS;
  Panel<T, D> nxt, acc;
  if (n > 0) panel_load(nxt, src, L);
  for (int i = 0; i < nstore || i < n; ++i) {
    if (i < nstore) panel_store(out + (ptrdiff_t)i * ostep * EL, S, L);
    if (i >= n) break;
    void* buf = lds[i & 1];
    if (ct) Ops::store_ct(buf, nxt, L); else Ops::store(buf, nxt, L);
    if (i + 1 < n) panel_load(nxt, src + (ptrdiff_t)(i + 1) * step * EL, L);
    __syncthreads();
    Ops::gemm3(acc, buf, S, L, true);
    S = acc;
  }
}

// Group matrices: [0, PG) forward totals, [PG, 2 PG) backward totals,
// [2 PG, 3 PG) forward carries, [3 PG, 4 PG) backward carries.
template <typename T, int D>
__device__ __forceinline__ T* grp_mat(const ProbDesc& P, int kind, int g) {
  return pf_mat<T, D>(P.grp, kind * P.PG + g);
}

template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) void k_carry_grp(Work W) {
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  Lane L;
  const int bwd = blockIdx.y;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
  int p, g;
  split_item(item, 0, W.rg.c_n, I.start, I.nprob, p, g);
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  const int c0 = g * P.CG;
  const int n = min(P.CG, P.P - c0);
  Panel<T, D> S;
  panel_identity(S, L);
  if (!bwd) {
    carry_chain<T, D, Ops>(S, pf_mat<T, D>(P.tf, c0), 1, n, false, pf_mat<T, D>(P.cf, c0), 1, n, lds, L);
    panel_store(grp_mat<T, D>(P, 0, g), S, L);
  } else {
    const int c1 = c0 + n - 1;  // the chain runs from the group's last chunk down
    carry_chain<T, D, Ops>(S, pf_mat<T, D>(P.tf, c1), -1, n, true, pf_mat<T, D>(P.cb, c1), -1, n, lds, L);
    panel_store(grp_mat<T, D>(P, 1, g), S, L);
  }
  __syncthreads();
  }
}

template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) void k_carry_top(Work W) {
  constexpr int NW = Mat<T, D>::NW;
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  __shared__ double red[2 * NW];
  Lane L;
  const int bwd = blockIdx.y;
  const Items I(W);
  for (int p = blockIdx.x; p < I.nprob; p += gridDim.x) {
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  Panel<T, D> S, acc;
  const int ng = P.PG;
  if (!bwd) {
    panel_identity(S, L);
    carry_chain<T, D, Ops>(S, grp_mat<T, D>(P, 0, 0), 1, ng, false, grp_mat<T, D>(P, 2, 0), 1, ng, lds, L);
    fidelity_epilogue<T, D>(P, S, L, red);
    // Unitarity residual of X_N: S^dag S from the conjugate transpose in LDS.
    __syncthreads();
    Ops::store_ct(lds[0], S, L);
    __syncthreads();
    Ops::gemm(acc, lds[0], S, L, true);
    residual_epilogue<T, D>(P, acc, L, red);
  } else {
    panel_load(S, reinterpret_cast<const T*>(P.Vint), L);
    carry_chain<T, D, Ops>(S, grp_mat<T, D>(P, 1, ng - 1), -1, ng - 1, false, grp_mat<T, D>(P, 3, ng - 1), -1, ng,
                      lds, L);
  }
  __syncthreads();
  }
}

// mc[c] = cb[c] cf[c]^dag for every chunk, the start of its backward scan, so
// that W_k = (local backward product) mc[c] xprev[k]^dag; cf[c] and cb[c] are
// formed here from the in-group carries and the group carries.
template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) void k_mc(Work W) {
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
  int p, c;
  split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  const int g = c / P.CG;
  Panel<T, D> a, b, x, y;
  // cf[c] = cf_loc[c] gcf[g] and cb[c] = cb_loc[c] gcb[g]
  panel_load(a, pf_mat<T, D>(P.cf, c), L);
  panel_load(b, pf_mat<T, D>(P.cb, c), L);
  panel_load(x, grp_mat<T, D>(P, 2, g), L);
  panel_load(y, grp_mat<T, D>(P, 3, g), L);
  Ops::store(lds[0], a, L);
  Ops::store(lds[1], b, L);
  __syncthreads();
  Ops::gemm3(a, lds[0], x, L, true);
  Ops::gemm3(b, lds[1], y, L, true);
  // mc[c] = cb[c] cf[c]^dag
  __syncthreads();
  Ops::store(lds[0], b, L);
  Ops::store(lds[1], a, L);
  __syncthreads();
  Ops::load_ct(x, lds[1], L);
  Ops::gemm(a, lds[0], x, L, true);
  panel_store(pf_mat<T, D>(P.mc, c), a, L);
  __syncthreads();
  }
}

// ---------------------------------------------------------------- adjoint / gradient

// The gradient from only the entries of Z = E + X2 C2 + S C1 that the
// controls read (s = 0, FP32, every control a weighted permutation: Pauli
// strings).  Control j reads Z[a][b] at b = col_j(a), once per column b, so
// the lane that holds column b of the panels (wavefront b / 16, lane b % 16
// of each lane group) forms z = Z[minv_j(b)][b] as the dot product of row
// minv_j(b) of X2 and of S (LDS) with its own entries of C2 and C1, the four
// lane groups each taking their 16 of the d rows and then summing.  E[a][b]
// of the first kSampleGather controls was gathered from LDS before S took
// E's place (sample_gather); later controls take it from the lane that holds
// it, inside the dot product.  That is 2 d m complex multiply-adds per column
// on the vector ALU in place of the last two products (d^3 each), then
// T_j = sum_b conj(z) val_j(minv_j(b)) in FP64 as in gradient_epilogue.
template <int D>
constexpr int kSampleGroup = 4;  // controls per reduction
// Controls whose entries E[minv_j(b)][b] are gathered (8 KB of LDS at D = 64,
// which still fits two workgroups per CU).
constexpr int kSampleGather = 16;

// Thread t: column t % D of controls t / D + 4 i.  The rows are loaded before
// the block's square is formed and the entries read after it, while E is
// still in LDS.
template <int D>
__device__ __forceinline__ void sample_rows(const ProbDesc& P, int (&ga)[kSampleGather / 4]) {
#pragma unroll
  for (int i = 0; i < kSampleGather / 4; ++i) {
    const int j = (int)threadIdx.x / D + 4 * i;
    ga[i] = j < P.m ? gp(P.minv)[(size_t)j * D + threadIdx.x % D] : 0;
  }
}

template <int D>
__device__ __forceinline__ void sample_gather(const ProbDesc& P, const int (&ga)[kSampleGather / 4], const void* elds,
                                              float* eg) {
  const float* er = static_cast<const float*>(elds);
  const float* ei = er + D * Mat<float, D>::SD;
  const int b = threadIdx.x % D;
#pragma unroll
  for (int i = 0; i < kSampleGather / 4; ++i) {
    const int j = (int)threadIdx.x / D + 4 * i;
    if (j < P.m) {
      const int off = lds_off<float, D>(ga[i], b);
      eg[2 * (j * D + b)] = er[off];
      eg[2 * (j * D + b) + 1] = ei[off];
    }
  }
}

// Partial sums of z over this lane group's rows; WITH_E also picks E[a][b]
// into (er, ei) in the lane that holds it (zero elsewhere), so that it is
// added after the sum over the lane groups, as the gathered entry is: the
// two forms give the same bits.
template <int D, bool WITH_E>
__device__ __forceinline__ void sampled_dot(float& zr, float& zi, float& er, float& ei, int a, const float* xr,
                                            const float* xi, const float* yr, const float* yi,
                                            const Panel<float, D>& E, const Panel<float, D>& C1,
                                            const Panel<float, D>& C2, const Lane& L) {
  constexpr int NV = D / 16;
  constexpr int SD = Mat<float, D>::SD;
  // LDS row a at the columns of this lane's panel rows 16 rb + 4 g + r
  const int base = a * SD + 4 * L.g;
  float pr[4] = {0.f, 0.f, 0.f, 0.f}, pi[4] = {0.f, 0.f, 0.f, 0.f};  // one chain per r
#pragma unroll
  for (int rb = 0; rb < NV; ++rb) {
    const f4 ar = Prec<float>::ld4(xr + base + 16 * rb), ai = Prec<float>::ld4(xi + base + 16 * rb);
    const f4 br = Prec<float>::ld4(yr + base + 16 * rb), bi = Prec<float>::ld4(yi + base + 16 * rb);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (WITH_E) {
        const bool own = 16 * rb + 4 * L.g + r == a;
        er = own ? E.re[rb][r] : er;
        ei = own ? E.im[rb][r] : ei;
      }
      pr[r] = fmaf(ar[r], C2.re[rb][r], pr[r]);
      pr[r] = fmaf(-ai[r], C2.im[rb][r], pr[r]);
      pr[r] = fmaf(br[r], C1.re[rb][r], pr[r]);
      pr[r] = fmaf(-bi[r], C1.im[rb][r], pr[r]);
      pi[r] = fmaf(ar[r], C2.im[rb][r], pi[r]);
      pi[r] = fmaf(ai[r], C2.re[rb][r], pi[r]);
      pi[r] = fmaf(br[r], C1.im[rb][r], pi[r]);
      pi[r] = fmaf(bi[r], C1.re[rb][r], pi[r]);
    }
  }
  zr = (pr[0] + pr[1]) + (pr[2] + pr[3]);
  zi = (pi[0] + pi[1]) + (pi[2] + pi[3]);
}

// The sampled step's reduction: each group's per-wavefront sums go to their
// own slot of the reduction array (epilogue_publish's layout), and one
// barrier publishes every kSampleSlots groups at once.
constexpr int kSampleSlots = 2 * kEpiDense / kSampleGroup<64>;

template <int NWAVES, int G>
__device__ __forceinline__ void sample_stash(int slot, double (&v)[2 * G], const Lane& L, double* red) {
  constexpr int V = 2 * G;
  constexpr int SH = 6 - __builtin_ctz(V);
  const double t = wave_sum_many<V>(v, L.lane);
  if ((L.lane & ((1 << SH) - 1)) == 0) red[slot * V * NWAVES + (L.lane >> SH) * NWAVES + L.w] = t;
}

template <int NWAVES, int G>
__device__ __forceinline__ void sample_flush(const ProbDesc& P, int k, int j0, int nj, const double* red) {
  if ((int)threadIdx.x < nj) {
    const int jj = threadIdx.x;
    const double* rg = red + (jj / G) * 2 * G * NWAVES;
    const int q = jj % G;
    double a = 0, b = 0;
    for (int w = 0; w < NWAVES; ++w) {
      a += rg[(2 * q) * NWAVES + w];
      b += rg[(2 * q + 1) * NWAVES + w];
    }
    grad_put(P, j0 + jj, k, a, b);
  }
}

template <int D, bool GATHERED>
__device__ __forceinline__ void sampled_gradient(const ProbDesc& P, int k, const Panel<float, D>& E,
                                                 const Panel<float, D>& C1, const Panel<float, D>& C2,
                                                 const void* x2lds, const void* slds, const float* eg,
                                                 double* red, const Lane& L) {
  constexpr int G = kSampleGroup<D>;
  const float* xr = static_cast<const float*>(x2lds);
  const float* xi = xr + D * Mat<float, D>::SD;
  const float* yr = static_cast<const float*>(slds);
  const float* yi = yr + D * Mat<float, D>::SD;
  const int b = 16 * L.w + L.c16;
  const float* mv = reinterpret_cast<const float*>(P.mval);
  static_assert(G * kSampleSlots <= 4 * D, "one thread per control of a block");
  float zr = 0.f, zi = 0.f;
  for (int j0 = 0, grp = 0; j0 < P.m; j0 += G, ++grp) {
    const int slot = grp % kSampleSlots;
    if (slot == 0 && grp > 0) __syncthreads();  // the previous block's sums are read
    // the group's table entries first: two round trips per group, not per control
    int ag[G], fl[G];
    float hrg[G], hig[G];
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      const int j = min(j0 + jj, P.m - 1);
      ag[jj] = gp(P.minv)[(size_t)j * D + b];
      fl[jj] = gp(P.mok)[j];
    }
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      const size_t e = (size_t)min(j0 + jj, P.m - 1) * D + ag[jj];
      hrg[jj] = gp(mv)[2 * e];
      hig[jj] = gp(mv)[2 * e + 1];
    }
    double v[2 * G];
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      // a control with the previous one's columns (in this group) reads the
      // same entries of Z: z is reused (uniform over the workgroup)
      if (jj == 0 || j0 + jj >= P.m || !(fl[jj] & 4)) {
        const int j = min(j0 + jj, P.m - 1);
        const bool gathered = GATHERED && j < kSampleGather;
        float er = 0.f, ei = 0.f;
        if constexpr (GATHERED) {
          if (gathered) sampled_dot<D, false>(zr, zi, er, ei, ag[jj], xr, xi, yr, yi, E, C1, C2, L);
          else sampled_dot<D, true>(zr, zi, er, ei, ag[jj], xr, xi, yr, yi, E, C1, C2, L);
        } else {
          sampled_dot<D, true>(zr, zi, er, ei, ag[jj], xr, xi, yr, yi, E, C1, C2, L);
        }
        zr += __shfl_xor(zr, 16, 64);
        zi += __shfl_xor(zi, 16, 64);
        zr += __shfl_xor(zr, 32, 64);
        zi += __shfl_xor(zi, 32, 64);
        if (gathered) {
          er = eg[2 * (j * D + b)];
          ei = eg[2 * (j * D + b) + 1];
        } else {  // one nonzero among the lane groups: the sum is exact
          er += __shfl_xor(er, 16, 64);
          ei += __shfl_xor(ei, 16, 64);
          er += __shfl_xor(er, 32, 64);
          ei += __shfl_xor(ei, 32, 64);
        }
        zr += er;
        zi += ei;
      }
      const float hr = hrg[jj], hi = hig[jj];
      double tr = 0, ti = 0;
      if (L.g == 0 && j0 + jj < P.m) {  // conj(z) h, once per column
        tr = (double)zr * hr + (double)zi * hi;
        ti = (double)zr * hi - (double)zi * hr;
      }
      v[2 * jj] = tr;
      v[2 * jj + 1] = ti;
    }
    sample_stash<D / 16, G>(slot, v, L, red);
    if (slot == kSampleSlots - 1 || j0 + G >= P.m) {
      __syncthreads();
      const int jb = j0 - slot * G;  // first control of the block
      sample_flush<D / 16, G>(P, k, jb, min(kSampleSlots * G, P.m - jb), red);
    }
  }
}

// Ops::gemm3 with P accumulator chain pairs where P > 1 (StdOps only).
template <int P, typename Ops, typename T, int D>
__device__ __forceinline__ void gemm3p(Panel<T, D>& acc, const void* lds, const Panel<T, D>& B, const Lane& L,
                                       bool zero_acc) {
  if constexpr (P > 1) Ops::template gemm3<P>(acc, lds, B, L, zero_acc);
  else Ops::gemm3(acc, lds, B, L, zero_acc);
}

template <typename T, int D, typename Ops>
constexpr bool kSampleLast = std::is_same<Ops, StdOps<float, D>>::value && D >= 32;

// One workgroup per slice.
//  1. W_k = bloc[k] xprev[k]^dag  (one product; bloc[k] carries mc[c]).
//  2. X = A_k^dag / 2^s in LDS buffer 0, E = W_k / 2^s in buffer 1.
//  3. The Taylor polynomial of degree qb of M = [[X, E], [0, X]] in delta
//     form, p(M) - I, by Paterson-Stockmeyer with M^2 as the step: the top
//     right block of exp(M) is the Frechet derivative L(X, E).
//  4. s squarings: [[I + D1, Q], [0, I + D1]]^2 gives D1 <- 2 D1 + D1^2 and
//     Q <- 2Q + D1 Q + Q D1.  Z_k = Q.
//  5. T_j = Tr(Z_k^dag Hc[j]) in FP64, grad = (2 dt / d^2) Im(conj(g) T_j).
// Two workgroups per CU (two waves per SIMD) where the LDS allows it, so
// that one workgroup's LDS and VALU work overlaps the other's MFMAs.  H_k is
// loaded together with the W factors where the extra registers cost no
// occupancy (FP32 at D = 64, FP64 at D = 32).
template <typename T, int D>
constexpr int kAdjWaves = ((sizeof(T) == 4 && D <= 64) || (sizeof(T) == 8 && D == 32)) ? 2 : 1;
template <typename T, int D>
constexpr bool kEarlyH = (sizeof(T) == 4 && D == 64) || (sizeof(T) == 8 && D == 32);

// MODE 0: every slice; where the sampled last step applies (kSampleLast), two
// instances split the slices: MODE 1 takes those where it does not apply,
// MODE 2 those where it does (s = 0, permutation controls), each returning at
// once for the others, so that neither carries the other's registers.
template <typename T, int D, typename Ops, int MODE = 0>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kAdjWaves<T, D>)))
void k_adjoint(Work W) {
  constexpr int NW = Mat<T, D>::NW;
  constexpr int AP = MODE == 2 ? 2 : 1;  // accumulator chain pairs of the sampling instance's products
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  __shared__ double red[2 * kEpiDense * 2 * NW];
  // sample_gather
  constexpr bool GATHER = MODE == 2;
  __shared__ __align__(16) float eg[GATHER ? 2 * kSampleGather * D : 1];
  Lane L;
  const Items I(W);
  if ((int)blockIdx.x >= I.total) return;  // (one item per workgroup)
  int p, k;
  split_item((int)blockIdx.x, W.rg.s_lo, W.rg.s_n, I.start, I.nprob, p, k);
  const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
  const int sqk = gp(P.sq)[k];
  int s, q, qb;
  unpack_sq(sqk, s, q, qb);
  if constexpr (MODE != 0) {
    const bool sampled = (sqk & kPlanSampled) != 0;  // uniform over the workgroup
    if (sampled != (MODE == 2)) return;
  }
  const bool mono = (sqk & kPlanMono) != 0;
  Panel<T, D> R1, R2, A1, A2;

  // 1. W = bloc[k] xprev[k]^dag (bloc carries mc[c]).  The slice's global
  //    loads (xprev, bloc and, where the registers allow, H_k) are issued
  //    together.
  HamRegs<T, D> ham;
  if constexpr (kEarlyH<T, D>) ham_load<T, D>(ham, pf_mat<T, D>(P.hk, k - W.rg.kbase));
  panel_load(A2, pf_mat<T, D>(P.xprev, k - W.rg.kbase), L);
  panel_load(R2, pf_mat<T, D>(P.bloc, k - W.rg.kbase), L);
  Ops::store(lds[0], R2, L);
  Ops::store(lds[1], A2, L);
  __syncthreads();
  Ops::load_ct(A2, lds[1], L);
  gemm3p<AP, Ops>(R2, lds[0], A2, L, true);  // R2 = W
  __syncthreads();

  // 2. E = W / 2^s, X = A^dag / 2^s
  const T scl = (T)ldexp(1.0, -s);
  panel_scale(R2, scl);
  Ops::store(lds[1], R2, L);
  if constexpr (kKeepH<D>) {
    if constexpr (!kEarlyH<T, D>) ham_load<T, D>(ham, pf_mat<T, D>(P.hk, k - W.rg.kbase));
    ham_put<T, D, Ops>(lds[0], ham, ldexp(P.dt, -s), -1.0, (P.flags & RUN_GENERAL) != 0);
  } else {
    assemble<T, D, Ops, (sizeof(T) == 4 ? 4 : 2)>(lds[0], P, k, ldexp(P.dt, -s), -1.0, nullptr, mono,
                                                  (P.flags & RUN_GENERAL) != 0);
  }
  __syncthreads();
  const void* X = lds[0];
  const void* E = lds[1];

  // 3. Paterson-Stockmeyer on the block.  With M^2 = [[X2, S], [0, X2]],
  //    X2 = X X and S = X E + E X, the delta block is p(M) - I = M + M^2 C,
  //    C = sum_{n=2..qb} M^(n-2) / n!.  C runs Horner in M^2 over the digits
  //    D_t = I / (2t+2)! + M / (2t+3)! (terms above degree qb dropped):
  //    C <- D_t + M^2 C = [[D_t11 + X2 C1, b_t E + X2 C2 + S C1], [0, .]].
  //    Each block product by M^2 takes three d x d products, the last one
  //    only the blocks used next.
  Panel<T, D> R3;
  int ga[kSampleGather / 4];
  if constexpr (GATHER) sample_rows<D>(P, ga);
  Ops::load(R1, X, L);  // R1 = X, R2 = E
  Ops::gemm3(A1, X, R1, L, true);  // A1 = X2
  gemm3p<AP, Ops>(A2, X, R2, L, true);
  gemm3p<AP, Ops>(A2, E, R1, L, false);  // A2 = S
  if constexpr (GATHER) sample_gather<D>(P, ga, E, eg);
  __syncthreads();                  // X and E are read: M^2 takes their place
  Ops::store(lds[0], A1, L);
  Ops::store(lds[1], A2, L);
  const int top = (qb - 2) / 2;  // index of the last digit
  int t;                         // next digit, folded in by a block product
  if (qb & 1) {                  // C = D_top = I / (qb-1)! + M / qb!
    t = top - 1;
    A1 = R1;
    panel_scale(A1, (T)inv_factorial(qb));
    panel_add_identity(A1, L, (T)inv_factorial(qb - 1));
    A2 = R2;
    panel_scale(A2, (T)inv_factorial(qb));
  } else if (top > 0) {  // D_top = I / qb!: C = D_{top-1} + M^2 / qb! without a product
    t = top - 2;
    panel_axpby(A1, (T)inv_factorial(qb - 1), R1, (T)inv_factorial(qb));
    panel_add_identity(A1, L, (T)inv_factorial(qb - 2));
    panel_axpby(A2, (T)inv_factorial(qb - 1), R2, (T)inv_factorial(qb));
  } else {  // qb = 2: C = I / 2
    t = -1;
    panel_zero(A1);
    panel_add_identity(A1, L, (T)0.5);
    panel_zero(A2);
  }
  __syncthreads();
  for (; t >= 0; --t) {
    const T a = (T)inv_factorial(2 * t + 2), b = (T)inv_factorial(2 * t + 3);
    R3 = R2;
    panel_scale(R3, b);
    Ops::gemm3(R3, lds[0], A2, L, false);
    Ops::gemm3(R3, lds[1], A1, L, false);  // R3 = b E + X2 C2 + S C1
    A2 = R1;
    panel_scale(A2, b);
    panel_add_identity(A2, L, a);
    Ops::gemm3(A2, lds[0], A1, L, false);  // A2 = a I + b X + X2 C1
    A1 = A2;
    A2 = R3;
  }
  if constexpr (MODE == 2) {
    // 4'-5'. only the entries of Z that the controls read
    sampled_gradient<D, GATHER>(P, k, R2, A1, A2, lds[0], lds[1], eg, red, L);
  } else {
  Ops::gemm3(R2, lds[0], A2, L, false);
  Ops::gemm3(R2, lds[1], A1, L, false);              // R2 = Q = E + X2 C2 + S C1
  if (s > 0) Ops::gemm3(R1, lds[0], A1, L, false);  // R1 = D1 = X + X2 C1
  A1 = R1;
  A2 = R2;

  // 4. squarings
  for (int j = 0; j < s; ++j) {
    __syncthreads();
    Ops::store(lds[0], A1, L);
    Ops::store(lds[1], A2, L);
    __syncthreads();
    Ops::gemm3(R2, lds[0], A2, L, true);   // D1 Q
    Ops::gemm3(R2, lds[1], A1, L, false);  // + Q D1
    panel_axpby(R2, (T)2, A2, (T)1);  // R2 = 2Q + D1 Q + Q D1
    if (j + 1 < s) {
      Ops::gemm3(R1, lds[0], A1, L, true);
      panel_axpby(A1, (T)1, R1, (T)2);
    }
    A2 = R2;
  }

  // 5. inner products with the controls (FP64), then the gradient
  gradient_epilogue<T, D>(P, k, A2, L, lds[0], red, mono);
  }
}

// ================================================================ segments: the Hermitian path at D <= 64
//
// For Hermitian H_k the costates need no stored products and no Frechet
// block.  With N_k = Q_{k-1} P_{k-1}^dag (Q, P of the header), W_k = U_k N_k and
// N_{k+1} = U_k N_k U_k^dag, and
//   Z_k = L(A_k^dag, W_k) = int_0^1 e^{sA_k} N_k e^{-sA_k} ds = sum_n C_n / (n + 1)!,
//   N_{k+1} = sum_n C_n / n!,   C_0 = N_k,  C_{n+1} = [A_k, C_n]
// (A_k anti-Hermitian).  Every step keeps Hermitian matrices Hermitian, and
// dF/du[j][k] = -(2 dt / d^2) |g| Tr(Hc[j] Z(Y_k)) reads only the Hermitian
// Y = (g N - (g N)^dag) / (2i |g|), whose commutator is one product:
// [A, C] = A C + (A C)^dag.  A slice costs m products with the one left factor
// A_k (m the degree at which the series' remainder at 2 |A_k| meets the unit
// roundoff) where the block form took a chain product, W, and six to twelve
// for the block, and reads nothing per slice but its amplitudes.
//
// Slices with s > 0 take the series on A_k / 2^s and double it s times,
// Z <- (Z + U Z U^dag) / 2 with U the propagator of the part covered so far, which
// starts from the exponential that k_seg_fwd has kept.
//
// The chunks are cut into segments of at most kSegMax slices, so that few
// problems still fill the chip: k_seg_fwd forms the segment totals, k_seg_join
// the chunk totals and the prefixes at the segment starts, k_seg_y each
// chunk's Y (after the carry), k_seg_grad the gradient of a segment from
// Y at its start, P_s Y P_s^dag (from P_s - I: the rounding of the products
// then scales with it and not with Y).  Panels and left factors carry Ops::C.
// Two workgroups per CU (two waves per SIMD) where registers and LDS allow it.
template <typename T, int D>
constexpr int kSegWaves = (sizeof(T) == 8 && D == 64) ? 1 : 2;
// The workspace has a second array for the exponentials of squared problems.
template <int D>
constexpr bool kKeepU = D >= 32;
// Workgroups that fill the chip's 256 CUs with kSegWaves wavefronts per SIMD.
template <typename T, int D>
constexpr int kSqGrid = 256 * 4 * kSegWaves<T, D> / (D / 16);

// Item -> (problem, chunk, segment), and the segment's slices [ka, kb).
struct SegItem {
  int p, c, s, ka, kb;
};
__device__ __forceinline__ SegItem seg_split(int item, const Range& rg, const Items& I, const ProbDesc* descs) {
  SegItem r;
  if (rg.c_n > 0) {
    const int sc = seg_count(descs[0].L, descs[0].SM);  // uniform launches share L
    const int per = rg.c_n * sc;
    r.p = item / per;
    const int x = item - r.p * per;
    r.c = rg.c_lo + x / sc;
    r.s = x % sc;
  } else {
    r.p = locate(I.start, I.nprob, item);
    const int x = item - gp(I.start)[r.p];
    const int sc = seg_count(descs[I.desc(r.p)].L, descs[I.desc(r.p)].SM);
    r.c = x / sc;
    r.s = x % sc;
  }
  const ProbDesc& P = descs[I.desc(r.p)];
  const int h = seg_len(P.L, P.SM);
  const int k1 = min(P.N, (r.c + 1) * P.L);
  r.ka = r.c * P.L + r.s * h;
  r.kb = min(k1, r.ka + h);
  return r;
}

// The row tables and amplitudes of one segment in LDS (row-table controls,
// where they fit): entries (j, a) in ENT, amplitudes u[j][ka + i] in SL * MAX.
template <typename T, int D>
struct SegTab {
  // two workgroups of the d = 64 FP32 gradient kernel share a CU's 160 KB
  // (four of the d = 32 FP64 one)
  static constexpr int ENT = (sizeof(T) == 4 && D == 64) ? 12 * D : (sizeof(T) == 8 && D == 32) ? 10 * D : 16 * D;
  static constexpr int MAXM = ENT / D;
  T vr[ENT], vi[ENT];
  unsigned char col[ENT];
  T u[MAXM * kSegMax];
};

template <typename T, int D>
__device__ __forceinline__ bool seg_tab_load(SegTab<T, D>& S, const ProbDesc& P, int ka, int kb, bool mono) {
  if (!mono || P.m > SegTab<T, D>::MAXM) return false;
  const T* mv = reinterpret_cast<const T*>(P.mval);
  for (int e = threadIdx.x; e < P.m * D; e += 4 * D) {
    S.col[e] = (unsigned char)gp(P.mcol)[e];
    S.vr[e] = gp(mv)[2 * e];
    S.vi[e] = gp(mv)[2 * e + 1];
  }
  const int n = kb - ka;
  for (int e = threadIdx.x; e < P.m * n; e += 4 * D) {
    const int j = e / n, i = e - j * n;
    S.u[j * kSegMax + i] = (T)gp(P.u)[(size_t)j * P.N + ka + i];
  }
  return true;
}

// X = -i c H_k as this wavefront's panel, H_k = H0 + sum_j u[j][k] Hc[j] with
// the sums of assemble(); lds (one planar matrix) and the tables are written
// and read inside: starts and ends with a barrier.
template <typename T, int D>
__device__ __forceinline__ void assemble_panel(Panel<T, D>& X, void* lds, const ProbDesc& P, int k, double c,
                                               bool mono, const SegTab<T, D>* tab, int ki, const Lane& L) {
  using v4 = typename Prec<T>::v4;
  constexpr int NV = D / 16;
  constexpr int NT = 4 * D;
  const T* H = reinterpret_cast<const T*>(P.Hint);
  T* pl = static_cast<T*>(lds);
  T* pi = pl + D * Mat<T, D>::SD;
  const int e0 = 4 * threadIdx.x;
  v4 hr[NV], hi[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    hr[v] = Prec<T>::gld4(H + e0 + 4 * NT * v);
    hi[v] = Prec<T>::gld4(H + D * D + e0 + 4 * NT * v);
  }
  if (!mono) {
    constexpr int G = sizeof(T) == 4 ? 2 : 1;  // controls loaded together
    for (int j0 = 0; j0 < P.m; j0 += G) {
      v4 ar[G][NV], ai[G][NV];
      T uw[G];
#pragma unroll
      for (int jj = 0; jj < G; ++jj) {
        const int j = min(j0 + jj, P.m - 1);
        uw[jj] = j0 + jj < P.m ? (T)gp(P.u)[(size_t)j * P.N + k] : (T)0;
        const T* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          ar[jj][v] = Prec<T>::gld4(Hj + 4 * NT * v);
          ai[jj][v] = Prec<T>::gld4(Hj + D * D + 4 * NT * v);
        }
      }
#pragma unroll
      for (int jj = 0; jj < G; ++jj)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            hr[v][i] = fma(uw[jj], ar[jj][v][i], hr[v][i]);
            hi[v][i] = fma(uw[jj], ai[jj][v][i], hi[v][i]);
          }
    }
  }
  __syncthreads();  // the buffer's last readers are done
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int e = e0 + 4 * NT * v;
    if constexpr (sizeof(T) == 4) {
      const int off = lds_off<T, D>(e / D, e % D);
      Prec<T>::st4(pl + off, hr[v]);
      Prec<T>::st4(pi + off, hi[v]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int off = lds_off<T, D>(e / D, e % D + i);
        pl[off] = hr[v][i];
        pi[off] = hi[v][i];
      }
    }
  }
  __syncthreads();
  if (mono) {
    // The thread of row a adds the row's entry of each control in turn; runs of
    // controls at the same column (X_i and Y_i) stay in registers.
    if ((int)threadIdx.x < D) {
      const int a = threadIdx.x;
      int off = -1;
      T sr = 0, si = 0;
      auto add = [&](int col, T uj, T vr, T vi) {
        const int o = lds_off<T, D>(a, col);
        if (o != off) {
          if (off >= 0) {
            pl[off] = sr;
            pi[off] = si;
          }
          off = o;
          sr = pl[o];
          si = pi[o];
        }
        sr = fma(uj, vr, sr);
        si = fma(uj, vi, si);
      };
      if (tab) {
        for (int j = 0; j < P.m; ++j)
          add(tab->col[j * D + a], tab->u[j * kSegMax + ki], tab->vr[j * D + a], tab->vi[j * D + a]);
      } else {
        const T* mv = reinterpret_cast<const T*>(P.mval);
        for (int j = 0; j < P.m; ++j) {
          const size_t idx = (size_t)j * D + a;
          add(gp(P.mcol)[idx], (T)gp(P.u)[(size_t)j * P.N + k], gp(mv)[2 * idx], gp(mv)[2 * idx + 1]);
        }
      }
      pl[off] = sr;
      pi[off] = si;
    }
    __syncthreads();
  }
  panel_from_lds(X, static_cast<const T*>(lds), L);
  __syncthreads();
  // c in two numbers of type T: in FP32 its rounding alone would be the same
  // relative error in every slice, and add up over the chain
  const T f = (T)c, fl = (T)(c - (double)f);
#pragma unroll
  for (int rb = 0; rb < NV; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const T xr = X.re[rb][r], xi = X.im[rb][r];
      X.re[rb][r] = fma(f, xi, fl * xi);  // -i c (xr + i xi)
      X.im[rb][r] = -fma(f, xr, fl * xr);
    }
}

// Coefficients of the degree-8 Taylor polynomial in three products (Bader,
// Blanes and Casas, Mathematics 7 (2019) 1174, eq. 8):
//   A4 = A2 (x1 A + x2 A2),  T8 = I + A + y2 A2 + (x3 A2 + A4)(x4 I + x5 A + x6 A2 + x7 A4).
struct T8 {
  static constexpr double r177 = 13.304134695650071;  // sqrt(177)
  static constexpr double x3 = 2.0 / 3.0, x1 = x3 * (1 + r177) / 88, x2 = x3 * (1 + r177) / 352,
                          x4 = (-271 + 29 * r177) / (315 * x3), x5 = 11 * (-1 + r177) / (1260 * x3),
                          x6 = 11 * (-9 + r177) / (5040 * x3), x7 = (89 - r177) / (5040 * x3 * x3),
                          y2 = (857 - 58 * r177) / 630;
};

// R = C (exp(A) - I) from the panel X = C A / 2^s (A anti-Hermitian), whose left
// factor is in lds already (and is replaced there): the Taylor polynomial of a
// degree of at least q in taylor_products(q) products, then s squarings.  part (a
// PF matrix, or null): receives C (exp(A / 2^s) - I) where s > 0.
//  * q <= 3: Horner in delta form with the one left factor, R <- (X + X R) / i;
//  * q = 4: X + A2 (I / 2 + X / 6 + A2 / 24);  q <= 8: T8;
//  * above: Paterson-Stockmeyer with A3 as the step.
template <typename T, int D, typename Ops>
__device__ __forceinline__ void taylor_delta(Panel<T, D>& R, const Panel<T, D>& X, void* lds, int s, int q,
                                             const Lane& L, T* part = nullptr) {
  constexpr T C = Ops::C, CI = (T)1 / Ops::C;
  Panel<T, D> acc;
  if (q <= 3) {
    R = X;
    panel_scale(R, (T)(1.0 / q));
    for (int i = q - 1; i >= 1; --i) {
      Ops::mul(acc, lds, R, L);
      const T ri = (T)(1.0 / i), rs = ri * CI;
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          R.re[rb][r] = fma(rs, acc.re[rb][r], ri * X.re[rb][r]);
          R.im[rb][r] = fma(rs, acc.im[rb][r], ri * X.im[rb][r]);
        }
    }
  } else {
    Panel<T, D> A2;
    Ops::mul(A2, lds, X, L);
    panel_scale(A2, CI);
    if (q <= 8) {
      __syncthreads();
      Ops::store_ct(lds, A2, L);  // A2 = A2^dag
      __syncthreads();
      // B = a I + b X + c A2 as the right factor of the next product
      const T a = q == 4 ? (T)0.5 : (T)0, b = (T)(q == 4 ? 1.0 / 6 : T8::x1), c = (T)(q == 4 ? 1.0 / 24 : T8::x2);
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb) {
        R.re[rb] = b * X.re[rb] + c * A2.re[rb];
        R.im[rb] = b * X.im[rb] + c * A2.im[rb];
      }
      panel_add_identity(R, L, a * C);
      Ops::mul(acc, lds, R, L);
      panel_scale(acc, CI);  // A4 (q = 4: A2 B)
      R = X;
      if (q == 4) {
        panel_fma(R, (T)1, acc);
      } else {
        panel_fma(R, (T)T8::y2, A2);
#pragma unroll
        for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const T ar = A2.re[rb][r], ai = A2.im[rb][r], pr = acc.re[rb][r], pi = acc.im[rb][r];
            acc.re[rb][r] = fma((T)T8::x3, ar, pr);  // the left factor x3 A2 + A4
            acc.im[rb][r] = fma((T)T8::x3, ai, pi);
            A2.re[rb][r] = fma((T)T8::x5, X.re[rb][r], fma((T)T8::x6, ar, (T)T8::x7 * pr));
            A2.im[rb][r] = fma((T)T8::x5, X.im[rb][r], fma((T)T8::x6, ai, (T)T8::x7 * pi));
          }
        __syncthreads();
        Ops::store(lds, acc, L);
        panel_add_identity(A2, L, (T)(T8::x4 * C));
        __syncthreads();
        Ops::mul(acc, lds, A2, L);
        panel_fma(R, CI, acc);
      }
    } else {
      Ops::mul(R, lds, A2, L);
      panel_scale(R, CI);  // A3
      __syncthreads();
      Ops::store_nct(lds, R, L);  // A3 = -A3^dag
      __syncthreads();
      const int top = (q - 1) / 3;
      panel_scale(R, q >= 3 * top + 3 ? (T)inv_factorial(3 * top + 3) : (T)0);
      for (int t = top;; --t) {  // R <- D_t + A3 R, D_t = X^0, X, X^2 over (3t)!, (3t+1)!, (3t+2)!
        const T b = 3 * t + 1 <= q ? (T)inv_factorial(3 * t + 1) : (T)0;
        const T c = 3 * t + 2 <= q ? (T)inv_factorial(3 * t + 2) : (T)0;
        panel_fma(R, b, X);
        panel_fma(R, c, A2);
        if (t == 0) break;
        panel_add_identity(R, L, (T)inv_factorial(3 * t) * C);
        Ops::mul(acc, lds, R, L);
        R = acc;
        panel_scale(R, CI);
      }
    }
  }
  if (s > 0 && part) panel_store(part, R, L);
  for (int j = 0; j < s; ++j) {
    __syncthreads();
    Ops::store(lds, R, L);
    __syncthreads();
    Ops::mul(acc, lds, R, L);
    panel_scale(R, (T)2);
    panel_fma(R, CI, acc);
  }
}

// The totals U_{kb-1} ... U_{ka} of the segments less I (into xprev at the
// segment's first slice).  The exponentials' products run on Ops; the chain's, whose
// errors add up over the N slices, always in precision T.
template <typename T, int D, typename Ops, bool PERSIST>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kSegWaves<T, D>))) void k_seg_fwd(Work W) {
  using Std = StdOps<T, D>;
  constexpr T CI = (T)1 / Ops::C;
  // one buffer for the assembly and every left factor: at d = 32 in FP64 two
  // would leave a CU six wavefronts
  __shared__ __align__(16) unsigned char la[Ops::BYTES > Std::BYTES ? Ops::BYTES : Std::BYTES];
  __shared__ SegTab<T, D> tab;
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    const SegItem g = seg_split(item, W.rg, I, W.descs);
    if (g.ka < g.kb) {
      const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
      const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
      const SegTab<T, D>* tb = seg_tab_load<T, D>(tab, P, g.ka, g.kb, mono) ? &tab : nullptr;
      // a gradient with squared slices: the exponentials before and after their
      // squarings, as k_seg_grad_sq takes them
      const bool keep = (P.flags & RUN_GRAD) && gp(P.squared)[0] != 0;
      Panel<T, D> S, X, R;
      for (int k = g.ka; k < g.kb; ++k) {
        int s, q, qb;
        unpack_sq(gp(P.sq)[k], s, q, qb);
        assemble_panel<T, D>(X, la, P, k, ldexp(P.dt * (double)Ops::C, -s), mono, tb, k - g.ka, L);
        Ops::store_nct(la, X, L);  // X = -X^dag
        __syncthreads();
        taylor_delta<T, D, Ops>(R, X, la, s, q, L, keep ? pf_mat<T, D>(P.delta, k - W.rg.kbase) : nullptr);
        if (kKeepU<D> && keep) panel_store(pf_mat<T, D>(P.hk, k - W.rg.kbase), R, L);
        panel_scale(R, CI);
        if (k == g.ka) {
          S = R;
        } else {
          __syncthreads();  // the exponential's last left factor has been read
          Std::store(la, R, L);
          __syncthreads();
          // S + I <- (Delta + I)(S + I): nothing is rounded at the size of I
          Std::gemm3(X, la, S, L, true);
          panel_fma(S, (T)1, R);
          panel_fma(S, (T)1, X);
        }
      }
      panel_store(pf_mat<T, D>(P.xprev, g.ka - W.rg.kbase), S, L);
    }
    if constexpr (!PERSIST) break;  // one item per workgroup: a single-trip loop
    __syncthreads();
  }
}

// Per chunk: the prefixes P_s at its segment starts, as P_s - I (into bloc at
// the segment's first slice), and the chunk total.
template <typename T, int D, bool PERSIST>
__global__ __launch_bounds__(4 * D) void k_seg_join(Work W) {
  using Ops = StdOps<T, D>;
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int k1 = min(P.N, (c + 1) * P.L), h = seg_len(P.L, P.SM);
    Panel<T, D> S, nxt, acc;
    int k = c * P.L;
    panel_load(S, pf_mat<T, D>(P.xprev, k - W.rg.kbase), L);
    panel_add_identity(S, L, (T)1);
    k += h;
    if (k < k1) panel_load(nxt, pf_mat<T, D>(P.xprev, k - W.rg.kbase), L);
    for (int i = 0; k < k1; ++i) {
      acc = S;
      panel_add_identity(acc, L, (T)-1);
      panel_store(pf_mat<T, D>(P.bloc, k - W.rg.kbase), acc, L);
      Ops::store(lds[i & 1], nxt, L);
      k += h;
      if (k < k1) panel_load(nxt, pf_mat<T, D>(P.xprev, k - W.rg.kbase), L);
      __syncthreads();
      // S <- S + (T - I) S, in four real products: the three-product form's
      // larger error in these factors doubled the gradient's, and T S rounds
      // every sum at the size of S (at d = 128 a chunk's residual |Y^dag Y - I|
      // was 4.5e-6 after two of them instead of 1.7e-6)
      Ops::gemm(acc, lds[i & 1], S, L, true);
      panel_fma(S, (T)1, acc);
    }
    if (!W.rg.recompute) panel_store(pf_mat<T, D>(P.tf, c), S, L);  // (k_reun follows in FP32)
    if constexpr (!PERSIST) break;  // one item per workgroup: a single-trip loop
    __syncthreads();
  }
}

// Per chunk, after the carry: N = Q_{k0-1} P_{k0-1}^dag at its start,
// N = tf[c]^dag cb[c] cf[c]^dag with cf[c] = cf_loc[c] gcf[g] and
// cb[c] = cb_loc[c] gcb[g], and from it Y = (w N - (w N)^dag) / (2i), w = g / |g|,
// into mc; for the complex dg/du the parts of N itself, N = Y' + i Y:
// Y into mc and Y' = (N + N^dag) / 2 into cb.
template <typename T, int D>
__global__ __launch_bounds__(4 * D) void k_seg_y(Work W) {
  using Ops = StdOps<T, D>;
  __shared__ __align__(16) unsigned char lds[2][Ops::BYTES];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int g = c / P.CG;
    Panel<T, D> a, b, x, y;
    panel_load(a, pf_mat<T, D>(P.cf, c), L);
    panel_load(b, pf_mat<T, D>(P.cb, c), L);
    panel_load(x, grp_mat<T, D>(P, 2, g), L);
    panel_load(y, grp_mat<T, D>(P, 3, g), L);
    Ops::store(lds[0], a, L);
    Ops::store(lds[1], b, L);
    __syncthreads();
    Ops::gemm3(a, lds[0], x, L, true);  // cf[c]
    Ops::gemm3(b, lds[1], y, L, true);  // cb[c]
    panel_load(x, pf_mat<T, D>(P.tf, c), L);
    __syncthreads();
    Ops::store_ct(lds[0], x, L);
    Ops::store(lds[1], a, L);
    __syncthreads();
    Ops::gemm3(y, lds[0], b, L, true);  // tf^dag cb
    Ops::load_ct(x, lds[1], L);
    __syncthreads();
    Ops::store(lds[0], y, L);
    __syncthreads();
    Ops::gemm3(a, lds[0], x, L, true);  // N
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
    for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double ar = (double)a.re[rb][r], ai = (double)a.im[rb][r];
        a.re[rb][r] = (T)(wr * ar - wi * ai);
        a.im[rb][r] = (T)(wr * ai + wi * ar);
      }
    Ops::store_ct(lds[1], a, L);
    __syncthreads();
    Ops::load(b, lds[1], L);  // (w N)^dag
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb) {
      x.re[rb] = (T)0.5 * (a.im[rb] - b.im[rb]);
      x.im[rb] = (T)0.5 * (b.re[rb] - a.re[rb]);
      y.re[rb] = (T)0.5 * (a.re[rb] + b.re[rb]);
      y.im[rb] = (T)0.5 * (a.im[rb] + b.im[rb]);
    }
    panel_store(pf_mat<T, D>(P.mc, c), x, L);
    if (raw) panel_store(pf_mat<T, D>(P.cb, c), y, L);
    __syncthreads();
  }
}

// The gradient entries of slice k from the Hermitian Z (planar in LDS):
// t_j = Tr(Hc[j] Z) in FP64, a real sum.  part: 0, Z of Y; 1, Z of Y'
// (RUN_RAWDG).
__device__ __forceinline__ void seg_grad_put(const ProbDesc& P, int j, int k, int part, double t) {
  const double dt = P.dt * gp(P.vscale)[0];
  if (P.flags & RUN_RAWDG) {
    // dg/du[j][k] = -i dt Tr(Z(N)^dag Hc[j]) with N = Y' + i Y
    gp(P.grad)[2 * ((size_t)j * P.N + k) + part] = -dt * t;
  } else {
    const double gr = gp(P.g)[0], gi = gp(P.g)[1];
    gp(P.grad)[(size_t)j * P.N + k] = -2.0 * dt / ((double)P.d * P.d) * sqrt(gr * gr + gi * gi) * t;
  }
}

constexpr int kSegEpi = 8;  // dense controls reduced together

template <typename T, int D>
__device__ __forceinline__ void seg_epilogue(const ProbDesc& P, int k, int part, const T* zl, double zscale,
                                             const SegTab<T, D>* tab, double* red, bool mono, const Lane& L) {
  using v4 = typename Prec<T>::v4;
  constexpr int NV = D / 16;
  constexpr int NT = 4 * D;
  constexpr int NW = D / 16;
  constexpr int SD = Mat<T, D>::SD;
  if (mono) {
    // lane group jj = t / D takes row a = t % D of controls jj + 4 i
    constexpr int CPT = 4;
    constexpr int GV = D / CPT;  // lanes per reduced value
    const int a = threadIdx.x % D, jj = threadIdx.x / D;
    const T* mv = reinterpret_cast<const T*>(P.mval);
    for (int j0 = 0; j0 < P.m; j0 += 4 * CPT) {
      double v[CPT];
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const int j = j0 + jj + 4 * i;
        v[i] = 0;
        if (j < P.m) {
          const int e = j * D + a;
          const int col = tab ? (int)tab->col[e] : gp(P.mcol)[e];
          const double x = (double)(tab ? tab->vr[e] : gp(mv)[2 * e]), y = (double)(tab ? tab->vi[e] : gp(mv)[2 * e + 1]);
          const int off = lds_off<T, D>(a, col);
          v[i] = (double)zl[off] * x + (double)zl[D * SD + off] * y;  // Re(conj(z) h)
        }
      }
      const double t = group_sum_many<CPT, D>(v, L.lane);
      const int j = j0 + jj + 4 * (a / GV);
      if (a % GV == 0 && j < P.m) seg_grad_put(P, j, k, part, zscale * t);
    }
    return;
  }
  const int e0 = 4 * threadIdx.x;
  const T* H = reinterpret_cast<const T*>(P.Hint);
  for (int j0 = 0, grp = 0; j0 < P.m; j0 += kSegEpi, ++grp) {
    double v[kSegEpi];
#pragma unroll
    for (int jj = 0; jj < kSegEpi; ++jj) {
      v[jj] = 0;
      if (j0 + jj < P.m) {
        const T* Hj = H + (size_t)(j0 + jj + 1) * 2 * D * D + e0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const int e = e0 + 4 * NT * q;
          const v4 hr = Prec<T>::gld4(Hj + 4 * NT * q), hi = Prec<T>::gld4(Hj + D * D + 4 * NT * q);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int off = lds_off<T, D>(e / D, e % D + i);
            v[jj] += (double)zl[off] * (double)hr[i] + (double)zl[D * SD + off] * (double)hi[i];
          }
        }
      }
    }
    const double t = wave_sum_many<kSegEpi>(v, L.lane);
    double* rg = red + (grp & 1) * kSegEpi * NW;
    if ((L.lane & 7) == 0) rg[(L.lane >> 3) * NW + L.w] = t;
    __syncthreads();
    if ((int)threadIdx.x < kSegEpi && j0 + (int)threadIdx.x < P.m) {
      double a = 0;
      for (int w = 0; w < NW; ++w) a += rg[threadIdx.x * NW + w];
      seg_grad_put(P, j0 + threadIdx.x, k, part, zscale * a);
    }
  }
}

// Y <- U Y U^dag = Y + G + G^dag + G D^dag with G = D Y, D = U - I: lds0 holds
// D, lds1 is free; ends with a barrier.
template <typename T, int D, typename Ops>
__device__ __forceinline__ void conjugate_by(Panel<T, D>& Y, T f, void* lds0, void* lds1, const Lane& L) {
  constexpr T CI = (T)1 / Ops::C;
  Panel<T, D> G, acc;
  Ops::mul(G, lds0, Y, L);
  panel_scale(G, CI);
  Ops::store(lds1, G, L);
  __syncthreads();
  Ops::mul_ct(acc, lds1, lds0, L);
  panel_fma(G, CI, acc);  // G + G D^dag
  Ops::load_ct(acc, lds1, L);
  panel_fma(G, (T)1, acc);
  panel_fma(Y, f, G);
  __syncthreads();
}

// The gradient of the slices [ka, kb) of segment sg of chunk c.  SQ: slices
// with s > 0 among them; without, their doublings would take the registers of
// every slice (133 of them spilled at d = 64 in FP32).
template <typename T, int D, typename Ops, bool SQ>
__device__ __forceinline__ void seg_grad_body(const ProbDesc& P, int c, int sg, int ka, int kb, int kbase, int part,
                                              bool mono, void* la, void* lb, SegTab<T, D>& tab, const Lane& L) {
  constexpr T C = Ops::C, CI = (T)1 / Ops::C;
  T* pt = static_cast<T*>(lb);  // planar
  const SegTab<T, D>* tb = seg_tab_load<T, D>(tab, P, ka, kb, mono) ? &tab : nullptr;
  Panel<T, D> Y, Z, Q, R;
  panel_load(Y, pf_mat<T, D>(part ? P.cb : P.mc, c), L);
  panel_scale(Y, C);
  if (sg > 0) {  // Y at the segment's start
    panel_load(R, pf_mat<T, D>(P.bloc, ka - kbase), L);
    panel_scale(R, C);
    Ops::store(la, R, L);
    __syncthreads();
    conjugate_by<T, D, Ops>(Y, (T)1, la, lb, L);
  }
  for (int k = ka; k < kb; ++k) {
    const int sqk = gp(P.sq)[k];
    int s, q, qb;
    unpack_sq(sqk, s, q, qb);
    const int m = plan_order(sqk);
    assemble_panel<T, D>(R, lb, P, k, ldexp(P.dt * (double)C, -s), mono, tb, k - ka, L);
    Ops::store_nct(la, R, L);  // A = -A^dag (every wavefront has left the previous slice's products)
    __syncthreads();
    // Q = C_n / n!, of norm at most (2 |A|)^n / n! |Y|: in FP16's range for
    // every plan.  It joins Y and Z while the next product runs.
    Q = Y;
    panel_zero(Y);
    panel_zero(Z);
    T yk = 1, zk = 1;
    auto gather = [&](int rb) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        Z.re[rb][r] = fma(zk, Q.re[rb][r], Z.re[rb][r]);
        Z.im[rb][r] = fma(zk, Q.im[rb][r], Z.im[rb][r]);
        if (SQ) {
          Y.re[rb][r] = fma(yk, Q.re[rb][r], Y.re[rb][r]);
          Y.im[rb][r] = fma(yk, Q.im[rb][r], Y.im[rb][r]);
        } else {
          Y.re[rb][r] += Q.re[rb][r];
          Y.im[rb][r] += Q.im[rb][r];
        }
      }
    };
    for (int n = 1; n <= m; ++n) {
      Ops::mul(R, la, Q, L, gather);
      if (n > 1) __syncthreads();  // the previous transpose has been read
      panel_to_lds_ct(pt, R, L);
      __syncthreads();
      panel_from_lds(Q, pt, L);
      const T ck = CI * (T)(1.0 / n);
      zk = (T)(1.0 / (n + 1));
      if (SQ && s > 0) yk = 0;  // Y waits for the whole slice's propagator
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          Q.re[rb][r] = (Q.re[rb][r] + R.re[rb][r]) * ck;
          Q.im[rb][r] = (Q.im[rb][r] + R.im[rb][r]) * ck;
        }
    }
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb) gather(rb);
    if constexpr (SQ) {
      if (s > 0) {
        panel_load(R, pf_mat<T, D>(P.delta, k - kbase), L);  // C (exp(A / 2^s) - I)
        for (int j = 0;; ++j) {
          __syncthreads();
          Ops::store(la, R, L);
          __syncthreads();
          if (j == s) break;
          conjugate_by<T, D, Ops>(Z, (T)0.5, la, lb, L);
          Ops::mul(Q, la, R, L);
          panel_scale(R, (T)2);
          panel_fma(R, CI, Q);
        }
        conjugate_by<T, D, Ops>(Y, (T)1, la, lb, L);
      }
    }
    __syncthreads();
    panel_to_lds_ct(pt, Z, L);  // Z = Z^dag
    __syncthreads();
    // (A is no longer needed: its buffer takes the sums)
    static_assert(2 * kSegEpi * (D / 16) * 8 <= Ops::BYTES, "sums");
    seg_epilogue<T, D>(P, k, part, pt, (double)CI, tb, static_cast<double*>(la), mono, L);
  }
}

// The same for the slices [wa, wb) of a segment that starts at ka, with slices of
// s > 0 among them, where k_seg_fwd has kept every slice's U - I (kKeepU): Y passes the
// slices by their propagators, those before wa too.  One panel V is Y or Z in turn
// (Y is put by while a slice's series runs) and one loop takes every conjugation, so
// that there is one instance of each product: the registers do not hold more.
template <typename T, int D, typename Ops>
__device__ __forceinline__ void seg_grad_pieces(const ProbDesc& P, int c, int sg, int ka, int wa, int wb, int kbase,
                                                int part, bool mono, void* la, void* lb, SegTab<T, D>& tab,
                                                const Lane& L) {
  constexpr T C = Ops::C, CI = (T)1 / Ops::C;
  T* pt = static_cast<T*>(lb);  // planar
  const SegTab<T, D>* tb = seg_tab_load<T, D>(tab, P, wa, wb, mono) ? &tab : nullptr;
  Panel<T, D> V, Q, R;
  panel_load(V, pf_mat<T, D>(part ? P.cb : P.mc, c), L);
  panel_scale(V, C);
  bool conj = sg > 0;  // V <- V + f (U V U^dag - V), U - I in R
  if (conj) {          // to Y at the segment's start
    panel_load(R, pf_mat<T, D>(P.bloc, ka - kbase), L);
    panel_scale(R, C);
  }
  // Where Y of slice k waits (this wavefront's panel): xprev's segment totals have been
  // joined, and bloc holds prefixes at segment starts only, which no k + 1 < wb is.
  auto yslot = [&](int k) { return part ? pf_mat<T, D>(P.bloc, k + 1 - kbase) : pf_mat<T, D>(P.xprev, k - kbase); };
  T f = 1;
  int k = ka, s = 0, j = 0;
  bool inside = false;  // V is Z of slice k, j of its s doublings done
#pragma unroll 1
  for (;;) {
    if (conj) {
      __syncthreads();  // la's last readers are done
      Ops::store(la, R, L);
      __syncthreads();
      conjugate_by<T, D, Ops>(V, f, la, lb, L);
    }
    if (inside) {
      if (conj && ++j < s) {
        Ops::mul(Q, la, R, L);
        panel_scale(R, (T)2);
        panel_fma(R, CI, Q);
        continue;
      }
      __syncthreads();
      panel_to_lds_ct(pt, V, L);  // Z = Z^dag
      __syncthreads();
      static_assert(2 * kSegEpi * (D / 16) * 8 <= Ops::BYTES, "sums");
      seg_epilogue<T, D>(P, k, part, pt, (double)CI, tb, static_cast<double*>(la), mono, L);
      if (k + 1 >= wb) break;
      panel_load(V, yslot(k), L);
      inside = false;
    } else if (k >= wa) {
      const int sqk = gp(P.sq)[k];
      int q, qb;
      unpack_sq(sqk, s, q, qb);
      const int m = plan_order(sqk);
      if (k + 1 < wb) panel_store(yslot(k), V, L);
      assemble_panel<T, D>(R, lb, P, k, ldexp(P.dt * (double)C, -s), mono, tb, k - wa, L);
      Ops::store_nct(la, R, L);  // A = -A^dag
      __syncthreads();
      Q = V;
      panel_zero(V);
      T zk = 1;
      auto gather = [&](int rb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          V.re[rb][r] = fma(zk, Q.re[rb][r], V.re[rb][r]);
          V.im[rb][r] = fma(zk, Q.im[rb][r], V.im[rb][r]);
        }
      };
      for (int n = 1; n <= m; ++n) {
        Ops::mul(R, la, Q, L, gather);
        if (n > 1) __syncthreads();  // the previous transpose has been read
        panel_to_lds_ct(pt, R, L);
        __syncthreads();
        panel_from_lds(Q, pt, L);
        const T ck = CI * (T)(1.0 / n);
        zk = (T)(1.0 / (n + 1));
#pragma unroll
        for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Q.re[rb][r] = (Q.re[rb][r] + R.re[rb][r]) * ck;
            Q.im[rb][r] = (Q.im[rb][r] + R.im[rb][r]) * ck;
          }
      }
#pragma unroll
      for (int rb = 0; rb < D / 16; ++rb) gather(rb);
      inside = true;
      conj = s > 0;
      f = (T)0.5;
      j = 0;
      if (conj) panel_load(R, pf_mat<T, D>(P.delta, k - kbase), L);  // C (exp(A / 2^s) - I)
      continue;
    }
    // Y to the next slice
    panel_load(R, pf_mat<T, D>(P.hk, k - kbase), L);
    conj = true;
    f = 1;
    ++k;
  }
}

// One workgroup per segment, and the problems without any s > 0 (*P.squared).
template <typename T, int D, typename Ops, bool PERSIST>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kSegWaves<T, D>))) void k_seg_grad(Work W) {
  constexpr int LB = StdOps<T, D>::BYTES > Ops::BYTES ? StdOps<T, D>::BYTES : Ops::BYTES;
  __shared__ __align__(16) unsigned char la[Ops::BYTES];
  __shared__ __align__(16) unsigned char lb[LB];
  __shared__ SegTab<T, D> tab;
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    const SegItem g = seg_split(item, W.rg, I, W.descs);
    if (g.ka < g.kb) {
      const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
      const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
      if (gp(P.squared)[0] == 0)
        seg_grad_body<T, D, Ops, false>(P, g.c, g.s, g.ka, g.kb, W.rg.kbase, blockIdx.y, mono, la, lb, tab, L);
    }
    if constexpr (!PERSIST) break;  // one item per workgroup: a single-trip loop
    __syncthreads();
  }
}

// Pieces that a segment of h slices is cut into: one per slice (whose workgroup takes Y
// through the slices before it: the same steps on the same numbers, two products per
// slice passed, against about 25 of a slice) if that takes less time in rounds of the
// grid.  Where several workgroups share a CU the last round's go the faster for being
// few, and cutting pays only if there is hardly more than one.  One problem of
// N = 1000 in FP64 (264 segments of four slices): d = 32 (grid 1024) 283 -> 179 us,
// d = 64 (grid 256) 1.55 -> 1.15 ms; eight problems of d = 32 883 -> 994 us.
__host__ __device__ inline int sq_pieces(int total, int h, int grid, bool shared) {
  if (shared && total >= grid + grid / 8) return 1;
  const int whole = (total + grid - 1) / grid * h * 25, cut = (total * h + grid - 1) / grid * (24 + h);
  return cut < whole - whole / 10 ? h : 1;
}

// The segments of the problems with squared slices, in turn over a grid that fills
// the chip (kSqGrid) and leaves at once when there is none.  The items are those of
// k_seg_grad (or their pieces), so that one squared problem of a batch spreads over
// all workgroups; a workgroup passes over the others' at one load each.  (Engine ticks
// cut in two: the engine's chunks have segments of two slices up to N = 2048.)
// With 256 workgroups at every d, dealt out by problem, 32 problems of d = 16, N = 1000
// with s = 2 took 1.38 ms in FP32 (now 0.34; the block form 0.37) and one such
// problem in a batch of 32 at d = 64 7.6 ms (now 2.8; the block form 6.0).
template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kSegWaves<T, D>))) void k_seg_grad_sq(Work W) {
  constexpr int LB = StdOps<T, D>::BYTES > Ops::BYTES ? StdOps<T, D>::BYTES : Ops::BYTES;
  __shared__ __align__(16) unsigned char la[Ops::BYTES];
  __shared__ __align__(16) unsigned char lb[LB];
  __shared__ SegTab<T, D> tab;
  Lane L;
  const Items I(W);
  if (I.nprob == 0 || gp(W.descs[I.desc(0)].squared)[1] == 0) return;
  const int cut = kKeepU<D> ? sq_pieces(I.total, W.dyn ? 2 : seg_len(W.descs[0].L, W.descs[0].SM), kSqGrid<T, D>, kSegWaves<T, D> > 1) : 1;
  for (int item = blockIdx.x; item < I.total * cut; item += gridDim.x) {
    const SegItem g = seg_split(item / cut, W.rg, I, W.descs);
    if (g.ka >= g.kb || gp(W.descs[I.desc(g.p)].squared)[0] == 0) continue;
    const ProbDesc P = W.descs[I.desc(g.p)];  // a copy: stores cannot alias it
    const int h = seg_len(P.L, P.SM), x = item % cut;
    const int wa = g.ka + h * x / cut, wb = min(g.kb, g.ka + h * (x + 1) / cut);
    if (wa >= wb) continue;
    const bool mono = (gp(P.sq)[g.ka] & kPlanMono) != 0;
    if constexpr (kKeepU<D>)
      seg_grad_pieces<T, D, Ops>(P, g.c, g.s, g.ka, wa, wb, W.rg.kbase, blockIdx.y, mono, la, lb, tab, L);
    else
      seg_grad_body<T, D, Ops, true>(P, g.c, g.s, g.ka, g.kb, W.rg.kbase, blockIdx.y, mono, la, lb, tab, L);
    __syncthreads();
  }
}

// ================================================================ d = 128
//
// A 128 x 128 complex matrix pair does not fit in LDS (one FP32 matrix is
// 132 KB with padding, one FP64 matrix 260 KB).  At D = 128 the state of every
// chain therefore lives in global scratch in PF layout (8 wavefronts, one
// 16-column panel each), each product accumulates one output panel per
// wavefront in registers, and the left factor is staged cooperatively into
// LDS, the whole matrix in FP32 and one 64-column half at a time in FP64.
// The grids are persistent (at most kScratchSlots workgroups), so that each
// workgroup owns a fixed scratch region.

template <typename T>
struct K128 {
  static constexpr int D = 128, NW = 8, RB = 8;
  static constexpr int HALVES = sizeof(T) == 8 ? 2 : 1;
  static constexpr int HC = D / HALVES;             // columns staged at once
  static constexpr int SD = HC + Prec<T>::PAD;      // LDS row stride
  static constexpr int LDS_ELEMS = 2 * D * SD;
  static constexpr int ELEMS = 2 * D * D;
  static constexpr int KBH = HC / 16;               // k blocks per staged part
  static constexpr int WPH = NW / HALVES;           // panels per staged part
};

// The three-product form in the FP32 expm and adjoint products at D = 128
// (their registers allow it; the FP64 kernels already spill).
template <typename T>
constexpr bool k128Gauss = sizeof(T) == 4;

// acc <- acc + a * (this wavefront's panel of the PF matrix M), one row block
// at a time so that no second panel is held in registers.
template <typename T>
__device__ __forceinline__ void panel_axpy_pf(Panel<T, 128>& acc, T a, const T* M, const Lane& L) {
#pragma unroll
  for (int rb = 0; rb < 8; ++rb) {
    typename Prec<T>::v4 re, im;
    pf_rb_load<T>(re, im, M, L.w, rb, L.lane);
    acc.re[rb] += a * re;
    acc.im[rb] += a * im;
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Stage part h (columns [h HC, (h+1) HC)) of M (CT = false) or of M^dag
// (CT = true) into LDS; M is a PF matrix.  Layout as for the D <= 64 LDS
// matrices, restricted to HC columns.
template <typename T, bool CT>
__device__ __forceinline__ void stage128(T* lds, const T* M, int h, const Lane& L) {
  using K = K128<T>;
  using v4 = typename Prec<T>::v4;
  T* lim = lds + K::D * K::SD;
  // Row blocks are loaded NB at a time, all NB loads in flight before the
  // LDS writes, so that the staging waits for RB / NB global round trips.
  constexpr int NB = sizeof(T) == 4 ? 4 : 2;
  if constexpr (!CT) {
    if (L.w / K::WPH != h) return;
    const int lw = L.w - h * K::WPH;
#pragma unroll
    for (int b0 = 0; b0 < K::RB; b0 += NB) {
      v4 re[NB], im[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) pf_rb_load<T>(re[i], im[i], M, L.w, b0 + i, L.lane);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int off = (16 * (b0 + i) + Prec<T>::rowmap(r, L.g)) * K::SD + 16 * lw + Prec<T>::perm(L.c16);
          lds[off] = re[i][r];
          lim[off] = im[i][r];
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    // M^dag[16w + c16][16 rb + rowmap(r, g)] = conj(M[16 rb + rowmap(r, g)][16w + c16])
    constexpr int RL = K::RB / K::HALVES;
#pragma unroll
    for (int b0 = 0; b0 < RL; b0 += NB) {
      v4 re[NB], im[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) pf_rb_load<T>(re[i], im[i], M, L.w, h * RL + b0 + i, L.lane);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        int off = (16 * L.w + L.c16) * K::SD + 16 * (b0 + i) + 4 * L.g;
        Prec<T>::st4(lds + off, re[i]);
        Prec<T>::st4(lim + off, -im[i]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// acc (+)= M B, M (or M^dag when CT) staged through LDS part by part, B this
// wavefront's panel of a PF matrix.  Every part is staged between two
// workgroup barriers, so M may have been written by any wavefront.  With
// stage = false and the whole matrix in one part (FP32), M is taken to be in
// LDS already from the previous product, which had the same left factor and
// no LDS writes since: one barrier (which also completes this wavefront's
// stores of B) and no staging.  G3 selects the three-product form of the
// complex product (as cgemm3m: T1 in acc.re, T3 in acc.im starting at
// acc.im + acc.re, T2 apart).
template <typename T, bool CT, bool G3 = false>
__device__ __forceinline__ void gemm128(Panel<T, 128>& acc, T* lds, const T* M, const T* B, const Lane& L,
                                        bool zero_acc, bool stage = true) {
  using K = K128<T>;
  using v4 = typename Prec<T>::v4;
  const T* lim = lds + K::D * K::SD;
  if (zero_acc) panel_zero(acc);
  v4 t2[G3 ? K::RB : 1];
  if constexpr (G3) {
#pragma unroll
    for (int rb = 0; rb < K::RB; ++rb) {
      t2[rb] = (v4){0, 0, 0, 0};
      if (!zero_acc) acc.im[rb] += acc.re[rb];
    }
  }
  const int base = L.c16 * K::SD + 4 * L.g;
#pragma unroll
  for (int h = 0; h < K::HALVES; ++h) {
    __syncthreads();
    if (stage || K::HALVES > 1) {
      stage128<T, CT>(lds, M, h, L);
      __syncthreads();
    }
    constexpr int STEPS = K::KBH * K::RB;
    v4 ar[2], ai[2], br[2], bi[2];
    ar[0] = Prec<T>::ld4(lds + base);
    ai[0] = Prec<T>::ld4(lim + base);
    pf_rb_load<T>(br[0], bi[0], B, L.w, h * K::KBH, L.lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      const int kbl = st / K::RB, mb = st % K::RB;
      const int cur = st & 1, kcur = kbl & 1;
      if (st + 1 < STEPS) {
        const int kn = (st + 1) / K::RB, mn = (st + 1) % K::RB;
        const int off = base + 16 * mn * K::SD + 16 * kn;
        ar[cur ^ 1] = Prec<T>::ld4(lds + off);
        ai[cur ^ 1] = Prec<T>::ld4(lim + off);
        if (mb == 0 && kbl + 1 < K::KBH) pf_rb_load<T>(br[kcur ^ 1], bi[kcur ^ 1], B, L.w, h * K::KBH + kbl + 1, L.lane);
      }
      if constexpr (G3) {
        const v4 as = ar[cur] + ai[cur];
        const v4 bs = br[kcur] + bi[kcur];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc.re[mb] = Prec<T>::mfma(ar[cur][r], br[kcur][r], acc.re[mb]);
          t2[mb] = Prec<T>::mfma(ai[cur][r], bi[kcur][r], t2[mb]);
          acc.im[mb] = Prec<T>::mfma(as[r], bs[r], acc.im[mb]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const T b_r = br[kcur][r];
          const T b_i = bi[kcur][r];
          acc.re[mb] = Prec<T>::mfma(ar[cur][r], b_r, acc.re[mb]);
          acc.im[mb] = Prec<T>::mfma(ar[cur][r], b_i, acc.im[mb]);
          acc.re[mb] = Prec<T>::mfma(-ai[cur][r], b_i, acc.re[mb]);
          acc.im[mb] = Prec<T>::mfma(ai[cur][r], b_r, acc.im[mb]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (G3) {
#pragma unroll
    for (int rb = 0; rb < K::RB; ++rb) {
      acc.im[rb] = acc.im[rb] - acc.re[rb] - t2[rb];
      acc.re[rb] = acc.re[rb] - t2[rb];
    }
  }
}

// out = M^dag (both PF), through LDS part by part.
template <typename T>
__device__ __forceinline__ void transpose128(T* out, T* lds, const T* M, const Lane& L) {
  using K = K128<T>;
  const T* lim = lds + K::D * K::SD;
  for (int h = 0; h < K::HALVES; ++h) {
    __syncthreads();
    stage128<T, true>(lds, M, h, L);
    __syncthreads();
    if (L.w / K::WPH == h) {
      const int lw = L.w - h * K::WPH;
      Panel<T, 128> P;
#pragma unroll
      for (int rb = 0; rb < K::RB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int off = (16 * rb + Prec<T>::rowmap(r, L.g)) * K::SD + 16 * lw + Prec<T>::perm(L.c16);
          P.re[rb][r] = lds[off];
          P.im[rb][r] = lim[off];
        }
      panel_store(out, P, L);
    }
  }
}

// X <- sgn * (-i) * c * H_k (this wavefront's panel, in registers) with
// H_k = H0 + sum_j u_jk Hc[j].  The matrix is read as chunks of four
// consecutive row elements, chunk t + 512 i by thread t, so that every
// 16-byte load is consecutive across lanes and a control's loads are all in
// flight together; the chunks then go through LDS (row-major, the layout of
// the staged left factors) to the panels, which are also stored to the PF
// matrix out.  FP32 takes all rows at once, FP64 one half of the rows per
// pass (one FP64 matrix does not fit in LDS); FP64 writes each half's rows of
// the panel to out and reads the panel back at the end, so that no panel is
// held across the passes.  Starts and ends with a workgroup barrier.
// With mono (every control has at most one nonzero per row) the chunks of H0
// go to LDS unscaled, one thread per row then adds the row's entry of each
// control in turn (the same sums, minus the structural zeros), and a last
// pass over the chunks applies the scale.
template <typename T>
__device__ __forceinline__ void assemble128(Panel<T, 128>& X, T* out, T* lds, const ProbDesc& P, int k, double c,
                                            double sgn, const Lane& L, bool mono) {
  using v4 = typename Prec<T>::v4;
  constexpr int D = 128, NT = 512;
  constexpr int PASSES = sizeof(T) == 4 ? 1 : 2;
  constexpr int NV = D * D / 4 / NT / PASSES;
  constexpr int ROWS = D / PASSES;
  constexpr int SD = D + Prec<T>::PAD;
  static_assert(2 * ROWS * SD <= K128<T>::LDS_ELEMS, "LDS too small");
  T* lim = lds + ROWS * SD;
  const T* H = reinterpret_cast<const T*>(P.Hint);
  // the factor in two numbers of type T (as in assemble_panel)
  const T f = (T)(sgn * c), fl = (T)(sgn * c - (double)f);
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int e0 = 4 * (threadIdx.x + pass * NV * NT);
    v4 hr[NV], hi[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      hr[v] = Prec<T>::gld4(H + e0 + 4 * NT * v);
      hi[v] = Prec<T>::gld4(H + D * D + e0 + 4 * NT * v);
    }
    if (!mono)
    for (int j = 0; j < P.m; ++j) {
      const T uj = (T)gp(P.u)[(size_t)j * P.N + k];
      const T* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
      v4 ar[NV], ai[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        ar[v] = Prec<T>::gld4(Hj + 4 * NT * v);
        ai[v] = Prec<T>::gld4(Hj + D * D + 4 * NT * v);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        hr[v] += uj * ar[v];
        hi[v] += uj * ai[v];
      }
    }
    __syncthreads();  // LDS free
    if (mono) {
      // H0 unscaled, then each row's control entries, then the scale
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = e0 + 4 * NT * v;
        const int row = e / D - pass * ROWS, col = e % D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int off = row * SD + ((col + i) & ~15) + Prec<T>::perm((col + i) & 15);
          lds[off] = hr[v][i];
          lim[off] = hi[v][i];
        }
      }
      __syncthreads();
      if ((int)threadIdx.x < ROWS) {
        const int a = pass * ROWS + threadIdx.x;
        const T* mv = reinterpret_cast<const T*>(P.mval);
        for (int j = 0; j < P.m; ++j) {
          const T uj = (T)gp(P.u)[(size_t)j * P.N + k];
          const size_t idx = (size_t)j * D + a;
          const int col = gp(P.mcol)[idx];
          const int off = (int)threadIdx.x * SD + (col & ~15) + Prec<T>::perm(col & 15);
          lds[off] += uj * gp(mv)[2 * idx];
          lim[off] += uj * gp(mv)[2 * idx + 1];
        }
      }
      __syncthreads();
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = e0 + 4 * NT * v;
        const int row = e / D - pass * ROWS, col = e % D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int off = row * SD + ((col + i) & ~15) + Prec<T>::perm((col + i) & 15);
          const T r = lds[off], im = lim[off];
          lds[off] = fma(f, im, fl * im);  // -i f (r + i im)
          lim[off] = -fma(f, r, fl * r);
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int e = e0 + 4 * NT * v;
        const int row = e / D - pass * ROWS, col = e % D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int off = row * SD + ((col + i) & ~15) + Prec<T>::perm((col + i) & 15);
          lds[off] = fma(f, hi[v][i], fl * hi[v][i]);  // -i f (hr + i hi)
          lim[off] = -fma(f, hr[v][i], fl * hr[v][i]);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8 / PASSES; ++i) {
      const int rb = pass * (8 / PASSES) + i;
      v4 re, im;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int off = (16 * i + Prec<T>::rowmap(r, L.g)) * SD + 16 * L.w + Prec<T>::perm(L.c16);
        re[r] = lds[off];
        im[r] = lim[off];
      }
      if constexpr (PASSES == 1) {
        X.re[rb] = re;
        X.im[rb] = im;
      } else {
        pf_rb_store<T>(out, re, im, L.w, rb, L.lane);
      }
    }
  }
  if constexpr (PASSES == 1) panel_store(out, X, L);
  else panel_load(X, out, L);  // own panel
  __syncthreads();
}

// The gradient epilogue at D = 128 (512 threads), as gradient_epilogue: Z goes
// through LDS so that thread t owns the chunks of four consecutive row
// elements t + 512 i and reads each control's chunks with 16-byte loads,
// consecutive across lanes.  The chunks are taken in two passes over the row
// halves (registers); FP32 stages all of Z once, FP64 stages the half of each
// pass (one FP64 matrix does not fit in LDS).  Z is read from the PF matrix
// Zpf, in which every wavefront has stored its own panel (so the staging
// needs no barrier before its reads and holds no panel in registers).
// With mono (every control has at most one nonzero per row) thread t takes
// row t % 128 of control j0 + t / 128 of each group of four controls and
// reads its one entry of Z from Zpf directly, after a barrier.  FP32 only:
// the branch doubles the FP64 adjoint's register spills, which costs more
// than the dense inner products.
template <typename T>
__device__ __forceinline__ void gradient_epilogue128(const ProbDesc& P, int k, const T* Zpf, const Lane& L,
                                                     T* lds, double* red, bool mono) {
  using v4 = typename Prec<T>::v4;
  constexpr int D = 128, NT = 512, NV = 4;
  static_assert(NT == kEpiGroup * D, "one (control, row) pair per thread");
  if (sizeof(T) == 4 && mono) {
    __syncthreads();  // every wavefront's panel of Z is in Zpf
    const int a = threadIdx.x % D, jj = threadIdx.x / D;
    const T* mv = reinterpret_cast<const T*>(P.mval);
    // PF position of row a: row block, and register / lane group within it
    const int rb = a >> 4, rr = a & 15;
    const int g = sizeof(T) == 4 ? rr >> 2 : rr & 3;
    const int r = sizeof(T) == 4 ? rr & 3 : rr >> 2;
    for (int j0 = 0, grp = 0; j0 < P.m; j0 += kEpiGroup, ++grp) {
      double v[2 * kEpiGroup];
      double tr = 0, ti = 0;
      if (j0 + jj < P.m) {
        const size_t idx = (size_t)(j0 + jj) * D + a;
        const int col = gp(P.mcol)[idx];
        const int lane = 16 * g + (col & 15);
        const double zr = (double)gp(Zpf)[pf_index<T, D>(col >> 4, 0, 4 * rb + r, lane)];
        const double zi = (double)gp(Zpf)[pf_index<T, D>(col >> 4, 1, 4 * rb + r, lane)];
        const double x = (double)gp(mv)[2 * idx], y = (double)gp(mv)[2 * idx + 1];
        tr = zr * x + zi * y;  // conj(z) h
        ti = zr * y - zi * x;
      }
#pragma unroll
      for (int q = 0; q < kEpiGroup; ++q) {
        v[2 * q] = q == jj ? tr : 0.0;
        v[2 * q + 1] = q == jj ? ti : 0.0;
      }
      epilogue_publish<8>(P, k, j0, grp, v, L, red);
    }
    return;
  }
  constexpr bool RESTAGE = sizeof(T) == 8;
  constexpr int ROWS = RESTAGE ? 64 : 128;  // rows staged at once
  constexpr int SD = D + Prec<T>::PAD;
  static_assert(2 * ROWS * SD <= K128<T>::LDS_ELEMS, "LDS too small");
  constexpr int LG = sizeof(T) == 4 ? 2 : 1;  // controls loaded together
  T* lim = lds + ROWS * SD;
  // Stage row blocks [rb0, rb0 + ROWS / 16) of Z, at local rows from 0.
  auto stage = [&](int rb0) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i) {
      v4 re, im;
      pf_rb_load<T>(re, im, Zpf, L.w, rb0 + i, L.lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int off = (16 * i + Prec<T>::rowmap(r, L.g)) * SD + 16 * L.w + Prec<T>::perm(L.c16);
        lds[off] = re[r];
        lim[off] = im[r];
      }
    }
    __syncthreads();
  };
  if (!RESTAGE) stage(0);
  const T* H = reinterpret_cast<const T*>(P.Hint);
  for (int j0 = 0, grp = 0; j0 < P.m; j0 += kEpiGroup, ++grp) {
    double v[2 * kEpiGroup];
#pragma unroll
    for (int i = 0; i < 2 * kEpiGroup; ++i) v[i] = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (RESTAGE) stage(4 * h);
      const int e0 = 4 * (threadIdx.x + h * NV * NT);
      const int row0 = RESTAGE ? 64 * h : 0;
      double zr[4 * NV], zi[4 * NV];
#pragma unroll
      for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = e0 + 4 * NT * q;
          const int col = e % D + i;
          const int off = (e / D - row0) * SD + (col & ~15) + Prec<T>::perm(col & 15);
          zr[4 * q + i] = (double)lds[off];
          zi[4 * q + i] = (double)lim[off];
        }
#pragma unroll
      for (int jb = 0; jb < kEpiGroup; jb += LG) {
        v4 hr[LG][NV], hi[LG][NV];
#pragma unroll
        for (int jj = 0; jj < LG; ++jj) {
          const int j = min(j0 + jb + jj, P.m - 1);
          const T* Hj = H + (size_t)(j + 1) * 2 * D * D + e0;
#pragma unroll
          for (int q = 0; q < NV; ++q) {
            hr[jj][q] = Prec<T>::gld4(Hj + 4 * NT * q);
            hi[jj][q] = Prec<T>::gld4(Hj + D * D + 4 * NT * q);
          }
        }
#pragma unroll
        for (int jj = 0; jj < LG; ++jj) {
          double tr = 0, ti = 0;
#pragma unroll
          for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double a = zr[4 * q + i], b = zi[4 * q + i];
              const double x = (double)hr[jj][q][i], y = (double)hi[jj][q][i];
              tr += a * x + b * y;  // conj(z) h
              ti += a * y - b * x;
            }
          v[2 * (jb + jj)] += tr;
          v[2 * (jb + jj) + 1] += ti;
        }
      }
    }
    epilogue_publish<8>(P, k, j0, grp, v, L, red);
  }
}

template <typename T>
__device__ __forceinline__ T* slot_mat(void* scratch, int i) {
  return reinterpret_cast<T*>(scratch) + ((size_t)blockIdx.x * kScratchMats + i) * K128<T>::ELEMS;
}

template <typename T>
__global__ __launch_bounds__(512) void k_expm128(Work W, void* scratch) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  Lane L;
  T* SX = slot_mat<T>(scratch, 0);
  T* SR = slot_mat<T>(scratch, 1);
  T* S2 = slot_mat<T>(scratch, 2);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, k;
    split_item(item, W.rg.s_lo, W.rg.s_n, I.start, I.nprob, p, k);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    int s, q, qb;
    const int sqk = gp(P.sq)[k];
    unpack_sq(sqk, s, q, qb);
    Panel<T, 128> acc;
    assemble128<T>(acc, SX, lds, P, k, ldexp(P.dt, -s), 1.0, L, (sqk & kPlanMono) != 0);  // SX: the left factor
    // For the adjoint: X = A_k / 2^s in PF layout (its X, A_k^dag / 2^s, is
    // the exact negation), one coalesced store of this wavefront's panel.
    if (P.flags & RUN_GRAD) panel_store(pf_mat<T, 128>(P.hk, k - W.rg.kbase), acc, L);
    // Paterson-Stockmeyer with X2 = X X as the step, X2 in slot 2, C in SR:
    //   p(X) - I = X + X2 C,  C = sum_{n=2..q} X^(n-2) / n!,  C <- D_t + X2 C,
    //   D_t = I / (2t+2)! + X / (2t+3)!
    // (as k_adjoint's block polynomial): expm_products(q) products, then s
    // squarings, all by one instance of the product.  (Inlined at each of its
    // uses it left FP64 276 spilled registers, which cost more than the products
    // that Horner's rule takes beyond these.)
    const int n = expm_products(q), top = (q - 2) / 2;
    const bool even = (q & 1) == 0;
    if (n == 0 && s > 0) panel_store(SR, acc, L);
#pragma unroll 1
    for (int i = 0; i < n + s; ++i) {
      const bool square = i >= n, inner = i > 0 && i < n;
      const int t = (even ? top - 1 : top) - i;  // inner: D_t, X at the last
      if (inner) {
        panel_load(acc, SX, L);
        if (i < n - 1) {
          panel_scale(acc, (T)inv_factorial(2 * t + 3));
          panel_add_identity(acc, L, (T)inv_factorial(2 * t + 2));
        }
      }
      gemm128<T, false, k128Gauss<T>>(acc, lds, square ? SR : (inner ? S2 : SX), square || inner ? SR : SX, L, !inner,
                                      i < 2 || !inner);
      if (square) {
        panel_axpy_pf(acc, (T)2, SR, L);
      } else if (i == 0 && q == 2) {
        panel_scale(acc, (T)0.5);
        panel_axpy_pf(acc, (T)1, SX, L);  // X + X2 / 2
      } else if (i == 0) {
        // C = I / (q-2)! + X / (q-1)! + X2 / q! or I / (q-1)! + X / q!
        panel_store(S2, acc, L);
        panel_scale(acc, even ? (T)inv_factorial(q) : (T)0);
        panel_axpy_pf(acc, (T)inv_factorial(even ? q - 1 : q), SX, L);
        panel_add_identity(acc, L, (T)inv_factorial(even ? q - 2 : q - 1));
      }
      if (i + 1 < n + s) panel_store(SR, acc, L);
    }
    panel_store(pf_mat<T, 128>(P.delta, k - W.rg.kbase), acc, L);
  }
}

// The re-unitarisation check of a forward chunk total at D = 128 (FP32): as
// reunitarise(), with G = Y^dag Y formed in FP64 on the vector ALU from Y
// staged in LDS (one FP64 matrix does not fit there): thread t owns the 4 x 8
// tile of G at rows 4 (t / 16), columns 8 (t % 16).  When r > tol, the factor
// (3I - G) / 2 is written in FP32 to Tpf (a PF matrix free during the forward
// scans) and Y <- Y (3I - G) / 2 replaces the chunk total at Ypf.
__device__ __noinline__ void reunitarise128(const ProbDesc& P, float* Ypf, float* Tpf, float* lds, double* red,
                                               const Lane& L) {
  using K = K128<float>;
  constexpr int D = 128, SD = K::SD;
  static_assert(2 * D * SD <= K::LDS_ELEMS, "LDS too small");
  float* yr = lds;
  float* yi = lds + D * SD;
  __syncthreads();  // every wavefront's panel of Y is stored; the LDS is free
#pragma unroll
  for (int rb = 0; rb < 8; ++rb) {
    typename Prec<float>::v4 re, im;
    pf_rb_load<float>(re, im, Ypf, L.w, rb, L.lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int off = (16 * rb + Prec<float>::rowmap(r, L.g)) * SD + 16 * L.w + L.c16;
      yr[off] = re[r];
      yi[off] = im[r];
    }
  }
  __syncthreads();
  const int i0 = 4 * (threadIdx.x / 16), j0 = 8 * (threadIdx.x % 16);
  double gr[4][8], gi[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) gr[a][b] = gi[a][b] = 0.0;
  for (int k = 0; k < D; ++k) {
    double ar[4], ai[4], br[8], bi[8];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      ar[a] = (double)yr[k * SD + i0 + a];
      ai[a] = (double)yi[k * SD + i0 + a];
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      br[b] = (double)yr[k * SD + j0 + b];
      bi[b] = (double)yi[k * SD + j0 + b];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 8; ++b) {  // conj(Y[k][i]) Y[k][j]
        gr[a][b] += ar[a] * br[b] + ai[a] * bi[b];
        gi[a][b] += ar[a] * bi[b] - ai[a] * br[b];
      }
  }
  const int d = P.d;
  double e2 = 0;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b)
      if (i0 + a < d && j0 + b < d) {
        const double xr = gr[a][b] - (i0 + a == j0 + b ? 1.0 : 0.0), xi = gi[a][b];
        e2 += xr * xr + xi * xi;
      }
  e2 = wave_sum(e2);
  if (L.lane == 0) red[L.w] = e2;
  __syncthreads();
  double tot = 0;
  for (int w = 0; w < 8; ++w) tot += red[w];
  const double res = sqrt(tot);
  if (threadIdx.x == 0)
    atomicMax(reinterpret_cast<unsigned long long*>(&P.diag[1]), (unsigned long long)__double_as_longlong(res));
  if (res > P.reun_tol) {
    // T = (3I - G) / 2 in PF layout: row i is register 4 (i / 16) + r of lane
    // group g (rowmap), column j is lane 16 g + j % 16 of panel j / 16
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int i = i0 + a, rr = i & 15;
      const int g = rr >> 2, r = rr & 3;  // FP32 rowmap(r, g) = 4 g + r
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int j = j0 + b;
        const int lane = 16 * g + (j & 15);
        gp(Tpf)[pf_index<float, D>(j >> 4, 0, 4 * (i >> 4) + r, lane)] =
            (float)(0.5 * ((i == j ? 3.0 : 0.0) - gr[a][b]));
        gp(Tpf)[pf_index<float, D>(j >> 4, 1, 4 * (i >> 4) + r, lane)] = (float)(-0.5 * gi[a][b]);
      }
    }
    __syncthreads();  // the factor is complete
    Panel<float, D> acc;
    gemm128<float, false>(acc, lds, Ypf, Tpf, L, true);  // Y (3I - G) / 2
    panel_store(Ypf, acc, L);
    if (threadIdx.x == 0) atomicAdd(reinterpret_cast<unsigned long long*>(&P.diag[2]), 1ull);
  }
  __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(512) void k_scan128(Work W, int dir) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  __shared__ double red[8];
  const int bwd = dir < 0 ? (int)blockIdx.y : dir;  // dir < 0: both passes, one per blockIdx.y
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int k0 = c * P.L;
    const int k1 = min(P.N, k0 + P.L);
    Panel<T, 128> acc;
    if (bwd) panel_load(acc, pf_mat<T, 128>(P.mc, c), L); else panel_identity(acc, L);
    if (!bwd) {
      panel_store(pf_mat<T, 128>(P.xprev, k0 - W.rg.kbase), acc, L);
      for (int k = k0; k < k1; ++k) {
        T* cur = pf_mat<T, 128>(P.xprev, k - W.rg.kbase);
        gemm128<T, false>(acc, lds, pf_mat<T, 128>(P.delta, k - W.rg.kbase), cur, L, true);
        panel_axpy_pf(acc, (T)1, cur, L);
        panel_store(k + 1 < k1 ? pf_mat<T, 128>(P.xprev, k + 1 - W.rg.kbase) : pf_mat<T, 128>(P.tf, c), acc, L);
      }
      if constexpr (sizeof(T) == 4) {
        if (P.reun_tol >= 0 && !W.rg.recompute)
          reunitarise128(P, pf_mat<T, 128>(P.tf, c), pf_mat<T, 128>(P.cf, c), reinterpret_cast<float*>(lds), red, L);
      }
    } else {
      panel_store(pf_mat<T, 128>(P.bloc, k1 - 1 - W.rg.kbase), acc, L);
      for (int k = k1 - 1; k >= k0; --k) {
        T* cur = pf_mat<T, 128>(P.bloc, k - W.rg.kbase);
        gemm128<T, true>(acc, lds, pf_mat<T, 128>(P.delta, k - W.rg.kbase), cur, L, true);
        panel_axpy_pf(acc, (T)1, cur, L);
        if (k > k0) panel_store(pf_mat<T, 128>(P.bloc, k - 1 - W.rg.kbase), acc, L);
      }
    }
    __syncthreads();
  }
}

// The grouped carry at D = 128 (the steps of k_carry_grp, k_carry_top and
// k_mc); every product reads both factors from stored PF matrices.
template <typename T>
__device__ __forceinline__ T* grp_mat128(const ProbDesc& P, int kind, int g) {
  return pf_mat<T, 128>(P.grp, kind * P.PG + g);
}

template <typename T>
__global__ __launch_bounds__(512) void k_carry_grp128(Work W, int dirs, void* scratch) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.total * dirs; item += gridDim.x) {
    const int bwd = item % dirs;
    int p, g;
    split_item(item / dirs, 0, W.rg.c_n, I.start, I.nprob, p, g);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int c0 = g * P.CG;
    const int c1 = min(P.P, c0 + P.CG) - 1;
    Panel<T, 128> acc;
    panel_identity(acc, L);
    if (!bwd) {
      panel_store(pf_mat<T, 128>(P.cf, c0), acc, L);
      for (int c = c0; c <= c1; ++c) {
        gemm128<T, false>(acc, lds, pf_mat<T, 128>(P.tf, c), pf_mat<T, 128>(P.cf, c), L, true);
        panel_store(c < c1 ? pf_mat<T, 128>(P.cf, c + 1) : grp_mat128<T>(P, 0, g), acc, L);
      }
    } else {
      panel_store(pf_mat<T, 128>(P.cb, c1), acc, L);
      for (int c = c1; c >= c0; --c) {
        gemm128<T, true>(acc, lds, pf_mat<T, 128>(P.tf, c), pf_mat<T, 128>(P.cb, c), L, true);  // tf[c]^dag cb_loc[c]
        panel_store(c > c0 ? pf_mat<T, 128>(P.cb, c - 1) : grp_mat128<T>(P, 1, g), acc, L);
      }
    }
    __syncthreads();
  }
  (void)scratch;
}

template <typename T>
__global__ __launch_bounds__(512) void k_carry_top128(Work W, int dirs, void* scratch) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  __shared__ double red[2 * 8];
  Lane L;
  const Items I(W);
  for (int item = blockIdx.x; item < I.nprob * dirs; item += gridDim.x) {
    const int bwd = item % dirs;
    const ProbDesc P = W.descs[I.desc(item / dirs)];  // a copy: stores cannot alias it
    const int ng = P.PG;
    Panel<T, 128> acc;
    if (!bwd) {
      panel_identity(acc, L);
      panel_store(grp_mat128<T>(P, 2, 0), acc, L);
      for (int g = 0; g < ng; ++g) {
        gemm128<T, false>(acc, lds, grp_mat128<T>(P, 0, g), grp_mat128<T>(P, 2, g), L, true);
        if (g + 1 < ng) panel_store(grp_mat128<T>(P, 2, g + 1), acc, L);
      }
      fidelity_epilogue<T, 128>(P, acc, L, red);
      T* SXN = slot_mat<T>(scratch, 0);
      panel_store(SXN, acc, L);
      gemm128<T, true>(acc, lds, SXN, SXN, L, true);
      residual_epilogue<T, 128>(P, acc, L, red);
    } else {
      panel_load(acc, reinterpret_cast<const T*>(P.Vint), L);
      panel_store(grp_mat128<T>(P, 3, ng - 1), acc, L);
      for (int g = ng - 1; g >= 1; --g) {
        gemm128<T, false>(acc, lds, grp_mat128<T>(P, 1, g), grp_mat128<T>(P, 3, g), L, true);
        panel_store(grp_mat128<T>(P, 3, g - 1), acc, L);
      }
    }
    __syncthreads();
  }
}

// mc[c] = cb[c] cf[c]^dag with cf[c] = cf_loc[c] gcf[g], cb[c] = cb_loc[c] gcb[g].
template <typename T>
__global__ __launch_bounds__(512) void k_mc128(Work W, void* scratch) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  Lane L;
  T* S0 = slot_mat<T>(scratch, 0);
  T* S1 = slot_mat<T>(scratch, 1);
  T* S2 = slot_mat<T>(scratch, 2);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, c;
    split_item(item, W.rg.c_lo, W.rg.c_n, I.start, I.nprob, p, c);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int g = c / P.CG;
    Panel<T, 128> acc;
    gemm128<T, false>(acc, lds, pf_mat<T, 128>(P.cf, c), grp_mat128<T>(P, 2, g), L, true);
    panel_store(S1, acc, L);  // cf[c]
    gemm128<T, false>(acc, lds, pf_mat<T, 128>(P.cb, c), grp_mat128<T>(P, 3, g), L, true);
    panel_store(S2, acc, L);  // cb[c]
    transpose128<T>(S0, lds, S1, L);
    gemm128<T, false>(acc, lds, S2, S0, L, true);
    panel_store(pf_mat<T, 128>(P.mc, c), acc, L);
    __syncthreads();
  }
}

// The sampled last step at D = 128 (FP32, s = 0, permutation controls, at most
// kSample128Max controls): as sampled_gradient, with the operands in scratch.
// X2 and S take the LDS in turn (the whole FP32 matrix fits), so every
// column set's partial sums stay in registers between the two passes: pass 1
// adds X2 C2, pass 2 S C1 and E; C1, C2 and E are read one row block of this
// wavefront's own panels at a time.
constexpr int kSample128Max = 16;

__device__ __forceinline__ void sampled_gradient128(const ProbDesc& P, int k, const Lane& L, float* lds, double* red,
                                                    const float* X2, const float* S, const float* C1,
                                                    const float* C2, const float* E, bool x2_staged) {
  using K = K128<float>;
  constexpr int MS = kSample128Max;
  constexpr int G = kEpiGroup;
  const float* lim = lds + K::D * K::SD;
  const int b = 16 * L.w + L.c16;
  const int m = P.m;
  int aj[MS];
  unsigned fresh = 0;  // bit j: control j starts a column set (else it reuses j - 1's)
#pragma unroll
  for (int j = 0; j < MS; ++j) {
    aj[j] = j < m ? gp(P.minv)[(size_t)j * K::D + b] : 0;
    if (j < m && (j % G == 0 || !(gp(P.mok)[j] & 4))) fresh |= 1u << j;
  }
  float zr[MS], zi[MS];
#pragma unroll
  for (int j = 0; j < MS; ++j) zr[j] = zi[j] = 0.f;
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1 || !x2_staged) {
      __syncthreads();
      stage128<float, false>(lds, pass == 0 ? X2 : S, 0, L);
      __syncthreads();
    }
    const float* Cp = pass == 0 ? C2 : C1;
#pragma unroll 1
    for (int rb = 0; rb < K::RB; ++rb) {
      f4 cr, ci, er, ei;
      pf_rb_load<float>(cr, ci, Cp, L.w, rb, L.lane);
      if (pass == 1) pf_rb_load<float>(er, ei, E, L.w, rb, L.lane);
      const int col = 16 * rb + 4 * L.g;
#pragma unroll
      for (int j = 0; j < MS; ++j) {
        if (fresh & (1u << j)) {  // uniform over the workgroup
          const f4 ar = Prec<float>::ld4(lds + aj[j] * K::SD + col), ai = Prec<float>::ld4(lim + aj[j] * K::SD + col);
          float pr = zr[j], pi = zi[j];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (pass == 1 && col + r == aj[j]) {
              pr += er[r];
              pi += ei[r];
            }
            pr = fmaf(ar[r], cr[r], pr);
            pr = fmaf(-ai[r], ci[r], pr);
            pi = fmaf(ar[r], ci[r], pi);
            pi = fmaf(ai[r], cr[r], pi);
          }
          zr[j] = pr;
          zi[j] = pi;
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < MS; ++j) {
    if (fresh & (1u << j)) {
      zr[j] += __shfl_xor(zr[j], 16, 64);
      zi[j] += __shfl_xor(zi[j], 16, 64);
      zr[j] += __shfl_xor(zr[j], 32, 64);
      zi[j] += __shfl_xor(zi[j], 32, 64);
    } else if (j > 0) {
      zr[j] = zr[j - 1];
      zi[j] = zi[j - 1];
    }
  }
  const float* mv = reinterpret_cast<const float*>(P.mval);
#pragma unroll
  for (int j0 = 0; j0 < MS; j0 += G) {
    if (j0 >= m) break;
    double v[2 * G];
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      const int j = j0 + jj;
      double tr = 0, ti = 0;
      if (L.g == 0 && j < m) {  // conj(z) h, once per column
        const size_t e = (size_t)j * K::D + aj[j];
        const float hr = gp(mv)[2 * e], hi = gp(mv)[2 * e + 1];
        tr = (double)zr[j] * hr + (double)zi[j] * hi;
        ti = (double)zr[j] * hi - (double)zi[j] * hr;
      }
      v[2 * jj] = tr;
      v[2 * jj + 1] = ti;
    }
    epilogue_publish<8, G>(P, k, j0, j0 / G, v, L, red);
  }
}

// Same steps as k_adjoint, with the chain state in scratch (see above).
template <typename T>
__global__ __launch_bounds__(512) void k_adjoint128(Work W, void* scratch) {
  __shared__ T lds[K128<T>::LDS_ELEMS];
  __shared__ double red[2 * kEpiGroup * 2 * 8];
  Lane L;
  T* S0 = slot_mat<T>(scratch, 0);
  T* S1 = slot_mat<T>(scratch, 1);
  T* SE = slot_mat<T>(scratch, 2);
  T* SX = slot_mat<T>(scratch, 3);
  T* SR1 = slot_mat<T>(scratch, 4);
  T* SR2 = slot_mat<T>(scratch, 5);
  const Items I(W);
  for (int item = blockIdx.x; item < I.total; item += gridDim.x) {
    int p, k;
    split_item(item, W.rg.s_lo, W.rg.s_n, I.start, I.nprob, p, k);
    const ProbDesc P = W.descs[I.desc(p)];  // a copy: stores cannot alias it
    const int sqk = gp(P.sq)[k];
    int s, q, qb;
    unpack_sq(sqk, s, q, qb);
    Panel<T, 128> acc;
    // W = bloc[k] xprev[k]^dag (bloc carries mc[c])
    transpose128<T>(S0, lds, pf_mat<T, 128>(P.xprev, k - W.rg.kbase), L);
    gemm128<T, false, k128Gauss<T>>(acc, lds, pf_mat<T, 128>(P.bloc, k - W.rg.kbase), S0, L, true);
    // E = W / 2^s
    panel_scale(acc, (T)ldexp(1.0, -s));
    panel_store(SE, acc, L);
    // X = A^dag / 2^s: the expm pass's A / 2^s negated (A = -i dt H_k with H_k
    // Hermitian), or its conjugate transpose for general generators (own
    // panel; the barrier at the start of the next product publishes SX)
    if (P.flags & RUN_GENERAL) {
      transpose128<T>(SX, lds, pf_mat<T, 128>(P.hk, k - W.rg.kbase), L);
    } else {
      panel_load(acc, pf_mat<T, 128>(P.hk, k - W.rg.kbase), L);
      panel_scale(acc, (T)-1);
      panel_store(SX, acc, L);
    }
    // The block polynomial by Paterson-Stockmeyer as in k_adjoint: M^2 =
    // [[X2, S], [0, X2]] into S0 (X2) and S1 (S), the running C = [[C1, C2],
    // [0, C1]] in SR1 and SR2.
    gemm128<T, false, k128Gauss<T>>(acc, lds, SX, SX, L, true);
    panel_store(S0, acc, L);
    gemm128<T, false, k128Gauss<T>>(acc, lds, SX, SE, L, true, false);
    gemm128<T, false, k128Gauss<T>>(acc, lds, SE, SX, L, false);
    panel_store(S1, acc, L);
    const int top = (qb - 2) / 2;
    int t;
    if (qb & 1) {  // C = I / (qb-1)! + M / qb!
      t = top - 1;
      panel_load(acc, SX, L);
      panel_scale(acc, (T)inv_factorial(qb));
      panel_add_identity(acc, L, (T)inv_factorial(qb - 1));
      panel_store(SR1, acc, L);
      panel_load(acc, SE, L);
      panel_scale(acc, (T)inv_factorial(qb));
      panel_store(SR2, acc, L);
    } else if (top > 0) {  // C = I / (qb-2)! + M / (qb-1)! + M^2 / qb!
      t = top - 2;
      panel_load(acc, SX, L);
      panel_scale(acc, (T)inv_factorial(qb - 1));
      panel_axpy_pf(acc, (T)inv_factorial(qb), S0, L);
      panel_add_identity(acc, L, (T)inv_factorial(qb - 2));
      panel_store(SR1, acc, L);
      panel_load(acc, SE, L);
      panel_scale(acc, (T)inv_factorial(qb - 1));
      panel_axpy_pf(acc, (T)inv_factorial(qb), S1, L);
      panel_store(SR2, acc, L);
    } else {  // qb = 2: C = I / 2
      t = -1;
      panel_zero(acc);
      panel_store(SR2, acc, L);
      panel_add_identity(acc, L, (T)0.5);
      panel_store(SR1, acc, L);
    }
    // Products with X2 as the left factor follow each other where they can
    // (S C1 first in a step), so that X2 stays in LDS between them (FP32).
    bool x2_staged = false;
    for (; t >= 0; --t) {  // C <- D_t + M^2 C (own panels of SR1, SR2 only)
      const T a = (T)inv_factorial(2 * t + 2), b = (T)inv_factorial(2 * t + 3);
      panel_load(acc, SE, L);
      panel_scale(acc, b);
      gemm128<T, false, k128Gauss<T>>(acc, lds, S1, SR1, L, false);
      gemm128<T, false, k128Gauss<T>>(acc, lds, S0, SR2, L, false);
      panel_store(SR2, acc, L);  // b E + S C1 + X2 C2
      panel_load(acc, SX, L);
      panel_scale(acc, b);
      panel_add_identity(acc, L, a);
      gemm128<T, false, k128Gauss<T>>(acc, lds, S0, SR1, L, false, false);
      panel_store(SR1, acc, L);  // a I + b X + X2 C1
      x2_staged = true;
    }
    if constexpr (sizeof(T) == 4) {
      if ((sqk & kPlanSampled) && P.m <= kSample128Max) {  // s = 0: only the entries the controls read
        sampled_gradient128(P, k, L, lds, red, S0, S1, SR1, SR2, SE, x2_staged);
        __syncthreads();
        continue;
      }
    }
    // Q = E + X2 C2 + S C1 and, when squaring follows, D1 = X + X2 C1 (into
    // S1 once every wavefront has staged S; Q waits in the own panel of SE).
    panel_load(acc, SE, L);
    gemm128<T, false, k128Gauss<T>>(acc, lds, S0, SR2, L, false, !x2_staged);
    gemm128<T, false, k128Gauss<T>>(acc, lds, S1, SR1, L, false);
    if (s > 0) {
      panel_store(SE, acc, L);
      panel_load(acc, SX, L);
      gemm128<T, false, k128Gauss<T>>(acc, lds, S0, SR1, L, false);
      panel_store(S1, acc, L);
      panel_load(acc, SE, L);
    }
    for (int j = 0; j < s; ++j) {
      panel_store(S0, acc, L);                        // Q
      gemm128<T, false, k128Gauss<T>>(acc, lds, S1, S0, L, true);   // D1 Q
      gemm128<T, false, k128Gauss<T>>(acc, lds, S0, S1, L, false);  // + Q D1
      panel_axpy_pf(acc, (T)2, S0, L);                // Q <- 2Q + D1 Q + Q D1
      if (j + 1 < s) {
        // Every wavefront's staging of the old Q and D1 ended before the
        // barrier inside the last product, so own panels may be replaced.
        panel_store(S0, acc, L);
        gemm128<T, false, k128Gauss<T>>(acc, lds, S1, S1, L, true);
        panel_axpy_pf(acc, (T)2, S1, L);              // D1 <- 2 D1 + D1^2
        panel_store(S1, acc, L);
        panel_load(acc, S0, L);
      }
    }
    panel_store(S0, acc, L);  // Z (own panel)
    gradient_epilogue128<T>(P, k, S0, L, lds, red, sizeof(T) == 4 && (sqk & kPlanMono));
    __syncthreads();
  }
}

#include "qoc_seg128.hpp"

// ---------------------------------------------------------------- launchers

// Work of an API launch over range rg: uniform counts when rg says so,
// otherwise the prefix arrays of the launch.
static inline Work slice_work(const Launch& L, const Range& rg) {
  return Work{L.descs, L.nprob, rg.s_n > 0 ? L.nprob * rg.s_n : L.total_slices, rg.s_n > 0 ? nullptr : L.slice_start,
              rg, nullptr};
}
static inline Work chunk_work(const Launch& L, const Range& rg) {
  return Work{L.descs, L.nprob, rg.c_n > 0 ? L.nprob * rg.c_n : L.total_chunks, rg.c_n > 0 ? nullptr : L.chunk_start,
              rg, nullptr};
}
static inline int grid_of(const Launch& L, int items, int cap) {
  if (L.dyn_grid > 0) return L.dyn_grid;
  return items < 1 ? 1 : (cap > 0 && items > cap ? cap : items);
}

// The general-generator path at D <= 64 (Ops: the LDS policy of the adjoint's
// products; the other stages run on StdOps).
template <typename T, int D, typename Ops>
static void stage_small(int stage, const Launch& L, const Range& rg, double ur) {
  using Std = StdOps<T, D>;
  constexpr int NT = Mat<T, D>::NT;
  hipStream_t st = L.stream;
  const int grad = (L.flags & RUN_GRAD) ? 1 : 0;
  const Range all = {0, L.uniformN, 0, L.uniformP, rg.kbase};
  switch (stage) {
    case ST_PLAN: {
      Work w = slice_work(L, all);
      hipLaunchKernelGGL(k_plan, dim3((w.total + 255) / 256), dim3(256), 0, st, w, ur, grad);
      break;
    }
    case ST_EXPM: {
      Work w = slice_work(L, rg);
      hipLaunchKernelGGL((k_expm<T, D, Std>), dim3(grid_of(L, w.total, 0)), dim3(NT), 0, st, w);
      break;
    }
    case ST_SCAN:
    case ST_BSCAN: {
      Work w = chunk_work(L, rg);
      // a recompute sweep runs the forward and backward passes of a segment
      // together (they are independent once mc is known)
      const bool both = stage == ST_SCAN && rg.recompute;
      const int dir = stage == ST_BSCAN ? 1 : (both ? -1 : 0);
      const dim3 grid(grid_of(L, w.total, 0), both ? 2 : 1);
      hipLaunchKernelGGL((k_scan_local<T, D, Std>), grid, dim3(NT), 0, st, w, dir);
      break;
    }
    case ST_MC: {
      Work w = chunk_work(L, all);
      hipLaunchKernelGGL((k_mc<T, D, Std>), dim3(grid_of(L, w.total, 0)), dim3(NT), 0, st, w);
      break;
    }
    case ST_ADJ: {
      Work w = slice_work(L, rg);
      const dim3 grid(grid_of(L, w.total, 0));
      if constexpr (kSampleLast<T, D, Ops>) {
        hipLaunchKernelGGL((k_adjoint<T, D, Ops, 2>), grid, dim3(NT), 0, st, w);
        hipLaunchKernelGGL((k_adjoint<T, D, Ops, 1>), grid, dim3(NT), 0, st, w);
      } else {
        hipLaunchKernelGGL((k_adjoint<T, D, Ops>), grid, dim3(NT), 0, st, w);
      }
      break;
    }
  }
}

// Preparation and carry at D <= 64, the same for both paths.
template <typename T, int D>
static void stage_common(int stage, const Launch& L, const Range& rg) {
  constexpr int NT = Mat<T, D>::NT;
  hipStream_t st = L.stream;
  const int dirs = (L.flags & RUN_BWD) ? 2 : 1;
  const Range all = {0, L.uniformN, 0, L.uniformP, rg.kbase};
  const Work dyn = L.dyn ? Work{L.descs, 0, 0, nullptr, Range{0, 0, 0, 0, 0}, L.dyn} : Work{};
  if (stage == ST_PREP) {
    Work w = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * (L.max_m + 2), nullptr,
                                Range{0, L.max_m + 2, 0, 0, 0}, nullptr};
    hipLaunchKernelGGL((k_prep<T, D>), dim3(grid_of(L, w.total, 0)), dim3(256), 0, st, w);
  } else {  // ST_CARRY
    int CG, PG;
    carry_groups(L.uniformP, CG, PG);
    Work wg = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * PG, nullptr, Range{0, 0, 0, PG, 0}, nullptr};
    hipLaunchKernelGGL((k_carry_grp<T, D, StdOps<T, D>>), dim3(grid_of(L, wg.total, 0), dirs), dim3(NT), 0, st, wg);
    Work w = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob, nullptr, all, nullptr};
    hipLaunchKernelGGL((k_carry_top<T, D, StdOps<T, D>>), dim3(grid_of(L, L.nprob, 0), dirs), dim3(NT), 0, st, w);
  }
}

// The Hermitian path at D <= 64 (segments; Ops: the policy of the products
// whose errors stay local).
template <typename T, int D, typename Ops>
static void stage_seg(int stage, const Launch& L, const Range& rg, double ur) {
  constexpr int NT = Mat<T, D>::NT;
  hipStream_t st = L.stream;
  const int grad = (L.flags & RUN_GRAD) ? 1 : 0;
  const Range all = {0, L.uniformN, 0, L.uniformP, rg.kbase};
  const Work dyn = L.dyn ? Work{L.descs, 0, 0, nullptr, Range{0, 0, 0, 0, 0}, L.dyn} : Work{};
  const int most = seg_max(D, L.chunk, sizeof(T) == 8);
  const Work segs = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * rg.c_n * seg_count(L.chunk, most), nullptr, rg, nullptr};
  switch (stage) {
    case ST_PLAN: {
      Work w = L.dyn ? dyn : slice_work(L, all);
      const int comm = (L.flags & RUN_STATE) ? 0 : PLAN_COMM;
      hipLaunchKernelGGL(k_plan, dim3(L.dyn ? L.dyn_grid : (w.total + 255) / 256), dim3(256), 0, st, w, ur,
                         grad | comm);
      break;
    }
    case ST_EXPM: {
      const dim3 grid(grid_of(L, segs.total, 0));
      if (L.dyn) hipLaunchKernelGGL((k_seg_fwd<T, D, Ops, true>), grid, dim3(NT), 0, st, segs);
      else hipLaunchKernelGGL((k_seg_fwd<T, D, Ops, false>), grid, dim3(NT), 0, st, segs);
      break;
    }
    case ST_SCAN: {
      Work w = L.dyn ? dyn : chunk_work(L, rg);
      const dim3 grid(grid_of(L, w.total, 0));
      if (L.dyn) hipLaunchKernelGGL((k_seg_join<T, D, true>), grid, dim3(NT), 0, st, w);
      else hipLaunchKernelGGL((k_seg_join<T, D, false>), grid, dim3(NT), 0, st, w);
      if constexpr (sizeof(T) == 4) {
        if (!rg.recompute) {
          if (L.dyn) hipLaunchKernelGGL((k_reun<D, true>), grid, dim3(NT), 0, st, w);
          else hipLaunchKernelGGL((k_reun<D, false>), grid, dim3(NT), 0, st, w);
        }
      }
      break;
    }
    case ST_MC: {
      Work w = L.dyn ? dyn : chunk_work(L, all);
      hipLaunchKernelGGL((k_seg_y<T, D>), dim3(grid_of(L, w.total, 0)), dim3(NT), 0, st, w);
      break;
    }
    case ST_ADJ: {
      const dim3 grid(grid_of(L, segs.total, 0), (L.flags & RUN_RAWDG) ? 2 : 1);
      if (L.dyn) hipLaunchKernelGGL((k_seg_grad<T, D, Ops, true>), grid, dim3(NT), 0, st, segs);
      else hipLaunchKernelGGL((k_seg_grad<T, D, Ops, false>), grid, dim3(NT), 0, st, segs);
      const int cap = kSqGrid<T, D>;
      const int items =
          segs.total * (kKeepU<D> && !L.dyn ? sq_pieces(segs.total, seg_len(L.chunk, most), cap, kSegWaves<T, D> > 1) : 1);
      const dim3 sq(L.dyn ? cap : std::max(1, std::min(items, cap)), grid.y);
      hipLaunchKernelGGL((k_seg_grad_sq<T, D, Ops>), sq, dim3(NT), 0, st, segs);
      break;
    }
  }
}

// One stage at D <= 64: SOps for Hermitian Hamiltonians, GOps for the adjoint
// of the block form (general generators).
template <typename T, int D, typename SOps, typename GOps>
static void stage_le64(int stage, const Launch& L, const Range& rg, double ur) {
  // The complex dg/du needs the series of two Hermitian parts: 2 m products,
  // which pays on the FP16 matrix cores only (FP64, m = 10: 20 against the
  // block form's 13; 256 problems of d = 16: 4.17 ms against 2.54).
  constexpr bool F16 = !std::is_same<SOps, StdOps<T, D>>::value;
  const bool block = (L.flags & RUN_GENERAL) || (!F16 && (L.flags & RUN_RAWDG));
  if (stage == ST_PREP || stage == ST_CARRY) stage_common<T, D>(stage, L, rg);
  else if (block) stage_small<T, D, GOps>(stage, L, rg, ur);
  else stage_seg<T, D, SOps>(stage, L, rg, ur);
}

// FP64, and general generators in FP32.
template <typename T>
static void stage_128(int stage, const Launch& L, const Range& rg, double ur) {
  hipStream_t st = L.stream;
  const int dirs = (L.flags & RUN_BWD) ? 2 : 1;
  const int grad = (L.flags & RUN_GRAD) ? 1 : 0;
  const Range all = {0, L.uniformN, 0, L.uniformP, rg.kbase};
  const Work dyn = L.dyn ? Work{L.descs, 0, 0, nullptr, Range{0, 0, 0, 0, 0}, L.dyn} : Work{};
  const int cap = kScratchSlots;
  switch (stage) {
    case ST_PREP: {
      Work w = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * (L.max_m + 2), nullptr,
                                  Range{0, L.max_m + 2, 0, 0, 0}, nullptr};
      hipLaunchKernelGGL((k_prep<T, 128>), dim3(grid_of(L, w.total, 0)), dim3(256), 0, st, w);
      break;
    }
    case ST_PLAN: {
      Work w = L.dyn ? dyn : slice_work(L, all);
      hipLaunchKernelGGL(k_plan, dim3(L.dyn ? L.dyn_grid : (w.total + 255) / 256), dim3(256), 0, st, w, ur,
                         grad | PLAN_PS);
      break;
    }
    case ST_EXPM: {
      Work w = L.dyn ? dyn : slice_work(L, rg);
      hipLaunchKernelGGL((k_expm128<T>), dim3(grid_of(L, w.total, cap)), dim3(512), 0, st, w, L.scratch);
      break;
    }
    case ST_SCAN:
    case ST_BSCAN: {
      Work w = L.dyn ? dyn : chunk_work(L, rg);
      const bool both = stage == ST_SCAN && rg.recompute && !L.dyn;
      const int dir = stage == ST_BSCAN ? 1 : (both ? -1 : 0);
      hipLaunchKernelGGL((k_scan128<T>), dim3(grid_of(L, w.total, 0), both ? 2 : 1), dim3(512), 0, st, w, dir);
      break;
    }
    case ST_CARRY: {
      int CG, PG;
      carry_groups(L.uniformP, CG, PG);
      Work wg = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * PG, nullptr, Range{0, 0, 0, PG, 0}, nullptr};
      hipLaunchKernelGGL(k_carry_grp128<T>, dim3(grid_of(L, wg.total * dirs, cap)), dim3(512), 0, st, wg, dirs,
                         L.scratch);
      Work w = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob, nullptr, all, nullptr};
      hipLaunchKernelGGL(k_carry_top128<T>, dim3(grid_of(L, L.nprob * dirs, cap)), dim3(512), 0, st, w, dirs,
                         L.scratch);
      break;
    }
    case ST_MC: {
      Work w = L.dyn ? dyn : chunk_work(L, all);
      hipLaunchKernelGGL(k_mc128<T>, dim3(grid_of(L, w.total, cap)), dim3(512), 0, st, w, L.scratch);
      break;
    }
    case ST_ADJ: {
      Work w = L.dyn ? dyn : slice_work(L, rg);
      hipLaunchKernelGGL((k_adjoint128<T>), dim3(grid_of(L, w.total, cap)), dim3(512), 0, st, w, L.scratch);
      break;
    }
  }
}

// Hermitian Hamiltonians at D = 128 in FP32.
static void stage_seg128(int stage, const Launch& L, const Range& rg, double ur) {
  hipStream_t st = L.stream;
  const int grad = (L.flags & RUN_GRAD) ? 1 : 0;
  const int parts = (L.flags & RUN_RAWDG) ? 2 : 1;
  const Range all = {0, L.uniformN, 0, L.uniformP, rg.kbase};
  const Work dyn = L.dyn ? Work{L.descs, 0, 0, nullptr, Range{0, 0, 0, 0, 0}, L.dyn} : Work{};
  const Work segs = L.dyn ? dyn : Work{L.descs, L.nprob, L.nprob * rg.c_n * seg_count(L.chunk, seg_max(128, L.chunk, false)), nullptr, rg, nullptr};
  const int cap = kScratchSlots;  // each workgroup owns a region of the scratch
  switch (stage) {
    case ST_PLAN: {
      Work w = L.dyn ? dyn : slice_work(L, all);
      hipLaunchKernelGGL(k_plan, dim3(L.dyn ? L.dyn_grid : (w.total + 255) / 256), dim3(256), 0, st, w, ur,
                         grad | PLAN_PS | ((L.flags & RUN_STATE) ? 0 : PLAN_COMM | PLAN_HORNER));
      break;
    }
    case ST_EXPM:
      hipLaunchKernelGGL(k_seg_fwd128, dim3(grid_of(L, segs.total, cap)), dim3(512), 0, st, segs, L.scratch);
      break;
    case ST_SCAN: {
      Work w = L.dyn ? dyn : chunk_work(L, rg);
      hipLaunchKernelGGL(k_seg_join128, dim3(grid_of(L, w.total, cap)), dim3(512), 0, st, w, L.scratch);
      break;
    }
    case ST_MC: {
      Work w = L.dyn ? dyn : chunk_work(L, all);
      hipLaunchKernelGGL(k_seg_y128, dim3(grid_of(L, w.total, cap)), dim3(512), 0, st, w, L.scratch);
      break;
    }
    case ST_ADJ: {
      const dim3 grid(std::min(grid_of(L, segs.total, cap), cap / parts), parts);
      hipLaunchKernelGGL(k_seg_grad128, grid, dim3(512), 0, st, segs, L.scratch);
      hipLaunchKernelGGL(k_seg_grad_sq128, grid, dim3(512), 0, st, segs, L.scratch);
      break;
    }
    case ST_BSCAN: break;  // (none)
    default: stage_128<float>(stage, L, rg, ur);  // preparation and carry
  }
}

hipError_t launch_stage(int precision, int D, int stage, const Launch& L, const Range& rg) {
  const double ur64 = 0x1p-53, ur32 = 0x1p-24;
  stage_mark(stage, true, L.stream);
  bool ok = true;
  if (precision == 0) {
    switch (D) {
      case 16: stage_le64<double, 16, StdOps<double, 16>, StdOps<double, 16>>(stage, L, rg, ur64); break;
      case 32: stage_le64<double, 32, StdOps<double, 32>, StdOps<double, 32>>(stage, L, rg, ur64); break;
      case 64: stage_le64<double, 64, StdOps<double, 64>, StdOps<double, 64>>(stage, L, rg, ur64); break;
      case 128: stage_128<double>(stage, L, rg, ur64); break;
      default: ok = false;
    }
  } else if (precision == 1) {
    switch (D) {
      case 16: stage_le64<float, 16, F16Ops<16>, StdOps<float, 16>>(stage, L, rg, ur32); break;
      case 32: stage_le64<float, 32, F16Ops<32>, StdOps<float, 32>>(stage, L, rg, ur32); break;
      case 64: stage_le64<float, 64, F16Ops<64>, StdOps<float, 64>>(stage, L, rg, ur32); break;
      case 128:
        if (L.flags & RUN_GENERAL) stage_128<float>(stage, L, rg, ur32);
        else stage_seg128(stage, L, rg, ur32);
        break;
      default: ok = false;
    }
  } else if (precision == 2) {
    // general generators: split-BF16 products in the adjoint (the Frechet
    // series and its trace contractions, the dominant kernel); the exponentials,
    // scans, carries and chunk products stay FP32, whose errors reach
    // Tr(V^dag X_N).  Hermitian Hamiltonians: the FP32 precision's kernels,
    // whose split-FP16 products are as cheap and keep six bits more.
    switch (D) {
      case 32: stage_le64<float, 32, F16Ops<32>, Bf3Ops<32>>(stage, L, rg, ur32); break;
      case 64: stage_le64<float, 64, F16Ops<64>, Bf3Ops<64>>(stage, L, rg, ur32); break;
      default: ok = false;
    }
  } else {
    ok = false;
  }
  stage_mark(stage, false, L.stream);
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---------------------------------------------------------------- state path: chunk totals

// The propagators of the state path's chunks less I, planar and row-major in tf
// (D <= 64):
// the identity carried through the chunk's slices as the states are, by the
// Taylor polynomial's action (q products per part of a slice, no exponential).
// In FP32 the sums over the slices are compensated (S and what their rounding
// dropped): of the chunk's errors only the products' stay, which scale with A_k.
// Each slice's factor also carries a scale of its own between 1 and 3/2: the
// entries that are the same in every slice then round differently in each, and
// their errors do not add up over the N slices.  1.04 ms at d = 64, m = 12, N =
// 2000, 32 problems in FP32: q products per slice on the FP16 matrix cores.
template <typename T, int D, typename Ops>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(kSegWaves<T, D>))) void k_state_total(
    const ProbDesc* descs, int chunks) {
  constexpr T C = Ops::C, CI = (T)1 / Ops::C;
  __shared__ __align__(16) unsigned char la[Ops::BYTES];
  __shared__ __align__(16) unsigned char lb[StdOps<T, D>::BYTES];
  __shared__ SegTab<T, D> tab;
  Lane L;
  const ProbDesc P = descs[blockIdx.x / chunks];  // a copy: stores cannot alias it
  const int c = blockIdx.x % chunks;
  const int k0 = c * P.L, k1 = min(P.N, k0 + P.L);
  const bool mono = (gp(P.sq)[k0] & kPlanMono) != 0;
  const SegTab<T, D>* tb = nullptr;
  constexpr bool COMP = sizeof(T) == 4;
  Panel<T, D> S, X, R, E;
  panel_zero(S);
  panel_zero(E);
  panel_add_identity(S, L, C);
  for (int k = k0; k < k1; ++k) {
    const int ki = (k - k0) % kSegMax;
    if (ki == 0) {
      __syncthreads();  // the tables have been read
      tb = seg_tab_load<T, D>(tab, P, k, min(k1, k + kSegMax), mono) ? &tab : nullptr;
    }
    int s, q, qb;
    unpack_sq(gp(P.sq)[k], s, q, qb);
    const double scale = COMP ? 1.0 + (k & 15) / 32.0 : 1.0;
    const T back = (T)(1.0 / ((double)C * scale));
    assemble_panel<T, D>(X, lb, P, k, ldexp(P.dt * (double)C * scale, -s), mono, tb, ki, L);
    Ops::store_nct(la, X, L);  // X = -X^dag
    __syncthreads();
    for (int r = 0; r < (1 << s); ++r) {
      R = S;
      for (int i = q; i > 1; --i) {
        Ops::mul(X, la, R, L);
        R = S;
        panel_fma(R, back * (T)(1.0 / i), X);
      }
      Ops::mul(X, la, R, L);
      if constexpr (COMP) {
        panel_scale(X, back);
        panel_fma(X, (T)1, E);
        auto add = [](T& a, T& e, T b) {  // a + e <- a + b (two-sum)
          const T t = a + b, z = t - a;
          e = (a - (t - z)) + (b - z);
          a = t;
        };
#pragma unroll
        for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            T a = S.re[rb][i], e;
            add(a, e, X.re[rb][i]);
            S.re[rb][i] = a;
            E.re[rb][i] = e;
            a = S.im[rb][i];
            add(a, e, X.im[rb][i]);
            S.im[rb][i] = a;
            E.im[rb][i] = e;
          }
      } else {
        panel_fma(S, back, X);
      }
    }
  }
  panel_add_identity(S, L, -C);
  panel_fma(S, (T)1, E);
  T* o = static_cast<T*>(P.tf) + (size_t)c * 2 * D * D;
#pragma unroll
  for (int rb = 0; rb < D / 16; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = (16 * rb + Prec<T>::rowmap(r, L.g)) * D + 16 * L.w + L.c16;
      o[e] = CI * S.re[rb][r];
      o[D * D + e] = CI * S.im[rb][r];
    }
}

hipError_t launch_state_totals(int precision, int D, const ProbDesc* descs, int B, int chunks, hipStream_t st) {
  const dim3 grid(B * chunks), nt(4 * D);
  switch (D + (precision == 0 ? 1000 : 0)) {
    case 16: hipLaunchKernelGGL((k_state_total<float, 16, F16Ops<16>>), grid, nt, 0, st, descs, chunks); break;
    case 32: hipLaunchKernelGGL((k_state_total<float, 32, F16Ops<32>>), grid, nt, 0, st, descs, chunks); break;
    case 64: hipLaunchKernelGGL((k_state_total<float, 64, F16Ops<64>>), grid, nt, 0, st, descs, chunks); break;
    case 1016: hipLaunchKernelGGL((k_state_total<double, 16, StdOps<double, 16>>), grid, nt, 0, st, descs, chunks); break;
    case 1032: hipLaunchKernelGGL((k_state_total<double, 32, StdOps<double, 32>>), grid, nt, 0, st, descs, chunks); break;
    case 1064: hipLaunchKernelGGL((k_state_total<double, 64, StdOps<double, 64>>), grid, nt, 0, st, descs, chunks); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#include "qoc_jac.hpp"

}  // namespace qoc
