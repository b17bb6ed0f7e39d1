// The COCG iteration with the lateral-Fourier preconditioner, carried out in
// lateral mode space.
//
// The preconditioner is the exact inverse of the flat-wire operator,
// P = A0^-1 with A = A0 - V (V the local potential and the nonlocal term;
// Eqs. (6), (8), (14)-(16)), so A z = r - V z for z = P r and the operator
// application of the recurrence p = z + beta p_old reads
//     q = A p = (r - V z) + beta q_old:
// no stencil and no electrode term are applied inside the iteration.  With
// q_old = (r_old - r) / alpha_old neither p nor q is stored.  One iteration is
//   plane pass   W = V z, plane by plane (Z -> z -> V z -> W), partials of z^T W;
//   mode pass    per lateral mode, along z:
//                  q  = (R - W) + (beta / alpha_old) (R_old - R),
//                  R' = R - alpha q,   Z = P R' (recursive z filter),
//                partials of rho' = r'^T z, sigma' = z^T q and |r'|^2
// with
//   beta  = -sigma alpha_old / rho_old   (z^T A p_old + beta p_old^T A p_old = 0),
//   alpha = rho / mu,  mu = p^T A p = z^T q = rho - z^T W + beta sigma.
// The solution correction of n steps is d = P t, t = sum_j alpha_j s_j with
// s_j = r_j + beta_j s_(j-1), a combination of the residuals r_0 .. r_(n-1):
// they are kept in a ring of vectors, folded into S and T when it is full,
// and d is formed once, when the residual is replaced.  An iteration moves 7
// vector streams (plane pass 2, mode pass 5).
//
// Why this beta and not rho / rho_old (the same number in exact arithmetic):
// it makes the new direction conjugate to the last one as computed, so the
// rounding that R_old - R brings into q is corrected from step to step instead
// of being carried along.  With rho / rho_old 5 of 5,664 solves of a 24 x 24 x 96
// chain with projectors took 500 to 2,700 iterations and a Na-like wire did not
// converge in complex64; with this one the most in 14,160 solves of the chain is
// 319 (mean 108.1; the recurrence with A p: 255 in 3,776, mean 109.9), and the
// wire takes 2,219 against 2,166.
//
// Real lateral basis.  Complex vectors are transformed with the real
// cos/sin pairs of the discrete Fourier transform along each lateral
// direction: position k < n/2 holds F(k) + F(-k), position n - k holds
// i (F(k) - F(-k)), the self-paired k = 0 and n/2 hold F(k).  The flat-wire
// operator is even in each lateral wave number, so it is diagonal in this
// basis too, and the bilinear form is
//     sum_x u v = (1/Nxy) sum_k w_k U_k V_k,   w = 1/2 per paired direction,
// without pairing a mode with its negative.
#include "fftreg.h"
#include "modal.h"

namespace {

__device__ __forceinline__ int rhs_of(const int* active, int slot) { return active ? active[slot] : slot; }

template <typename T> IOBM_HD cplx<T> mul_i(cplx<T> a) { return mk(-a.im, a.re); }   // i a
template <typename T> IOBM_HD cplx<T> mul_mi(cplx<T> a) { return mk(a.im, -a.re); }  // -i a

template <typename T> __device__ __forceinline__ const T* potential(const double* Vd, const float* Vf);
template <> __device__ __forceinline__ const double* potential<double>(const double* Vd, const float*) { return Vd; }
template <> __device__ __forceinline__ const float* potential<float>(const double*, const float* Vf) { return Vf; }

// Vector type for pairs of elements in global accesses (16 bytes).
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  typedef float4 type;
  static constexpr int n = 2;
  static __device__ __forceinline__ zf get(const float4& v, int k) { return k ? mk(v.z, v.w) : mk(v.x, v.y); }
  static __device__ __forceinline__ void set(float4& v, int k, zf c) {
    if (k) { v.z = c.re; v.w = c.im; } else { v.x = c.re; v.y = c.im; }
  }
};
template <> struct Vec16<double> {
  typedef double2 type;
  static constexpr int n = 1;
  static __device__ __forceinline__ zd get(const double2& v, int) { return mk(v.x, v.y); }
  static __device__ __forceinline__ void set(double2& v, int, zd c) { v.x = c.re; v.y = c.im; }
};

// ------------------------------------------------------------- plane pass ---
// What a plane kernel does with each plane of a right-hand side:
//   PM_FULL  Z -> W in place: inverse transform, times V, forward transform;
//   PM_INV   Z -> z in place (the first half, before the nonlocal projection);
//   PM_VFWD  z -> W in place (the second half: V z plus the nonlocal term);
//   PM_FWD   r -> R in place (a replaced residual);
//   PM_ACC   x += inverse transform of D (x not read where xset = 0).
// PM_FULL and PM_VFWD write the plane's partial of z^T V z and, on plane 0 of
// a right-hand side, advance its scalars by one step.
enum { PM_FULL = 0, PM_INV = 1, PM_VFWD = 2, PM_FWD = 3, PM_ACC = 4 };
constexpr bool pm_inv(int mode) { return mode == PM_FULL || mode == PM_INV || mode == PM_ACC; }
constexpr bool pm_fwd(int mode) { return mode == PM_FULL || mode == PM_VFWD || mode == PM_FWD; }
constexpr bool pm_sum(int mode) { return mode == PM_FULL || mode == PM_VFWD; }

// Scalars of the step that begins: the sums of the mode pass's block partials
// (fixed order), and the last step's rho and alpha moved to *_old.  A group
// of G threads takes them in two steps around a block barrier: NS strided
// sums of each value into LDS (read at the kernel's start, beside the plane:
// one thread adding them in turn would expose a load latency per block of
// modes), then threads t < 5 write one field each.
constexpr int kAdvValues = 4;  // rho and sigma (|r|^2 is read at a check only, k_modal_check)
constexpr int adv_subs(int G) { return G / kAdvValues < 1 ? 1 : (G / kAdvValues > 16 ? 16 : G / kAdvValues); }
template <int G>
__device__ __forceinline__ void advance_sums(double* sub, const double* part, int nmb, int t) {
  constexpr int NS = adv_subs(G);
  if (t < NS * kAdvValues) {
    const int v = t % kAdvValues, s = t / kAdvValues;
    double a = 0;
#pragma unroll 4
    for (int k = s; k < nmb; k += NS) a += part[MODAL_PART * k + v];
    sub[t] = a;
  }
}
template <int G>
__device__ __forceinline__ void advance_scalars(ModalScal& s, const double* sub, int t) {
  if (t < kAdvValues) {
    double v = 0;
    for (int k = 0; k < adv_subs(G); ++k) v += sub[k * kAdvValues + t];
    switch (t) {
      case 0: s.rho_old.re = s.rho.re; s.rho.re = v; break;
      case 1: s.rho_old.im = s.rho.im; s.rho.im = v; break;
      case 2: s.sigma.re = v; break;
      default: s.sigma.im = v; break;
    }
  } else if (t == kAdvValues) {
    s.alpha_old = s.alpha;
    s.step += 1;
  }
}

// Vector k of the ring (a chain of selects: the slot is uniform, and indexing
// the kernel arguments would put them in scratch memory).
template <typename T>
__device__ __forceinline__ cplx<T>* ring_at(cplx<T>* const (&ring)[ModalRing<T>::n], int k) {
  cplx<T>* p = ring[0];
#pragma unroll
  for (int i = 1; i < ModalRing<T>::n; ++i)
    if (k == i) p = ring[i];
  return p;
}

// Cos/sin positions -> twice the Fourier coefficients of one line, and back
// (all N values of the line in registers).
template <typename T, int N>
__device__ __forceinline__ void cs_to_fourier(cplx<T>* v) {
  v[0] = (T)2 * v[0];
  if constexpr (N % 2 == 0) v[N / 2] = (T)2 * v[N / 2];
#pragma unroll
  for (int k = 1; 2 * k < N; ++k) {
    const cplx<T> u = v[k], w = mul_mi(v[N - k]);
    v[k] = u + w;
    v[N - k] = u - w;
  }
}
template <typename T, int N>
__device__ __forceinline__ void fourier_to_cs(cplx<T>* v) {
#pragma unroll
  for (int k = 1; 2 * k < N; ++k) {
    const cplx<T> a = v[k], b = v[N - k];
    v[k] = a + b;
    v[N - k] = mul_i(a - b);
  }
}

// Element k of a line of n cos/sin positions as twice its Fourier
// coefficient (p = position k, q = position (n - k) % n), and element k of
// the cos/sin line from the Fourier coefficients.
template <typename T>
__device__ __forceinline__ cplx<T> cs_f(int k, int n, cplx<T> p, cplx<T> q) {
  if (k == 0 || 2 * k == n) return (T)2 * p;
  return 2 * k < n ? p + mul_mi(q) : q + mul_i(p);
}
template <typename T>
__device__ __forceinline__ cplx<T> f_cs(int k, int n, cplx<T> p, cplx<T> q) {
  if (k == 0 || 2 * k == n) return p;
  return 2 * k < n ? p + q : mul_i(q - p);
}

__device__ __forceinline__ float swap_pair(float x) {  // the value of the other lane of a pair (lane ^ 1)
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xf, 0xf, true));
}
__device__ __forceinline__ double swap_pair(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <typename T> __device__ __forceinline__ cplx<T> swap_pair(cplx<T> c) { return mk(swap_pair(c.re), swap_pair(c.im)); }

// Threads per line: complex128 lines of 24 points and more take two adjacent
// lanes (a whole 48-point complex128 line and the transform's scratch exceed
// the register file).  N is then a multiple of 4.
template <typename T, int N>
constexpr int line_split() { return (sizeof(T) == 8 && N >= 24) ? 2 : 1; }

// Inverse transform of a line of cos/sin positions in LDS (elements at
// a[i stride]); the result, unscaled by 2 N, is left in v: all N values, or
// with two lanes per line the values [half M, half M + M), M = N / 2.
template <typename T, int N, int SPLIT>
__device__ __forceinline__ void inverse_line(const cplx<T>* a, int stride, int half, cplx<T>* v) {
  if constexpr (SPLIT == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = a[i * stride];
    cs_to_fourier<T, N>(v);
    line_fft<T, N, +1>(v);
  } else {
    constexpr int M = N / 2;
#pragma unroll
    for (int m = 0; m < M; ++m) {  // even (half 0) or odd samples
      const int k = 2 * m + half;
      const cplx<T> p = a[k * stride], q = a[(m == 0 && !half ? 0 : N - k) * stride];
      v[m] = cs_f(k, N, p, q);
    }
    line_fft<T, M, +1>(v);
#pragma unroll
    for (int k = 0; k < M; ++k) {
      const cplx<T> o = swap_pair(v[k]);
      const cplx<T> t = mul_tw<T, N, +1>(half ? v[k] : o, k);
      const cplx<T> e = half ? o : v[k];
      v[k] = half ? e - t : e + t;
    }
  }
}

// Forward transform of a line held as inverse_line leaves it; with two lanes
// per line the result is distributed as v[k] = X(2 k + half).
template <typename T, int N, int SPLIT>
__device__ __forceinline__ void forward_regs(cplx<T>* v, int half) {
  if constexpr (SPLIT == 1) {
    line_fft<T, N, -1>(v);
  } else {
    constexpr int M = N / 2;
#pragma unroll
    for (int k = 0; k < M; ++k) {
      const cplx<T> o = swap_pair(v[k]);
      v[k] = half ? mul_tw<T, N, -1>(o - v[k], k) : v[k] + o;
    }
    line_fft<T, M, -1>(v);
  }
}

// add(voxel, sum_p B[voxel][p] W[p]) for the support voxels of plane z, shared
// by nt threads; only the projectors that are nonzero in the voxel's block of
// 256, the values of four voxels in flight together.
template <typename T, class Add>
__device__ __forceinline__ void add_nonlocal(const KBPlane<T>& kb, const cplx<T>* W, int z, int t, int nt, Add add) {
  constexpr int UB = 4;  // voxels in flight per thread
  const int u1 = kb.uplane[z + 1];
  for (int u0 = kb.uplane[z] + t; u0 < u1; u0 += UB * nt) {
    int u[UB], lo[UB], hi[UB], vox[UB], most = 0;
#pragma unroll
    for (int i = 0; i < UB; ++i) {
      u[i] = min(u0 + i * nt, u1 - 1);
      lo[i] = kb.prange[2 * (u[i] >> 8)];
      hi[i] = kb.prange[2 * (u[i] >> 8) + 1];
      vox[i] = kb.uvox[u[i]];
    }
    cplx<T> acc[UB];
#pragma unroll
    for (int i = 0; i < UB; ++i) {
      acc[i] = mk<T>(0, 0);
      most = max(most, hi[i] - lo[i]);
    }
    for (int p0 = 0; p0 < most; p0 += 4) {
      T b[UB][4];
#pragma unroll
      for (int i = 0; i < UB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) b[i][j] = kb.Bt[(long long)max(min(lo[i] + p0 + j, hi[i] - 1), 0) * kb.nu + u[i]];
#pragma unroll
      for (int i = 0; i < UB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int p = lo[i] + p0 + j;
          const T bv = p < hi[i] ? b[i][j] : (T)0;
          const cplx<T> w = W[min(p, kb.npad - 1)];
          acc[i].re += bv * w.re;
          acc[i].im += bv * w.im;
        }
    }
#pragma unroll
    for (int i = 0; i < UB; ++i)
      if (u0 + i * nt < u1) add(vox[i], acc[i]);
  }
}

// Square planes (N x N, N in the register-FFT list), PPB planes per block,
// SPLIT N threads per plane: each thread (pair) transforms one row and then
// one column in registers, the plane going through one padded LDS copy.
// Bound: PM_FULL carries four line transforms per element against two
// streams and is limited by vector arithmetic (complex64, N = 48: 4,340 vector
// instructions per wavefront and plane, which take 92% of the SIMDs' issue
// cycles over the launch), nearly as much by memory: 4.4 TB/s at 48 x 48 x 128
// with 768 states, 0.54 ms per launch.
template <typename T, int N, int PPB, int MODE>
__global__ void __launch_bounds__((line_split<T, N>() * N * PPB)) __attribute__((amdgpu_waves_per_eu(2)))
    k_plane_reg(PlaneArgs<T> A) {
  typedef typename Vec16<T>::type VT;
  constexpr int PE = Vec16<T>::n;
  constexpr int NN = N * N;
  constexpr int SPLIT = line_split<T, N>();
  constexpr int TP = SPLIT * N;           // threads per plane
  constexpr int EPT = NN / PE / TP;       // 16-byte accesses per thread: N / (PE SPLIT)
  constexpr int ROWS = PE * SPLIT;        // rows covered by one access of every thread
  constexpr int M = SPLIT == 1 ? N : N / 2;  // values per thread of a line
  __shared__ cplx<T> sm[PPB][N][N + 1];
  const int pl = threadIdx.x / TP, lt = threadIdx.x - pl * TP;
  const int gp = blockIdx.x * PPB + pl;
  // a group past the last plane repeats it and stores nothing, so that no load
  // sits under a branch
  const int gq = min(gp, A.nplanes - 1);
  const int slot = gq / A.nz, z = gq - slot * A.nz;
  const int rhs = rhs_of(A.active, slot);
  const bool ok = gp < A.nplanes;
  const long long off = ((long long)rhs * A.nz + z) * NN;
  cplx<T>* vec = A.vec + off;
  const int li = lt / SPLIT, half = lt % SPLIT;
  const int r0 = lt * PE / N, c0 = lt * PE - r0 * N;  // first element of the thread's accesses
  constexpr bool HAS_INV = pm_inv(MODE), HAS_FWD = pm_fwd(MODE);
  const T scale = (T)(0.25 / NN);
  double d_re = 0, d_im = 0;
  __shared__ double adv[pm_sum(MODE) ? PPB : 1][adv_subs(TP) * kAdvValues];
  const bool advance = pm_sum(MODE) && ok && z == 0;
  if (advance) advance_sums<TP>(adv[pl], A.part + (long long)rhs * A.nmb * MODAL_PART, A.nmb, lt);
  // stage the plane in LDS, all of a thread's loads in flight together
  {
    VT buf[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) buf[e] = reinterpret_cast<const VT*>(vec)[lt + e * TP];
    if constexpr (MODE == PM_VFWD) {
      const T* V = potential<T>(A.Vd, A.Vf) + (long long)z * NN + lt * PE;
      T pot[EPT * PE];
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int k = 0; k < PE; ++k) pot[e * PE + k] = V[e * TP * PE + k];
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int k = 0; k < PE; ++k) {
          const cplx<T> c = Vec16<T>::get(buf[e], k), u = pot[e * PE + k] * c;
          d_re += (double)c.re * u.re - (double)c.im * u.im;
          d_im += (double)c.re * u.im + (double)c.im * u.re;
          sm[pl][e * ROWS + r0][c0 + k] = u;
        }
      asm volatile("" : "+v"(d_re), "+v"(d_im));  // the sums are taken here (see the inverse path)
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int k = 0; k < PE; ++k) sm[pl][e * ROWS + r0][c0 + k] = Vec16<T>::get(buf[e], k);
    }
  }
  __syncthreads();
  if constexpr (MODE == PM_VFWD) {
    if (A.kb.nu) {
      // the nonlocal term on this plane's support voxels, B W; W of the
      // plane's right-hand side staged in LDS
      extern __shared__ char kb_lds[];
      cplx<T>* Wl = reinterpret_cast<cplx<T>*>(kb_lds) + pl * A.kb.npad;
      const double* W = A.kb.W + (long long)slot * 2 * A.kb.npad;
      for (int p = lt; p < A.kb.npad; p += TP) Wl[p] = mk<T>((T)W[2 * p], (T)W[2 * p + 1]);
      __syncthreads();
      add_nonlocal(A.kb, Wl, z, lt, TP, [&](int el, cplx<T> acc) {
        el -= z * NN;
        sm[pl][el / N][el % N] = sm[pl][el / N][el % N] + acc;
      });
      __syncthreads();
    }
  }
  cplx<T> v[M];
  if constexpr (HAS_INV) {
    inverse_line<T, N, SPLIT>(&sm[pl][li][0], 1, half, v);  // row li
#pragma unroll
    for (int i = 0; i < M; ++i) sm[pl][li][i + half * M] = v[i];
    __syncthreads();
    inverse_line<T, N, SPLIT>(&sm[pl][0][li], N + 1, half, v);  // column li
    if constexpr (MODE == PM_FULL) {
      // V of this column in batches: all of it in flight during the transform
      // would not fit the registers (N = 48: 380 B of scratch per lane)
      const T* V = potential<T>(A.Vd, A.Vf) + (long long)z * NN + li;
      constexpr int VB = M % 3 == 0 ? M / 3 : M / 2;
#pragma unroll
      for (int i0 = 0; i0 < M; i0 += VB) {
        T pot[VB];
#pragma unroll
        for (int i = 0; i < VB; ++i) pot[i] = V[(i0 + i + half * M) * N];
#pragma unroll
        for (int i = 0; i < VB; ++i) {
          const cplx<T> c = scale * v[i0 + i], u = pot[i] * c;
          d_re += (double)c.re * u.re - (double)c.im * u.im;
          d_im += (double)c.re * u.im + (double)c.im * u.re;
          v[i0 + i] = u;
        }
        // the sums are taken here: left to the end they would keep every
        // operand alive through the forward transform (scratch)
        asm volatile("" : "+v"(d_re), "+v"(d_im));
      }
    } else {
#pragma unroll
      for (int i = 0; i < M; ++i) v[i] = scale * v[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < M; ++i) v[i] = sm[pl][i + half * M][li];  // column li
  }
  if constexpr (HAS_FWD) {
    forward_regs<T, N, SPLIT>(v, half);
    if constexpr (SPLIT == 1) {
      fourier_to_cs<T, N>(v);
#pragma unroll
      for (int i = 0; i < N; ++i) sm[pl][i][li] = v[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = sm[pl][li][i];  // row li
      line_fft<T, N, -1>(v);
      fourier_to_cs<T, N>(v);
#pragma unroll
      for (int i = 0; i < N; ++i) sm[pl][li][i] = v[i];
    } else {
#pragma unroll
      for (int k = 0; k < M; ++k) sm[pl][2 * k + half][li] = v[k];
      __syncthreads();
      // row li of the cos/sin positions along y, from the Fourier rows li and -li
      const int lj = li ? N - li : 0;
#pragma unroll
      for (int k = 0; k < M; ++k) v[k] = f_cs(li, N, sm[pl][li][k + half * M], sm[pl][lj][k + half * M]);
      __syncthreads();
      forward_regs<T, N, SPLIT>(v, half);
#pragma unroll
      for (int k = 0; k < M; ++k) sm[pl][li][2 * k + half] = v[k];
    }
  } else {
#pragma unroll
    for (int i = 0; i < M; ++i) sm[pl][i + half * M][li] = v[i];
  }
  __syncthreads();
  if (ok) {
    if constexpr (MODE == PM_ACC) {
      const int xr = lt / N, xc = lt - xr * N;
      zd* x = A.x + off + lt;
      constexpr int XPT = NN / TP, XB = XPT % 8 == 0 ? 8 : 4;
      const bool have = A.xset[rhs] != 0;
#pragma unroll
      for (int e0 = 0; e0 < XPT; e0 += XB) {
        zd xv[XB];
        if (have) {
#pragma unroll
          for (int e = 0; e < XB; ++e) xv[e] = x[(e0 + e) * TP];
        } else {
#pragma unroll
          for (int e = 0; e < XB; ++e) xv[e] = mk(0.0, 0.0);
        }
#pragma unroll
        for (int e = 0; e < XB; ++e) x[(e0 + e) * TP] = xv[e] + cvt<double>(sm[pl][(e0 + e) * SPLIT + xr][xc]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int r = e * ROWS + r0;
        VT o;
#pragma unroll
        for (int k = 0; k < PE; ++k) {
          cplx<T> c = sm[pl][r][c0 + k];
          if constexpr (HAS_FWD && SPLIT > 1) c = f_cs(c0 + k, N, c, sm[pl][r][c0 + k ? N - c0 - k : 0]);
          Vec16<T>::set(o, k, c);
        }
        reinterpret_cast<VT*>(vec)[lt + e * TP] = o;
      }
    }
  }
  if constexpr (pm_sum(MODE)) {
    // per-plane sum in a fixed order: 8 strided sums, then those in order
    __shared__ double red[2][TP * PPB];
    __shared__ double red8[2][8 * PPB];
    red[0][threadIdx.x] = d_re;
    red[1][threadIdx.x] = d_im;
    __syncthreads();
    if (lt < 8) {
      double a = 0, b = 0;
      for (int i = lt; i < TP; i += 8) { a += red[0][pl * TP + i]; b += red[1][pl * TP + i]; }
      red8[0][pl * 8 + lt] = a;
      red8[1][pl * 8 + lt] = b;
    }
    __syncthreads();
    if (lt == 0 && ok) {
      double a = 0, b = 0;
      for (int i = 0; i < 8; ++i) { a += red8[0][pl * 8 + i]; b += red8[1][pl * 8 + i]; }
      double* dp = A.dpart + ((long long)rhs * A.ndp + z) * 2;
      dp[0] = a;
      dp[1] = b;
    }
    if (advance) advance_scalars<TP>(A.sc[rhs], adv[pl], lt);
  }
}

// The plane pass of a pair at a lateral Bloch vector: G plane pairs per block,
// N threads per plane, the primary's plane beside its shadow's.  Plain Fourier
// modes; the shadow's transforms run with the opposite sign, as those of its
// conjugate (V is real), conjugated on the way in and out.  The partials are
// those of z~^T V z.  The same bounds and memory traffic as k_plane_reg.
// A solve of 48 x 48 x 128 pairs: 47.7 ms with the real-space recurrence, 30.6 ms.
template <int N, int G, int MODE>
__global__ void __launch_bounds__(2 * N * G) __attribute__((amdgpu_waves_per_eu(2))) k_plane_pair(PlaneArgs<float> A) {
  constexpr int NN = N * N, EPT = N / 2;
  __shared__ zf sm[2 * G][N][N + 1];
  const int pl = threadIdx.x / N, lt = threadIdx.x - pl * N, shadow = pl & 1;
  const int gp = blockIdx.x * G + (pl >> 1), total = A.nplanes / 2;
  const int gq = min(gp, total - 1);  // a group past the last pair repeats it and stores nothing
  const int pair = gq / A.nz, z = gq - pair * A.nz;
  const int rhs = rhs_of(A.active, 2 * pair + shadow);
  const bool ok = gp < total;
  const long long off = ((long long)rhs * A.nz + z) * NN;
  zf* vec = A.vec + off;
  const float cj = shadow ? -1.0f : 1.0f;
  const int r0 = 2 * lt / N, c0 = 2 * lt - r0 * N;
  double d_re = 0, d_im = 0;
  __shared__ double adv[MODE == PM_FULL ? G : 1][adv_subs(N) * kAdvValues];
  const bool advance = MODE == PM_FULL && ok && z == 0 && !shadow;
  if (advance) advance_sums<N>(adv[pl >> 1], A.part + (long long)rhs * A.nmb * MODAL_PART, A.nmb, lt);
  {
    float4 buf[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) buf[e] = reinterpret_cast<const float4*>(vec)[lt + e * N];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      sm[pl][2 * e + r0][c0] = mk(buf[e].x, cj * buf[e].y);
      sm[pl][2 * e + r0][c0 + 1] = mk(buf[e].z, cj * buf[e].w);
    }
  }
  __syncthreads();
  zf v[N];
  if constexpr (MODE != PM_FWD) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = sm[pl][lt][i];
    line_fft<float, N, +1>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) sm[pl][lt][i] = v[i];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = sm[pl][i][lt];  // column lt
  if constexpr (MODE != PM_FWD) {
    line_fft<float, N, +1>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = (float)(1.0 / NN) * v[i];
  }
  if constexpr (MODE == PM_FULL) {
    if (shadow) {
#pragma unroll
      for (int i = 0; i < N; ++i) sm[pl][i][lt] = v[i];
    }
    __syncthreads();
    const float* V = A.Vf + (long long)z * NN + lt;
    constexpr int VB = N % 3 == 0 ? N / 3 : N / 2;
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += VB) {
      float pot[VB];
#pragma unroll
      for (int i = 0; i < VB; ++i) pot[i] = V[(i0 + i) * N];
#pragma unroll
      for (int i = 0; i < VB; ++i) {
        const zf u = pot[i] * v[i0 + i], p = sm[pl | 1][i0 + i][lt];  // conj(z~); the shadow's own sums are not used
        d_re += (double)p.re * u.re + (double)p.im * u.im;
        d_im += (double)p.re * u.im - (double)p.im * u.re;
        v[i0 + i] = u;
      }
      asm volatile("" : "+v"(d_re), "+v"(d_im));  // the sums are taken here (see k_plane_reg)
    }
    __syncthreads();
  }
  if constexpr (MODE != PM_ACC) {
    line_fft<float, N, -1>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) sm[pl][i][lt] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = sm[pl][lt][i];  // row lt
    line_fft<float, N, -1>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) sm[pl][lt][i] = v[i];
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) sm[pl][i][lt] = v[i];
  }
  __syncthreads();
  if (ok) {
    if constexpr (MODE == PM_ACC) {
      zd* x = A.x + off + lt;
      constexpr int XB = N % 8 == 0 ? 8 : 4;
#pragma unroll
      for (int e0 = 0; e0 < N; e0 += XB) {
        zd xv[XB];
#pragma unroll
        for (int e = 0; e < XB; ++e) xv[e] = x[(e0 + e) * N];
#pragma unroll
        for (int e = 0; e < XB; ++e) {
          const zf c = sm[pl][e0 + e][lt];
          x[(e0 + e) * N] = xv[e] + mk((double)c.re, (double)(cj * c.im));
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const zf a = sm[pl][2 * e + r0][c0], b = sm[pl][2 * e + r0][c0 + 1];
        reinterpret_cast<float4*>(vec)[lt + e * N] = make_float4(a.re, cj * a.im, b.re, cj * b.im);
      }
    }
  }
  if constexpr (MODE == PM_FULL) {
    // per-plane sum in a fixed order: 8 strided sums, then those in order
    __shared__ double red[2][2 * N * G];
    __shared__ double red8[2][16 * G];
    red[0][threadIdx.x] = d_re;
    red[1][threadIdx.x] = d_im;
    __syncthreads();
    if (lt < 8) {
      double a = 0, b = 0;
      for (int i = lt; i < N; i += 8) { a += red[0][pl * N + i]; b += red[1][pl * N + i]; }
      red8[0][pl * 8 + lt] = a;
      red8[1][pl * 8 + lt] = b;
    }
    __syncthreads();
    if (lt == 0 && ok && !shadow) {
      double a = 0, b = 0;
      for (int i = 0; i < 8; ++i) { a += red8[0][pl * 8 + i]; b += red8[1][pl * 8 + i]; }
      double* dp = A.dpart + ((long long)rhs * A.ndp + z) * 2;
      dp[0] = a;
      dp[1] = b;
    }
    if (advance) advance_scalars<N>(A.sc[rhs], adv[pl >> 1], lt);
  }
}

// Any other plane size: one plane per block in LDS (two copies and, with TW,
// the twiddle tables: see lds_holds), mixed-radix Stockham stages along x and y.
template <typename T, int MODE, bool TW>
__global__ void __launch_bounds__(256) k_plane_lds(PlaneArgs<T> A, FFTPlan2D plan, const cplx<T>* __restrict__ twx,
                                                   const cplx<T>* __restrict__ twy) {
  extern __shared__ char smem_raw[];
  const int nx = plan.x.n, ny = plan.y.n, nxy = nx * ny;
  cplx<T>* a = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* b = a + nxy;
  cplx<T>* tx = b + nxy;
  cplx<T>* ty = tx + (TW ? nx : 0);
  double* red = reinterpret_cast<double*>(ty + (TW ? ny : 0));  // [2][4]
  double* adv = red + 8;                             // [16][5]
  const int slot = blockIdx.x / A.nz, z = blockIdx.x - slot * A.nz;
  const int rhs = rhs_of(A.active, slot);
  const long long off = ((long long)rhs * A.nz + z) * nxy;
  cplx<T>* vec = A.vec + off;
  const T* V = potential<T>(A.Vd, A.Vf) + (long long)z * nxy;
  double d_re = 0, d_im = 0;
  constexpr bool HAS_INV = pm_inv(MODE), HAS_FWD = pm_fwd(MODE);
  const bool advance = pm_sum(MODE) && z == 0;
  if (advance) advance_sums<256>(adv, A.part + (long long)rhs * A.nmb * MODAL_PART, A.nmb, threadIdx.x);
  const float inx = 1.0f / (float)nx;
  if constexpr (TW) {
    for (int i = threadIdx.x; i < nx; i += blockDim.x) tx[i] = twx[i];
    for (int i = threadIdx.x; i < ny; i += blockDim.x) ty[i] = twy[i];
  }
  auto fft = [&](cplx<T>* in, cplx<T>* tmp, int sign) -> cplx<T>* {
    if constexpr (TW) return fft2d_lds(in, tmp, plan, tx, ty, sign);
    else return fft2d_lds(in, tmp, plan, twx, twy, sign);
  };
  for (int p = threadIdx.x; p < nxy; p += blockDim.x) {
    cplx<T> c = vec[p];
    if constexpr (MODE == PM_VFWD) {
      const cplx<T> u = V[p] * c;
      d_re += (double)c.re * u.re - (double)c.im * u.im;
      d_im += (double)c.re * u.im + (double)c.im * u.re;
      c = u;
    }
    a[p] = c;
  }
  __syncthreads();
  if constexpr (MODE == PM_VFWD) {
    if (A.kb.nu) {
      cplx<T>* Wl = reinterpret_cast<cplx<T>*>(adv + 16 * kAdvValues);  // [npad]
      const double* W = A.kb.W + (long long)slot * 2 * A.kb.npad;
      for (int p = threadIdx.x; p < A.kb.npad; p += blockDim.x) Wl[p] = mk<T>((T)W[2 * p], (T)W[2 * p + 1]);
      __syncthreads();
      add_nonlocal(A.kb, Wl, z, threadIdx.x, blockDim.x, [&](int el, cplx<T> acc) { a[el - z * nxy] = a[el - z * nxy] + acc; });
      __syncthreads();
    }
  }
  cplx<T>* src = a;
  if constexpr (HAS_INV) {
    for (int p = threadIdx.x; p < nxy; p += blockDim.x) {
      const int j = small_quotient(p, inx), i = p - j * nx;
      const int jm = (j ? ny - j : 0) * nx, im = i ? nx - i : 0, jp = j * nx;
      b[p] = cs_f(j, ny, cs_f(i, nx, a[jp + i], a[jp + im]), cs_f(i, nx, a[jm + i], a[jm + im]));
    }
    __syncthreads();
    src = fft(b, a, +1);
    const T scale = (T)(0.25 / nxy);
    if constexpr (MODE == PM_ACC) {
      zd* x = A.x + off;
      const bool have = A.xset[rhs] != 0;
      for (int p = threadIdx.x; p < nxy; p += blockDim.x) {
        const zd d = cvt<double>(scale * src[p]);
        x[p] = have ? x[p] + d : d;
      }
    } else if constexpr (MODE != PM_FULL) {
      for (int p = threadIdx.x; p < nxy; p += blockDim.x) vec[p] = scale * src[p];
    } else {
      for (int p = threadIdx.x; p < nxy; p += blockDim.x) {
        const cplx<T> c = scale * src[p], u = V[p] * c;
        d_re += (double)c.re * u.re - (double)c.im * u.im;
        d_im += (double)c.re * u.im + (double)c.im * u.re;
        src[p] = u;
      }
      __syncthreads();
    }
  }
  if constexpr (HAS_FWD) {
    cplx<T>* f = fft(src, src == a ? b : a, -1);
    for (int p = threadIdx.x; p < nxy; p += blockDim.x) {
      const int j = small_quotient(p, inx), i = p - j * nx;
      const int jm = (j ? ny - j : 0) * nx, im = i ? nx - i : 0, jp = j * nx;
      vec[p] = f_cs(j, ny, f_cs(i, nx, f[jp + i], f[jp + im]), f_cs(i, nx, f[jm + i], f[jm + im]));
    }
  }
  if constexpr (pm_sum(MODE)) {
    for (int o = 32; o > 0; o >>= 1) {
      d_re += __shfl_xor(d_re, o);
      d_im += __shfl_xor(d_im, o);
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { red[2 * wv] = d_re; red[2 * wv + 1] = d_im; }
    __syncthreads();
    if (threadIdx.x == 0) {
      double sr = 0, si = 0;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) { sr += red[2 * w]; si += red[2 * w + 1]; }
      double* dp = A.dpart + ((long long)rhs * A.ndp + z) * 2;
      dp[0] = sr;
      dp[1] = si;
    }
    if (advance) advance_scalars<256>(A.sc[rhs], adv, threadIdx.x);
  }
}

// -------------------------------------------------------------- mode pass ---
// ZS_STEP   one iteration's update and preconditioner (see the top of the file);
// ZS_START  Z = P R of a replaced residual (ring slot 0), the step count reset;
// ZS_FOLD   D = P t, the correction of the steps since the last replacement.
enum { ZS_STEP = 0, ZS_START = 1, ZS_FOLD = 2 };

// a / b, and whether b is nonzero and the quotient finite
__device__ __forceinline__ bool quotient(zd a, zd b, zd& r) {
  const double d = b.re * b.re + b.im * b.im;
  r = mk((a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d);
  if (d > 0 && isfinite(r.re) && isfinite(r.im)) return true;
  r = mk(0.0, 0.0);
  return false;
}

// Coefficients of the ring's residuals in t (the correction) and s (the
// direction) over the steps base .. n-1 of one right-hand side:
//   t_j = alpha_j + beta_(j+1) t_(j+1),  s_j = prod_(l > j) beta_l,
// and of the folded s of step base-1 (t_prev, s_prev).
template <int NR>
__device__ __forceinline__ void ring_coeffs(const zd* ha, const zd* hb, int base, int n, zd* t, zd* s, zd& t_prev,
                                            zd& s_prev) {
  zd ct = mk(0.0, 0.0), cs = mk(1.0, 0.0);
#pragma unroll
  for (int q = NR - 1; q >= 0; --q) {
    const int j = base + q;
    if (j >= n) { t[q] = s[q] = mk(0.0, 0.0); continue; }
    if (j < n - 1) {
      const zd b1 = hb[(j + 1) % NR];
      ct = ha[j % NR] + b1 * ct;
      cs = b1 * cs;
    } else {
      ct = ha[j % NR];
    }
    t[q] = ct;
    s[q] = cs;
  }
  const zd b0 = base < n ? hb[base % NR] : mk(0.0, 0.0);
  t_prev = b0 * ct;
  s_prev = b0 * cs;
}

// Recursive z filter in mode space.  Lane = lateral mode, wavefront = chunk
// of L planes held in registers:
//   causal      F(z) = sum_k al_k F(z-1-k) + sum_k fb_k  r(z-k)
//   anti-causal B(z) = sum_k al_k B(z+1+k) + sum_k fbb_k r(z+1+k),
//   out(z) = F(z) + B(z).
// Each chunk runs both recursions from a zero state; the states that enter it
// follow from the other chunks' end states and the state propagator M^L
// (tabulated per mode), and their homogeneous responses are added.  Block =
// MB modes x C chunks of one right-hand side (MB C <= 512).  The inputs of a step (W,
// R, R_old) are each read once, the boundary planes of R' pass between
// chunks through LDS.  Bound: memory (5 streams); the per-element work is
// about 8 nf complex multiply-adds and three FP64 dot products (59% of the issue
// cycles at 48 x 48 x 128; wavefronts wait a third of theirs).  Measured, with
// the starts and folds: 4.9 TB/s (48 x 48 x 128, 768 states), where the passes
// it stands for (operator, residual update, z filter, r^T z) took 12 of the
// operator-applying iteration's 14 streams; a solve there 68.7 -> 48.1 ms.
// Chunks of 16 planes instead of 8: 16 x 16 x 48 0.92 against 0.87 ms, 24 x 24 x
// 96 38 against 32 ms, 48 x 48 x 128 the same.
//
// PAIR (a lateral Bloch vector, plain Fourier modes): block = the same modes of
// a primary and its shadow, one after the other, with the primary's scalars
// and filter; the shadow is stored at the negative of its own modes, so that
// its operator and the products rho' = r~^T z and sigma' = (q~^T z + q^T z~) / 2
// (z and q kept in registers from the primary) are elementwise.  The mean of
// the two makes both directions conjugate alike: with q~^T z alone one of 180
// states of a 16 x 16 x 96 grid did not converge, of 1,932 with the mean every one.
template <typename T, int L, int NF, int MODE, int MB, bool PAIR>
__global__ void __launch_bounds__(512) k_zstep(ModeArgsZ<T> A) {
  constexpr int NR = ModalRing<T>::n;
  extern __shared__ char smem_raw[];
  const int C = blockDim.y;
  cplx<T>* hf = reinterpret_cast<cplx<T>*>(smem_raw);  // [C][NF][MB] first planes of each chunk
  cplx<T>* hl = hf + C * NF * MB;                      // [C][NF][MB] last NF - 1 planes
  cplx<T>* sc = hl + C * NF * MB;                      // [C][NF][MB] causal end states
  cplx<T>* sb = sc + C * NF * MB;                      // [C][NF][MB] anti-causal begin states
  double* red = reinterpret_cast<double*>(smem_raw);   // [C][5 (PAIR: 6)][MB], after the states are read
  const int slot = blockIdx.x / A.nmb, mb = blockIdx.x - slot * A.nmb;
  const int lane = threadIdx.x;
  // uniform over a wavefront where one holds a single chunk
  const int c = MB == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.y) : threadIdx.y;
  const int rhs = __builtin_amdgcn_readfirstlane(rhs_of(A.active, PAIR ? 2 * slot : slot));  // scalar: so are the vectors' addresses
  const int m = mb * MB + lane, nxy = A.nxy, nz = A.nz;
  const bool live = m < nxy;
  const int z0 = c * L;
  // byte offsets of the own planes within a right-hand side's vector (32 bits
  // beside a scalar base: at most 2^20 points of 16 bytes).
  // Loads are unconditional from clamped (always valid) addresses and masked
  // afterwards: a load under a branch of its own is waited for on its own
  const bool whole = live && z0 + L <= nz;
  unsigned off[L];
#pragma unroll
  for (int i = 0; i < L; ++i) off[i] = (unsigned)(min(z0 + i, nz - 1) * nxy + min(m, nxy - 1)) * (unsigned)sizeof(cplx<T>);
  auto in = [&](int i) -> bool { return live && z0 + i < nz; };
  auto mask = [&](cplx<T>* v) {  // zero outside the region
    if (!whole) {
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (!in(i)) v[i] = mk<T>(0, 0);
    }
  };
  auto load = [&](const cplx<T>* src, cplx<T>* v) {
#pragma unroll
    for (int i = 0; i < L; ++i) v[i] = *reinterpret_cast<const cplx<T>*>(reinterpret_cast<const char*>(src) + off[i]);
  };
  auto store = [&](cplx<T>* dst, const cplx<T>* v) {
    if (whole) {
#pragma unroll
      for (int i = 0; i < L; ++i) *reinterpret_cast<cplx<T>*>(reinterpret_cast<char*>(dst) + off[i]) = v[i];
    } else {
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (in(i)) *reinterpret_cast<cplx<T>*>(reinterpret_cast<char*>(dst) + off[i]) = v[i];
    }
  };
  ModalScal& S = A.sc[rhs];
  const int step = __builtin_amdgcn_readfirstlane(S.step);
  constexpr bool STEP = MODE == ZS_STEP;
  double d[5] = {0, 0, 0, 0, 0}, n2_prim = 0;
  cplx<T> zp[PAIR ? L : 1], qp[PAIR && STEP ? L : 1];  // Z and q of the primary
  __shared__ zd sco[2];
#pragma unroll 1
  for (int shadow = 0; shadow < (PAIR ? 2 : 1); ++shadow) {
  const int rv = rhs + shadow;  // the vectors' right-hand side
  const long long base = (long long)rv * nxy * nz;
  // own inputs; rr[NF - 1 + i] is plane z0 + i
  cplx<T> rr[L + 2 * NF - 1];
  cplx<T> q[STEP ? L : 1];
  if constexpr (STEP) {
    const int k = step;
    const cplx<T>* X = ring_at<T>(A.ring, k > 0 ? (k - 1) % NR : 0) + base;
    cplx<T> xo[L];
    load(ring_at<T>(A.ring, k % NR) + base, rr + NF - 1);
    load(A.w + base, q);
    load(X, xo);
    // z^T W of this right-hand side, summed in a fixed order, and the
    // step's scalars: by the first wavefront, while the loads are in flight
    if (c < 64 / MB && !shadow) {
      const int wl = c * MB + lane;
      zd dl = mk(0.0, 0.0);
      const double* dp = A.dpart + (long long)rhs * A.ndp * 2;
      for (int j = wl; j < A.ndp; j += 64) dl = dl + mk(dp[2 * j], dp[2 * j + 1]);
      for (int o = 32; o > 0; o >>= 1) dl = dl + mk(__shfl_xor(dl.re, o), __shfl_xor(dl.im, o));
      zd beta = mk(0.0, 0.0), g = mk(0.0, 0.0), alpha;
      bool good = true;
      if (k > 0) good = quotient(-(S.sigma * S.alpha_old), S.rho_old, beta) && quotient(-S.sigma, S.rho_old, g);
      good = quotient(S.rho, S.rho - dl + beta * S.sigma, alpha) && good;
      if (wl == 0) {
        sco[0] = alpha;
        sco[1] = g;  // beta / alpha_old
        if (mb == 0) {
          S.alpha = alpha;
          A.ha[(long long)rhs * NR + k % NR] = alpha;
          A.hb[(long long)rhs * NR + k % NR] = beta;
          if (!good) S.flag = 1;
        }
      }
    }
    __syncthreads();
    const cplx<T> at_ = cvt<T>(sco[0]), ct = cvt<T>(sco[1]);
    mask(rr + NF - 1);
    mask(q);
    mask(xo);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const cplx<T> r = rr[NF - 1 + i];
      q[i] = cfma(ct, xo[i] - r, r - q[i]);
      rr[NF - 1 + i] = cfma(-at_, q[i], r);
    }
    store(ring_at<T>(A.ring, (k + 1) % NR) + base, rr + NF - 1);
  } else if constexpr (MODE == ZS_START) {
    load(A.ring[0] + base, rr + NF - 1);
    mask(rr + NF - 1);
    if (mb == 0 && c == 0 && lane == 0 && !shadow) {
      S.step = -1;  // the next plane pass makes it 0
      S.base = 0;
      S.flag = 0;
      S.alpha = mk(0.0, 0.0);
    }
  } else {
    const int n = step + 1, b0 = __builtin_amdgcn_readfirstlane(S.base);
#pragma unroll
    for (int i = 0; i < L; ++i) rr[NF - 1 + i] = mk<T>(0, 0);
    auto add = [&](const cplx<T>* v, cplx<T> f) {
      cplx<T> t[L];
      load(v, t);
#pragma unroll
      for (int i = 0; i < L; ++i) rr[NF - 1 + i] = cfma(f, t[i], rr[NF - 1 + i]);
    };
    zd ct[NR], cs[NR], tp, sp;
    ring_coeffs<NR>(A.ha + (long long)rhs * NR, A.hb + (long long)rhs * NR, b0, n, ct, cs, tp, sp);
#pragma unroll
    for (int j = 0; j < NR; ++j)
      if (b0 + j < n) add(ring_at<T>(A.ring, (b0 + j) % NR) + base, cvt<T>(ct[j]));
    if (b0 > 0) {
      add(A.fold_s + rv * A.fold_stride, cvt<T>(tp));
      add(A.fold_t + rv * A.fold_stride, mk<T>(1, 0));
    }
    mask(rr + NF - 1);
  }
  // filter coefficients of this mode: [al | fb | fbb | M^L] (coalesced)
  constexpr int NC = 3 * NF + NF * NF;
  cplx<T> cf[NC];
  {
    const cplx<T>* ft = A.ft + (long long)A.e_rhs[rhs] * NC * nxy;
#pragma unroll
    for (int k = 0; k < NC; ++k) cf[k] = ft[(unsigned)(k * nxy + min(m, nxy - 1))];
  }
  const cplx<T>*al = cf, *fb = cf + NF, *fbb = cf + 2 * NF, *ML = cf + 3 * NF;
  // boundary planes between neighbouring chunks
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    hf[(c * NF + k) * MB + lane] = rr[NF - 1 + k];
    if (k < NF - 1) hl[(c * NF + k) * MB + lane] = rr[L + k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    rr[NF - 1 + L + k] = c + 1 < C ? hf[((c + 1) * NF + k) * MB + lane] : mk<T>(0, 0);
    if (k < NF - 1) rr[k] = c > 0 ? hl[((c - 1) * NF + k) * MB + lane] : mk<T>(0, 0);
  }
  cplx<T> y[L];
  {
    cplx<T> h[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) h[k] = mk<T>(0, 0);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      cplx<T> F = cfma(al[0], h[0], fb[0] * rr[NF - 1 + i]);
#pragma unroll
      for (int k = 1; k < NF; ++k) F = cfma(al[k], h[k], cfma(fb[k], rr[NF - 1 + i - k], F));
#pragma unroll
      for (int k = NF - 1; k > 0; --k) h[k] = h[k - 1];
      h[0] = F;
      y[i] = F;
    }
#pragma unroll
    for (int k = 0; k < NF; ++k) sc[(c * NF + k) * MB + lane] = h[k];
#pragma unroll
    for (int k = 0; k < NF; ++k) h[k] = mk<T>(0, 0);
#pragma unroll
    for (int i = L - 1; i >= 0; --i) {
      cplx<T> B = cfma(al[0], h[0], fbb[0] * rr[NF + i]);
#pragma unroll
      for (int k = 1; k < NF; ++k) B = cfma(al[k], h[k], cfma(fbb[k], rr[NF + i + k], B));
#pragma unroll
      for (int k = NF - 1; k > 0; --k) h[k] = h[k - 1];
      h[0] = B;
      y[i] = y[i] + B;
    }
#pragma unroll
    for (int k = 0; k < NF; ++k) sb[(c * NF + k) * MB + lane] = h[k];
  }
  __syncthreads();
  // the true states entering this chunk from both sides
  auto incoming = [&](const cplx<T>* st, int from, int to, int dir, cplx<T>* h) {
#pragma unroll
    for (int k = 0; k < NF; ++k) h[k] = mk<T>(0, 0);
    for (int cc = from; cc != to; cc += dir) {
      cplx<T> t[NF];
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        t[i] = st[(cc * NF + i) * MB + lane];
#pragma unroll
        for (int j = 0; j < NF; ++j) t[i] = cfma(ML[i * NF + j], h[j], t[i]);
      }
#pragma unroll
      for (int i = 0; i < NF; ++i) h[i] = t[i];
    }
  };
  auto respond = [&](cplx<T>* h, cplx<T>& out) {  // one plane of the homogeneous recursion
    cplx<T> F = al[0] * h[0];
#pragma unroll
    for (int k = 1; k < NF; ++k) F = cfma(al[k], h[k], F);
#pragma unroll
    for (int k = NF - 1; k > 0; --k) h[k] = h[k - 1];
    h[0] = F;
    out = out + F;
  };
  if (c > 0) {
    cplx<T> h[NF];
    incoming(sc, 0, c, 1, h);
#pragma unroll
    for (int i = 0; i < L; ++i) respond(h, y[i]);
  }
  if (c < C - 1) {
    cplx<T> h[NF];
    incoming(sb, C - 1, c, -1, h);
#pragma unroll
    for (int i = L - 1; i >= 0; --i) respond(h, y[i]);
  }
  store(A.w + base, y);
  if constexpr (MODE != ZS_FOLD) {
    // bilinear products: rho' = r'^T z, sigma' = z^T q, |r'|^2
    // (past the region r and q vanish, and with them every product)
    if constexpr (PAIR) {
      if (!shadow) {
        n2_prim = 0;
#pragma unroll
        for (int i = 0; i < L; ++i) {
          zp[i] = y[i];
          if constexpr (STEP) qp[i] = q[i];
          const cplx<T> r = rr[NF - 1 + i];
          n2_prim += (double)r.re * r.re + (double)r.im * r.im;
        }
        __syncthreads();  // the states in LDS are read
        continue;
      }
    }
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const cplx<T> r = rr[NF - 1 + i], zz = PAIR ? zp[PAIR ? i : 0] : y[i];
      d[0] += (double)r.re * zz.re - (double)r.im * zz.im;
      d[1] += (double)r.re * zz.im + (double)r.im * zz.re;
      if constexpr (STEP) {
        const cplx<T> v = q[i];
        d[2] += (double)v.re * zz.re - (double)v.im * zz.im;
        d[3] += (double)v.re * zz.im + (double)v.im * zz.re;
        if constexpr (PAIR) {  // the mean of q~^T z and q^T z~
          const cplx<T> qq = qp[i], zs = y[i];
          d[2] += (double)qq.re * zs.re - (double)qq.im * zs.im;
          d[3] += (double)qq.re * zs.im + (double)qq.im * zs.re;
        }
      }
      d[4] += (double)r.re * r.re + (double)r.im * r.im;
    }
  } else if constexpr (PAIR) {
    __syncthreads();  // the states in LDS are read
  }
  }
  if constexpr (MODE != ZS_FOLD) {
    if constexpr (PAIR) {
      d[2] *= 0.5;
      d[3] *= 0.5;
    }
    // weight of the mode in the bilinear form
    const int iy = m / A.nx, ix = m - iy * A.nx;
    const double w = (PAIR ? 1.0
                           : ((ix == 0 || 2 * ix == A.nx) ? 1.0 : 0.5) * ((iy == 0 || 2 * iy * A.nx == nxy) ? 1.0 : 0.5)) /
                     nxy;
    constexpr int ND = PAIR ? 6 : 5;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 5; ++k) red[(c * ND + k) * MB + lane] = w * d[k];
    if constexpr (PAIR) red[(c * ND + 5) * MB + lane] = w * n2_prim;
    __syncthreads();
    // the threads of chunk c sum the values c, c + C, ...: chunks in order, then lanes
    for (int k = c; k < ND; k += C) {
      double s = 0;
      for (int cc = 0; cc < C; ++cc) s += red[(cc * ND + k) * MB + lane];
      for (int o = MB / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
      // of a pair, |r|^2 of the shadow goes to its own partials
      const int row = PAIR && k == 4 ? rhs + 1 : rhs, to = k == 5 ? 4 : k;
      if (lane == 0) A.part[((long long)row * A.nmb + mb) * MODAL_PART + to] = s;
    }
  }
}

// S = s_(n-1), T = t_(n-1) from the ring's residuals (and the previous S, T)
// for the right-hand sides whose ring is full; the others are left alone.
template <typename T>
__global__ void __launch_bounds__(256) k_ring_fold(ModeArgsZ<T> A, long long vol) {
  constexpr int NR = ModalRing<T>::n;
  const int rhs = rhs_of(A.active, blockIdx.y);
  const int own = A.pair ? rhs & ~1 : rhs;  // whose scalars
  const int n = A.sc[own].step + 1, b0 = A.sc[own].base;
  if (n - b0 != NR - 1) return;
  zd ct[NR], cs[NR], tp, sp;
  ring_coeffs<NR>(A.ha + (long long)own * NR, A.hb + (long long)own * NR, b0, n, ct, cs, tp, sp);
  cplx<T>* S = A.fold_s + rhs * A.fold_stride;
  cplx<T>* Tv = A.fold_t + rhs * A.fold_stride;
  const cplx<T>* R[NR - 1];
#pragma unroll
  for (int j = 0; j < NR - 1; ++j) R[j] = ring_at<T>(A.ring, (b0 + j) % NR) + (long long)rhs * vol;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < vol; i += (long long)gridDim.x * blockDim.x) {
    cplx<T> s = mk<T>(0, 0), t = mk<T>(0, 0);
    if (b0 > 0) {
      s = cvt<T>(sp) * S[i];
      t = cfma(cvt<T>(tp), S[i], Tv[i]);
    }
#pragma unroll
    for (int j = 0; j < NR - 1; ++j) {
      const cplx<T> r = R[j][i];
      s = cfma(cvt<T>(cs[j]), r, s);
      t = cfma(cvt<T>(ct[j]), r, t);
    }
    S[i] = s;
    Tv[i] = t;
  }
}

// The new base of the folded right-hand sides (after every block of
// k_ring_fold has read the old one).
__global__ void k_ring_rebase(ModalScal* sc, const int* active, int nact, int nr, bool pair) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nact || (pair && i % 2)) return;
  ModalScal& s = sc[rhs_of(active, i)];
  if (s.step + 1 - s.base == nr - 1) s.base = s.step + 1;
}

// No steps since the last replacement.
__global__ void k_modal_drop(ModalScal* sc, const int* active, int nact) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nact) return;
  ModalScal& s = sc[rhs_of(active, i)];
  s.step = -1;
  s.base = 0;
}

// |r|^2 and the breakdown flag of the last mode pass per right-hand side,
// for the host's convergence check.
__global__ void __launch_bounds__(256) k_modal_check(const ModalScal* __restrict__ sc, const double* __restrict__ part,
                                                     int nmb, const int* __restrict__ active, int nact,
                                                     double* __restrict__ rn2, int* __restrict__ flag, bool pair) {
  const int slot = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (slot >= nact) return;  // whole wavefronts
  const int rhs = rhs_of(active, slot);
  double n2 = 0;
  for (int k = lane; k < nmb; k += 64) n2 += part[((long long)rhs * nmb + k) * MODAL_PART + 4];
  for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
  if (lane == 0) {
    rn2[rhs] = n2;
    flag[rhs] = sc[pair ? rhs & ~1 : rhs].flag;
  }
}

// Filter table [energy][3 nf + nf^2][mode] in the iteration precision:
// al_k = -q_(nf-1-k), fb_k, fbb_k, and the state propagator M^L of
// (F(z), F(z-1), ...), formed in FP64.
// The order is a template argument so that the matrices stay in registers
// (12 -> 3.4 us at nf = 2; with a run-time order they were in scratch memory).
template <typename T, int nf>
__global__ void __launch_bounds__(64) k_filter_table(int nE, int nxy, int L, const ModeData* __restrict__ modes,
                                                     cplx<T>* __restrict__ ft) {
  const long long g = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (g >= (long long)nE * nxy) return;
  const int e = (int)(g / nxy), m = (int)(g - (long long)e * nxy);
  const ModeData& md = modes[g];
  cplx<T>* o = ft + (long long)e * (3 * nf + nf * nf) * nxy + m;
  zd M[nf * nf], P[nf * nf], t[nf * nf];
#pragma unroll
  for (int i = 0; i < nf * nf; ++i) M[i] = mk(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < nf; ++k) {
    M[k] = -md.q[nf - 1 - k];
    if (k > 0) M[k * nf + k - 1] = mk(1.0, 0.0);
    o[(long long)k * nxy] = cvt<T>(M[k]);
    o[(long long)(nf + k) * nxy] = cvt<T>(md.fb[k]);
    o[(long long)(2 * nf + k) * nxy] = cvt<T>(md.fbb[k]);
  }
#pragma unroll
  for (int i = 0; i < nf * nf; ++i) P[i] = M[i];
  for (int p = 1; p < L; p *= 2) {  // L is a power of two
#pragma unroll
    for (int i = 0; i < nf; ++i)
#pragma unroll
      for (int j = 0; j < nf; ++j) {
        zd s = mk(0.0, 0.0);
#pragma unroll
        for (int k = 0; k < nf; ++k) s = s + P[i * nf + k] * P[k * nf + j];
        t[i * nf + j] = s;
      }
#pragma unroll
    for (int i = 0; i < nf * nf; ++i) P[i] = t[i];
  }
#pragma unroll
  for (int i = 0; i < nf * nf; ++i) o[(long long)(3 * nf + i) * nxy] = cvt<T>(P[i]);
}

template <typename T> const cplx<T>* twx_of(iobm_ctx c);
template <> const zd* twx_of<double>(iobm_ctx c) { return c->twx_d; }
template <> const zf* twx_of<float>(iobm_ctx c) { return c->twx_f; }
template <typename T> const cplx<T>* twy_of(iobm_ctx c);
template <> const zd* twy_of<double>(iobm_ctx c) { return c->twy_d; }
template <> const zf* twy_of<float>(iobm_ctx c) { return c->twy_f; }

template <typename T, int N, int PPB>
void plane_reg(iobm_ctx c, int mode, const PlaneArgs<T>& A) {
  const dim3 grid((A.nplanes + PPB - 1) / PPB), blk(line_split<T, N>() * N * PPB);
  const size_t sh = mode == PM_VFWD ? (size_t)PPB * A.kb.npad * sizeof(cplx<T>) : 0;  // W of each plane's rhs
#define IOBM_PR(MM) hipLaunchKernelGGL((k_plane_reg<T, N, PPB, MM>), grid, blk, sh, c->stream, A)
  switch (mode) {
    case PM_FULL: IOBM_PR(PM_FULL); break;
    case PM_INV: IOBM_PR(PM_INV); break;
    case PM_VFWD: IOBM_PR(PM_VFWD); break;
    case PM_FWD: IOBM_PR(PM_FWD); break;
    default: IOBM_PR(PM_ACC); break;
  }
#undef IOBM_PR
}

template <int N, int G>
void plane_pair(iobm_ctx c, int mode, const PlaneArgs<float>& A) {
  const dim3 grid((A.nplanes / 2 + G - 1) / G), blk(2 * N * G);
#define IOBM_PP(MM) hipLaunchKernelGGL((k_plane_pair<N, G, MM>), grid, blk, 0, c->stream, A)
  switch (mode) {
    case PM_FULL: IOBM_PP(PM_FULL); break;
    case PM_FWD: IOBM_PP(PM_FWD); break;
    default: IOBM_PP(PM_ACC); break;
  }
#undef IOBM_PP
}

template <typename T>
hipError_t launch_plane(iobm_ctx c, int mode, const PlaneArgs<T>& A) {
  if (A.nplanes <= 0) return hipSuccess;
  if constexpr (sizeof(T) == 4)
    if (A.pair) {
      switch (c->g.nx) {
        case 8: plane_pair<8, 8>(c, mode, A); break;
        case 12: plane_pair<12, 8>(c, mode, A); break;
        case 16: plane_pair<16, 4>(c, mode, A); break;
        case 24: plane_pair<24, 2>(c, mode, A); break;
        case 32: plane_pair<32, 1>(c, mode, A); break;
        default: plane_pair<48, 1>(c, mode, A); break;
      }
      return hipGetLastError();
    }
  if (fft_reg_available<T>(c)) {
    constexpr bool dbl = sizeof(T) == 8;
    switch (c->g.nx) {
      case 8: plane_reg<T, 8, 8>(c, mode, A); break;
      case 12: plane_reg<T, 12, 16>(c, mode, A); break;
      case 16: plane_reg<T, 16, 4>(c, mode, A); break;
      case 24: plane_reg<T, 24, dbl ? 4 : 8>(c, mode, A); break;
      case 32: plane_reg<T, 32, dbl ? 1 : 2>(c, mode, A); break;
      default: plane_reg<T, 48, dbl ? 2 : 1>(c, mode, A); break;
    }
    return hipGetLastError();
  }
  const size_t sh = 2 * (size_t)c->g.nxy * sizeof(cplx<T>) + (8 + 16 * kAdvValues) * sizeof(double) +
                    (mode == PM_VFWD ? A.kb.npad * sizeof(cplx<T>) : 0);
  const size_t tables = (size_t)(c->g.nx + c->g.ny) * sizeof(cplx<T>);
  const bool tw = lds_holds(sh + tables);
#define IOBM_PL1(MM, TW)                                                                                             \
  hipLaunchKernelGGL((k_plane_lds<T, MM, TW>), dim3(A.nplanes), dim3(256), sh + (TW ? tables : 0), c->stream, A, c->plan, \
                     twx_of<T>(c), twy_of<T>(c))
#define IOBM_PL(MM)              \
  do {                           \
    if (tw) IOBM_PL1(MM, true);  \
    else IOBM_PL1(MM, false);    \
  } while (0)
  switch (mode) {
    case PM_FULL: IOBM_PL(PM_FULL); break;
    case PM_INV: IOBM_PL(PM_INV); break;
    case PM_VFWD: IOBM_PL(PM_VFWD); break;
    case PM_FWD: IOBM_PL(PM_FWD); break;
    default: IOBM_PL(PM_ACC); break;
  }
#undef IOBM_PL
#undef IOBM_PL1
  return hipGetLastError();
}

// Modes per block of the mode pass for chunks of L planes: as many as leave
// at most 512 threads.
int zstep_modes(int nz, int L) {
  const int C = (nz + L - 1) / L;
  return C <= 8 ? 64 : (C <= 16 ? 32 : 16);
}

template <typename T>
hipError_t launch_zstep(iobm_ctx c, int mode, const ModeArgsZ<T>& A, int nact) {
  if (nact <= 0) return hipSuccess;
  constexpr int L = kModalChunk;
  const int nf = c->g.nf, MB = zstep_modes(c->g.nz, L);
  // whole wavefronts (the kernel sums across 64 lanes): a chunk past the last
  // plane is empty
  const int cw = 64 / MB, C = ((c->g.nz + L - 1) / L + cw - 1) / cw * cw;
  if (C * MB > 512) return hipErrorInvalidValue;
  const size_t st = (size_t)4 * C * nf * MB * sizeof(cplx<T>), rd = (size_t)C * (A.pair ? 6 : 5) * MB * sizeof(double);
  const size_t sh = st > rd ? st : rd;
  const dim3 grid((A.pair ? nact / 2 : nact) * A.nmb), blk(MB, C);
#define IOBM_Z1(NFF, MM, BB)                                                                             \
  do {                                                                                                   \
    if constexpr (sizeof(T) == 4)                                                                        \
      if (A.pair) {                                                                                      \
        hipLaunchKernelGGL((k_zstep<T, L, NFF, MM, BB, true>), grid, blk, sh, c->stream, A);             \
        break;                                                                                           \
      }                                                                                                  \
    hipLaunchKernelGGL((k_zstep<T, L, NFF, MM, BB, false>), grid, blk, sh, c->stream, A);                \
  } while (0)
#define IOBM_Z2(NFF, BB)                             \
  switch (mode) {                                    \
    case ZS_STEP: IOBM_Z1(NFF, ZS_STEP, BB); break;   \
    case ZS_START: IOBM_Z1(NFF, ZS_START, BB); break; \
    default: IOBM_Z1(NFF, ZS_FOLD, BB); break;        \
  }
#define IOBM_Z3(BB)                    \
  switch (nf) {                        \
    case 1: IOBM_Z2(1, BB); break;     \
    case 2: IOBM_Z2(2, BB); break;     \
    default: IOBM_Z2(3, BB); break;    \
  }
  switch (MB) {
    case 64: IOBM_Z3(64); break;
    case 32: IOBM_Z3(32); break;
    default: IOBM_Z3(16); break;
  }
#undef IOBM_Z3
#undef IOBM_Z2
#undef IOBM_Z1
  return hipGetLastError();
}

}  // namespace

// =================================================================== host ===
int modal_mode_blocks(iobm_ctx c) {
  const int mb = zstep_modes(c->g.nz, kModalChunk);
  return (c->g.nxy + mb - 1) / mb;
}

template <typename T>
hipError_t modal_setup(iobm_ctx c, Modal<T>& M) {
  const long long n = (long long)M.nE * c->g.nxy;
  const dim3 grid((unsigned)((n + 63) / 64)), blk(64);
#define IOBM_FT(NFF) \
  hipLaunchKernelGGL((k_filter_table<T, NFF>), grid, blk, 0, c->stream, M.nE, c->g.nxy, kModalChunk, c->modes_d, M.ft)
  switch (c->g.nf) {
    case 1: IOBM_FT(1); break;
    case 2: IOBM_FT(2); break;
    default: IOBM_FT(3); break;
  }
#undef IOBM_FT
  return hipGetLastError();
}

template <typename T>
static ModeArgsZ<T> mode_args(iobm_ctx c, const Modal<T>& M, const int* active) {
  ModeArgsZ<T> A;
  A.nz = c->g.nz;
  A.nx = c->g.nx;
  A.nxy = c->g.nxy;
  A.nmb = M.nmb;
  A.ndp = M.ndp;
  for (int i = 0; i < ModalRing<T>::n; ++i) A.ring[i] = M.ring[i];
  A.w = M.w;
  A.ft = M.ft;
  A.e_rhs = M.e_rhs;
  A.active = active;
  A.sc = M.sc;
  A.part = M.part;
  A.dpart = M.dpart;
  A.ha = M.ha;
  A.hb = M.hb;
  A.fold_s = M.fold_s;
  A.fold_t = M.fold_t;
  A.fold_stride = M.fold_stride;
  A.pair = M.pair;
  return A;
}

template <typename T>
static PlaneArgs<T> plane_args(iobm_ctx c, const Modal<T>& M, cplx<T>* vec, int nact, const int* active) {
  PlaneArgs<T> A;
  A.nz = c->g.nz;
  A.nplanes = nact * c->g.nz;
  A.nmb = M.nmb;
  A.ndp = M.ndp;
  A.vec = vec;
  A.active = active;
  A.Vd = c->V_d;
  A.Vf = c->V_f;
  A.sc = M.sc;
  A.part = M.part;
  A.dpart = M.dpart;
  A.pair = M.pair;
  return A;
}

template <typename T>
hipError_t modal_start(iobm_ctx c, const Modal<T>& M, int nact, const int* active) {
  if (nact <= 0) return hipSuccess;
  const double stream = (double)nact * c->g.npts * sizeof(cplx<T>);
  int rec = prof_start(c, IOBM_K_FFT_PLANES);
  hipError_t e = launch_plane<T>(c, PM_FWD, plane_args<T>(c, M, M.ring[0], nact, active));
  prof_stop(c, rec, 2.0 * stream);
  if (e != hipSuccess) return e;
  rec = prof_start(c, IOBM_K_ZFILTER);
  e = launch_zstep<T>(c, ZS_START, mode_args<T>(c, M, active), nact);
  prof_stop(c, rec, 2.0 * stream);
  return e;
}

template <typename T>
hipError_t modal_step(iobm_ctx c, const Modal<T>& M, int nact, const int* active, bool fold) {
  if (nact <= 0) return hipSuccess;
  const double stream = (double)nact * c->g.npts * sizeof(cplx<T>);
  PlaneArgs<T> P = plane_args<T>(c, M, M.w, nact, active);
  const ModeArgsZ<T> A = mode_args<T>(c, M, active);
  const bool kb = c->kb.ncen > 0;
  int rec = prof_start(c, kb ? IOBM_K_FFT_PLANES : IOBM_K_FFT_PLANES_UPD);
  hipError_t e = launch_plane<T>(c, kb ? PM_INV : PM_FULL, P);
  prof_stop(c, rec, 2.0 * stream);
  if (e != hipSuccess) return e;
  if (kb) {
    // C = B^T z, W = h^3 D C, and C^T W as one more partial of z^T V z
    e = launch_kb_coeffs<T>(c, M.w, nact, active, M.dpart + 2 * (long long)c->g.nz, 2 * (long long)M.ndp, &P.kb);
    if (e != hipSuccess) return e;
    rec = prof_start(c, IOBM_K_FFT_PLANES_UPD);
    e = launch_plane<T>(c, PM_VFWD, P);
    prof_stop(c, rec, 2.0 * stream);
    if (e != hipSuccess) return e;
  }
  rec = prof_start(c, IOBM_K_ZFILTER);
  e = launch_zstep<T>(c, ZS_STEP, A, nact);
  prof_stop(c, rec, 5.0 * stream);
  if (e != hipSuccess || !fold) return e;
  const long long vol = c->g.npts;
  const unsigned bx = (unsigned)std::min<long long>(256, (vol + 255) / 256);
  hipLaunchKernelGGL(k_ring_fold<T>, dim3(bx, nact), dim3(256), 0, c->stream, A, vol);
  hipLaunchKernelGGL(k_ring_rebase, dim3((nact + 255) / 256), dim3(256), 0, c->stream, M.sc, active, nact,
                     (int)ModalRing<T>::n, M.pair);
  return hipGetLastError();
}

template <typename T>
hipError_t modal_correct(iobm_ctx c, const Modal<T>& M, zd* x, const int* xset, int nact, const int* active,
                         double ring_reads, int nfirst) {
  if (nact <= 0) return hipSuccess;
  const double pts = (double)c->g.npts;
  int rec = prof_start(c, IOBM_K_ZFILTER);
  hipError_t e = launch_zstep<T>(c, ZS_FOLD, mode_args<T>(c, M, active), nact);
  prof_stop(c, rec, (ring_reads + nact) * pts * sizeof(cplx<T>));
  if (e != hipSuccess) return e;
  PlaneArgs<T> P = plane_args<T>(c, M, M.w, nact, active);
  P.x = x;
  P.xset = xset;
  rec = prof_start(c, IOBM_K_ACCUMULATE);
  e = launch_plane<T>(c, PM_ACC, P);
  prof_stop(c, rec, pts * ((double)nact * (sizeof(cplx<T>) + sizeof(zd)) + (double)(nact - nfirst) * sizeof(zd)));
  return e;
}

template <typename T>
hipError_t modal_drop(iobm_ctx c, const Modal<T>& M, int nact, const int* active) {
  if (nact <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_modal_drop, dim3((nact + 255) / 256), dim3(256), 0, c->stream, M.sc, active, nact);
  return hipGetLastError();
}

template <typename T>
hipError_t modal_check(iobm_ctx c, const Modal<T>& M, int nact, const int* active, double* rn2, int* flag) {
  if (nact <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_modal_check, dim3((nact + 3) / 4), dim3(256), 0, c->stream, M.sc, M.part, M.nmb, active, nact,
                     rn2, flag, M.pair);
  return hipGetLastError();
}

#define IOBM_MODAL_INST(T)                                                                                       \
  template hipError_t modal_setup<T>(iobm_ctx, Modal<T>&);                                                       \
  template hipError_t modal_start<T>(iobm_ctx, const Modal<T>&, int, const int*);                                \
  template hipError_t modal_step<T>(iobm_ctx, const Modal<T>&, int, const int*, bool);                           \
  template hipError_t modal_correct<T>(iobm_ctx, const Modal<T>&, zd*, const int*, int, const int*, double, int); \
  template hipError_t modal_drop<T>(iobm_ctx, const Modal<T>&, int, const int*);                                  \
  template hipError_t modal_check<T>(iobm_ctx, const Modal<T>&, int, const int*, double*, int*);
IOBM_MODAL_INST(float)
IOBM_MODAL_INST(double)
#undef IOBM_MODAL_INST
