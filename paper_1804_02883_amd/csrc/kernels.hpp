// HIP kernels of the hybrid LB/EPD step (gfx950).
//
// Layout everywhere: structure-of-arrays planes, row-major [y][x] with x
// contiguous, nx x ny sites per plane, plane stride `plane` elements.
// T is the storage/arithmetic type (float or double); all grid-wide sums are
// accumulated in double and finished by the last block to arrive, in a fixed
// order, so results are deterministic.
#pragma once
#include "fft.hpp"

namespace epdlb {

// Device scalars shared between kernels (double).
enum Scal : int {
  kMeanA = 0, kMeanB = 1, kMeanS = 2,  // site means of the current omega planes
  kQS = 3, kGaugeS = 4,                 // Q_S and the constant it was computed with
  kQPf = 5, kQPb = 6,                   // Q_P from the forward and backward chains
  kGext = 7,                            // reverse-Poiseuille force amplitude, lattice units
  // surrogate mode (maxima of non-negative values, updated atomically)
  kNnResid = 8,                         // max |sum Phi - 1| of surrogate steps since the last check
  kResidEx = 9,                         // max |sum Phi - 1| of the last exact step
  kNnErrLast = 10,                      // max |Phi_NN - Phi_exact| (A, B) at the last exact step
  kNnErr = 11,                          // the same, maximum over all exact steps
  kNnErrUse = 12,                       // the same, over exact steps that ended surrogate steps
  kNumScal = 13
};

// ---------------------------------------------------------------------------
// XCD-aware tile order.  Workgroups are handed to the 8 XCDs of an MI355X
// round-robin by linear id, and each XCD has its own L2.  Remapping so that
// XCD k processes the k-th contiguous range of logical tiles keeps
// neighbouring tiles (which share cache lines and halos) in one L2.
// ---------------------------------------------------------------------------
constexpr int kNumXcd = 8;

// Replicas of one grid shape share a launch: replica z's planes, tables and
// scalars sit `rs` bytes after replica z-1's (blockIdx.z = z).
template <class X>
__device__ __forceinline__ X* sh(X* p, long off) {
  return (X*)((const char*)p + off);
}
__device__ __forceinline__ int xcd_tile(int linear, int total) {
  if (total % kNumXcd) return linear;
  return (linear % kNumXcd) * (total / kNumXcd) + linear / kNumXcd;
}

// ---------------------------------------------------------------------------
// Deterministic grid reduction: per-block sums -> partials -> last block.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Reduces NV per-thread values over the block; thread 0 gets the sums.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* red /*[16*NV]*/) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) red[wid * NV + i] = v[i];
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += red[w * NV + i];
      v[i] = s;
    }
  }
}

// Writes this block's NV sums to partials[slot*NV + i].  A later kernel
// (or a later stage of the consumer) adds the partials in slot order, so the
// grid-wide sums are deterministic and need no device-scope fences here.
template <int NV>
__device__ __forceinline__ void block_partial(double (&v)[NV], double* red, double* partials, int slot) {
  block_sum<NV>(v, red);
  if (threadIdx.x == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) partials[slot * NV + i] = v[i];
}

// Sums nslots partials of NV values each, in slot order, over one block.
// Each thread loads four of its slots at a time before adding them in order,
// so the loads of a batch are in flight together.
template <int NV>
__device__ __forceinline__ void sum_partials(const double* partials, int nslots, double (&acc)[NV],
                                             double* red) {
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  const int step = blockDim.x;
  for (int s0 = threadIdx.x; s0 < nslots; s0 += 4 * step) {
    double v[4][NV];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int s = s0 + k * step;
#pragma unroll
      for (int i = 0; i < NV; ++i) v[k][i] = s < nslots ? partials[s * NV + i] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (s0 + k * step < nslots)
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] += v[k][i];
  }
  block_sum<NV>(acc, red);
}

// The scalars of the field statistics from their sums.
__device__ __forceinline__ void finish_stats(double* scal, const double (&acc)[4], long n, double dA) {
  scal[kGaugeS] = scal[kMeanS];  // the constant the exponentials were taken with
  scal[kMeanA] = acc[0] / double(n);
  scal[kMeanB] = acc[1] / double(n);
  scal[kMeanS] = acc[2] / double(n);
  scal[kQS] = acc[3] * dA;
}

// Finishes the field statistics: partials of (sum w_A, sum w_B, sum w_S,
// sum exp(-(w_S - gauge))) -> means, Q_S and the gauge it used.  One block.
inline __global__ void __launch_bounds__(256) k_finish_stats(const double* partials, int nslots, double* scal,
                                                      long n, double dA, long rs) {
  __shared__ double red[16 * 4];
  partials = sh(partials, long(blockIdx.z) * rs);
  scal = sh(scal, long(blockIdx.z) * rs);
  double acc[4];
  sum_partials<4>(partials, nslots, acc, red);
  if (threadIdx.x == 0) finish_stats(scal, acc, n, dA);
}

// ---------------------------------------------------------------------------
// Chain propagators.  K = K_x K_y = K_y K_x, so each contour step applies its
// two one-dimensional convolutions in alternating order: even steps x then y,
// odd steps y then x.  The last convolution of step a and the first one of
// step a+1 then share an orientation and run in ONE kernel with q_{a+1}
// stored in between: N + 1 launches for N contour steps, both chains per
// launch (blockIdx.y = chain; 0 forward, 1 backward).
// ---------------------------------------------------------------------------
template <typename T> struct PropArgs {
  const T* wA;            // first pass
  const T* wB;
  T* EA;                  // first pass: exp(-(w_A - c_A)/2), written for the later ones
  T* EB;                  // exp(-(w_B - c_B)/2)
  T* EJ;                  // the same of the junction segment (A fraction fracJ); nullptr: none
  const T* E[2][2];       // factor plane of chain c at step a (+0/+1): EA, EB or EJ
  const double* scal;     // kMeanA, kMeanB: gauge constants
  T* q[2];                // q_1..q_N of chain c at q[c] + (j-1)*plane
  T* tmp;                 // 2 planes (per chain): data between the two convolutions of a step
  const T* mult_x;        // exp(-R_G^2 kx^2 ds)/nx in FFT order
  const T* mult_y;        // exp(-R_G^2 ky^2 ds)/ny
  const T2<T>* tw_x;      // exp(-2 pi i e/nx)
  const T2<T>* tw_y;
  int nx, ny;
  long plane;
  int a;                  // contour step finished by the first convolution
  int second;             // then x E(step a+1), convolution 2, store tmp
  int last;               // partial sums of q_N for Q_P
  T frac[2];              // first pass: A fraction of chain c's segment at step 0
  T fracJ;
  bool plain;             // convolutions set no constant aside (see convolve)
  double* partials;       // last: per-block sums of q_N, chain c at [c*gridDim.x]
  int nf;                 // transforms per block (row kernels)
  int nrep;               // replicas in the launch (gridDim.z)
  long rs;                // replica stride in bytes
  __device__ void shift(long o) {
    wA = sh(wA, o), wB = sh(wB, o), EA = sh(EA, o), EB = sh(EB, o), scal = sh(scal, o);
    if (EJ) EJ = sh(EJ, o);
    for (int c = 0; c < 2; ++c)
      for (int k = 0; k < 2; ++k) E[c][k] = sh(E[c][k], o);
    q[0] = sh(q[0], o), q[1] = sh(q[1], o), tmp = sh(tmp, o), mult_x = sh(mult_x, o);
    mult_y = sh(mult_y, o), tw_x = sh(tw_x, o), tw_y = sh(tw_y, o);
    partials = sh(partials, o);
  }
};


template <typename T>
__device__ __forceinline__ T boltz(T wa, T wb, T a, T ca, T cb) {
  const T x = a * (wa - ca) + (T(1) - a) * (wb - cb);
  return exp(T(-0.5) * x);
}

// Element at a 32-bit byte offset (a plane is below 4 GiB), so that accesses
// take a scalar base and one offset register.
template <typename X> __device__ __forceinline__ X ld(const void* base, unsigned off) {
  return *reinterpret_cast<const X*>(static_cast<const char*>(base) + off);
}
template <typename X> __device__ __forceinline__ void st(void* base, unsigned off, X v) {
  *reinterpret_cast<X*>(static_cast<char*>(base) + off) = v;
}

template <int R, typename T> __device__ __forceinline__ void add_const(T* re, T* im, T v) {
#pragma unroll
  for (int m = 0; m < R; ++m) {
    re[m] += v;
    im[m] += v;
  }
}

// Convolution with the real, even multiplier g in the lane layout.  The kernel's
// sum is 1 (g = 1/L at k = 0, exact in binary), so a constant passes unchanged, and
// with BASE what is transformed is the difference from 1: the transforms' rounding
// then scales with the fluctuation of q, not with q itself.  The mean of q is at
// least 1 (Jensen, the potentials' means taken out), so the sum of squares that the
// rounding scales with never grows.  Velocity after 4 steps at 1024 x 512, N = 64,
// FP32, against 64 bits, 8 seeds: 1.2e-6 to 2.1e-6 without, 7.6e-7 to 9.0e-7 with,
// at no measurable cost.  Without: the plain convolution.
template <typename T, int L, int R, bool BASE, class V>
__device__ __forceinline__ void convolve(T* re, T* im, int j, const V& lds, const Twiddles<T, L, R>& twf,
                                         const Twiddles<T, L, R>& twi, const T* g) {
  if constexpr (BASE) add_const<R>(re, im, T(-1));
  fft_forward<T, L, R>(re, im, j, lds, twf);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    re[m] *= g[m];
    im[m] *= g[m];
  }
  fft_inverse<T, L, R>(re, im, j, lds, twi);
  if constexpr (BASE) add_const<R>(re, im, T(1));
}

// Whether a column pass changes its lane mapping (see ColMap).  The plain passes
// keep one mapping, in which the compiler contracts products and sums as it did
// when their bits were set.
template <int L, int R, bool BASE> constexpr bool col_remap() { return BASE && col_mapped<L, R>(); }

// The same over the columns of a block (ColMap); g in the wave mapping.
template <typename T, int L, int R, bool BASE>
__device__ __forceinline__ void convolve_cols(T* re, T* im, const ColMap<T, L, R>& c, const Twiddles<T, L, R>& twf,
                                              const Twiddles<T, L, R>& twi, const T* g) {
  if constexpr (BASE) add_const<R>(re, im, T(-1));
  col_forward<T, L, R, 0>(re, im, c, twf);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    re[m] *= g[m];
    im[m] *= g[m];
  }
  col_inverse<T, L, R, 0>(re, im, c, twi);
  if constexpr (BASE) add_const<R>(re, im, T(1));
}

// x-oriented kernel: rows 2rp and 2rp+1 of one chain packed as one complex
// row (the multiplier is real and even, so the two real rows stay apart).
//
// The passes are short and latency-bound, so the code path of a launch is kept
// short and straight: the first pass is an instantiation of its own, the
// factors come from one plane per step (the junction segment has one too),
// every load is unconditional (a transform past the end repeats the last one
// and stores nothing).  With a branch per element that picked the factor's
// plane or evaluated the junction's, and 64-bit addresses (2,360 instructions
// in the 256-row pass), a pass took, in alternation with the other kind: 256 x 256
// 5.5 us, now 4.5; 512 x 512 8.0, now 6.6; 1024 x 512 9.8, now 9.3; 128 x 128 5.1,
// now 3.9; FP64 256 x 128 6.0, now 4.5 (same shapes, same results bit for bit).
template <typename T, int L, int R, bool FIRST, bool BASE>
__global__ void __launch_bounds__(512) k_prop_row(PropArgs<T> P) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, true, 1>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[16 * 1];
  const int f = threadIdx.x / TL, j = threadIdx.x % TL;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  P.shift(long(blockIdx.z) * P.rs);
  const int c = blockIdx.y;
  const int want = blockIdx.x * P.nf + f, rp = min(want, P.ny / 2 - 1);
  const bool active = want == rp;
  const unsigned r0 = (unsigned(2 * rp) * L + j) * sizeof(T), r1 = r0 + L * sizeof(T);
  constexpr unsigned kStep = TL * sizeof(T);  // element j + TL m lies m steps on
  T* tmp = P.tmp + c * P.plane;
  T re[R], im[R], ea[R], eb[R];
  if constexpr (FIRST) {
    // the factors from the potentials; the factor planes of the later passes:
    // A's from the forward chain's blocks, B's from the backward chain's
    const T ca = T(P.scal[kMeanA]), cb = T(P.scal[kMeanB]);
    const T fr0 = c == 0 ? P.frac[0] : P.frac[1];
    T* Ep = c == 0 ? P.EA : P.EB;
    const T pure = c == 0 ? T(1) : T(0);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const unsigned o0 = r0 + m * kStep, o1 = r1 + m * kStep;
      const T wa0 = ld<T>(P.wA, o0), wb0 = ld<T>(P.wB, o0), wa1 = ld<T>(P.wA, o1), wb1 = ld<T>(P.wB, o1);
      const T p0 = boltz(wa0, wb0, pure, ca, cb), p1 = boltz(wa1, wb1, pure, ca, cb);
      if (active) {
        st(Ep, o0, p0);
        st(Ep, o1, p1);
        if (c == 0 && P.EJ) {
          st(P.EJ, o0, boltz(wa0, wb0, P.fracJ, ca, cb));
          st(P.EJ, o1, boltz(wa1, wb1, P.fracJ, ca, cb));
        }
      }
      re[m] = fr0 == pure ? p0 : boltz(wa0, wb0, fr0, ca, cb);
      im[m] = fr0 == pure ? p1 : boltz(wa1, wb1, fr0, ca, cb);
    }
  } else {
    const T* E0 = c == 0 ? P.E[0][0] : P.E[1][0];
#pragma unroll
    for (int m = 0; m < R; ++m) {
      re[m] = ld<T>(tmp, r0 + m * kStep);
      im[m] = ld<T>(tmp, r1 + m * kStep);
    }
#pragma unroll
    for (int m = 0; m < R; ++m) {
      ea[m] = ld<T>(E0, r0 + m * kStep);
      eb[m] = ld<T>(E0, r1 + m * kStep);
    }
  }
  Twiddles<T, L, R> twf, twi;
  load_fwd_twiddles(twf, j, P.tw_x);
  load_inv_twiddles(twi, j, P.tw_x);
  T g[R];
#pragma unroll
  for (int m = 0; m < R; ++m) g[m] = P.mult_x[j + TL * m];
  convolve<T, L, R, BASE>(re, im, j, lds, twf, twi, g);
  double qsum = 0.0;
  if constexpr (!FIRST) {
    T* qo = (c == 0 ? P.q[0] : P.q[1]) + long(P.a) * P.plane;
#pragma unroll
    for (int m = 0; m < R; ++m) {
      re[m] *= ea[m];
      im[m] *= eb[m];
      qsum += double(re[m]) + double(im[m]);
    }
    if (active)
#pragma unroll
      for (int m = 0; m < R; ++m) {
        st(qo, r0 + m * kStep, re[m]);
        st(qo, r1 + m * kStep, im[m]);
      }
    if (P.second) {
      const T* E0 = c == 0 ? P.E[0][0] : P.E[1][0];
      const T* E1 = c == 0 ? P.E[0][1] : P.E[1][1];
      if (E1 != E0) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
          ea[m] = ld<T>(E1, r0 + m * kStep);
          eb[m] = ld<T>(E1, r1 + m * kStep);
        }
      }
#pragma unroll
      for (int m = 0; m < R; ++m) {
        re[m] *= ea[m];
        im[m] *= eb[m];
      }
      convolve<T, L, R, BASE>(re, im, j, lds, twf, twi, g);
    }
  }
  if ((FIRST || P.second) && active) {
#pragma unroll
    for (int m = 0; m < R; ++m) {
      st(tmp, r0 + m * kStep, re[m]);
      st(tmp, r1 + m * kStep, im[m]);
    }
  }
  if (!FIRST && P.last) {
    double v[1] = {active ? qsum : 0.0};
    block_partial<1>(v, red, P.partials + c * gridDim.x, blockIdx.x);
  }
}

// y-oriented kernel: columns 2cp and 2cp+1 packed as one complex column; NF
// transforms per block interleaved lane by lane so that each global access
// of a wavefront covers NF consecutive column pairs.
template <typename T, int L, int R, int NF, bool BASE>
__global__ void __launch_bounds__(512) k_prop_col(PropArgs<T> P) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, false, NF>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[16 * 1];
  const int f = threadIdx.x % NF, j = threadIdx.x / NF;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  constexpr bool kMap = col_remap<L, R, BASE>();
  const int jw = kMap ? int(threadIdx.x) % TL : j;  // the lane within the transform between the exchanges
  P.shift(long(blockIdx.z) * P.rs);
  const int lt = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int c = lt / gridDim.x, tile = lt % gridDim.x;
  const int want = tile * NF + f, cp = min(want, P.nx / 2 - 1);
  const bool active = want == cp;
  const unsigned o0 = (unsigned(j) * P.nx + 2 * cp) * sizeof(T), step = unsigned(TL) * P.nx * sizeof(T);
  T* tmp = P.tmp + c * P.plane;
  const T* E0 = c == 0 ? P.E[0][0] : P.E[1][0];
  T re[R], im[R];
  T2<T> e[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const T2<T> v = ld<T2<T>>(tmp, o0 + m * step);
    re[m] = v.x;
    im[m] = v.y;
  }
#pragma unroll
  for (int m = 0; m < R; ++m) e[m] = ld<T2<T>>(E0, o0 + m * step);
  Twiddles<T, L, R> twf, twi;
  load_fwd_twiddles(twf, jw, P.tw_y);
  if constexpr (kMap)
    load_col_inv_twiddles(twi, jw, j, P.tw_y);
  else
    load_inv_twiddles(twi, j, P.tw_y);
  T g[R];
#pragma unroll
  for (int m = 0; m < R; ++m) g[m] = P.mult_y[jw + TL * m];
  auto conv = [&] {
    if constexpr (kMap) {
      T2<T>* buf = reinterpret_cast<T2<T>*>(smem_raw);
      const ColMap<T, L, R> cm{{buf, f}, {buf, int(threadIdx.x) / TL}, j, jw};
      convolve_cols<T, L, R, BASE>(re, im, cm, twf, twi, g);
    } else {
      convolve<T, L, R, BASE>(re, im, j, lds, twf, twi, g);
    }
  };
  conv();
  double qsum = 0.0;
  T* qo = (c == 0 ? P.q[0] : P.q[1]) + long(P.a) * P.plane;
#pragma unroll
  for (int m = 0; m < R; ++m) {
    re[m] *= e[m].x;
    im[m] *= e[m].y;
    qsum += double(re[m]) + double(im[m]);
  }
  auto store = [&](T* p) {
#pragma unroll
    for (int m = 0; m < R; ++m) {
      T2<T> o;
      o.x = re[m];
      o.y = im[m];
      st(p, o0 + m * step, o);
    }
  };
  if (active) store(qo);
  if (P.second) {
    const T* E1 = c == 0 ? P.E[0][1] : P.E[1][1];
    if (E1 != E0) {
#pragma unroll
      for (int m = 0; m < R; ++m) e[m] = ld<T2<T>>(E1, o0 + m * step);
    }
#pragma unroll
    for (int m = 0; m < R; ++m) {
      re[m] *= e[m].x;
      im[m] *= e[m].y;
    }
    conv();
    if (active) store(tmp);
  }
  if (P.last) {
    double v[1] = {active ? qsum : 0.0};
    block_partial<1>(v, red, P.partials + c * gridDim.x, tile);
  }
}

// ---------------------------------------------------------------------------
// Chain propagators of a small grid in one launch: one workgroup per chain
// (blockIdx.x) and replica keeps its plane on one CU for all N contour steps.
// At these sizes a convolution is cheapest as a product with the circulant
// matrix of the kernel's real-space values (c_x, c_y): MFMA in the planes' own
// precision, no exchanges.  Wave w owns the 16 columns from 16 w, all rows:
//   x:  D = Q C_x, rows of Q from LDS (16-byte reads), C_x in registers;
//   y:  C_y D, where the output layout of the first product is the operand
//       layout of the second up to the order of the summed rows, which the
//       registers of C_y follow: no data moves between the two;
// then x E, store q_{a+1}, x E of the next step, back to LDS (two buffers, one
// barrier per step).  A circulant matrix takes L/4 registers of a wave: the
// element at (row, column) depends on their difference only.
// What bounds it: the matrix pipes of one CU (64 x 64 FP32: 128 MFMAs of 32
// cycles per wave and step, 1.7 of the 2.8 us measured; 32 x 32 FP64 1.8 us),
// where a launch per step took 4.1-5.7 us whatever the size.
// ---------------------------------------------------------------------------
template <typename T> struct Mfma16;
template <> struct Mfma16<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  typedef float lds4 __attribute__((ext_vector_type(4), aligned(16)));  // four values of a row, as they lie in LDS
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of register i in lane group g (16 lanes)
  static __device__ __forceinline__ int row(int g, int i) { return 4 * g + i; }
};
template <> struct Mfma16<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  typedef double lds4 __attribute__((ext_vector_type(4), aligned(16)));  // two 16-byte reads (acc asks for 32-byte alignment)
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int i) { return 4 * i + g; }
};

template <typename T> struct ResArgs {
  const T* wA;
  const T* wB;
  const double* scal;  // kMeanA, kMeanB
  T* q[2];             // q_1..q_N of chain c
  const T* cx;         // kernel of the x convolution at distance 0..nx-1
  const T* cy;
  double* partials;    // sum of q_N of chain c at [c]
  long plane;
  int N;
  double fAN;          // f_A N: segment j has A fraction clip(f_A N - j, 0, 1)
  // nstat > 0: the field statistics of k_advect_update are still partial sums
  // (at most 64 slots here, so that the sums are k_finish_stats' bit for bit);
  // both workgroups add them, chain 0's writes the scalars
  const double* stat;
  int nstat;
  double* scal_out;
  double dA;
  long rs;
  __device__ void shift(long o) {
    wA = sh(wA, o), wB = sh(wB, o), scal = sh(scal, o), q[0] = sh(q[0], o), q[1] = sh(q[1], o);
    cx = sh(cx, o), cy = sh(cy, o), partials = sh(partials, o), stat = sh(stat, o), scal_out = sh(scal_out, o);
  }
};

template <typename T, int LX, int LY>
__global__ void __launch_bounds__(4 * LX) k_prop_res(ResArgs<T> P) {
  using M = Mfma16<T>;
  using A4 = typename M::acc;
  constexpr int KX = LX / 16, KY = LY / 16;
  constexpr int S = LX + (sizeof(T) == 4 ? 4 : 2);  // row stride: 16 rows' 16-byte reads on distinct banks
  using X4 = typename M::lds4;
  static_assert(alignof(X4) == 16 && S * sizeof(T) % alignof(X4) == 0, "rows start at multiples of the reads' alignment");
  __shared__ __attribute__((aligned(16))) T buf[2][LY * S];
  __shared__ double red[16 * 4];
  __shared__ double mean_s[2];
  P.shift(long(blockIdx.z) * P.rs);
  const int c = blockIdx.x;
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int x0 = (threadIdx.x >> 6) * 16;
  if (P.nstat > 0) {
    double acc[4];
    sum_partials<4>(P.stat, P.nstat, acc, red);
    if (threadIdx.x == 0) {
      mean_s[0] = acc[0] / double(P.plane);
      mean_s[1] = acc[1] / double(P.plane);
      if (c == 0) finish_stats(P.scal_out, acc, P.plane, P.dA);
    }
  } else if (threadIdx.x == 0) {
    mean_s[0] = P.scal[kMeanA];
    mean_s[1] = P.scal[kMeanB];
  }
  __syncthreads();
  const T ca = T(mean_s[0]), cb = T(mean_s[1]);
  T cx[KX][4], cy[KY][4];
#pragma unroll
  for (int k = 0; k < KX; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) cx[k][i] = P.cx[(x0 + n - (16 * k + 4 * g + i)) & (LX - 1)];
#pragma unroll
  for (int k = 0; k < KY; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) cy[k][i] = P.cy[(16 * k + n - M::row(g, i)) & (LY - 1)];
  // this lane's sites: column x0 + n, rows 16 m + row(g, i)
  auto site = [&](int m, int i) { return (16 * m + M::row(g, i)) * LX + x0 + n; };
  T ea[KY][4], eb[KY][4];
#pragma unroll
  for (int m = 0; m < KY; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T wa = P.wA[site(m, i)], wb = P.wB[site(m, i)];
      ea[m][i] = boltz(wa, wb, T(1), ca, cb);
      eb[m][i] = boltz(wa, wb, T(0), ca, cb);
    }
  auto frac = [&](int step) {
    const double v = P.fAN - double(c == 0 ? step : P.N - 1 - step);
    return T(v < 0.0 ? 0.0 : (v > 1.0 ? 1.0 : v));
  };
  auto times_e = [&](A4 (&v)[KY], T fr) {
#pragma unroll
    for (int m = 0; m < KY; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (fr == T(1)) v[m][i] *= ea[m][i];
        else if (fr == T(0)) v[m][i] *= eb[m][i];
        else v[m][i] *= boltz(P.wA[site(m, i)], P.wB[site(m, i)], fr, ca, cb);
      }
  };
  // the products act on the difference from 1, which passes a convolution unchanged (see convolve)
  auto to_lds = [&](T* b, const A4 (&v)[KY]) {
#pragma unroll
    for (int m = 0; m < KY; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) b[(16 * m + M::row(g, i)) * S + x0 + n] = v[m][i] - T(1);
  };
  A4 v[KY];
#pragma unroll
  for (int m = 0; m < KY; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) v[m][i] = T(1);
  times_e(v, frac(0));
  to_lds(buf[0], v);
  double qsum = 0.0;
  for (int s = 0; s < P.N; ++s) {
    __syncthreads();
    const T* b = buf[s & 1];
    // the KY products of a step of the sum are independent: their MFMAs go back to back
    A4 d[KY];
#pragma unroll
    for (int m = 0; m < KY; ++m) d[m] = A4{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int k = 0; k < KX; ++k) {
      A4 a[KY];
#pragma unroll
      for (int m = 0; m < KY; ++m) a[m] = *reinterpret_cast<const X4*>(b + (16 * m + n) * S + 16 * k + 4 * g);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < KY; ++m) d[m] = M::mma(a[m][i], cx[k][i], d[m]);
    }
#pragma unroll
    for (int m = 0; m < KY; ++m) v[m] = A4{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int k = 0; k < KY; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < KY; ++m) v[m] = M::mma(cy[(m - k + KY) % KY][i], d[k][i], v[m]);
#pragma unroll
    for (int m = 0; m < KY; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[m][i] += T(1);
    const T fr = frac(s);
    times_e(v, fr);
    T* qo = (c == 0 ? P.q[0] : P.q[1]) + long(s) * P.plane;
#pragma unroll
    for (int m = 0; m < KY; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) qo[site(m, i)] = v[m][i];
    if (s + 1 < P.N) {
      times_e(v, frac(s + 1));
      to_lds(buf[(s + 1) & 1], v);
    } else {
#pragma unroll
      for (int m = 0; m < KY; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) qsum += double(v[m][i]);
    }
  }
  double r[1] = {qsum};
  block_partial<1>(r, red, P.partials, c);
}

// ---------------------------------------------------------------------------
// Densities (contour integrals, solvent) and S = sum_I Phi_I/D_I - S~.
// ---------------------------------------------------------------------------
template <typename T> struct DensArgs {
  const double* qpart;  // per-block sums of q_N from the last column pass, 2 chains
  int nqpart;           // blocks per chain
  double dA;
  double* scal_out;     // scal: receives Q_P (both chains)
  const T* q[2];
  const T* wS;
  const T* stilde;
  T* phi;        // 3 planes
  T* S;
  const double* scal;
  const T* wnA;  // node weights, N+1 each
  const T* wnB;
  long n;        // sites
  int N;
  double V, phiP, phiSbar, invDA, invDB, invDS;
  int nrep;
  long rs;
  __device__ void shift(long o) {
    qpart = sh(qpart, o), scal_out = sh(scal_out, o), q[0] = sh(q[0], o), q[1] = sh(q[1], o);
    wS = sh(wS, o), stilde = sh(stilde, o), phi = sh(phi, o), scal = sh(scal, o);
    wnA = sh(wnA, o), wnB = sh(wnB, o);
    if (S) S = sh(S, o);
  }
};

template <typename T>
__global__ void __launch_bounds__(256) k_density(DensArgs<T> P) {
  __shared__ double red[16 * 2];
  __shared__ double qp_s;
  P.shift(long(blockIdx.z) * P.rs);
  {
    // Q_P from the column-pass partials, in fixed order (same in every block)
    double acc[2];
    double tmp[2] = {0.0, 0.0};
    for (int s = threadIdx.x; s < P.nqpart; s += blockDim.x) {
      tmp[0] += P.qpart[s];
      tmp[1] += P.qpart[P.nqpart + s];
    }
    acc[0] = tmp[0];
    acc[1] = tmp[1];
    block_sum<2>(acc, red);
    if (threadIdx.x == 0) {
      qp_s = acc[0] * P.dA;
      if (blockIdx.x == 0) {
        P.scal_out[kQPf] = acc[0] * P.dA;
        P.scal_out[kQPb] = acc[1] * P.dA;
      }
    }
    __syncthreads();
  }
  const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= P.n) return;
  const int N = P.N;
  T sA = T(0), sB = T(0);
  // node 0: q_0 = 1, node N: q'_0 = 1
  {
    const T prod = P.q[1][long(N - 1) * P.n + i];
    sA += P.wnA[0] * prod;
    sB += P.wnB[0] * prod;
  }
  // eight nodes' loads in flight: where the grid is small a load's latency per
  // node is what the kernel takes
  for (int j0 = 1; j0 < N; j0 += 8) {
    T f[8], b[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = min(j0 + k, N - 1);
      f[k] = P.q[0][long(j - 1) * P.n + i];
      b[k] = P.q[1][long(N - j - 1) * P.n + i];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = j0 + k;
      if (j < N) {
        const T prod = f[k] * b[k];
        sA += P.wnA[j] * prod;
        sB += P.wnB[j] * prod;
      }
    }
  }
  {
    const T prod = P.q[0][long(N - 1) * P.n + i];
    sA += P.wnA[N] * prod;
    sB += P.wnB[N] * prod;
  }
  const T cP = T(P.V * P.phiP / qp_s);
  const T cS = T(P.V * P.phiSbar / P.scal[kQS]);
  const T pA = cP * sA, pB = cP * sB;
  const T pS = cS * exp(-(P.wS[i] - T(P.scal[kGaugeS])));
  P.phi[i] = pA;
  P.phi[P.n + i] = pB;
  P.phi[2 * P.n + i] = pS;
  if (P.S) P.S[i] = pA * T(P.invDA) + pB * T(P.invDB) + pS * T(P.invDS) - P.stilde[i];
}

// ---------------------------------------------------------------------------
// Site means of omega and Q_S (used at seeding and after host uploads).
// ---------------------------------------------------------------------------
template <typename T> struct StatArgs {
  const T* w;   // 3 planes
  long n;
  double* scal;
  double* partials;
  int nrep;
  long rs;
  __device__ void shift(long o) { w = sh(w, o), scal = sh(scal, o), partials = sh(partials, o); }
};

template <typename T>
__global__ void __launch_bounds__(256) k_field_stats(StatArgs<T> P) {
  __shared__ double red[16 * 4];
  P.shift(long(blockIdx.z) * P.rs);
  const double cS = P.scal[kMeanS];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (long i = long(blockIdx.x) * blockDim.x + threadIdx.x; i < P.n; i += long(gridDim.x) * blockDim.x) {
    v[0] += double(P.w[i]);
    v[1] += double(P.w[P.n + i]);
    const T ws = P.w[2 * P.n + i];
    v[2] += double(ws);
    v[3] += double(exp(-(ws - T(cS))));
  }
  block_partial<4>(v, red, P.partials, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Advection (donor cell) + chemical potential + EPD field update, fused.
// Tile TX x TY outputs; inputs staged with a 2-site halo in LDS.
// ---------------------------------------------------------------------------
constexpr int kTX = 32, kTY = 8;
constexpr int kHX = kTX + 4, kHY = kTY + 4;   // input region (halo 2)
constexpr int kMX = kTX + 2, kMY = kTY + 2;   // mu region (halo 1)

template <typename T> struct UpdArgs {
  const T* phi;    // 3 planes Phi^n
  const T* w;      // 3 planes omega^n
  const T* u;      // 2 planes u^{n-1} (lattice units)
  T* wout;         // 3 planes omega^{n+1}
  T* stilde;       // sum_I Phi~_I / D_I
  const double* scal;
  double* partials;
  int nx, ny;
  long n;
  T chi[3][3];
  T kappa;
  T coef[3];       // D_I dt / dx^2
  T invD[3];
  int advect;      // 0: no flow coupling
  int nrep;
  long rs;
  __device__ void shift(long o) {
    phi = sh(phi, o), w = sh(w, o), u = sh(u, o), wout = sh(wout, o), stilde = sh(stilde, o);
    scal = sh(scal, o), partials = sh(partials, o);
  }
};

// One Euler-forward convection step at LDS position (lx, ly) of a tile holding
// phi[3], omega[3], ux, uy: donor-cell flux form for Phi (face velocity the
// mean of the two cell velocities, upwind cell by its sign), upwind form for
// the auxiliary convection of omega (App. C, first comment).
template <typename T>
__device__ __forceinline__ void advect_site(const T (&sIn)[8][kHY][kHX], int lx, int ly, T (&pt)[3], T (&wt)[3]) {
  const T uxc = sIn[6][ly][lx], uyc = sIn[7][ly][lx];
  // face velocities
  const T uxe = T(0.5) * (uxc + sIn[6][ly][lx + 1]);
  const T uxw = T(0.5) * (sIn[6][ly][lx - 1] + uxc);
  const T uyn = T(0.5) * (uyc + sIn[7][ly + 1][lx]);
  const T uys = T(0.5) * (sIn[7][ly - 1][lx] + uyc);
#pragma unroll
  for (int I = 0; I < 3; ++I) {
    const T c = sIn[I][ly][lx];
    const T Je = uxe >= T(0) ? uxe * c : uxe * sIn[I][ly][lx + 1];
    const T Jw = uxw >= T(0) ? uxw * sIn[I][ly][lx - 1] : uxw * c;
    const T Jn = uyn >= T(0) ? uyn * c : uyn * sIn[I][ly + 1][lx];
    const T Js = uys >= T(0) ? uys * sIn[I][ly - 1][lx] : uys * c;
    pt[I] = c - (Je - Jw) - (Jn - Js);
    const T w = sIn[3 + I][ly][lx];
    const T upx = uxc > T(0) ? uxc : T(0), umx = uxc < T(0) ? uxc : T(0);
    const T upy = uyc > T(0) ? uyc : T(0), umy = uyc < T(0) ? uyc : T(0);
    wt[I] = w - (upx * (w - sIn[3 + I][ly][lx - 1]) + umx * (sIn[3 + I][ly][lx + 1] - w)) -
            (upy * (w - sIn[3 + I][ly - 1][lx]) + umy * (sIn[3 + I][ly + 1][lx] - w));
  }
}

// Loads the tile at (tx0, ty0) with a halo of 2 into sIn (velocities zero
// when the flow does not advect).  Launched with kTX * kTY threads; every
// thread issues all its loads before the first LDS write, so the block waits
// for one memory round trip instead of one per pass.
template <typename T>
__device__ __forceinline__ void load_advect_tile(const UpdArgs<T>& P, int tx0, int ty0, T (&sIn)[8][kHY][kHX]) {
  constexpr int kThr = kTX * kTY, kIt = (kHX * kHY + kThr - 1) / kThr;
  T v[kIt][8];
  long gi[kIt];
#pragma unroll
  for (int it = 0; it < kIt; ++it) {
    const int e = threadIdx.x + it * kThr;
    if (e < kHX * kHY) {
      const int lx = e % kHX, ly = e / kHX;
      const int gx = (tx0 + lx - 2 + P.nx) & (P.nx - 1);
      const int gy = (ty0 + ly - 2 + P.ny) & (P.ny - 1);
      gi[it] = long(gy) * P.nx + gx;
#pragma unroll
      for (int I = 0; I < 3; ++I) {
        v[it][I] = P.phi[I * P.n + gi[it]];
        v[it][3 + I] = P.w[I * P.n + gi[it]];
      }
      v[it][6] = P.advect ? P.u[gi[it]] : T(0);
      v[it][7] = P.advect ? P.u[P.n + gi[it]] : T(0);
    }
  }
#pragma unroll
  for (int it = 0; it < kIt; ++it) {
    const int e = threadIdx.x + it * kThr;
    if (e < kHX * kHY) {
      const int lx = e % kHX, ly = e / kHX;
#pragma unroll
      for (int k = 0; k < 8; ++k) sIn[k][ly][lx] = v[it][k];
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_advect_update(UpdArgs<T> P) {
  __shared__ T sIn[8][kHY][kHX];   // phi[3], w[3], ux, uy
  __shared__ T sMu[3][kMY][kMX];
  __shared__ T sWt[3][kMY][kMX];
  __shared__ double red[16 * 4];
  P.shift(long(blockIdx.z) * P.rs);
  const int lt = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int tx0 = (lt % gridDim.x) * kTX, ty0 = (lt / gridDim.x) * kTY;
  const int tid = threadIdx.x;
  load_advect_tile(P, tx0, ty0, sIn);
  __syncthreads();
  // advected fields and mu~ on the halo-1 region, 34 x 10 sites: the first
  // pass gives each 32-lane half of a wave one row of 32 sites, so that every
  // LDS access of the stencil is 32 consecutive words of one row (no bank
  // conflicts); the second covers rows 8-9 and then columns 32-33
  static_assert(kTX == 32 && kTY == 8 && kMX == 34 && kMY == 10, "halo-1 pass mapping");
  for (int pass = 0; pass < 2; ++pass) {
    int mx, my;
    if (pass == 0) {
      mx = tid & 31, my = tid >> 5;
    } else if (tid < 64) {
      mx = tid & 31, my = 8 + (tid >> 5);
    } else if (tid < 84) {
      mx = 32 + ((tid - 64) & 1), my = (tid - 64) >> 1;
    } else {
      break;
    }
    T pt[3], wt[3];
    advect_site(sIn, mx + 1, my + 1, pt, wt);  // position in sIn
    const T tot = pt[0] + pt[1] + pt[2];
#pragma unroll
    for (int I = 0; I < 3; ++I) {
      T acc = T(0);
#pragma unroll
      for (int J = 0; J < 3; ++J)
        if (J != I) acc += P.chi[I][J] * pt[J];
      sMu[I][my][mx] = acc - wt[I] + P.kappa * (tot - T(1));
      sWt[I][my][mx] = wt[I];
    }
    if (mx >= 1 && mx <= kTX && my >= 1 && my <= kTY) {
      const long gi = long(ty0 + my - 1) * P.nx + (tx0 + mx - 1);
      P.stilde[gi] = pt[0] * P.invD[0] + pt[1] * P.invD[1] + pt[2] * P.invD[2];
    }
  }
  __syncthreads();
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  const T cS = T(P.scal[kMeanS]);
  {
    const int ox = tid % kTX, oy = tid / kTX;  // 256 threads = 32 x 8 outputs
    const int mx = ox + 1, my = oy + 1;
    const long gi = long(ty0 + oy) * P.nx + (tx0 + ox);
#pragma unroll
    for (int I = 0; I < 3; ++I) {
      const T lap = sMu[I][my][mx + 1] + sMu[I][my][mx - 1] + sMu[I][my + 1][mx] +
                    sMu[I][my - 1][mx] - T(4) * sMu[I][my][mx];
      const T wn = sWt[I][my][mx] - P.coef[I] * lap;
      P.wout[I * P.n + gi] = wn;
      v[I] = double(wn);
      if (I == 2) v[3] = double(exp(-(wn - cS)));
    }
  }
  block_partial<4>(v, red, P.partials, lt);
}

// The convection step alone: Phi~ -> phit and the auxiliary-convected omega
// -> wt (3 planes each), for the Phi -> omega inversion that follows it.
template <typename T>
__global__ void __launch_bounds__(256) k_advect_only(UpdArgs<T> P, T* __restrict__ phit, T* __restrict__ wt) {
  __shared__ T sIn[8][kHY][kHX];
  const int lt = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int tx0 = (lt % gridDim.x) * kTX, ty0 = (lt / gridDim.x) * kTY;
  load_advect_tile(P, tx0, ty0, sIn);
  __syncthreads();
  const int ox = threadIdx.x % kTX, oy = threadIdx.x / kTX;  // 256 threads = 32 x 8 sites
  T pt[3], w[3];
  advect_site(sIn, ox + 2, oy + 2, pt, w);
  const long gi = long(ty0 + oy) * P.nx + (tx0 + ox);
#pragma unroll
  for (int I = 0; I < 3; ++I) {
    phit[I * P.n + gi] = pt[I];
    wt[I * P.n + gi] = w[I];
  }
}

// ---------------------------------------------------------------------------
// Force reconstruction in k-space: row FFT of S, column FFT x multiplier x
// inverse, row inverse giving f_x + i f_y; external force; lattice units.
// ---------------------------------------------------------------------------
template <typename T> struct ForceArgs {
  const T* S;
  T2<T>* spec;          // nx*ny complex work plane
  T* F;                 // 2 planes (lattice units)
  const T2<T>* tw_x;
  const T2<T>* tw_y;
  int nx, ny;
  long n;
  double kx0, ky0;      // 2 pi/(nx dx), 2 pi/(ny dx)
  double pref;          // (kT/v)/dt / (nx ny)
  double conv;          // dt^2/dx (physical -> lattice), 0 if uncoupled
  const double* scal;   // kGext: external force amplitude in lattice units
  int nf;
  int nrep;
  long rs;
  __device__ void shift(long o) {
    S = sh(S, o), spec = sh(spec, o), F = sh(F, o), tw_x = sh(tw_x, o), tw_y = sh(tw_y, o);
    scal = sh(scal, o);
  }
};

template <typename T, int L, int R>
__global__ void __launch_bounds__(512) k_force_row_fwd(ForceArgs<T> P) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, true, 1>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int f = threadIdx.x / TL, j = threadIdx.x % TL;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  P.shift(long(blockIdx.z) * P.rs);
  const int y = blockIdx.x * P.nf + f;
  const bool active = y < P.ny;
  Twiddles<T, L, R> twf;
  load_fwd_twiddles(twf, j, P.tw_x);
  T re[R], im[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    re[m] = active ? P.S[long(y) * P.nx + j + TL * m] : T(0);
    im[m] = T(0);
  }
  fft_forward<T, L, R>(re, im, j, lds, twf);
  if (active) {
#pragma unroll
    for (int m = 0; m < R; ++m) {
      T2<T> o;
      o.x = re[m];
      o.y = im[m];
      P.spec[long(y) * P.nx + j + TL * m] = o;
    }
  }
}

template <typename T, int L, int R, int NF>
__global__ void __launch_bounds__(512) k_force_col(ForceArgs<T> P) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, false, NF>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int f = threadIdx.x % NF, j = threadIdx.x / NF;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  P.shift(long(blockIdx.z) * P.rs);
  const int kxi = xcd_tile(blockIdx.x, gridDim.x) * NF + f;   // column = x wavenumber index
  const bool active = kxi < P.nx;
  Twiddles<T, L, R> twf, twi;
  load_fwd_twiddles(twf, j, P.tw_y);
  load_inv_twiddles(twi, j, P.tw_y);
  T re[R], im[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    T2<T> v;
    v.x = T(0);
    v.y = T(0);
    if (active) v = P.spec[long(j + TL * m) * P.nx + kxi];
    re[m] = v.x;
    im[m] = v.y;
  }
  fft_forward<T, L, R>(re, im, j, lds, twf);
  const int mx = kxi < P.nx / 2 ? kxi : kxi - P.nx;
  const double kx = P.kx0 * mx;
  const bool nyq_x = (kxi == P.nx / 2);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int kyi = j + TL * m;
    const int my = kyi < P.ny / 2 ? kyi : kyi - P.ny;
    const double ky = P.ky0 * my;
    const double k2 = kx * kx + ky * ky;
    const double inv = k2 > 0.0 ? P.pref / k2 : 0.0;
    const T al = nyq_x ? T(0) : T(inv * kx);
    const T be = (kyi == P.ny / 2) ? T(0) : T(inv * ky);
    const T sr = re[m], si = im[m];
    // G = i al S + i (i be S) = (i al - be) S: real part f_x, imaginary part f_y
    re[m] = -al * si - be * sr;
    im[m] = al * sr - be * si;
  }
  fft_inverse<T, L, R>(re, im, j, lds, twi);
  if (active) {
#pragma unroll
    for (int m = 0; m < R; ++m) {
      T2<T> o;
      o.x = re[m];
      o.y = im[m];
      P.spec[long(j + TL * m) * P.nx + kxi] = o;
    }
  }
}

template <typename T, int L, int R>
__global__ void __launch_bounds__(512) k_force_row_inv(ForceArgs<T> P) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, true, 1>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int f = threadIdx.x / TL, j = threadIdx.x % TL;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  P.shift(long(blockIdx.z) * P.rs);
  const int y = blockIdx.x * P.nf + f;
  const bool active = y < P.ny;
  Twiddles<T, L, R> twi;
  load_inv_twiddles(twi, j, P.tw_x);
  T re[R], im[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    T2<T> v;
    v.x = T(0);
    v.y = T(0);
    if (active) v = P.spec[long(y) * P.nx + j + TL * m];
    re[m] = v.x;
    im[m] = v.y;
  }
  fft_inverse<T, L, R>(re, im, j, lds, twi);
  if (active) {
    const T conv = T(P.conv);
    const double g = P.scal[kGext];
    const T fext = T(y < P.ny / 2 ? -g : g);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const long i = long(y) * P.nx + j + TL * m;
      P.F[i] = re[m] * conv + fext;
      P.F[P.n + i] = im[m] * conv;
    }
  }
}

// ---------------------------------------------------------------------------
// D2Q9 lattice Boltzmann: pull stream + BGK collision with second-order force.
// Populations are stored as deviations g_i = f_i - w_i from the rest state
// (rho = 1, u = 0) so that FP32 keeps the small momentum of slow flows.
// ---------------------------------------------------------------------------
template <typename T> struct LbArgs {
  const T* fin;    // 9 planes g* = f* - w (previous post-collision)
  T* fout;         // 9 planes
  const T* F;      // 2 planes
  T* rho;
  T* u;            // 2 planes
  int nx, ny;
  long n;
  T omega;         // BGK: 1/tau
  T fpre;          // BGK: 1 - 1/(2 tau)
  T gs, gb, gg;    // multi-relaxation: shear, bulk and non-hydrodynamic factors
  T umax2;         // flow-speed guard: |u|^2 above this sets guard[kGuardMach]
  unsigned* guard; // kNumGuard flags of the replica, set (never cleared) by the kernel
  int nrep;
  long rs;
  __device__ void shift(long o) {
    fin = sh(fin, o), fout = sh(fout, o), F = sh(F, o), rho = sh(rho, o), u = sh(u, o);
    guard = sh(guard, o);
  }
};

// Stability flags of one replica, raised by the LB kernel and reported by the
// host at the next synchronisation: the flow speed above the guard, a
// negative post-collision population, a density or velocity that is not finite.
enum Guard : int { kGuardMach = 0, kGuardNegative = 1, kGuardNonFinite = 2, kNumGuard = 3 };

// Flags of one lane over the sites it updates; raised in memory by lb_raise.
struct LbFlags {
  bool nonfinite = false, fast = false, neg = false;
};
template <typename T>
__device__ __forceinline__ void lb_check(LbFlags& fl, T rho, T usq, T umax2, T fmin) {
  const bool nf = !isfinite(rho) || !isfinite(usq);
  fl.nonfinite |= nf;
  fl.fast |= !nf && usq > umax2;
  fl.neg |= !nf && fmin < T(0);
}
// Lanes that found a condition store its flag (a rare path; all store 1).
__device__ __forceinline__ void lb_raise(unsigned* guard, const LbFlags& fl) {
  if (fl.nonfinite) guard[kGuardNonFinite] = 1u;
  if (fl.fast) guard[kGuardMach] = 1u;
  if (fl.neg) guard[kGuardNegative] = 1u;
}

// MRT = false: BGK collision with relaxation time tau and the second-order
// force term.  MRT = true: the multi-relaxation collision in moment space
// (moments of the deviations g = f - w, so rho - 1 and the stress minus its
// rest value keep full precision):
//   u = (j + F/2)/rho,  Pi_eq = rho/3 I + rho u u,  N = Pi - Pi_eq,
//   Pi* = Pi_eq + gs (N - tr(N)/2 I) + gb tr(N)/2 I
//         + (1 + gs)/2 [u F + F u - (u.F) I] + (1 + gb)/2 (u.F) I,
//   f*_i = H_i(rho, j + F, Pi*) + gg (f_i - H_i(rho, j, Pi)),
// H_i(rho, j, Pi) = w_i [rho + 3 j.c_i + 4.5 (Pi - rho/3 I):(c_i c_i - I/3)],
// the populations that carry exactly (rho, j, Pi).
// Pull streaming of one site: g_k(x) = g*_k(x - c_k) from the previous buffer;
// c = (0,0),(1,0),(0,1),(-1,0),(0,-1),(1,1),(-1,1),(-1,-1),(1,-1).
template <typename T>
__device__ __forceinline__ void lb_pull(const LbArgs<T>& P, int x, int y, T (&g)[9]) {
  const int xm = (x - 1) & (P.nx - 1), xp = (x + 1) & (P.nx - 1);
  const long ym = long((y - 1) & (P.ny - 1)) * P.nx, yp = long((y + 1) & (P.ny - 1)) * P.nx;
  const long yc = long(y) * P.nx;
  g[0] = P.fin[0 * P.n + yc + x];
  g[1] = P.fin[1 * P.n + yc + xm];
  g[2] = P.fin[2 * P.n + ym + x];
  g[3] = P.fin[3 * P.n + yc + xp];
  g[4] = P.fin[4 * P.n + yp + x];
  g[5] = P.fin[5 * P.n + ym + xm];
  g[6] = P.fin[6 * P.n + ym + xp];
  g[7] = P.fin[7 * P.n + yp + xp];
  g[8] = P.fin[8 * P.n + yp + xm];
}

// Collision of the pulled populations g of site i with the force (Fx, Fy);
// stores f*, rho, u and records the guard's conditions in fl.
template <typename T, bool MRT>
__device__ __forceinline__ void lb_collide(const LbArgs<T>& P, long i, const T (&g)[9], T Fx, T Fy, LbFlags& fl) {
  // sum_i w_i = 1 and sum_i w_i c_i = 0, so the deviations carry rho - 1 and the momentum
  const T drho = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
  const T rho = T(1) + drho;
  const T jx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
  const T jy = (g[2] - g[4]) + (g[5] + g[6]) - (g[7] + g[8]);
  const T ir = T(1) / rho;
  const T ux = (jx + T(0.5) * Fx) * ir;
  const T uy = (jy + T(0.5) * Fy) * ir;
  const T usq = ux * ux + uy * uy;
  constexpr int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  constexpr int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  if constexpr (MRT) {
    // second moments of g: sum_i w_i c_i c_i = I/3, so Pi - rho/3 I = Sg - drho/3 I
    const T sxx = (g[1] + g[3]) + ((g[5] + g[6]) + (g[7] + g[8]));
    const T syy = (g[2] + g[4]) + ((g[5] + g[6]) + (g[7] + g[8]));
    const T sxy = (g[5] - g[6]) + (g[7] - g[8]);
    const T third = T(1.0 / 3.0);
    // A = Pi - rho/3 I (pre-collision), B = Pi* - rho/3 I (post-collision)
    const T axx = sxx - third * drho, ayy = syy - third * drho, axy = sxy;
    const T nxx = axx - rho * ux * ux, nyy = ayy - rho * uy * uy, nxy = axy - rho * ux * uy;
    const T htr = T(0.5) * (nxx + nyy);
    const T uF = ux * Fx + uy * Fy;
    const T cs_ = T(0.5) * (T(1) + P.gs), cb_ = T(0.5) * (T(1) + P.gb);
    const T bxx = rho * ux * ux + P.gs * (nxx - htr) + P.gb * htr + cs_ * (T(2) * ux * Fx - uF) + cb_ * uF;
    const T byy = rho * uy * uy + P.gs * (nyy - htr) + P.gb * htr + cs_ * (T(2) * uy * Fy - uF) + cb_ * uF;
    const T bxy = rho * ux * uy + P.gs * nxy + cs_ * (ux * Fy + uy * Fx);
    const T jxs = jx + Fx, jys = jy + Fy;
    // The moving populations from the expansion; the rest population is their
    // complement to rho - 1, its exact value: the rounded weights would
    // otherwise leave the stress term a trace of about eps |rho u u| per step,
    // a systematic drift of the mass.
    T o[9];
#pragma unroll
    for (int k = 1; k < 9; ++k) {
      const T w = k < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0);
      const T qx = T(cx[k] * cx[k]) - third, qy = T(cy[k] * cy[k]) - third, qxy = T(2 * cx[k] * cy[k]);
      const T hpost = w * (drho + T(3) * (T(cx[k]) * jxs + T(cy[k]) * jys) +
                           T(4.5) * (bxx * qx + byy * qy + bxy * qxy));
      const T hpre = w * (drho + T(3) * (T(cx[k]) * jx + T(cy[k]) * jy) +
                          T(4.5) * (axx * qx + ayy * qy + axy * qxy));
      o[k] = hpost + P.gg * (g[k] - hpre);
    }
    o[0] = drho - (((o[1] + o[2]) + (o[3] + o[4])) + ((o[5] + o[6]) + (o[7] + o[8])));
    T fmin = o[0] + T(4.0 / 9.0);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      P.fout[k * P.n + i] = o[k];
      fmin = min(fmin, o[k] + (k == 0 ? T(4.0 / 9.0) : (k < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0))));
    }
    lb_check(fl, rho, usq, P.umax2, fmin);
    P.rho[i] = rho;
    P.u[i] = ux;
    P.u[P.n + i] = uy;
    return;
  }
  T fmin = T(1);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const T w = k == 0 ? T(4.0 / 9.0) : (k < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0));
    const T cu = T(cx[k]) * ux + T(cy[k]) * uy;
    // f^eq - w = w (rho - 1) + w rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2)
    const T geq = w * drho + w * rho * (T(3) * cu + T(4.5) * cu * cu - T(1.5) * usq);
    const T cF = T(cx[k]) * Fx + T(cy[k]) * Fy;
    const T cmuF = (T(cx[k]) - ux) * Fx + (T(cy[k]) - uy) * Fy;
    const T src = w * (T(3) * cmuF + T(9) * cu * cF);
    const T o = g[k] - (g[k] - geq) * P.omega + P.fpre * src;
    P.fout[k * P.n + i] = o;
    fmin = min(fmin, o + w);
  }
  lb_check(fl, rho, usq, P.umax2, fmin);
  P.rho[i] = rho;
  P.u[i] = ux;
  P.u[P.n + i] = uy;
}

// An LB state that varies along y only: rows[p * ny + y] over the rows of plane
// p = blockIdx.y, the 9 populations, then u (2), then rho.
constexpr int kLbRowPlanes = 12;
template <typename T>
__global__ void __launch_bounds__(256) k_lb_rows(const double* rows, int nx, int ny, T* f, T* u, T* rho) {
  const long n = long(nx) * ny, i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (i >= n) return;
  T* d = p < 9 ? f + p * n : (p < 11 ? u + (p - 9) * n : rho);
  d[i] = T(rows[p * ny + int(i / nx)]);
}

template <typename T, bool MRT>
__global__ void __launch_bounds__(256) k_lb(LbArgs<T> P) {
  P.shift(long(blockIdx.z) * P.rs);
  const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= P.n) return;
  const int x = int(i & (P.nx - 1)), y = int(i / P.nx);
  T g[9];
  lb_pull(P, x, y, g);
  LbFlags fl;
  lb_collide<T, MRT>(P, i, g, P.F[i], P.F[P.n + i], fl);
  lb_raise(P.guard, fl);
}

// The row-inverse force pass fused with the LB step of the same rows: the
// x-inverse FFT of the force spectrum gives (f_x, f_y) of nf rows per block,
// stored as the lattice force F (as k_force_row_inv does) and handed to the LB
// step of those sites in registers (as k_lb does with F from memory).  The
// populations the LB pulls (neighbouring rows of the previous buffer, which
// no block of this launch writes) are loaded before the transform, so their
// latency overlaps it.
template <typename T, int L, int R, bool MRT>
__global__ void __launch_bounds__(512) k_force_inv_lb(ForceArgs<T> P, LbArgs<T> B) {
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, true, 1>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int f = threadIdx.x / TL, j = threadIdx.x % TL;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  P.shift(long(blockIdx.z) * P.rs);
  B.shift(long(blockIdx.z) * B.rs);
  const int y = blockIdx.x * P.nf + f;
  const bool active = y < P.ny;
  Twiddles<T, L, R> twi;
  load_inv_twiddles(twi, j, P.tw_x);
  T re[R], im[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    T2<T> v;
    v.x = T(0);
    v.y = T(0);
    if (active) v = P.spec[long(y) * P.nx + j + TL * m];
    re[m] = v.x;
    im[m] = v.y;
  }
  T g[R][9];
  if (active) {
#pragma unroll
    for (int m = 0; m < R; ++m) lb_pull(B, j + TL * m, y, g[m]);
  }
  fft_inverse<T, L, R>(re, im, j, lds, twi);
  if (!active) return;
  const T conv = T(P.conv);
  const double ge = P.scal[kGext];
  const T fext = T(y < P.ny / 2 ? -ge : ge);
  LbFlags fl;
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const long i = long(y) * P.nx + j + TL * m;
    const T Fx = re[m] * conv + fext, Fy = im[m] * conv;
    P.F[i] = Fx;
    P.F[P.n + i] = Fy;
    lb_collide<T, MRT>(B, i, g[m], Fx, Fy, fl);
  }
  lb_raise(B.guard, fl);
}

}  // namespace epdlb
