// Chain propagators and densities on a three-dimensional periodic grid
// (Sec. II: the split step, the density integrals and Eq. phi_s, with the
// heat kernel exp(-R_G^2 |k|^2 ds) of three dimensions).
//
// The heat kernel separates, K = K_x K_y K_z, and the factors commute, so a
// contour step q -> E K (E q), E = exp(-(w_j - c_j)/2), is three real
// one-dimensional convolutions, in the order x, y, z on even steps and z, y, x
// on odd ones.  The last convolution of step a and the first of step a + 1
// then run along the same axis and share a pass: convolve, multiply by E_a,
// store q_{a+1}, multiply by E_{a+1}, convolve.  Two real lines ride in one
// complex transform (the multiplier is real and even), both chains in one
// launch (blockIdx.y), and the planes between the passes stay real: a contour
// step moves 6 planes per chain (the shared pass: scratch and factor in, q and
// scratch out; the y pass: scratch in and out).
//
// What bounds it: HBM at large sizes (launch latency below about 64^3, where a
// pass is 4-5 us).  As one three-dimensional complex transform pair per step, a
// chain at a time, a step moved 22 planes per chain in 5 launches.  Measured at
// 256^3 FP32, N = 32: 320 launches of 120 us, 39.4 ms per evaluation, before;
// 65 launches of 84-86 us in the mean (events at their own start and end; 403 MB
// each, 4.7-4.8 TB/s, where a copy reaches 5.05), 6.75-7.04 ms, now, by card (6.45
// on the best).  Under the kernel trace: 89-90 us along y and z, 104 along x, 132-136
// the first.  128^3: 4.99 -> 1.07-1.13 ms (FP32), 9.32 -> 1.74 ms (FP64).
//
// The sums (gauge, Q_P, Q_S) are FP64 block partials in fixed slots, added in
// slot order.
#pragma once
#include "kernels.hpp"

namespace epdlb {
namespace epd3 {

constexpr int kThreads = 256;
constexpr int kRedBlocks = 1024;
constexpr int kMaxLen = 512;

// One pass of the propagators: lines of length L along one axis.
template <typename T> struct PassArgs {
  const T* wA;          // first pass (and grids of one site)
  const T* wB;
  T* EA;                // first pass: exp(-(w_A - c_A)/2), written for the later ones
  T* EB;
  T* EJ;                // the same of the junction segment (A fraction fracJ); nullptr: none
  const T* E[2][2];     // factor plane of chain c at step a (+0/+1): EA, EB or EJ
  const double* sums;   // field sums: [0] w_A, [1] w_B
  double inv_n;
  T* q[2];              // mid: the plane q_{a+1} of each chain
  T* tmp;               // 2 planes (per chain): data between two passes
  const T2<T>* tw;      // the twiddles of TwTables<T, L, R>
  const T* mult;        // exp(-R_G^2 k^2 ds)/L in FFT order: L values, then what their rounding left
  long n;               // sites, the plane stride
  long units;           // pairs of lines
  long rows;            // contiguous lines: their number (the last pair may be half empty)
  long inner, gs, st;   // strided lines: pair u starts at (u / inner) gs + 2 (u % inner), element stride st
  int conv;             // first pass: convolve (0: a grid with one axis, whose first pass only forms E)
  int mid;              // after the convolution: x E(step a), store q_{a+1}
  int second;           // then x E(step a + 1) and convolve again (2: no convolution, one axis)
  int last;             // with mid: partial sums of q_N
  T frac[2];            // first pass: A fraction of chain c's segment at step 0
  T fracJ;
  double* partials;     // last: per-block sums of q_N of the forward chain
};

// Transforms per block of a pass over strided lines.  Wide: 256 or 512 lanes, and
// neighbouring lanes on neighbouring pairs: 128-byte segments (a whole cache
// line) for lengths up to 256 in FP32 and 512 in FP64 (64 bytes at 512 in FP32,
// where 16 pairs would need 1,024 lanes).  Narrow: one wave (at least four pairs),
// for grids whose wide blocks would leave CUs idle.
template <typename T, int L, int R> constexpr int strided_nf(bool wide) {
  constexpr int tl = L / R;
  constexpr int seg = sizeof(T) == 4 ? 16 : 8;   // pairs of one 128-byte segment
  if (!wide) return tl * 4 <= 64 ? 64 / tl : 4;
  return tl * seg <= 256 ? 256 / tl : (tl * seg <= 512 ? seg : 512 / tl);
}
// Values per lane: whole short lines, else 8.
template <int L> constexpr int values_per_lane() { return L < 8 ? L : 8; }

// Convolution with the multiplier g + gl.  Every contour step applies the same
// operator, so an error of the rounded multiplier, or of a twiddle, adds up
// over the steps coherently, as rounding errors of the data do not.  Measured
// at 256^3 FP32, N = 32, relative error of Phi_A: 5.7e-7 with rounded
// multipliers and twiddles from two preloaded ones by products, 3.4e-7 with
// both as here (3.8-4.9e-7 with the three-dimensional transform), at no cost in time: the
// twiddle table lies in LDS and frees the registers the preloaded ones held.
template <typename T, int L, int R, class V, class TW>
__device__ __forceinline__ void convolve_exact(T* re, T* im, int j, const V& lds, const TW& tw, const T* g,
                                               const T* gl) {
  fft_forward<T, L, R>(re, im, j, lds, tw);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    if constexpr (sizeof(T) == 4) {
      re[m] = fma(re[m], g[m], re[m] * gl[m]);
      im[m] = fma(im[m], g[m], im[m] * gl[m]);
    } else {
      re[m] *= g[m];
      im[m] *= g[m];
    }
  }
  fft_inverse<T, L, R>(re, im, j, lds, tw);
}

// CONTIG: lines along x, two neighbouring rows per transform, nf = blockDim /
// (L/R) transforms per block.  Otherwise lines along y or z, columns x, x + 1
// per transform, NF transforms per block interleaved lane by lane.  The code path
// is kept straight as in the two-dimensional passes: the first pass is an
// instantiation of its own, factors come from one plane per step, every load is
// unconditional (a transform past the end repeats the last one and stores
// nothing), offsets are 32 bits (a plane is at most 2^27 sites).  With the factor
// chosen by a branch per value, 64 x 32 x 16 FP64 at N = 16 took 0.237 ms, and
// 0.196 ms now.  FP32 is held to 128 registers, four waves per SIMD: at 256^3 the
// 129th cost 8.08 against 6.45 ms on the same card.
template <typename T, int L, int R, bool CONTIG, int NF, bool FIRST>
__global__ void __launch_bounds__(512, sizeof(T) == 4 ? 4 : 2) k_p3_pass(PassArgs<T> P) {
  static_assert(CONTIG || !FIRST, "the first pass runs along x");
  constexpr int TL = L / R;
  using V = LdsView<T, L, R, CONTIG, NF>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[16];
  const int f = CONTIG ? int(threadIdx.x) / TL : int(threadIdx.x) % NF;
  const int j = CONTIG ? int(threadIdx.x) % TL : int(threadIdx.x) / NF;
  const int nf = CONTIG ? int(blockDim.x) / TL : NF;
  V lds{reinterpret_cast<T2<T>*>(smem_raw), f};
  const int lt = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int c = lt / gridDim.x, tile = lt % gridDim.x;
  const unsigned want = unsigned(tile) * nf + f, u = min(want, unsigned(P.units) - 1u);
  const bool active = want == u;
  // element m of this lane: byte offset o0 + m step, and o1 + m step in the
  // second line (strided lines: the pair is one aligned access at o0)
  unsigned o0, o1 = 0, step;
  bool two = active;
  if constexpr (CONTIG) {
    o0 = (2u * u * L + j) * unsigned(sizeof(T));
    const bool has = 2u * u + 1u < unsigned(P.rows);
    o1 = has ? o0 + L * unsigned(sizeof(T)) : o0;
    two = active && has;
    step = TL * sizeof(T);
  } else {
    const unsigned in = unsigned(P.inner), g = u / in;
    o0 = (g * unsigned(P.gs) + 2u * (u - g * in) + unsigned(j) * unsigned(P.st)) * unsigned(sizeof(T));
    step = unsigned(TL) * unsigned(P.st) * unsigned(sizeof(T));
  }
  auto load2 = [&](const T* p, int m, T& a, T& b) {
    if constexpr (CONTIG) {
      a = ld<T>(p, o0 + m * step);
      b = ld<T>(p, o1 + m * step);
    } else {
      const T2<T> v = ld<T2<T>>(p, o0 + m * step);
      a = v.x;
      b = v.y;
    }
  };
  auto store2 = [&](T* p, int m, T a, T b) {
    if constexpr (CONTIG) {
      if (active) st(p, o0 + m * step, a);
      if (two) st(p, o1 + m * step, b);
    } else if (active) {
      T2<T> v;
      v.x = a;
      v.y = b;
      st(p, o0 + m * step, v);
    }
  };
  T* tmp = P.tmp + c * P.n;
  T re[R], im[R], ea[R], eb[R];
  if constexpr (FIRST) {
    // the factor planes of the later passes: A's from the forward chain's
    // blocks, B's from the backward chain's
    const T ca = T(P.sums[0] * P.inv_n), cb = T(P.sums[1] * P.inv_n);
    const T fr0 = c == 0 ? P.frac[0] : P.frac[1];
    const T pure = c == 0 ? T(1) : T(0);
    T* Ep = c == 0 ? P.EA : P.EB;
#pragma unroll
    for (int m = 0; m < R; ++m) {
      T ua, ub, va, vb;
      load2(P.wA, m, ua, ub);
      load2(P.wB, m, va, vb);
      const T p0 = boltz(ua, va, pure, ca, cb), p1 = boltz(ub, vb, pure, ca, cb);
      store2(Ep, m, p0, p1);
      if (c == 0 && P.EJ) store2(P.EJ, m, boltz(ua, va, P.fracJ, ca, cb), boltz(ub, vb, P.fracJ, ca, cb));
      re[m] = fr0 == pure ? p0 : boltz(ua, va, fr0, ca, cb);
      im[m] = fr0 == pure ? p1 : boltz(ub, vb, fr0, ca, cb);
    }
  } else {
    const T* E0 = c == 0 ? P.E[0][0] : P.E[1][0];
#pragma unroll
    for (int m = 0; m < R; ++m) load2(tmp, m, re[m], im[m]);
    if (P.mid) {  // loaded before the transform, so that the latency overlaps it
#pragma unroll
      for (int m = 0; m < R; ++m) load2(E0, m, ea[m], eb[m]);
    }
  }
  // twiddles into LDS, behind the transforms' buffer
  T2<T>* twl = reinterpret_cast<T2<T>*>(smem_raw) + (L > R ? V::size_elems(nf) : 0);
  for (int i = threadIdx.x; i < TwTables<T, L, R>::kElems; i += blockDim.x) twl[i] = P.tw[i];
  if constexpr (V::kSync != kSyncBlock && L > R) __syncthreads();  // the exchanges have no barrier of the block
  const TwTables<T, L, R> tw{twl};
  T g[R], gl[R];
#pragma unroll
  for (int m = 0; m < R; ++m) {
    g[m] = P.mult[j + TL * m];
    gl[m] = sizeof(T) == 4 ? P.mult[L + j + TL * m] : T(0);
  }
  if (!FIRST || P.conv) convolve_exact<T, L, R>(re, im, j, lds, tw, g, gl);
  double qsum = 0.0;
  if (!FIRST && P.mid) {
    T* qo = c == 0 ? P.q[0] : P.q[1];
#pragma unroll
    for (int m = 0; m < R; ++m) {
      re[m] *= ea[m];
      im[m] *= eb[m];
      store2(qo, m, re[m], im[m]);
      qsum += (active ? double(re[m]) : 0.0) + (two ? double(im[m]) : 0.0);
    }
    if (P.second) {
      const T* E0 = c == 0 ? P.E[0][0] : P.E[1][0];
      const T* E1 = c == 0 ? P.E[0][1] : P.E[1][1];
      if (E1 != E0) {
#pragma unroll
        for (int m = 0; m < R; ++m) load2(E1, m, ea[m], eb[m]);
      }
#pragma unroll
      for (int m = 0; m < R; ++m) {
        re[m] *= ea[m];
        im[m] *= eb[m];
      }
      if (P.second == 1) convolve_exact<T, L, R>(re, im, j, lds, tw, g, gl);
    }
  }
  if (FIRST || !P.mid || P.second) {
#pragma unroll
    for (int m = 0; m < R; ++m) store2(tmp, m, re[m], im[m]);
  }
  if (!FIRST && P.last && c == 0) {
    double v[1] = {qsum};
    block_partial<1>(v, red, P.partials, tile);
  }
}

// A grid of one site: K is the identity, q_{j+1} = E_j^2 q_j.
template <typename T>
__global__ void k_p3_one(PassArgs<T> P, T* q, int chain, int first) {
  if (threadIdx.x || blockIdx.x) return;
  const T ca = T(P.sums[0] * P.inv_n), cb = T(P.sums[1] * P.inv_n);
  const T e = boltz(P.wA[0], P.wB[0], P.frac[chain], ca, cb);
  q[0] = e * (e * (first ? T(1) : P.tmp[chain]));
  P.tmp[chain] = q[0];
  if (P.last && chain == 0) P.partials[0] = double(q[0]);
}

// Block sums over grid-stride elements, FP64, in fixed slots [block][NV].
// gauge = nullptr: of the NV planes of a (n apart); else of exp(-(a - c)) with
// c the mean from gauge[0].  Four elements per thread in flight.
template <typename T, int NV>
__global__ void __launch_bounds__(kThreads) k_p3_sums(const T* __restrict__ a, long n, const double* __restrict__ gauge,
                                                      double inv_n, double* __restrict__ part) {
  __shared__ double red[16 * NV];
  const T c = gauge ? T(gauge[0] * inv_n) : T(0);
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  const long step = long(gridDim.x) * blockDim.x;
  for (long i0 = long(blockIdx.x) * blockDim.x + threadIdx.x; i0 < n; i0 += 4 * step) {
    T x[4][NV];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int v = 0; v < NV; ++v) x[k][v] = i0 + k * step < n ? a[v * n + i0 + k * step] : T(0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k * step < n)
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += double(gauge ? exp(-(x[k][v] - c)) : x[k][v]);
  }
  block_partial<NV>(acc, red, part, blockIdx.x);
}

// out[v] = sum over blocks of part[block][v] in slot order.  One block.
template <int NV>
__global__ void __launch_bounds__(kThreads) k_p3_finish(const double* __restrict__ part, int nb,
                                                        double* __restrict__ out) {
  __shared__ double red[16 * NV];
  double acc[NV];
  sum_partials<NV>(part, nb, acc, red);
  if (threadIdx.x == 0)
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = acc[v];
}

struct DensArgs {
  int N;
  long n;
  double V_over_dV;   // V / dV = number of sites
  double phiP;
  const double* wAn;  // node weights, N + 1 each
  const double* wBn;
  const double* sums; // [0] sum wA, [1] sum wB, [2] sum wS, [3] sum q_N, [4] sum exp(-(wS - cS))
  double inv_n;
};

// Phi_A = (V phibar_P / Q_P) sum_j wA_j q_j qb_{N-j}, Phi_B likewise, Phi_S =
// V (1 - phibar_P) exp(-(wS - cS)) / Q_S, with Q = dV * sum (dV cancels).
// q and qb hold the planes q_1 .. q_N (q_0 = 1).
template <typename T>
__global__ void __launch_bounds__(kThreads) k_p3_density(const T* __restrict__ q, const T* __restrict__ qb,
                                                         const T* __restrict__ wS, T* __restrict__ phi,
                                                         DensArgs D) {
  const double sP = D.V_over_dV * D.phiP / D.sums[3];
  const double sS = D.V_over_dV * (1.0 - D.phiP) / D.sums[4];
  const T cS = T(D.sums[2] * D.inv_n);
  for (long i = long(blockIdx.x) * blockDim.x + threadIdx.x; i < D.n; i += long(gridDim.x) * blockDim.x) {
    const T q0 = qb[long(D.N - 1) * D.n + i], qN = q[long(D.N - 1) * D.n + i];
    T sa = T(D.wAn[0]) * q0, sb = T(D.wBn[0]) * q0;
#pragma unroll 8
    for (int j = 1; j < D.N; ++j) {
      const T pr = q[long(j - 1) * D.n + i] * qb[long(D.N - j - 1) * D.n + i];
      sa += T(D.wAn[j]) * pr;
      sb += T(D.wBn[j]) * pr;
    }
    sa += T(D.wAn[D.N]) * qN;
    sb += T(D.wBn[D.N]) * qN;
    phi[i] = T(sP) * sa;
    phi[D.n + i] = T(sP) * sb;
    phi[2 * D.n + i] = T(sS) * exp(-(wS[i] - cS));
  }
}

}  // namespace epd3
}  // namespace epdlb
