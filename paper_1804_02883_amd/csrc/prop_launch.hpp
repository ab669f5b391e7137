// Launches of the two-dimensional propagator passes by transform length L, values
// per lane R and, for columns, transforms per block NF.
#pragma once
#include "kernels.hpp"
#include "launch.hpp"

namespace epdlb {

// The shapes a pass comes with (FP64 columns with NF = 4 only).
template <typename T, int L, int R>
constexpr bool fft_ok() {
  return (R == 8 || R == 4 || ((R == 16 || R == 2) && sizeof(T) == 4)) && L >= R;
}
constexpr int kMaxColThreads = 512;
template <typename T, int L, int R, int NF>
constexpr bool col_ok() {
  return fft_ok<T, L, R>() && NF * (L / R) <= kMaxColThreads && (sizeof(T) == 4 || NF == 4);
}

template <typename T, int L, int R, class K>
hipError_t run_prop_row(K k, const PropArgs<T>& a, hipStream_t s) {
  using V = LdsView<T, L, R, true, 1>;
  const size_t lds = 2 * size_t(V::size_elems(a.nf)) * sizeof(T);
  hipError_t e = prep_lds(k, lds);
  if (e != hipSuccess) return e;
  const int tiles = (a.ny / 2 + a.nf - 1) / a.nf;
  launch_k(k, dim3(tiles, 2, a.nrep), dim3(a.nf * (L / R)), lds, s, a);
  return hipGetLastError();
}

template <typename T, int L, int R, int NF, bool REMAP, class K>
hipError_t run_prop_col(K k, const PropArgs<T>& a, hipStream_t s) {
  const size_t elems = REMAP ? NF * ColView<T, L, R>::kLen : LdsView<T, L, R, false, NF>::size_elems(NF);
  const size_t lds = elems * sizeof(T2<T>);
  hipError_t e = prep_lds(k, lds);
  if (e != hipSuccess) return e;
  const int tiles = (a.nx / 2 + NF - 1) / NF;
  launch_k(k, dim3(tiles, 2, a.nrep), dim3(NF * (L / R)), lds, s, a);
  return hipGetLastError();
}

// Transforms per block of a first pass: one wave, or one transform.
inline int first_nf(int L, int R, int ny) { return clampi(64 * R / L, 1, ny / 2); }

// The plain passes (PropArgs::plain) of FP32 surrogate runs at R = 2, 4 or 16
// (prop_plain.hip).
hipError_t plain_prop_row(int L, int R, const PropArgs<float>& a, bool first, hipStream_t s);
hipError_t plain_prop_col(int L, int R, const PropArgs<float>& a, hipStream_t s);
// FP64 surrogate runs keep R = 8.
inline hipError_t plain_prop_row(int, int, const PropArgs<double>&, bool, hipStream_t) { return hipErrorInvalidValue; }
inline hipError_t plain_prop_col(int, int, const PropArgs<double>&, hipStream_t) { return hipErrorInvalidValue; }
inline bool plain_elsewhere(bool plain, int R) { return plain && (R == 2 || R == 4 || R == 16); }

}  // namespace epdlb
