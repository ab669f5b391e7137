// The plain propagator passes at R = 2, 4 and 16, which a surrogate context takes when
// a tuned or given shape asks for them.  They are a translation unit of their own, so
// that they are loaded only then and the other kernels stay close together: with these
// hundred kernels among them a 256 x 256 step took 0.3 %, a surrogate step of 512 x 512
// 0.7 % longer (1,854 -> 1,859 us per 10 steps, 5,645 -> 5,688 per 50).
#include "prop_launch.hpp"

namespace epdlb {
namespace {

template <int L, int R> hipError_t row(const PropArgs<float>& a, bool first, hipStream_t s) {
  if constexpr (fft_ok<float, L, R>()) {
    if (!first) return run_prop_row<float, L, R>(k_prop_row<float, L, R, false, false>, a, s);
    PropArgs<float> f = a;
    f.nf = first_nf(L, R, a.ny);
    return run_prop_row<float, L, R>(k_prop_row<float, L, R, true, false>, f, s);
  }
  return hipErrorInvalidValue;
}

template <int L, int R, int NF> hipError_t col_n(const PropArgs<float>& a, hipStream_t s) {
  if constexpr (col_ok<float, L, R, NF>())
    return run_prop_col<float, L, R, NF, col_remap<L, R, false>()>(k_prop_col<float, L, R, NF, false>, a, s);
  return hipErrorInvalidValue;
}
template <int L, int R> hipError_t col(const PropArgs<float>& a, hipStream_t s) {
  switch (a.nf) {
    case 4: return col_n<L, R, 4>(a, s);
    case 8: return col_n<L, R, 8>(a, s);
    case 16: return col_n<L, R, 16>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int L> hipError_t rows(int R, const PropArgs<float>& a, bool first, hipStream_t s) {
  switch (R) {
    case 2: return row<L, 2>(a, first, s);
    case 4: return row<L, 4>(a, first, s);
    case 16: return row<L, 16>(a, first, s);
  }
  return hipErrorInvalidValue;
}
template <int L> hipError_t cols(int R, const PropArgs<float>& a, hipStream_t s) {
  switch (R) {
    case 2: return col<L, 2>(a, s);
    case 4: return col<L, 4>(a, s);
    case 16: return col<L, 16>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t plain_prop_row(int L, int R, const PropArgs<float>& a, bool first, hipStream_t s) {
  switch (L) {
    case 32: return rows<32>(R, a, first, s);
    case 64: return rows<64>(R, a, first, s);
    case 128: return rows<128>(R, a, first, s);
    case 256: return rows<256>(R, a, first, s);
    case 512: return rows<512>(R, a, first, s);
    case 1024: return rows<1024>(R, a, first, s);
  }
  return hipErrorInvalidValue;
}

hipError_t plain_prop_col(int L, int R, const PropArgs<float>& a, hipStream_t s) {
  switch (L) {
    case 16: return cols<16>(R, a, s);
    case 32: return cols<32>(R, a, s);
    case 64: return cols<64>(R, a, s);
    case 128: return cols<128>(R, a, s);
    case 256: return cols<256>(R, a, s);
    case 512: return cols<512>(R, a, s);
    case 1024: return cols<1024>(R, a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace epdlb
