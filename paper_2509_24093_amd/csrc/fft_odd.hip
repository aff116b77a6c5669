// Column DFT passes of the lengths R = P * 2^j between the powers of two, for
// P = CGCONV_TU_P = 3, 5 or 7 (see fft_pass.h): the outer passes of
// zero-padded plans.  Built once per P.
#include "fft_pass.h"

namespace cgconv {
namespace {

template <int INM, int OUTM, int DIR>
hipError_t launch_odd(const PassDesc& d, hipStream_t s) {
  constexpr int P = CGCONV_TU_P;
  switch (d.R / P) {  // R = 12 .. 384 (P = 3), 10 .. 320 (5), 56 .. 448 (7)
    case 2: if constexpr (P == 5) return launch_r<2 * P, INM, OUTM, DIR>(d, s); else break;
    case 4: if constexpr (P < 7) return launch_r<4 * P, INM, OUTM, DIR>(d, s); else break;
    case 8: return launch_r<8 * P, INM, OUTM, DIR>(d, s);
    case 16: return launch_r<16 * P, INM, OUTM, DIR>(d, s);
    case 32: return launch_r<32 * P, INM, OUTM, DIR>(d, s);
    case 64: return launch_r<64 * P, INM, OUTM, DIR>(d, s);
    case 128: if constexpr (P == 3) return launch_r<128 * P, INM, OUTM, DIR>(d, s); else break;
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <>
hipError_t launch_fft_pass_odd<CGCONV_TU_P>(const PassDesc& d, hipStream_t s) {
  if (d.R % CGCONV_TU_P != 0) return hipErrorInvalidValue;
  if (d.dir < 0) {
    if (d.out_mode != OUT_COMPLEX) return hipErrorInvalidValue;
    switch (d.in_mode) {
      case IN_PAIR_F32_PAD: return launch_odd<IN_PAIR_F32_PAD, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_BF16_PAD: return launch_odd<IN_PAIR_BF16_PAD, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_F32_SCALED_REV_PAD:
        if (!d.a.in_scale) return hipErrorInvalidValue;
        return launch_odd<IN_PAIR_F32_SCALED_REV_PAD, OUT_COMPLEX, -1>(d, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (d.in_mode != IN_COMPLEX) return hipErrorInvalidValue;
  switch (d.out_mode) {
    case OUT_SPLIT_F32: return launch_odd<IN_COMPLEX, OUT_SPLIT_F32, 1>(d, s);
    case OUT_SPLIT_BF16: return launch_odd<IN_COMPLEX, OUT_SPLIT_BF16, 1>(d, s);
    case OUT_SPLIT_F32_SCALED:
      if (!d.a.out_scale) return hipErrorInvalidValue;
      return launch_odd<IN_COMPLEX, OUT_SPLIT_F32_SCALED, 1>(d, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace cgconv
