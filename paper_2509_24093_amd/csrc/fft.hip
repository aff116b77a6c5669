// Column DFT passes of power-of-two lengths (see fft_pass.h), and the entry
// point that picks the kernel of a pass.
#include "fft_pass.h"

namespace cgconv {
namespace {

template <int INM, int OUTM, int DIR>
hipError_t launch_modes(const PassDesc& d, hipStream_t s) {
  switch (d.R) {
    case 2: return launch_r<2, INM, OUTM, DIR>(d, s);
    case 4: return launch_r<4, INM, OUTM, DIR>(d, s);
    case 8: return launch_r<8, INM, OUTM, DIR>(d, s);
    case 16: return launch_r<16, INM, OUTM, DIR>(d, s);
    case 32: return launch_r<32, INM, OUTM, DIR>(d, s);
    case 64: return launch_r<64, INM, OUTM, DIR>(d, s);
    case 128: return launch_r<128, INM, OUTM, DIR>(d, s);
    case 256: return launch_r<256, INM, OUTM, DIR>(d, s);
    case 512: return launch_r<512, INM, OUTM, DIR>(d, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_fft_pass(const PassDesc& d, hipStream_t s) {
  if ((d.R & (d.R - 1)) != 0)
    return d.R % 3 == 0 ? launch_fft_pass_odd<3>(d, s) : d.R % 5 == 0 ? launch_fft_pass_odd<5>(d, s)
                                                                     : launch_fft_pass_odd<7>(d, s);
  if (d.dir < 0) {
    if (d.out_mode != OUT_COMPLEX) return hipErrorInvalidValue;
    switch (d.in_mode) {
      case IN_PAIR_F32: return launch_modes<IN_PAIR_F32, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_BF16: return launch_modes<IN_PAIR_BF16, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_F32_SCALED_REV:
        if (!d.a.in_scale) return hipErrorInvalidValue;
        return launch_modes<IN_PAIR_F32_SCALED_REV, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_F32_PAD: return launch_modes<IN_PAIR_F32_PAD, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_BF16_PAD: return launch_modes<IN_PAIR_BF16_PAD, OUT_COMPLEX, -1>(d, s);
      case IN_PAIR_F32_SCALED_REV_PAD:
        if (!d.a.in_scale) return hipErrorInvalidValue;
        return launch_modes<IN_PAIR_F32_SCALED_REV_PAD, OUT_COMPLEX, -1>(d, s);
      case IN_COMPLEX: return launch_modes<IN_COMPLEX, OUT_COMPLEX, -1>(d, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (d.in_mode != IN_COMPLEX) return hipErrorInvalidValue;
  switch (d.out_mode) {
    case OUT_COMPLEX: return launch_modes<IN_COMPLEX, OUT_COMPLEX, 1>(d, s);
    case OUT_SPLIT_F32: return launch_modes<IN_COMPLEX, OUT_SPLIT_F32, 1>(d, s);
    case OUT_SPLIT_BF16: return launch_modes<IN_COMPLEX, OUT_SPLIT_BF16, 1>(d, s);
    case OUT_SPLIT_F32_SCALED:
      if (!d.a.out_scale) return hipErrorInvalidValue;
      return launch_modes<IN_COMPLEX, OUT_SPLIT_F32_SCALED, 1>(d, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace cgconv
