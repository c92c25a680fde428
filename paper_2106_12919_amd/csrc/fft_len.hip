// The transform kernels of one unit of axis lengths (PIC_FFT_UNIT, see kFftLengths).
#include "fft_kernels.h"

namespace pic {

template <typename T, int U>
const FftOps<T>* fft_ops(int n) {
  constexpr int second = U + kFftUnits;
  static_assert(second + kFftUnits >= kFftLengthCount, "at most two lengths per unit");
  if (n == kFftLengths[U]) return &FftLength<T, kFftLengths[U]>::ops;
  if constexpr (second < kFftLengthCount)
    if (n == kFftLengths[second]) return &FftLength<T, kFftLengths[second]>::ops;
  return nullptr;
}

template const FftOps<float>* fft_ops<float, PIC_FFT_UNIT>(int);
template const FftOps<double>* fft_ops<double, PIC_FFT_UNIT>(int);

}  // namespace pic
