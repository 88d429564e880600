// Numbers of the light frames (fltop_beam_light.inc): plain C++, the same on the host, where the choice
// of a build needs them and tests run them under the sanitizers.  (Constant-expression functions are
// device functions as well.)
#ifndef FLTOP_LIGHT_H_
#define FLTOP_LIGHT_H_

#include <cstdint>

namespace fltop {

constexpr int kLightBins = 256;  // bins of their selection, 16 bits each

// Bin of a candidate whose score lies `x` bins below the reference.  What has no mass lies infinitely
// far below, masked tokens farther than any integer counts, and a score may come out a little above
// the reference: the clamp has to come before the conversion, whose result is undefined outside the
// integer's range.
constexpr uint32_t light_bin(float x) {
    return (uint32_t)__builtin_fminf(__builtin_fmaxf(x, 0.0f), (float)(kLightBins - 1));
}

}  // namespace fltop

#endif
