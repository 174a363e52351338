// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(7) X(15) X(25) X(36) X(50) X(70) X(90) X(112) X(144) X(175) X(210) X(245) X(294) X(343) X(392) \
    X(448) X(504) X(588) X(672) X(735) X(810) X(900) X(1008)
KBN_ANY_UNIT(kbn_any_passes_3, KBN_LENS)
