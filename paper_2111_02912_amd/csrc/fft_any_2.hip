// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(6) X(14) X(24) X(35) X(49) X(64) X(84) X(108) X(140) X(168) X(200) X(243) X(288) X(336) X(384) \
    X(441) X(500) X(576) X(648) X(729) X(800) X(896) X(1000)
KBN_ANY_UNIT(kbn_any_passes_2, KBN_LENS)
