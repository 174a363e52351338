// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(9) X(18) X(28) X(42) X(56) X(75) X(98) X(125) X(150) X(189) X(224) X(252) X(315) X(360) X(405) \
    X(480) X(540) X(625) X(686) X(756) X(864) X(960)
KBN_ANY_UNIT(kbn_any_passes_5, KBN_LENS)
