// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(5) X(12) X(21) X(32) X(48) X(63) X(81) X(105) X(135) X(162) X(196) X(240) X(280) X(324) X(378) \
    X(432) X(490) X(567) X(640) X(720) X(784) X(882) X(980)
KBN_ANY_UNIT(kbn_any_passes_1, KBN_LENS)
