// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(8) X(16) X(27) X(40) X(54) X(72) X(96) X(120) X(147) X(180) X(216) X(250) X(300) X(350) X(400) \
    X(450) X(525) X(600) X(675) X(750) X(840) X(945) X(1024)
KBN_ANY_UNIT(kbn_any_passes_4, KBN_LENS)
