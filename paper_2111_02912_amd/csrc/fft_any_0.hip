// FFT passes of one group of grid lengths (see fft_any.h; the groups only
// spread the compile time).
#include "fft_any.h"

#define KBN_LENS(X) \
    X(4) X(10) X(20) X(30) X(45) X(60) X(80) X(100) X(126) X(160) X(192) X(225) X(270) X(320) X(375) \
    X(420) X(486) X(560) X(630) X(700) X(768) X(875) X(972)
KBN_ANY_UNIT(kbn_any_passes_0, KBN_LENS)
