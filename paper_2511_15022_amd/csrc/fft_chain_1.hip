// chain FFT kernels, part 1
#define CGH_CHAIN_PART 1
#include "fft_chain_part.h"
