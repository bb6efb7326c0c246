// chain FFT kernels, part 6
#define CGH_CHAIN_PART 6
#include "fft_chain_part.h"
