// chain FFT kernels, part 2
#define CGH_CHAIN_PART 2
#include "fft_chain_part.h"
