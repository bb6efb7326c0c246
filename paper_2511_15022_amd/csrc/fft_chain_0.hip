// chain FFT kernels, part 0
#define CGH_CHAIN_PART 0
#include "fft_chain_part.h"
