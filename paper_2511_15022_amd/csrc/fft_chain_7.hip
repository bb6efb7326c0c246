// chain FFT kernels, part 7
#define CGH_CHAIN_PART 7
#include "fft_chain_part.h"
