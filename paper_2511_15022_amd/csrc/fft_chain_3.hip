// chain FFT kernels, part 3
#define CGH_CHAIN_PART 3
#include "fft_chain_part.h"
