// chain FFT kernels, part 4
#define CGH_CHAIN_PART 4
#include "fft_chain_part.h"
