// chain FFT kernels, part 5
#define CGH_CHAIN_PART 5
#include "fft_chain_part.h"
