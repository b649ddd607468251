// Strided FFT passes with 64-bit offsets (strided_wide), apart from fft.hip so
// that its code object holds the kernels of the usual sizes only.
#define NUFFT_FFT_WIDE
#include "fft.hip"
