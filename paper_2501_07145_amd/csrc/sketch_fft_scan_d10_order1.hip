// Tuned sketch/FFT/scan kernels for D = 1024, signature order 1.
#define RFSF_LOG2D 10
#define RFSF_ORDER 1
#include "sketch_fft_scan_inst.inc"
