// Tuned sketch/FFT/scan kernels for transforms of 2048 points held by one wavefront (Plan<2048>), signature order 2.
#define RFSF_LOG2D 2048
#define RFSF_ORDER 2
#include "sketch_fft_scan_inst.inc"
