// Host-side launch of the tuned sketch/FFT/scan kernel. The instantiations for one transform
// length live in one translation unit each (sketch_fft_scan_d<log2 D>.hip) so that they
// compile in parallel; this header declares their entry points and holds the shared template.
#pragma once

#include "rfsf_internal.h"

namespace rfsf {
namespace tuned {

#define RFSF_DECLARE_DISPATCH(LOG2D)                                                                       \
    hipError_t dispatch_levels_##LOG2D(int M, int order, const float *dphi, const uint32_t *table, int64_t n_seq,     \
                                       int64_t L, const int64_t *lengths, int F, int Dout, float *out, int64_t ld_out, hipStream_t stream, TimeCut cut);
RFSF_DECLARE_DISPATCH(6)
RFSF_DECLARE_DISPATCH(7)
RFSF_DECLARE_DISPATCH(8)
RFSF_DECLARE_DISPATCH(9)
RFSF_DECLARE_DISPATCH(10_order1)
RFSF_DECLARE_DISPATCH(10_order2)
RFSF_DECLARE_DISPATCH(10_order3)
RFSF_DECLARE_DISPATCH(12)
RFSF_DECLARE_DISPATCH(13)
RFSF_DECLARE_DISPATCH(100)
RFSF_DECLARE_DISPATCH(200)
RFSF_DECLARE_DISPATCH(500)
RFSF_DECLARE_DISPATCH(1000)
RFSF_DECLARE_DISPATCH(2048_order1)
RFSF_DECLARE_DISPATCH(2048_order2)
RFSF_DECLARE_DISPATCH(2048_order3)
#undef RFSF_DECLARE_DISPATCH
#define RFSF_DISPATCH_BY_ORDER(LOG2D)                                                                      \
    inline hipError_t dispatch_levels_##LOG2D(int M, int order, const float *dphi, const uint32_t *table, int64_t n_seq, \
                                              int64_t L, const int64_t *lengths, int F, int Dout, float *out, int64_t ld_out, \
                                              hipStream_t stream, TimeCut cut)                             \
    {                                                                                                      \
        const auto f = order == 3 ? dispatch_levels_##LOG2D##_order3                                       \
                                  : order == 2 ? dispatch_levels_##LOG2D##_order2 : dispatch_levels_##LOG2D##_order1; \
        return f(M, order, dphi, table, n_seq, L, lengths, F, Dout, out, ld_out, stream, cut);             \
    }
RFSF_DISPATCH_BY_ORDER(10)
RFSF_DISPATCH_BY_ORDER(2048)
#undef RFSF_DISPATCH_BY_ORDER

}  // namespace tuned
}  // namespace rfsf
