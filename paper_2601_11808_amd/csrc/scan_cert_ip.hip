#include "scan_cert.h"

namespace sivf {

void launch_scan_cert_ip(hipStream_t st, const Dev &S, const SearchBufs &W, const float *q, int np_stride, int kcap, int k,
                         const int32_t *k_per_query, int npairs) {
    launch_cert<1>(st, S, W, q, np_stride, kcap, k, k_per_query, npairs);
}

}  // namespace sivf
