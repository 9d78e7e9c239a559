// The dense convolution's choice of kernel and tile (csrc/alcs_dense_plan.h) as a C function.
#include "alcs_dense_plan.h"

extern "C" void dense_plan(const int *shape, int cus, int *out) {
    const alcs::DensePlan p = alcs::dense_plan(shape[0], shape[1], shape[2], shape[3], shape[4], shape[5], shape[6], cus);
    const int k = shape[5], stride = shape[6], pad = k / 2;
    const long long P = (long long)((shape[3] + 2 * pad - k) / stride + 1) * ((shape[4] + 2 * pad - k) / stride + 1);
    out[7] = alcs::dense_few(p, shape[0] * P, shape[2], cus);
    out[0] = p.kind; out[1] = p.bm; out[2] = p.bn; out[3] = p.npt; out[4] = p.npos; out[5] = p.threads; out[6] = p.lds;
}
