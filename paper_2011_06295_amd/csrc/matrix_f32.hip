// The matrix kernel for fp32 layers (the kinds are compiled apart, side by side).
#include "matrix_kernel.h"

namespace sc {

int launch_matrix_f32(const MatrixPlan& p, const MatrixArgs& a, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (p.MK * 100 + p.NP * 10 + p.KS) {
        case 121: return launch_fly<float, 1, 2, 1>(a, p, s);
        case 221: return launch_fly<float, 2, 2, 1>(a, p, s);
        case 224: return launch_fly<float, 2, 2, 4>(a, p, s);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace sc
