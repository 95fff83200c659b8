// The matrix kernel for binary16 layers (the kinds are compiled apart, side by side).
#include "matrix_kernel.h"

namespace sc {

int launch_matrix_f16(const MatrixPlan& p, const MatrixArgs& a, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (p.MK * 100 + p.NP * 10 + p.KS) {
        case 221: return launch_fly<_Float16, 2, 2, 1>(a, p, s);
        case 241: return launch_fly<_Float16, 2, 4, 1>(a, p, s);
        case 224: return launch_fly<_Float16, 2, 2, 4>(a, p, s);
        case 118: return launch_fly<_Float16, 1, 1, 8>(a, p, s);
        case 128: return launch_fly<_Float16, 1, 2, 8>(a, p, s);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace sc
