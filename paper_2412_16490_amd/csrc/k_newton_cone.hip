// Launchers of the dual Newton polish, circular-cone form: the lanes per QP that
// newton_group (bodex_qp.hip) chooses for each contact count.
#include "bodex_launch.h"
#include "bodex_newton_kernels.h"

namespace bodex {

template <int MM, int... GS>
static hipError_t run(const KArgs& a, int gs, hipStream_t st) {
    const size_t lds = newton_lds<MM>(a.slots);
    const bool known = (... || (gs == GS && (newton_kernel<MM, GS, true>
                                             <<<dim3(a.n_tiles * GS), dim3(kWave), lds, st>>>(a), true)));
    if (!known) return hipErrorInvalidValue;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((newton_out_kernel<MM, true>), dim3(a.n_tiles), dim3(kWave), newton_out_lds<MM>(a.slots), st, a);
    return hipGetLastError();
}

hipError_t launch_newton_cone(int mm, int gs, const KArgs& a, hipStream_t st) {
    switch (mm) {
        case 4: return run<4, 4>(a, gs, st);
        case 5: return run<5, 8>(a, gs, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace bodex
