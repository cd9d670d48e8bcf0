// phi and the recombination vector on the device: the one-wavefront kernel around
// locate_device.hpp.
#include "locate_device.hpp"

namespace draco {

__global__ __launch_bounds__(kW) void cyc_locate_kernel(const double2* __restrict__ gamma,
                                                        const double2* __restrict__ roots, int P, int s, double tau,
                                                        const double2* __restrict__ b0,
                                                        int32_t* __restrict__ spec_state, LocateOut out) {
    __shared__ LocateSmem sm;
    const int lane = threadIdx.x;
    for (int j = lane; j < P; j += kW) {
        sm.gam[j] = gamma[j];
        sm.root[j] = roots[j];
    }
    wave_sync();
    const bool clean = locate_wave(sm, P, s, tau, b0, out, lane);
    if (lane == 0 && spec_state != nullptr) spec_state[0] = clean ? 1 : 0;
}

hipError_t launch_cyc_locate(const double2* gamma, const double2* roots, int P, int s, double tau, const double2* b0,
                             uint64_t* mask_out, int32_t* status_out, double2* b_out, int32_t* idx_out,
                             int32_t* nu_out, int32_t* spec_state, hipStream_t stream) {
    const LocateOut out{mask_out, status_out, b_out, idx_out, nu_out};
    hipLaunchKernelGGL(cyc_locate_kernel, dim3(1), dim3(kW), 0, stream, gamma, roots, P, s, tau, b0, spec_state, out);
    return hipGetLastError();
}

}  // namespace draco
