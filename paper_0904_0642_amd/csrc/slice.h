// slice.h -- what the slice update kernels share: the guarded norm of a
// projected SU(2) block, the place of a sweep's partial sums, the step of the
// device's sweep counter.
#pragma once

#include "geometry.h"

namespace su3hb {

// 1/k for the norm k = sqrt(k2) of a projected SU(2) block; false for a
// degenerate projection (k <= 1e-300), which no hit accepts.  Norms from
// 2^-500 up take rsqrt_refined; smaller ones the exact square root, so the
// degenerate test is the one of the definition.
__device__ __forceinline__ bool inv_norm(double k2, double &ik)
{
    if (k2 >= 0x1p-1000) {
        ik = rsqrt_refined(k2);
        return true;
    }
    const double k = sqrt(k2);
    if (!(k > 1e-300)) return false;
    ik = 1.0 / k;
    return true;
}

// The partial sums of block b in a measured slice of the place-th measured
// sweep.
template <int D, int NC>
__device__ __forceinline__ double *meas_of_block(const UpdateArgs &a, uint32_t place, uint32_t b)
{
    return a.meas + ((size_t(place) * D + uint32_t(a.mu)) * a.total_blocks + b) * NC;
}

// The sweep counter's step at the end of each parity (one thread per launch;
// kSweepWords in layout.h).
__device__ __forceinline__ void advance_sweep(const UpdateArgs &a, int D, uint32_t sweep)
{
    if (a.mu != D - 1 || blockIdx.x != 0 || threadIdx.x != 0) return;
    a.sweep[1 - a.parity] = sweep + uint32_t(a.parity);
    if (a.meas != nullptr) a.sweep[3 - a.parity] = a.sweep[2 + a.parity] + uint32_t(a.parity);
}

// Between a wave's LDS writes and its lanes' reads of them: the wave's LDS
// operations complete in order.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// XCD of the calling wave (hardware register XCC_ID, 4 bits).
__device__ __forceinline__ uint32_t xcc_id()
{
    return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kBarrierXcds - 1u);
}

}  // namespace su3hb
