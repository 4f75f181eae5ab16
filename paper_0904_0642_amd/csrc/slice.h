// slice.h -- what the slice update kernels share: the guarded norm of a
// projected SU(2) block, the rotation of a link's rows, the place of a sweep's partial sums, the step of the
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

// U <- R_IJ(r) U and W <- R_IJ(r) W: the 2x2 matrix r mixes rows I and J.
template <typename H, int I, int J>
__device__ __forceinline__ void rotate_rows(mat3<H> &U, mat3<H> &W, const cx<H> &r00, const cx<H> &r01,
                                            const cx<H> &r10, const cx<H> &r11)
{
    const H z = H(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<H> ui = U.e[I][c], uj = U.e[J][c];
        cx<H> ni{z, z}, nj{z, z};
        cfma(ni, r00, ui); cfma(ni, r01, uj);
        cfma(nj, r10, ui); cfma(nj, r11, uj);
        U.e[I][c] = ni;
        U.e[J][c] = nj;
        const cx<H> wi = W.e[I][c], wj = W.e[J][c];
        cx<H> mi{z, z}, mj{z, z};
        cfma(mi, r00, wi); cfma(mi, r01, wj);
        cfma(mj, r10, wi); cfma(mj, r11, wj);
        W.e[I][c] = mi;
        W.e[J][c] = mj;
    }
}

// Overrelaxation on rows (I, J): the reflection that keeps Re Tr(U A).  With
// the block of W = U A equal to k V (V in SU(2)) the block becomes k V^dag:
// U <- R_IJ(r) U with r = V^dag V^dag.  The projection is FP64 as in the
// heatbath; the rotation is in H.  No random numbers.
template <typename H, int I, int J>
__device__ __forceinline__ void su2_reflect(mat3<H> &U, mat3<H> &W, int &attempts, int &accepts)
{
    const double a0 = double(H(0.5) * (W.e[I][I].re + W.e[J][J].re));
    const double a1 = double(H(0.5) * (W.e[I][J].im + W.e[J][I].im));
    const double a2 = double(H(0.5) * (W.e[I][J].re - W.e[J][I].re));
    const double a3 = double(H(0.5) * (W.e[I][I].im - W.e[J][J].im));
    double ik;
    if (!inv_norm(fma(a0, a0, fma(a1, a1, fma(a2, a2, a3 * a3))), ik)) return;  // degenerate: no reflection
    ++attempts;
    ++accepts;
    const double b0 = a0 * ik, b1 = a1 * ik, b2 = a2 * ik, b3 = a3 * ik;
    // V^dag = [[b0 - i b3, -b2 - i b1], [b2 - i b1, b0 + i b3]], r = V^dag V^dag
    const cx<double> V00{b0, -b3}, V01{-b2, -b1}, V10{b2, -b1}, V11{b0, b3};
    cx<double> q00{0.0, 0.0}, q01{0.0, 0.0}, q10{0.0, 0.0}, q11{0.0, 0.0};
    cfma(q00, V00, V00); cfma(q00, V01, V10);
    cfma(q01, V00, V01); cfma(q01, V01, V11);
    cfma(q10, V10, V00); cfma(q10, V11, V10);
    cfma(q11, V10, V01); cfma(q11, V11, V11);
    rotate_rows<H, I, J>(U, W, cx<H>{H(q00.re), H(q00.im)}, cx<H>{H(q01.re), H(q01.im)},
                         cx<H>{H(q10.re), H(q10.im)}, cx<H>{H(q11.re), H(q11.im)});
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
__device__ __forceinline__ void advance_sweep(const UpdateArgs &a, int D, uint32_t sweep, uint32_t thread = 0)
{
    if (a.mu != D - 1 || blockIdx.x != 0 || threadIdx.x != thread) return;
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
