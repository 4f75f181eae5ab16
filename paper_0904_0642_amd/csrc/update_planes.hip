// update_planes.hip -- slice updates of middle-sized lattices and batches: the
// planes of a link's staple on waves of their own.
//
// One thread per link (update.hip) leaves SIMDs idle up to some 64 thousand
// links and waits for the staples of D - 1 planes one after another; sharing
// a link among lanes (split.h) costs twice the work (the lines between the
// three: layout.h).  Here a block takes 64
// links with D waves, a lane per link in each: wave t < D - 1 makes both
// staples of plane t and, while its loads are on the way, the second hits'
// draws of subgroup t; the last wave draws the first hits meanwhile, sums the
// staples from LDS and updates.  Every number is formed by the operations of
// update_link in their order, so the links are the same bits.
#include "kernels.h"
#include "split.h"

namespace su3hb {

// A block's 64 links in LDS: the staples element by element (2 t forward, 2 t
// + 1 backward), the second hits' draws, and on two layers the weight and the
// measurement class of every staple.
template <int D, int PREC>
struct PlanesLds {
    using R = typename Store<PREC>::real;
    cx<R> m[2 * (D - 1) * 9][kPlanesLinks];
    Draw<R> second[3][kPlanesLinks];
    LogEntry table[128];
    R weight[2 * (D - 1)][kPlanesLinks];
    uint32_t cls[2 * (D - 1)][kPlanesLinks];
};

template <typename R>
__device__ __forceinline__ Draw<R> planes_draw(uint32_t lid, uint32_t sweep, uint32_t sub, uint32_t hit, uint32_t k0,
                                               uint32_t k1, const LogEntry *tbl)
{
    const uint32_t word = (sub << 16) | (hit << 1);
    return Draw<R>{draw_proposal(lid, sweep, word, k0, k1, tbl), draw_direction<R>(lid, sweep, word, k0, k1)};
}

// su2_heatbath with the draws of hits 0 and 1 in hand.
template <typename H, int I, int J, int SUB>
__device__ __forceinline__ void planes_heatbath(mat3<H> &U, mat3<H> &W, const Draw<H> &first, const Draw<H> &second,
                                                uint32_t lid, uint32_t sweep, int nhit, uint32_t k0, uint32_t k1,
                                                const LogEntry *tbl, int &attempts, int &accepts)
{
    double a[4], ik;
    a[0] = double(H(0.5) * (W.e[I][I].re + W.e[J][J].re));
    a[1] = double(H(0.5) * (W.e[I][J].im + W.e[J][I].im));
    a[2] = double(H(0.5) * (W.e[I][J].re - W.e[J][I].re));
    a[3] = double(H(0.5) * (W.e[I][I].im - W.e[J][J].im));
    if (!inv_norm(fma(a[0], a[0], fma(a[1], a[1], fma(a[2], a[2], a[3] * a[3]))), ik)) return;
    const double inv_alpha = 1.5 * ik;
    Direction<H> d = first.d;
    double delta = -first.p.e * inv_alpha;
    bool ok = first.p.q <= 1.0 - 0.5 * delta;
    int tried = 1;
    if (!ok && nhit > 1) {
        d = second.d;
        delta = -second.p.e * inv_alpha;
        ok = second.p.q <= 1.0 - 0.5 * delta;
        tried = 2;
        if (!ok) {
            for (; tried < nhit && !ok; ++tried) {
                const Proposal n =
                    draw_proposal(lid, sweep, (uint32_t(SUB) << 16) | (uint32_t(tried) << 1), k0, k1, tbl);
                delta = -n.e * inv_alpha;
                ok = n.q <= 1.0 - 0.5 * delta;
            }
            if (ok) d = draw_direction<H>(lid, sweep, (uint32_t(SUB) << 16) | (uint32_t(tried - 1) << 1), k0, k1);
        }
    }
    attempts += tried;
    if (!ok) return;
    ++accepts;
    cx<H> r00, r01, r10, r11;
    heatbath_rotation<H>(a, ik, delta, d, r00, r01, r10, r11);
    rotate_rows<H, I, J>(U, W, r00, r01, r10, r11);
}

// The sum of a link's weighted staples.
template <int D, int PREC>
__device__ __forceinline__ mat3<typename Store<PREC>::real> planes_sum(const PlanesLds<D, PREC> &s, uint32_t lane,
                                                                       bool single)
{
    using R = typename Store<PREC>::real;
    mat3<R> A;
    set_zero(A);
#pragma unroll
    for (int t = 0; t < D - 1; ++t) {
        R wf = R(1), wb = R(1);
        if (!single) {
            wf = s.weight[2 * t][lane];
            wb = s.weight[2 * t + 1][lane];
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const cx<R> f = s.m[18 * t + e][lane], b = s.m[18 * t + 9 + e][lane];
            cx<R> &v = A.e[e / 3][e % 3];
            v.re = fma(wf, f.re, fma(wb, b.re, v.re));
            v.im = fma(wf, f.im, fma(wb, b.im, v.im));
        }
    }
    return A;
}

// The unweighted sum of the planes nu < mu (NC = 3: of class k).
template <int D, int PREC, int NC>
__device__ __forceinline__ mat3<typename Store<PREC>::real> planes_low(const PlanesLds<D, PREC> &s, uint32_t lane,
                                                                       int mu, uint32_t k)
{
    using R = typename Store<PREC>::real;
    mat3<R> A;
    set_zero(A);
#pragma unroll 1
    for (int t = 0; t < mu; ++t) {
        const bool tf = NC == 1 || s.cls[2 * t][lane] == k, tb = NC == 1 || s.cls[2 * t + 1][lane] == k;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const cx<R> f = s.m[18 * t + e][lane], b = s.m[18 * t + 9 + e][lane];
            cx<R> &v = A.e[e / 3][e % 3];
            if (NC == 1) {
                v.re = f.re + (b.re + v.re);
                v.im = f.im + (b.im + v.im);
            } else {
                if (tf) {
                    v.re += f.re;
                    v.im += f.im;
                }
                if (tb) {
                    v.re += b.re;
                    v.im += b.im;
                }
            }
        }
    }
    return A;
}

// One slice.  Bound by one chain per block (a load, a staple, the sum and the
// update) and, where two or three blocks share a CU, by the rate of FP64
// arithmetic beside it: 16^4 FP64-18 (32768 links, two blocks on each CU) 16.1 us
// shared by lanes, 17.6 us one thread per link, 13.5 us here; 24 x 16^3 FP32-12
// (49152 links, three) 14.3, 13.3 and 11.3 us.  The second hits' draws on the
// waves of the planes: without them 13.9 and 10.2 us (16^4) for 13.6 and 9.9; all
// loads of a plane ahead of them, or four FP32 blocks on a CU, spill registers
// (15.0 us and 12.6 us); a higher priority for the updating wave changes nothing.
template <int D, int PREC, int NC>
__global__ void __launch_bounds__(64 * D, 2) update_planes_kernel(UpdateArgs a)
{
    using R = typename Store<PREC>::real;
    __shared__ PlanesLds<D, PREC> s;
    const uint32_t sweep = a.sweep[a.parity];
    const uint32_t lane = threadIdx.x & 63u, t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t group = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (group >= a.total_blocks) return;
    const RepDesc &rep = a.reps[a.nrep == 1 ? 0 : find_replica(a.reps, a.nrep, group, kPlanesBlocks)];
    const SplitSite<D> site(rep, (group - rep.planes_block0) * kPlanesLinks + lane, a.parity);
    const Site<D> &x = site.x;
    const uint32_t layer = site.layer;
    const int p = a.parity, q = 1 - p;
    const bool single = rep.nlat == 1;
    const double beta0 = a.use_rep_beta ? rep.beta0 : a.beta0;
    const uint32_t lid = split_lid<D>(rep, site, a.mu);
    for (uint32_t i = threadIdx.x; i < 128u; i += 64u * D) s.table[i] = kLogTable[i];
    if (t < uint32_t(D) - 1u) {
        const uint32_t glued = single ? 0u : rep.glued;
        const double beta1 = a.use_rep_beta ? rep.beta1 : a.beta1;
        const int nu = int(t) + (int(t) >= a.mu ? 1 : 0);
        const Step fm = step_fwd<D>(rep, x, a.mu, glued);
        const Step fn = step_fwd<D>(rep, x, nu, glued), bn = step_bwd<D>(rep, x, nu, glued);
        const uint32_t s_pm = x.s + uint32_t(fm.ds), l_pm = layer ^ fm.flip;
        const uint32_t s_pn = x.s + uint32_t(fn.ds), l_pn = layer ^ fn.flip;
        const uint32_t s_mn = x.s + uint32_t(bn.ds), l_mn = layer ^ bn.flip;
        const uint32_t s_pmmn = s_pm + uint32_t(bn.ds), l_pmmn = l_pm ^ bn.flip;
        const mat3<R> f3 = load_rows01<PREC>(link_ref<D, PREC>(a.links, rep, layer, nu, p, x.s));
        // the first plane reads U_mu(x + nu) whole, the others rebuild row 2
        // (as update_link)
        const LinkRef r2 = link_ref<D, PREC>(a.links, rep, l_pn, a.mu, q, s_pn);
        const mat3<R> f1 = load_rows01<PREC>(link_ref<D, PREC>(a.links, rep, l_pm, nu, q, s_pm));
        mat3<R> f2 = load_rows01<PREC>(r2);
        if (Store<PREC>::NE == 9 && t == 0) {
#pragma unroll
            for (int e = 6; e < Store<PREC>::NE; ++e) f2.e[2][e - 6] = load_elem<PREC>(r2, e);
        }
        __syncthreads();
        if (a.nhit > 1) {
            // wave t draws for subgroup t, the last one also for those left
            const uint32_t last = t == uint32_t(D) - 2u ? 2u : t;
            for (uint32_t sub = t; sub <= last; ++sub)
                s.second[sub][lane] = planes_draw<R>(lid, sweep, sub, 1, rep.key0, rep.key1, s.table);
        }
        if (!(Store<PREC>::NE == 9 && t == 0)) third_row(f2);
        const mat3<R> mf = forward_staple(f1, f2, f3);
#pragma unroll
        for (int e = 0; e < 9; ++e) s.m[18 * t + e][lane] = mf.e[e / 3][e % 3];
        const mat3<R> b2 = load_rows01<PREC>(link_ref<D, PREC>(a.links, rep, l_mn, a.mu, q, s_mn));
        const mat3<R> b1 = load_link<PREC>(link_ref<D, PREC>(a.links, rep, l_pmmn, nu, p, s_pmmn));
        const mat3<R> b3 = load_link<PREC>(link_ref<D, PREC>(a.links, rep, l_mn, nu, q, s_mn));
        const mat3<R> mb = backward_staple(b1, b2, b3);
#pragma unroll
        for (int e = 0; e < 9; ++e) s.m[18 * t + 9 + e][lane] = mb.e[e / 3][e % 3];
        if (!single) {
            const uint32_t tags_f = layer + l_pm + l_pn + layer, tags_b = l_mn + l_pmmn + layer + l_mn;
            s.weight[2 * t][lane] = R(tags_f == 0 ? beta0 : beta1);
            s.weight[2 * t + 1][lane] = R(tags_b == 0 ? beta0 : beta1);
            s.cls[2 * t][lane] = layer == 0 ? (tags_f == 0 ? 0u : 1u) : 2u;
            s.cls[2 * t + 1][lane] = l_mn == 0 ? (tags_b == 0 ? 0u : 1u) : 2u;
        }
        __syncthreads();
        return;
    }

    const LinkRef uptr = link_ref<D, PREC>(a.links, rep, layer, a.mu, p, x.s);
    mat3<R> U = load_link<PREC>(uptr);
    __syncthreads();
    Draw<R> first[3] = {};
    if (a.nhit > 0) {
#pragma unroll
        for (uint32_t sub = 0; sub < 3; ++sub)
            first[sub] = planes_draw<R>(lid, sweep, sub, 0, rep.key0, rep.key1, s.table);
    }
    __syncthreads();
    mat3<R> A = planes_sum<D, PREC>(s, lane, single);
    if (single) scale(A, R(beta0));
    mat3<R> W = mul_nn(U, A);
    const double tr_old = double(W.e[0][0].re) + double(W.e[1][1].re) + double(W.e[2][2].re);
    int att[3] = {0, 0, 0}, acc[3] = {0, 0, 0};
    if (a.nhit > 0) {
        planes_heatbath<R, 0, 1, 0>(U, W, first[0], s.second[0][lane], lid, sweep, a.nhit, rep.key0, rep.key1, s.table,
                                    att[0], acc[0]);
        planes_heatbath<R, 0, 2, 1>(U, W, first[1], s.second[1][lane], lid, sweep, a.nhit, rep.key0, rep.key1, s.table,
                                    att[1], acc[1]);
        planes_heatbath<R, 1, 2, 2>(U, W, first[2], s.second[2][lane], lid, sweep, a.nhit, rep.key0, rep.key1, s.table,
                                    att[2], acc[2]);
    } else {
        su2_reflect<R, 0, 1>(U, W, att[0], acc[0]);
        su2_reflect<R, 0, 2>(U, W, att[1], acc[1]);
        su2_reflect<R, 1, 2>(U, W, att[2], acc[2]);
    }
    SplitSums<NC> sums;
    if (site.valid) {
        sums.dtrace = (double(W.e[0][0].re) + double(W.e[1][1].re) + double(W.e[2][2].re) - tr_old) * (1.0 / 3.0);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            sums.att[i] = att[i];
            sums.acc[i] = acc[i];
        }
        sums.upd = 1;
    }
    mat3<double> Ud = widen<double>(U);
    reunitarize(Ud);
    if (split_measures<NC>(a, rep)) {
        const mat3<R> Us = stored_form_r<PREC>(Ud);
#pragma unroll 1
        for (int k = 0; k < NC; ++k) {
            const double v = double(re_tr_nn(Us, planes_low<D, PREC, NC>(s, lane, a.mu, uint32_t(k)))) * (1.0 / 3.0);
            if (site.valid) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (c == k) sums.plaq[c] = v;
            }
        }
    }
    if (site.valid) store_link<PREC, false>(uptr, Ud);
    split_flush<D, NC, 1>(a, group, a.meas != nullptr ? a.sweep[3] : 0u, sums);
    advance_sweep(a, D, sweep, 64u * (D - 1));
}

template <int D, int PREC>
static hipError_t launch_planes_t(hipStream_t st, const UpdateArgs &a)
{
    const dim3 grid((a.total_blocks + 7) / 8 * 8), block(64 * D);
    if (a.meas != nullptr && a.parity == 1 && a.meas_classes == 3)
        return launch_kernel(update_planes_kernel<D, PREC, 3>, grid, block, st, a);
    return launch_kernel(update_planes_kernel<D, PREC, 1>, grid, block, st, a);
}

template <int D>
hipError_t launch_planes_d(int prec, hipStream_t st, const UpdateArgs &a)
{
    switch (prec) {
    case kFP64_18: return launch_planes_t<D, kFP64_18>(st, a);
    case kFP32_18: return launch_planes_t<D, kFP32_18>(st, a);
    case kFP32_12: return launch_planes_t<D, kFP32_12>(st, a);
    case kFP64_12: return launch_planes_t<D, kFP64_12>(st, a);
    default: return hipErrorInvalidValue;
    }
}

#ifdef SU3HB_DIM  // as in update.hip
template hipError_t launch_planes_d<SU3HB_DIM>(int, hipStream_t, const UpdateArgs &);
#else
extern template hipError_t launch_planes_d<3>(int, hipStream_t, const UpdateArgs &);
extern template hipError_t launch_planes_d<4>(int, hipStream_t, const UpdateArgs &);

hipError_t launch_update_planes(int D, int prec, hipStream_t st, const UpdateArgs &a)
{
    switch (D) {
    case 3: return launch_planes_d<3>(prec, st, a);
    case 4: return launch_planes_d<4>(prec, st, a);
    default: return hipErrorInvalidValue;
    }
}
#endif

}  // namespace su3hb
