// split.h -- one link's update shared by lanes and waves.
//
// A slice of a small lattice has fewer links than the chip has lanes, and one
// thread per link (update.hip) then waits for its own serial chain: the
// staples of D - 1 planes one after another, three subgroup draws, the
// rotations.  Here a block of four waves takes 16 links and divides that chain.
//   Staples: lane (t, l) = (lane / 16, lane % 16) takes plane t of link l, so
//     that 16 lanes read 16 consecutive links (256 bytes of a packet); the
//     2 (D - 1) staples of a link meet in LDS.
//   Update: lane (l, c) = (lane / 4, lane % 4) takes column c of U and of
//     W = U A of link l (lane 3 doubles column 2).  A subgroup rotation acts
//     on each column by itself; what a subgroup needs of the other columns,
//     and the draws, come from the neighbouring lanes of the quad by DPP.
//   Draws: lane (l, c) makes the proposals of hits 0 and 1 of subgroup c and
//     their directions, which do not depend on the links, on waves that have
//     nothing else to do.
// Every number is formed by the operations of update_link in their order
// (the staples of a link are summed plane by plane, the backward one first),
// so the links are the same bits.
#pragma once

#include "slice.h"

namespace su3hb {

// Value of lane K of the calling lane's quad.
template <int K>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_mov_dpp(int(v), K * 0x55, 0xf, 0xf, true));
}

template <int K>
__device__ __forceinline__ float quad_lane(float v)
{
    return __uint_as_float(quad_lane<K>(__float_as_uint(v)));
}

template <int K>
__device__ __forceinline__ double quad_lane(double v)
{
    return __hiloint2double(int(quad_lane<K>(uint32_t(__double2hiint(v)))),
                            int(quad_lane<K>(uint32_t(__double2loint(v)))));
}

template <int K, typename T>
__device__ __forceinline__ cx<T> quad_lane(const cx<T> &v)
{
    return cx<T>{quad_lane<K>(v.re), quad_lane<K>(v.im)};
}

// One of three values by a lane's column (by value: a choice between places
// would put them in scratch memory).
template <typename T>
__device__ __forceinline__ cx<T> pick(uint32_t c, cx<T> v0, cx<T> v1, cx<T> v2)
{
    return cx<T>{c == 0 ? v0.re : c == 1 ? v1.re : v2.re, c == 0 ? v0.im : c == 1 ? v1.im : v2.im};
}

// What a subgroup's draw needs of the random numbers: e = ln u1 + cos^2(2 pi
// u2) ln u3 and q = u4^2 of a proposal, and the direction that follows it.
struct Proposal {
    double e, q;
};

template <typename H>
struct Direction {
    H cth, sth, sph, cph;
};

template <typename H>
struct Draw {
    Proposal p;
    Direction<H> d;
};

__device__ __forceinline__ Proposal draw_proposal(uint32_t lid, uint32_t sweep, uint32_t word, uint32_t k0,
                                                  uint32_t k1, const LogEntry *tbl)
{
    const uint4 r = philox4x32_10(make_uint4(lid, sweep, word, kTagUpdate), k0, k1);
    const double c2 = cos2_turn(u01(r.y));
    const double r4 = u01(r.w);
    return Proposal{fma(c2, log_unit(u01(r.z), tbl), log_unit(u01(r.x), tbl)), r4 * r4};
}

template <typename H>
__device__ __forceinline__ Direction<H> draw_direction(uint32_t lid, uint32_t sweep, uint32_t word, uint32_t k0,
                                                       uint32_t k1)
{
    Direction<H> d;
    const uint4 q = philox4x32_10(make_uint4(lid, sweep, word | 1u, kTagUpdate), k0, k1);
    d.cth = H(2.0 * u01(q.x) - 1.0);
    d.sth = sqrt_nonneg<H>(max(H(0), H(1) - d.cth * d.cth));
    sincos_turn<H>(u01(q.y), &d.sph, &d.cph);
    return d;
}

template <int SUB, typename H>
__device__ __forceinline__ Draw<H> quad_draw(const Draw<H> &v)
{
    return Draw<H>{{quad_lane<SUB>(v.p.e), quad_lane<SUB>(v.p.q)},
                   {quad_lane<SUB>(v.d.cth), quad_lane<SUB>(v.d.sth), quad_lane<SUB>(v.d.sph),
                    quad_lane<SUB>(v.d.cph)}};
}

// 1 - x in an operation of its own (x is a product that must not be fused).
__device__ __forceinline__ double one_minus(double x)
{
#pragma clang fp contract(off)
    return 1.0 - x;
}

// The projection of W's 2x2 block (I, J): quaternion a, and 1/k; false for a
// degenerate one.
template <typename H, int I, int J>
__device__ __forceinline__ bool quad_project(const cx<H> w[3], double a[4], double &ik)
{
    const cx<H> wii = quad_lane<I>(w[I]), wij = quad_lane<J>(w[I]);
    const cx<H> wji = quad_lane<I>(w[J]), wjj = quad_lane<J>(w[J]);
    a[0] = double(H(0.5) * (wii.re + wjj.re));
    a[1] = double(H(0.5) * (wij.im + wji.im));
    a[2] = double(H(0.5) * (wij.re - wji.re));
    a[3] = double(H(0.5) * (wii.im - wjj.im));
    return inv_norm(fma(a[0], a[0], fma(a[1], a[1], fma(a[2], a[2], a[3] * a[3]))), ik);
}

template <typename H, int I, int J>
__device__ __forceinline__ void rotate_column(cx<H> v[3], const cx<H> &r00, const cx<H> &r01, const cx<H> &r10,
                                              const cx<H> &r11)
{
    const cx<H> vi = v[I], vj = v[J];
    cx<H> ni{H(0), H(0)}, nj{H(0), H(0)};
    cfma(ni, r00, vi); cfma(ni, r01, vj);
    cfma(nj, r10, vi); cfma(nj, r11, vj);
    v[I] = ni;
    v[J] = nj;
}

// The rotation R = X V^dag of an accepted draw (su2_heatbath).
template <typename H>
__device__ __forceinline__ void heatbath_rotation(const double a[4], double ik, double delta, const Direction<H> &d,
                                                  cx<H> &r00, cx<H> &r01, cx<H> &r10, cx<H> &r11)
{
    const double x0d = one_minus(delta);
    const H x0 = H(x0d);
    const H rad = sqrt_nonneg<H>(H(fmax(0.0, 1.0 - x0d * x0d)));
    const H x1 = rad * d.sth * d.cph, x2 = rad * d.sth * d.sph, x3 = rad * d.cth;
    const H b0 = H(a[0] * ik), b1 = H(a[1] * ik), b2 = H(a[2] * ik), b3 = H(a[3] * ik);
    const cx<H> X00{x0, x3}, X01{x2, x1}, X10{-x2, x1}, X11{x0, -x3};
    const cx<H> V00{b0, -b3}, V01{-b2, -b1}, V10{b2, -b1}, V11{b0, b3};
    r00 = r01 = r10 = r11 = cx<H>{H(0), H(0)};
    cfma(r00, X00, V00); cfma(r00, X01, V10);
    cfma(r01, X00, V01); cfma(r01, X01, V11);
    cfma(r10, X10, V00); cfma(r10, X11, V10);
    cfma(r11, X10, V01); cfma(r11, X11, V11);
}

// One subgroup heatbath on the columns u, w of a quad's link (su2_heatbath).
// own: the lane's draws for hits 0 and 1.  Later hits are
// tried four at a time, one per lane; the first accepted one counts, as in the
// loop over hits.
template <typename H, int I, int J, int SUB>
__device__ __forceinline__ void quad_heatbath(cx<H> u[3], cx<H> w[3], const Draw<H> own[2], uint32_t lid,
                                              uint32_t sweep, int nhit, uint32_t k0, uint32_t k1,
                                              const LogEntry *tbl, int &attempts, int &accepts)
{
    Draw<H> v = quad_draw<SUB>(own[0]);
    double a[4], ik;
    if (!quad_project<H, I, J>(w, a, ik)) return;
    const double inv_alpha = 1.5 * ik;
    double delta = -v.p.e * inv_alpha;
    bool ok = v.p.q <= 1.0 - 0.5 * delta;
    int tried = 1;
    if (!ok && nhit > 1) {
        v = quad_draw<SUB>(own[1]);
        delta = -v.p.e * inv_alpha;
        ok = v.p.q <= 1.0 - 0.5 * delta;
        tried = 2;
    }
    if (!ok) {
        const uint32_t lane = threadIdx.x & 63u, quad = lane & ~3u;
        for (int base = 2; base < nhit; base += 4) {
            const int hit = base + int(lane & 3u);
            const Proposal n =
                draw_proposal(lid, sweep, (uint32_t(SUB) << 16) | (uint32_t(hit) << 1), k0, k1, tbl);
            const double nd = -n.e * inv_alpha;
            const bool good = hit < nhit && n.q <= 1.0 - 0.5 * nd;
            const uint32_t m = uint32_t(__ballot(good) >> quad) & 15u;
            tried = min(base + 4, nhit);
            if (m) {
                const uint32_t k = uint32_t(__builtin_ctz(m));
                delta = __shfl(nd, int(quad + k));
                tried = base + int(k) + 1;
                ok = true;
                break;
            }
        }
        if (ok)
            v.d = draw_direction<H>(lid, sweep, (uint32_t(SUB) << 16) | (uint32_t(tried - 1) << 1), k0, k1);
    }
    attempts += tried;
    if (!ok) return;
    ++accepts;
    cx<H> r00, r01, r10, r11;
    heatbath_rotation<H>(a, ik, delta, v.d, r00, r01, r10, r11);
    rotate_column<H, I, J>(u, r00, r01, r10, r11);
    rotate_column<H, I, J>(w, r00, r01, r10, r11);
}

// One subgroup reflection (su2_reflect).
template <typename H, int I, int J>
__device__ __forceinline__ void quad_reflect(cx<H> u[3], cx<H> w[3], int &attempts, int &accepts)
{
    double a[4], ik;
    if (!quad_project<H, I, J>(w, a, ik)) return;
    ++attempts;
    ++accepts;
    const double b0 = a[0] * ik, b1 = a[1] * ik, b2 = a[2] * ik, b3 = a[3] * ik;
    const cx<double> V00{b0, -b3}, V01{-b2, -b1}, V10{b2, -b1}, V11{b0, b3};
    cx<double> q00{0.0, 0.0}, q01{0.0, 0.0}, q10{0.0, 0.0}, q11{0.0, 0.0};
    cfma(q00, V00, V00); cfma(q00, V01, V10);
    cfma(q01, V00, V01); cfma(q01, V01, V11);
    cfma(q10, V10, V00); cfma(q10, V11, V10);
    cfma(q11, V10, V01); cfma(q11, V11, V11);
    const cx<H> r00{H(q00.re), H(q00.im)}, r01{H(q01.re), H(q01.im)}, r10{H(q10.re), H(q10.im)},
        r11{H(q11.re), H(q11.im)};
    rotate_column<H, I, J>(u, r00, r01, r10, r11);
    rotate_column<H, I, J>(w, r00, r01, r10, r11);
}

// Places of a block's 16 links in LDS: the staples element by
// element, 16 links to a row; rows are padded so that the three columns that
// a quad reads lie in different banks.  Two layers: the weight and the
// measurement class of every staple follow.
template <int D, int PREC>
struct SplitLds {
    using R = typename Store<PREC>::real;
    static constexpr int kStaples = 2 * (D - 1);
    static constexpr int kRow = sizeof(R) == 8 ? 20 : 24;
    static constexpr size_t kMatrixBytes = size_t(kStaples) * 9 * kRow * sizeof(cx<R>);
    static constexpr size_t kWeightBytes = size_t(kStaples) * kSplitLinks * (sizeof(R) + sizeof(uint32_t));
    static constexpr size_t kBytes = kMatrixBytes + kWeightBytes;
    cx<R> *m;
    R *weight;
    uint32_t *cls;

    __device__ __forceinline__ explicit SplitLds(char *base)
        : m(reinterpret_cast<cx<R> *>(base)), weight(reinterpret_cast<R *>(base + kMatrixBytes)),
          cls(reinterpret_cast<uint32_t *>(weight + kStaples * kSplitLinks))
    {
    }
    // element e of staple j (2 t forward, 2 t + 1 backward) of link l
    __device__ __forceinline__ cx<R> &at(uint32_t j, uint32_t e, uint32_t l) { return m[(j * 9u + e) * kRow + l]; }
};

// One step along a direction that differs between the lanes.
template <int D, bool FWD>
__device__ __forceinline__ Step step_lane(const RepDesc &rep, const Site<D> &x, uint32_t dir, uint32_t glued)
{
    uint32_t st = rep.stride[0], n = uint32_t(rep.n[0]);
#pragma unroll
    for (uint32_t i = 1; i < uint32_t(D); ++i) {
        st = dir == i ? rep.stride[i] : st;
        n = dir == i ? uint32_t(rep.n[i]) : n;
    }
    const bool wrap = ((FWD ? x.hi : x.lo) >> dir) & 1u;
    const int32_t span = int32_t((n - 1u) * st);
    Step s;
    s.ds = FWD ? (wrap ? -span : int32_t(st)) : (wrap ? span : -int32_t(st));
    s.flip = wrap ? ((glued >> dir) & 1u) : 0u;
    return s;
}

// (F1 (F3 F2)^dag) and ((B2 B1)^dag B3): the operations of acc_plane_staples.
template <typename R>
__device__ __forceinline__ mat3<R> two_rows(const mat3<R> &a, const mat3<R> &b)
{
    mat3<R> m;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            cx<R> s{R(0), R(0)};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma(s, a.e[j][k], b.e[k][i]);
            m.e[j][i] = s;
        }
    third_row(m);
    return m;
}

template <typename R>
__device__ __forceinline__ mat3<R> forward_staple(const mat3<R> &f1, const mat3<R> &f2, const mat3<R> &f3)
{
    const mat3<R> M = two_rows(f3, f2);
    mat3<R> q;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<R> s{R(0), R(0)};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma_nc(s, f1.e[r][k], M.e[j][k]);
            q.e[r][j] = s;
        }
    third_row(q);
    return q;
}

template <typename R>
__device__ __forceinline__ mat3<R> backward_staple(const mat3<R> &b1, const mat3<R> &b2, const mat3<R> &b3)
{
    const mat3<R> N = two_rows(b2, b1);
    mat3<R> q;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<R> s{R(0), R(0)};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma_cn(s, N.e[k][r], b3.e[k][j]);
            q.e[r][j] = s;
        }
    third_row(q);
    return q;
}

// What a wave's links add to the counters and the measurement; lanes 0 of the
// quads hold the values.
template <int NC>
struct SplitSums {
    int att[3] = {0, 0, 0}, acc[3] = {0, 0, 0}, upd = 0;
    double dtrace = 0.0, plaq[NC] = {};
};

// A lane's link: its site and place.
template <int D>
struct SplitSite {
    Site<D> x;
    uint32_t layer;
    bool valid;

    __device__ __forceinline__ SplitSite(const RepDesc &rep, uint32_t lt, int p)
    {
        // lanes past the last link work on it too and leave no trace
        const uint32_t total = rep.nlat * rep.Vh;
        valid = lt < total;
        lt = min(lt, total - 1u);
        layer = lt >= rep.Vh ? 1u : 0u;
        x.template from_half<true>(rep, lt - layer * rep.Vh, p, layer);
    }
};

// The forward or the backward staples of 16 links, first .. first + 15, into
// LDS, by one wave; POLICY: of the loads.
template <int D, int PREC, bool FWD, int POLICY>
__device__ __forceinline__ void split_staples(const UpdateArgs &a, const RepDesc &rep, uint32_t first,
                                              SplitLds<D, PREC> lds)
{
    using R = typename Store<PREC>::real;
    constexpr uint32_t NT = D - 1;
    const uint32_t l = threadIdx.x & 15u, t = (threadIdx.x >> 4) & 3u;
    const uint32_t mu = uint32_t(a.mu);
    const int p = a.parity, q = 1 - p;
    const SplitSite<D> s(rep, first + l, p);
    const Site<D> &x = s.x;
    const uint32_t layer = s.layer;
    const bool single = rep.nlat == 1;
    const uint32_t glued = single ? 0u : rep.glued;
    const double beta0 = a.use_rep_beta ? rep.beta0 : a.beta0;
    const double beta1 = a.use_rep_beta ? rep.beta1 : a.beta1;
    const Step fm = step_fwd<D>(rep, x, a.mu, glued);
    const uint32_t s_pm = x.s + uint32_t(fm.ds), l_pm = layer ^ fm.flip;
#pragma unroll
    for (uint32_t t0 = 0; t0 < NT; t0 += 4) {
        const uint32_t tp = t0 + t;
        if (tp >= NT) break;
        const uint32_t nu = tp + (tp >= mu ? 1u : 0u);
        const Step bn = step_lane<D, false>(rep, x, nu, glued);
        const uint32_t l_mn = layer ^ bn.flip, l_pmmn = l_pm ^ bn.flip;
        if constexpr (FWD) {
            const Step fn = step_lane<D, true>(rep, x, nu, glued);
            const uint32_t s_pn = x.s + uint32_t(fn.ds), l_pn = layer ^ fn.flip;
            const mat3<R> f3 = load_rows01<PREC, POLICY>(link_ref<D, PREC>(a.links, rep, layer, int(nu), p, x.s));
            // the first plane reads U_mu(x + nu) whole, the others rebuild
            // row 2 (as update_link)
            const LinkRef r2 = link_ref<D, PREC>(a.links, rep, l_pn, a.mu, q, s_pn);
            const mat3<R> f1 = load_rows01<PREC, POLICY>(link_ref<D, PREC>(a.links, rep, l_pm, int(nu), q, s_pm));
            mat3<R> f2 = load_rows01<PREC, POLICY>(r2);
            if (Store<PREC>::NE == 9 && tp == 0) {
#pragma unroll
                for (int e = 6; e < Store<PREC>::NE; ++e) f2.e[2][e - 6] = load_elem<PREC, POLICY>(r2, e);
            } else {
                third_row(f2);
            }
            const mat3<R> m = forward_staple(f1, f2, f3);
#pragma unroll
            for (uint32_t e = 0; e < 9; ++e) lds.at(2 * tp, e, l) = m.e[e / 3][e % 3];
            if (!single) {
                const uint32_t tags = layer + l_pm + l_pn + layer;
                lds.weight[2 * tp * kSplitLinks + l] = R(tags == 0 ? beta0 : beta1);
                lds.cls[2 * tp * kSplitLinks + l] = layer == 0 ? (tags == 0 ? 0u : 1u) : 2u;
            }
        } else {
            const uint32_t s_mn = x.s + uint32_t(bn.ds), s_pmmn = s_pm + uint32_t(bn.ds);
            const mat3<R> b2 = load_rows01<PREC, POLICY>(link_ref<D, PREC>(a.links, rep, l_mn, a.mu, q, s_mn));
            const mat3<R> b1 = load_link<PREC, POLICY>(link_ref<D, PREC>(a.links, rep, l_pmmn, int(nu), p, s_pmmn));
            const mat3<R> b3 = load_link<PREC, POLICY>(link_ref<D, PREC>(a.links, rep, l_mn, int(nu), q, s_mn));
            const mat3<R> m = backward_staple(b1, b2, b3);
            const uint32_t j = 2 * tp + 1;
#pragma unroll
            for (uint32_t e = 0; e < 9; ++e) lds.at(j, e, l) = m.e[e / 3][e % 3];
            if (!single) {
                const uint32_t tags = l_mn + l_pmmn + layer + l_mn;
                lds.weight[j * kSplitLinks + l] = R(tags == 0 ? beta0 : beta1);
                lds.cls[j * kSplitLinks + l] = l_mn == 0 ? (tags == 0 ? 0u : 1u) : 2u;
            }
        }
    }
}

// The Philox word of a hit of the lane's subgroup (lane % 4, at most 2).
__device__ __forceinline__ uint32_t split_word(uint32_t hit)
{
    return (min(threadIdx.x & 3u, 2u) << 16) | (hit << 1);
}

template <int D>
__device__ __forceinline__ uint32_t split_lid(const RepDesc &rep, const SplitSite<D> &s, int mu)
{
    return ((rep.lat2test ? 0u : s.layer * rep.V) + s.x.s) * uint32_t(D) + uint32_t(mu);
}

// Column c of a link's staple sum A, and of its part with nu < mu (NC = 3: by
// class).
template <int PREC, int NC>
struct SplitColumn {
    cx<typename Store<PREC>::real> A[3], low[NC][3];
};

template <int NC>
__device__ __forceinline__ bool split_measures(const UpdateArgs &a, const RepDesc &rep)
{
    return a.meas != nullptr && a.parity == 1 && (NC == 3 || rep.nlat == 1);
}

// The lane's column from the staples in LDS.
template <int D, int PREC, int NC>
__device__ __forceinline__ SplitColumn<PREC, NC> split_sum(const UpdateArgs &a, const RepDesc &rep,
                                                           SplitLds<D, PREC> lds)
{
    using R = typename Store<PREC>::real;
    const uint32_t l = (threadIdx.x & 63u) >> 2, c = min(threadIdx.x & 3u, 2u);
    const bool single = rep.nlat == 1, measure = split_measures<NC>(a, rep);
    const double beta0 = a.use_rep_beta ? rep.beta0 : a.beta0;
    SplitColumn<PREC, NC> col;
    auto &A = col.A;
    auto &low = col.low;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        A[i] = cx<R>{R(0), R(0)};
#pragma unroll
        for (int k = 0; k < NC; ++k) low[k][i] = cx<R>{R(0), R(0)};
    }
#pragma unroll
    for (uint32_t t = 0; t < uint32_t(D) - 1u; ++t) {
        R wf = R(1), wb = R(1);
        uint32_t cf = 0, cb = 0;
        if (!single) {
            wf = lds.weight[2 * t * kSplitLinks + l];
            wb = lds.weight[(2 * t + 1) * kSplitLinks + l];
            cf = lds.cls[2 * t * kSplitLinks + l];
            cb = lds.cls[(2 * t + 1) * kSplitLinks + l];
        }
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i) {
            const cx<R> f = lds.at(2 * t, i * 3 + c, l), b = lds.at(2 * t + 1, i * 3 + c, l);
            A[i].re = fma(wf, f.re, fma(wb, b.re, A[i].re));
            A[i].im = fma(wf, f.im, fma(wb, b.im, A[i].im));
            if (NC == 1) {
                if (measure && int(t) < a.mu) low[0][i] = A[i];
            } else if (measure && int(t) < a.mu) {
#pragma unroll
                for (uint32_t k = 0; k < uint32_t(NC); ++k) {
                    if (cf == k) {
                        low[k][i].re += f.re;
                        low[k][i].im += f.im;
                    }
                    if (cb == k) {
                        low[k][i].re += b.re;
                        low[k][i].im += b.im;
                    }
                }
            }
        }
    }
    if (single) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            A[i].re *= R(beta0);
            A[i].im *= R(beta0);
        }
    }
    return col;
}

// The update of the wave's 16 links.
template <int D, int PREC, int NC>
__device__ __forceinline__ void split_update(const UpdateArgs &a, const RepDesc &rep, const SplitSite<D> &s,
                                             uint32_t sweep, const SplitColumn<PREC, NC> &col,
                                             const mat3<typename Store<PREC>::real> &U,
                                             const Draw<typename Store<PREC>::real> draw[2], const LinkRef &uptr,
                                             const LogEntry *tbl, SplitSums<NC> &sums)
{
    using R = typename Store<PREC>::real;
    const uint32_t c4 = threadIdx.x & 3u, c = min(c4, 2u);
    const bool measure = split_measures<NC>(a, rep);
    const auto &low = col.low;
    cx<R> u[3], w[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        u[i] = pick(c, U.e[i][0], U.e[i][1], U.e[i][2]);
        w[i] = cx<R>{R(0), R(0)};
#pragma unroll
        for (int k = 0; k < 3; ++k) cfma(w[i], U.e[i][k], col.A[k]);
    }
    const bool counted = a.stats != nullptr;
    double tr_old = 0.0;
    if (counted) tr_old = double(quad_lane<0>(w[0].re)) + double(quad_lane<1>(w[1].re)) + double(quad_lane<2>(w[2].re));

    int att[3] = {0, 0, 0}, acc[3] = {0, 0, 0};
    if (a.nhit > 0) {
        const uint32_t lid = split_lid<D>(rep, s, a.mu);
        quad_heatbath<R, 0, 1, 0>(u, w, draw, lid, sweep, a.nhit, rep.key0, rep.key1, tbl, att[0], acc[0]);
        quad_heatbath<R, 0, 2, 1>(u, w, draw, lid, sweep, a.nhit, rep.key0, rep.key1, tbl, att[1], acc[1]);
        quad_heatbath<R, 1, 2, 2>(u, w, draw, lid, sweep, a.nhit, rep.key0, rep.key1, tbl, att[2], acc[2]);
    } else {
        quad_reflect<R, 0, 1>(u, w, att[0], acc[0]);
        quad_reflect<R, 0, 2>(u, w, att[1], acc[1]);
        quad_reflect<R, 1, 2>(u, w, att[2], acc[2]);
    }
    const bool mine = c4 == 0 && s.valid;
    if (counted) {
        const double tr =
            double(quad_lane<0>(w[0].re)) + double(quad_lane<1>(w[1].re)) + double(quad_lane<2>(w[2].re));
        if (mine) {
            sums.dtrace += (tr - tr_old) * (1.0 / 3.0);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                sums.att[i] += att[i];
                sums.acc[i] += acc[i];
            }
            ++sums.upd;
        }
    }

    // reunitarisation of rows 0 and 1, gathered in every lane of the quad
    mat3<double> Ud;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const cx<double> v{double(u[i].re), double(u[i].im)};
        Ud.e[i][0] = quad_lane<0>(v);
        Ud.e[i][1] = quad_lane<1>(v);
        Ud.e[i][2] = quad_lane<2>(v);
    }
    reunitarize(Ud);
    if (measure) {
        // Re Tr(U' A_low): row i of U' meets column i of A_low in lane i, the
        // running sum goes from lane to lane (the order of re_tr_nn)
        const mat3<R> Us = stored_form_r<PREC>(Ud);
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            R sum = R(0);
#define SU3HB_ROW(I)                                                                                  \
    {                                                                                                 \
        R v = sum;                                                                                    \
        for (int j = 0; j < 3; ++j)                                                                   \
            v = fma(Us.e[I][j].re, low[k][j].re, fma(-Us.e[I][j].im, low[k][j].im, v));               \
        sum = quad_lane<I>(v);                                                                        \
    }
            SU3HB_ROW(0)
            SU3HB_ROW(1)
            SU3HB_ROW(2)
#undef SU3HB_ROW
            if (mine) sums.plaq[k] += double(sum) * (1.0 / 3.0);
        }
    }
    if (mine) store_link<PREC, false>(uptr, Ud);
}

// A wave's counters into a slot of the statistics, its measurement into the
// partial sums of its group, of the place-th measured sweep.
template <int D, int NC, int FIRST = 4>
__device__ __forceinline__ void split_flush(const UpdateArgs &a, uint32_t group, uint32_t place, SplitSums<NC> &v)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (a.meas != nullptr && a.parity == 1) {
#pragma unroll
        for (int off = FIRST; off < 64; off <<= 1)
#pragma unroll
            for (int k = 0; k < NC; ++k) v.plaq[k] += __shfl_xor(v.plaq[k], off);
        if (lane == 0) {
            double *m = meas_of_block<D, NC>(a, place, group);
#pragma unroll
            for (int k = 0; k < NC; ++k) m[k] = v.plaq[k];
        }
    }
    if (a.stats == nullptr) return;
#pragma unroll
    for (int off = FIRST; off < 64; off <<= 1) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            v.att[i] += __shfl_xor(v.att[i], off);
            v.acc[i] += __shfl_xor(v.acc[i], off);
        }
        v.upd += __shfl_xor(v.upd, off);
        v.dtrace += __shfl_xor(v.dtrace, off);
    }
    if (lane == 0) {
        StatSlot *sl = &a.stats[group % kStatSlots];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            atomicAdd(&sl->attempts[i], (unsigned long long)v.att[i]);
            atomicAdd(&sl->accepts[i], (unsigned long long)v.acc[i]);
        }
        atomicAdd(&sl->updates, (unsigned long long)v.upd);
        unsafeAtomicAdd(&sl->dtrace, v.dtrace);
    }
}

}  // namespace su3hb
