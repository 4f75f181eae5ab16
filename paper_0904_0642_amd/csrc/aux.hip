// aux.hip -- plaquette measurement (paper Sec. 2.4 measurement step) with
// FP64 accumulation, start configurations (Sec. 2.3 istart), conversion
// between the canonical FP64 layout and the internal storage, SU(3) input
// validation, and small counter kernels.
#include "geometry.h"
#include "kernels.h"

namespace su3hb {

// ---------------------------------------------------------------------------
// plaquettes

// Reduce NV doubles over the block; thread 0 returns the sums.  Fixed order
// for a fixed block size, so repeated measurements agree bit for bit.
template <int NV>
__device__ __forceinline__ void block_sum(double v[NV])
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] += __shfl_xor(v[i], off);
    __shared__ double s[4][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < NV; ++i) s[wave][i] = v[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        for (int w = 1; w < nw; ++w)
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] += s[w][i];
    }
}

// Plane k of D(D-1)/2 as (mu, nu), mu < nu, in the order (0,1), (0,2), ...
template <int D>
__device__ __forceinline__ void plane_dirs(int k, int &mu, int &nu)
{
    mu = 0;
    nu = 1;
#pragma unroll
    for (int m = 0, c = 0; m < D; ++m)
#pragma unroll
        for (int n = m + 1; n < D; ++n, ++c)
            if (c == k) {
                mu = m;
                nu = n;
            }
}

// One thread per (site, plane) item (`spt` items per thread, strided by the
// block size; items plane-major, so a wave reads consecutive sites):
// (1/3) Re Tr[U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag] = (1/3) Re Tr(T1 T2^dag)
// with T1 = U_mu(x) U_nu(x+mu), T2 = U_nu(x) U_mu(x+nu); products in FP64.
// Partial sums per block: [spacelike, timelike, layer0, layer1, beta-weighted].
template <int D, int PREC>
__global__ void __launch_bounds__(256) plaquette_kernel(PlaqArgs a)
{
    constexpr int NPL = D * (D - 1) / 2;
    const uint32_t lb = blockIdx.x;
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (lb < a.total_blocks) {
        const int r = a.nrep == 1 ? 0 : find_replica(a.reps, a.nrep, lb, kPlaquetteBlocks);
        const RepDesc &rep = a.reps[r];
        const uint32_t glued = rep.nlat == 2 ? rep.glued : 0u;
        const double beta0 = a.use_rep_beta ? rep.beta0 : a.beta0;
        const double beta1 = a.use_rep_beta ? rep.beta1 : a.beta1;
        void *links = const_cast<void *>(a.links);
        // items can outnumber links ((D-1)/2 per link): 64-bit item index
        const uint32_t nsite = rep.nlat * rep.V;
        const uint64_t nitem = uint64_t(nsite) * uint64_t(NPL);
        const uint64_t first = uint64_t(lb - rep.plq_block0) * blockDim.x * rep.plq_spt + threadIdx.x;
        for (uint32_t j = 0; j < rep.plq_spt; ++j) {
            const uint64_t it = first + uint64_t(j) * blockDim.x;
            if (it >= nitem) break;
            const int k = int(it / nsite);
            const uint32_t lt = uint32_t(it - uint64_t(k) * nsite);
            const uint32_t layer = lt >= rep.V ? 1u : 0u;
            const uint32_t rem = lt - layer * rep.V;
            const int p = rem >= rep.Vh ? 1 : 0;
            const uint32_t h = rem - uint32_t(p) * rep.Vh;
            Site<D> x;
            x.from_half(rep, h, p, layer);
            const int q = 1 - p;
            int mu, nu;
            plane_dirs<D>(k, mu, nu);
            const Step fm = step_fwd<D>(rep, x, mu, glued);
            const Step fn = step_fwd<D>(rep, x, nu, glued);
            const uint32_t s_pm = x.s + uint32_t(fm.ds), l_pm = layer ^ fm.flip;
            const uint32_t s_pn = x.s + uint32_t(fn.ds), l_pn = layer ^ fn.flip;
            const mat3<double> t1 =
                mul_nn(widen<double>(load_link<PREC>(link_ref<D, PREC>(links, rep, layer, mu, p, x.s))),
                       widen<double>(load_link<PREC>(link_ref<D, PREC>(links, rep, l_pm, nu, q, s_pm))));
            const mat3<double> t2 =
                mul_nn(widen<double>(load_link<PREC>(link_ref<D, PREC>(links, rep, layer, nu, p, x.s))),
                       widen<double>(load_link<PREC>(link_ref<D, PREC>(links, rep, l_pn, mu, q, s_pn))));
            const double P = re_tr_na(t1, t2) * (1.0 / 3.0);
            if (nu == D - 1) v[1] += P; else v[0] += P;
            if (layer == 0) v[2] += P; else v[3] += P;
            const uint32_t tags = layer + l_pm + l_pn + layer;
            v[4] += (tags == 0 ? beta0 : beta1) * P;
        }
    }
    block_sum<5>(v);
    if (threadIdx.x == 0 && lb < a.total_blocks)
#pragma unroll
        for (int i = 0; i < 5; ++i) a.partials[size_t(lb) * 5 + i] = v[i];
}

// One thread per site: all its planes one after another, so that a link comes
// from the memory side once and from L2 for its other planes.  A wave takes 64
// consecutive half-lattice indices of one parity, the next wave the other
// parity of the same ones; XCD k takes a contiguous run of blocks.  The loops
// over the planes stay loops: unrolled, every plane's loads are hoisted.  Per
// plane of the lattice (plaquette_kernel) every link crossed the memory side
// D - 1 times: 32^4 FP64-12 330 -> 160 us with the order below.
// Strips: from four dimensions on the tiles go kPlaqStrip steps of x_{D-2} at
// a time along the whole of x_{D-1}, where such a strip's row is whole tiles.
// Lexicographically, the links at x + e_{D-1} lay a whole x_{D-1} layer ahead
// (32^4 FP64-18: 19 MB) and an XCD's L2 (4 MB) no longer had them.  Measured at
// 32^4 and 64^3 x 32, lexicographic -> strips, whole calls: FP64-18 330 -> 303 and
// 2700 -> 2542 us, FP64-12 186 -> 180 and 1449 -> 1343 us, FP32-18 186 -> 133 and
// 1519 -> 1010 us, FP32-12 118 -> 118 and 910 -> 860 us.  Strips of two and eight
// steps are slower or equal; in three dimensions, where whole layers stay in
// L2, the divisions cost more than they give (64^3 FP64-18 45 -> 51 us).
constexpr uint32_t kPlaqStrip = 4;

template <int D>
__device__ __forceinline__ uint32_t strip_tile(const RepDesc &rep, uint32_t t)
{
    const uint32_t sites = kPlaqStrip * rep.stride[D - 2];
    if (sites % (2u * kTile) || uint32_t(rep.n[D - 2]) % kPlaqStrip) return t;
    const uint32_t row = sites / (2u * kTile), last = uint32_t(rep.n[D - 1]);
    const uint32_t strip = t / (row * last), rem = t - strip * (row * last), x = rem / row;
    return (x * (uint32_t(rep.n[D - 2]) / kPlaqStrip) + strip) * row + (rem - x * row);
}

template <int D, int PREC>
__global__ void __launch_bounds__(256, 2) plaquette_site_kernel(PlaqArgs a)
{
    using R = typename Store<PREC>::real;
    const uint32_t per = (a.total_blocks + 7u) >> 3, lb = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if (lb >= a.total_blocks) return;
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const int r = a.nrep == 1 ? 0 : find_replica(a.reps, a.nrep, lb, kPlaquetteBlocks);
    const RepDesc &rep = a.reps[r];
    const uint32_t glued = rep.nlat == 2 ? rep.glued : 0u;
    const double beta0 = a.use_rep_beta ? rep.beta0 : a.beta0;
    const double beta1 = a.use_rep_beta ? rep.beta1 : a.beta1;
    void *links = const_cast<void *>(a.links);
    const uint32_t tiles = rep.Vhp / kTile, waves = rep.nlat * 2u * tiles;
    const uint32_t w0 = ((lb - rep.plq_block0) * rep.plq_spt) * (blockDim.x >> 6) + (threadIdx.x >> 6);
    for (uint32_t j = 0; j < rep.plq_spt; ++j) {
        const uint32_t w = w0 + j * (blockDim.x >> 6);
        if (w >= waves) break;
        const uint32_t layer = w >= 2u * tiles ? 1u : 0u, wl = w - layer * 2u * tiles;
        const int p = int(wl & 1u), q = 1 - p;
        uint32_t tile = __builtin_amdgcn_readfirstlane(wl >> 1);
        if constexpr (D >= 4) tile = strip_tile<D>(rep, tile);
        const uint32_t h = tile * kTile + (threadIdx.x & 63u);
        if (h >= rep.Vh) continue;
        Site<D> x;
        x.template from_half<true>(rep, h, p, layer);
#pragma unroll 1
        for (int mu = 0; mu < D - 1; ++mu) {
            const Step fm = step_fwd<D>(rep, x, mu, glued);
            const uint32_t s_pm = x.s + uint32_t(fm.ds), l_pm = layer ^ fm.flip;
            const mat3<R> umu = load_link<PREC>(link_ref<D, PREC>(links, rep, layer, mu, p, x.s));
#pragma unroll 1
            for (int nu = mu + 1; nu < D; ++nu) {
                const Step fn = step_fwd<D>(rep, x, nu, glued);
                const uint32_t s_pn = x.s + uint32_t(fn.ds), l_pn = layer ^ fn.flip;
                const mat3<R> b = load_link<PREC>(link_ref<D, PREC>(links, rep, l_pm, nu, q, s_pm));
                const mat3<R> c = load_link<PREC>(link_ref<D, PREC>(links, rep, layer, nu, p, x.s));
                const mat3<R> d = load_link<PREC>(link_ref<D, PREC>(links, rep, l_pn, mu, q, s_pn));
                // FP64-18: all loads before the first product.  Left to itself the
                // compiler put them between the products, one link in flight at
                // a time; the registers this takes leave two waves per SIMD for
                // three (32^4 303 -> 236 us, 64^3 x 32 2542 -> 2397 us).  The
                // other storages lose more by that than they gain (64^3 x 32
                // FP32-18 1010 -> 1076, FP32-12 860 -> 875, FP64-12 1343 ->
                // 1374 us).
                if constexpr (PREC == kFP64_18) __builtin_amdgcn_sched_barrier(0);
                const double P = re_tr_na(mul_nn(widen<double>(umu), widen<double>(b)),
                                          mul_nn(widen<double>(c), widen<double>(d))) *
                                 (1.0 / 3.0);
                if (nu == D - 1) v[1] += P; else v[0] += P;
                if (layer == 0) v[2] += P; else v[3] += P;
                const uint32_t tags = layer + l_pm + l_pn + layer;
                v[4] += (tags == 0 ? beta0 : beta1) * P;
            }
        }
    }
    block_sum<5>(v);
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) a.partials[size_t(lb) * 5 + i] = v[i];
}

// Fused measurement: meas[mu][b][c] holds the block sums of (1/3) Re Tr U_p
// over the planes (nu, mu), nu < mu, written by the parity-1 update slices,
// in nc classes: nc = 1 for one layer; nc = 3 for two layers (0: base site in
// layer 0 and all links in layer 0, 1: base in layer 0 otherwise, 2: base in
// layer 1).  One block per sweep adds them up in a fixed order.
__global__ void __launch_bounds__(1024) measure_finalize_kernel(const double *meas, int D, uint32_t nblocks, int nc,
                                                                 double V, int nlat, double beta0, double beta1,
                                                                 double *series, uint32_t *sweep)
{
    meas += size_t(blockIdx.x) * D * nblocks * nc;
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // [spacelike, timelike] x class
    const uint32_t bd = blockDim.x;
    for (int mu = 1; mu < D; ++mu) {
        for (int c = 0; c < nc; ++c) {
            // eight independent partial sums (fixed assignment, so the result
            // is reproducible) keep eight loads in flight per thread
            const double *m = meas + size_t(mu) * nblocks * nc + c;
            double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            uint32_t b = threadIdx.x;
            for (; b + 7 * bd < nblocks; b += 8 * bd) {
#pragma unroll
                for (int k = 0; k < 8; ++k) s[k] += m[size_t(b + k * bd) * nc];
            }
            for (; b < nblocks; b += bd) s[0] += m[size_t(b) * nc];
            v[(mu == D - 1 ? 3 : 0) + c] += ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < 6; ++i) v[i] += __shfl_xor(v[i], off);
    __shared__ double sh[16][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < 6; ++i) sh[wave][i] = v[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < int(blockDim.x >> 6); ++w)
#pragma unroll
            for (int i = 0; i < 6; ++i) v[i] += sh[w][i];
        plaquette_row(v, D, V, nlat, beta0, beta1, series + size_t(blockIdx.x) * 6);
        if (blockIdx.x == 0) sweep[2] = 0u;
    }
}

hipError_t launch_measure_finalize(hipStream_t st, const double *meas, int n, int D, uint32_t nblocks, int nc,
                                   double V, int nlat, double beta0, double beta1, double *series, uint32_t *sweep)
{
    if (nc != 1 && nc != 3) return hipErrorInvalidValue;
    return launch_kernel(measure_finalize_kernel, dim3(n), dim3(1024), st, meas, D, nblocks, nc, V, nlat, beta0,
                         beta1, series, sweep);
}

// One block per replica: fixed-order sum of its block partials, normalised.
__global__ void __launch_bounds__(256) plaquette_finalize_kernel(const RepDesc *reps, int D,
                                                                  const double *partials, double *out)
{
    const RepDesc &rep = reps[blockIdx.x];
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (uint32_t b = threadIdx.x; b < rep.plq_blocks; b += blockDim.x)
#pragma unroll
        for (int i = 0; i < 5; ++i) v[i] += partials[size_t(rep.plq_block0 + b) * 5 + i];
    block_sum<5>(v);
    if (threadIdx.x == 0) {
        const double nV = double(rep.nlat) * double(rep.V);
        const double nspace = nV * (D - 1) * (D - 2) / 2.0;
        const double ntime = nV * (D - 1);
        const double nlayer = double(rep.V) * D * (D - 1) / 2.0;
        const double nan = __builtin_nan("");
        double o[6];
        o[0] = (v[0] + v[1]) / (nspace + ntime);
        o[1] = nspace > 0 ? v[0] / nspace : nan;
        o[2] = v[1] / ntime;
        o[3] = v[2] / nlayer;
        o[4] = rep.nlat == 2 ? v[3] / nlayer : nan;
        o[5] = v[4];
        for (int i = 0; i < 6; ++i) out[size_t(blockIdx.x) * 6 + i] = o[i];
    }
}

template <int D, int PREC>
static hipError_t launch_plaquette_t(dim3 g, dim3 b, hipStream_t st, const PlaqArgs &a)
{
    if (a.by_site) return launch_kernel(plaquette_site_kernel<D, PREC>, dim3((g.x + 7) / 8 * 8), b, st, a);
    return launch_kernel(plaquette_kernel<D, PREC>, g, b, st, a);
}

hipError_t launch_plaquette(int D, int prec, dim3 g, dim3 b, hipStream_t st, const PlaqArgs &a)
{
#define SU3HB_CASE(DD)                                                            \
    case DD:                                                                      \
        switch (prec) {                                                           \
        case kFP64_18: return launch_plaquette_t<DD, kFP64_18>(g, b, st, a);      \
        case kFP32_18: return launch_plaquette_t<DD, kFP32_18>(g, b, st, a);      \
        case kFP32_12: return launch_plaquette_t<DD, kFP32_12>(g, b, st, a);      \
        case kFP64_12: return launch_plaquette_t<DD, kFP64_12>(g, b, st, a);      \
        default: return hipErrorInvalidValue;                                     \
        }
    switch (D) {
        SU3HB_CASE(2)
        SU3HB_CASE(3)
        SU3HB_CASE(4)
        SU3HB_CASE(5)
        SU3HB_CASE(6)
    default: return hipErrorInvalidValue;
    }
#undef SU3HB_CASE
}

hipError_t launch_plaquette_finalize(hipStream_t st, const RepDesc *reps, int nrep, int D,
                                     const double *partials, double *out)
{
    return launch_kernel(plaquette_finalize_kernel, dim3(nrep), dim3(256), st, reps, D, partials, out);
}

// ---------------------------------------------------------------------------
// start configurations

// Haar SU(3): two rows of complex Gaussians (Box-Muller on three Philox
// blocks of the start stream), Gram-Schmidt and the cross product.
template <int D, int PREC>
__global__ void __launch_bounds__(256) start_kernel(void *links, const RepDesc *reps, int r,
                                                     uint32_t nthreads, int mode)
{
    const uint32_t lt = blockIdx.x * blockDim.x + threadIdx.x;
    if (lt >= nthreads) return;
    const RepDesc &rep = reps[r];
    const uint32_t h = lt % rep.Vh;
    const uint32_t t2 = lt / rep.Vh;
    const int p = int(t2 & 1u);
    const uint32_t t3 = t2 >> 1;
    const int mu = int(t3 % uint32_t(D));
    const uint32_t layer = t3 / uint32_t(D);
    Site<D> x;
    x.from_half(rep, h, p, layer);
    mat3<double> u;
    if (mode == 1) {
        set_zero(u);
        u.e[0][0].re = u.e[1][1].re = u.e[2][2].re = 1.0;
    } else {
        const uint32_t lid = ((rep.lat2test ? 0u : layer * rep.V) + x.s) * uint32_t(D) + uint32_t(mu);
        double uu[12];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint4 w = philox4x32_10(make_uint4(lid, 0u, uint32_t(j), kTagStart), rep.key0, rep.key1);
            uu[4 * j + 0] = u01(w.x);
            uu[4 * j + 1] = u01(w.y);
            uu[4 * j + 2] = u01(w.z);
            uu[4 * j + 3] = u01(w.w);
        }
        double g[12];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double rho = sqrt(-2.0 * log(uu[2 * k]));
            double sn, cs;
            sincospi(2.0 * uu[2 * k + 1], &sn, &cs);  // sin, cos of 2 pi u
            g[2 * k] = rho * cs;
            g[2 * k + 1] = rho * sn;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            u.e[0][c] = cx<double>{g[2 * c], g[2 * c + 1]};
            u.e[1][c] = cx<double>{g[6 + 2 * c], g[7 + 2 * c]};
        }
        reunitarize(u);
    }
    store_link<PREC>(link_ref<D, PREC>(links, rep, layer, mu, p, x.s), u);
}

// ---------------------------------------------------------------------------
// canonical <-> internal

template <int D>
__device__ __forceinline__ void site_from_number(const RepDesc &rep, uint32_t s, Site<D> &x, int &p)
{
    int sum = 0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        x.x[i] = int((s / rep.stride[i]) % uint32_t(rep.n[i]));
        sum += x.x[i];
    }
    x.s = s;
    x.set_edges(rep);
    p = sum & 1;
}

template <int D, int PREC>
__global__ void __launch_bounds__(256) pack_kernel(const void *links, const RepDesc *reps, int r, uint64_t c0,
                                                    uint32_t count, double *dst)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const RepDesc &rep = reps[r];
    const uint64_t f = c0 + t;
    const uint32_t layer = uint32_t(f / rep.V);
    const uint32_t s = uint32_t(f - uint64_t(layer) * rep.V);
    Site<D> x;
    int p;
    site_from_number<D>(rep, s, x, p);
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
        const mat3<double> u = widen<double>(
            load_link<PREC>(link_ref<D, PREC>(const_cast<void *>(links), rep, layer, mu, p, s)));
        double *o = dst + (size_t(t) * D + mu) * 18;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            o[2 * e] = u.e[e / 3][e % 3].re;
            o[2 * e + 1] = u.e[e / 3][e % 3].im;
        }
    }
}

template <int D, int PREC>
__global__ void __launch_bounds__(256) unpack_kernel(void *links, const RepDesc *reps, int r, uint64_t c0,
                                                      uint32_t count, const double *src)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const RepDesc &rep = reps[r];
    const uint64_t f = c0 + t;
    const uint32_t layer = uint32_t(f / rep.V);
    const uint32_t s = uint32_t(f - uint64_t(layer) * rep.V);
    Site<D> x;
    int p;
    site_from_number<D>(rep, s, x, p);
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
        const double *in = src + (size_t(t) * D + mu) * 18;
        mat3<double> u;
#pragma unroll
        for (int e = 0; e < 9; ++e) u.e[e / 3][e % 3] = cx<double>{in[2 * e], in[2 * e + 1]};
        store_link<PREC>(link_ref<D, PREC>(links, rep, layer, mu, p, s), u);
    }
}

#define SU3HB_DISPATCH(KERNEL, ...)                                                        \
    switch (D) {                                                                            \
    case 2: SU3HB_PREC(KERNEL, 2, __VA_ARGS__)                                             \
    case 3: SU3HB_PREC(KERNEL, 3, __VA_ARGS__)                                             \
    case 4: SU3HB_PREC(KERNEL, 4, __VA_ARGS__)                                             \
    case 5: SU3HB_PREC(KERNEL, 5, __VA_ARGS__)                                             \
    case 6: SU3HB_PREC(KERNEL, 6, __VA_ARGS__)                                             \
    default: return hipErrorInvalidValue;                                                  \
    }
#define SU3HB_PREC(KERNEL, DD, ...)                                                        \
    switch (prec) {                                                                        \
    case kFP64_18: return launch_kernel(KERNEL<DD, kFP64_18>, __VA_ARGS__);                \
    case kFP32_18: return launch_kernel(KERNEL<DD, kFP32_18>, __VA_ARGS__);                \
    case kFP32_12: return launch_kernel(KERNEL<DD, kFP32_12>, __VA_ARGS__);                \
    case kFP64_12: return launch_kernel(KERNEL<DD, kFP64_12>, __VA_ARGS__);                \
    default: return hipErrorInvalidValue;                                                  \
    }

hipError_t launch_start(int D, int prec, hipStream_t st, void *links, const RepDesc *reps, int r,
                        uint32_t nthreads, int mode)
{
    if (nthreads == 0) return hipSuccess;
    const dim3 g((nthreads + 255) / 256), b(256);
    SU3HB_DISPATCH(start_kernel, g, b, st, links, reps, r, nthreads, mode)
}

hipError_t launch_pack(int D, int prec, hipStream_t st, const void *links, const RepDesc *reps, int r,
                       uint64_t c0, uint32_t count, double *dst)
{
    if (count == 0) return hipSuccess;
    const dim3 g((count + 255) / 256), b(256);
    SU3HB_DISPATCH(pack_kernel, g, b, st, links, reps, r, c0, count, dst)
}

hipError_t launch_unpack(int D, int prec, hipStream_t st, void *links, const RepDesc *reps, int r,
                         uint64_t c0, uint32_t count, const double *src)
{
    if (count == 0) return hipSuccess;
    const dim3 g((count + 255) / 256), b(256);
    SU3HB_DISPATCH(unpack_kernel, g, b, st, links, reps, r, c0, count, src)
}

// ---------------------------------------------------------------------------
// validation of canonical input

__global__ void __launch_bounds__(256) validate_kernel(const double *src, uint64_t nmat,
                                                        unsigned long long *maxdef)
{
    const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    double d = 0.0;
    if (t < nmat) {
        const double *in = src + t * 18;
        mat3<double> u;
        bool finite = true;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            u.e[e / 3][e % 3] = cx<double>{in[2 * e], in[2 * e + 1]};
            finite = finite && isfinite(in[2 * e]) && isfinite(in[2 * e + 1]);
        }
        if (!finite) {
            d = __builtin_inf();
        } else {
            const mat3<double> uu = mul_na(u, u);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const double re = uu.e[i][j].re - (i == j ? 1.0 : 0.0);
                    d = fmax(d, fmax(fabs(re), fabs(uu.e[i][j].im)));
                }
            // det via the first row and the cofactors
            cx<double> m0{0, 0}, m1{0, 0}, m2{0, 0};
            cfma(m0, u.e[1][1], u.e[2][2]);
            cfma(m0, cx<double>{-u.e[1][2].re, -u.e[1][2].im}, u.e[2][1]);
            cfma(m1, u.e[1][2], u.e[2][0]);
            cfma(m1, cx<double>{-u.e[1][0].re, -u.e[1][0].im}, u.e[2][2]);
            cfma(m2, u.e[1][0], u.e[2][1]);
            cfma(m2, cx<double>{-u.e[1][1].re, -u.e[1][1].im}, u.e[2][0]);
            cx<double> det{0, 0};
            cfma(det, u.e[0][0], m0);
            cfma(det, u.e[0][1], m1);
            cfma(det, u.e[0][2], m2);
            d = fmax(d, sqrt((det.re - 1.0) * (det.re - 1.0) + det.im * det.im));
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) d = fmax(d, __shfl_xor(d, off));
    if ((threadIdx.x & 63) == 0) atomicMax(maxdef, (unsigned long long)__double_as_longlong(d));
}

hipError_t launch_validate(hipStream_t st, const double *src, uint64_t nmat, unsigned long long *maxdef)
{
    if (nmat == 0) return hipSuccess;
    return launch_kernel(validate_kernel, dim3(uint32_t((nmat + 255) / 256)), dim3(256), st, src, nmat,
                         maxdef);
}

// ---------------------------------------------------------------------------
// statistics and counters

__global__ void stats_zero_kernel(StatSlot *slots)
{
    StatSlot &s = slots[threadIdx.x];
    for (int i = 0; i < 3; ++i) {
        s.attempts[i] = 0;
        s.accepts[i] = 0;
    }
    s.updates = 0;
    s.dtrace = 0.0;
}

__global__ void stats_reduce_kernel(StatSlot *slots, StatSlot *out)
{
    __shared__ unsigned long long si[kStatSlots][7];
    __shared__ double sd[kStatSlots];
    const int t = threadIdx.x;
    for (int i = 0; i < 3; ++i) {
        si[t][i] = slots[t].attempts[i];
        si[t][3 + i] = slots[t].accepts[i];
    }
    si[t][6] = slots[t].updates;
    sd[t] = slots[t].dtrace;
    slots[t] = StatSlot{};  // empty for the next call
    __syncthreads();
    for (int w = kStatSlots / 2; w > 0; w >>= 1) {
        if (t < w) {
            for (int i = 0; i < 7; ++i) si[t][i] += si[t + w][i];
            sd[t] += sd[t + w];
        }
        __syncthreads();
    }
    if (t == 0) {
        for (int i = 0; i < 3; ++i) {
            out->attempts[i] = si[0][i];
            out->accepts[i] = si[0][3 + i];
        }
        out->updates = si[0][6];
        out->dtrace = sd[0];
    }
}

__global__ void counter_add_kernel(uint32_t *ctr, uint32_t add)
{
    if (threadIdx.x == 0) atomicAdd(ctr, add);
}

__global__ void counter_set_kernel(uint32_t *ctr, uint32_t value)
{
    if (threadIdx.x == 0) atomicExch(ctr, value);
}

__global__ void measure_begin_kernel(uint32_t *sweep)
{
    if (threadIdx.x == 0) sweep[2] = 0u;
}

__global__ void u32_zero_kernel(uint32_t *p, int n)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 0u;
}

__global__ void u64_zero_kernel(unsigned long long *p, int n)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) atomicExch(&p[t], 0ull);
}

// One replica descriptor, passed by value, written to device memory (so a
// captured graph carries the descriptor in its kernel arguments).
__global__ void rep_set_kernel(RepDesc r, RepDesc *dst)
{
    if (threadIdx.x == 0) *dst = r;
}

hipError_t launch_rep_set(hipStream_t st, const RepDesc &r, RepDesc *dst)
{
    return launch_kernel(rep_set_kernel, dim3(1), dim3(64), st, r, dst);
}

hipError_t launch_stats_zero(hipStream_t st, StatSlot *slots)
{
    return launch_kernel(stats_zero_kernel, dim3(1), dim3(kStatSlots), st, slots);
}

hipError_t launch_stats_reduce(hipStream_t st, StatSlot *slots, StatSlot *out)
{
    return launch_kernel(stats_reduce_kernel, dim3(1), dim3(kStatSlots), st, slots, out);
}

hipError_t launch_counter_add(hipStream_t st, uint32_t *ctr, uint32_t add)
{
    return launch_kernel(counter_add_kernel, dim3(1), dim3(64), st, ctr, add);
}

hipError_t launch_counter_set(hipStream_t st, uint32_t *ctr, uint32_t value)
{
    return launch_kernel(counter_set_kernel, dim3(1), dim3(64), st, ctr, value);
}

hipError_t launch_measure_begin(hipStream_t st, uint32_t *sweep)
{
    return launch_kernel(measure_begin_kernel, dim3(1), dim3(64), st, sweep);
}

hipError_t launch_u32_zero(hipStream_t st, uint32_t *p, int n)
{
    return launch_kernel(u32_zero_kernel, dim3((n + 255) / 256), dim3(256), st, p, n);
}

hipError_t launch_u64_zero(hipStream_t st, unsigned long long *p, int n)
{
    return launch_kernel(u64_zero_kernel, dim3((n + 63) / 64), dim3(64), st, p, n);
}

}  // namespace su3hb
