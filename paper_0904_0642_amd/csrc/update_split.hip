// update_split.hip -- slice updates of small lattices and batches: every
// link's update is shared by the lanes of a wave (split.h).
#include "kernels.h"
#include "split.h"

namespace su3hb {

// One slice, four waves to 16 links: wave 0 loads the links, draws the
// directions of hits 0 and 1 and updates, waves 1 and 2 make the forward and
// the backward staples, wave 3 copies the logarithm's table and makes the
// proposals of hits 0 and 1.  Bound by that chain (a load, a staple, the sum
// and the update, about 11 thousand cycles) and by the launch (3 to 4 us), not
// by memory or by the rate of arithmetic: 30x22x18 FP32-12 12.8 -> 7.6 us a
// slice, 8^4 FP64-18 14.9 -> 6.9 us.  One wave for all four parts took 11.7 us
// for the same 8^4 slice.  Waves that have done their part meet wave 0 at the
// one barrier of the block and leave.
template <int D, int PREC, int NC>
__global__ void __launch_bounds__(256, 2) update_split_kernel(UpdateArgs a)
{
    using R = typename Store<PREC>::real;
    __shared__ LogEntry table[128];
    __shared__ Proposal s_proposal[2][64];
    __shared__ __align__(16) char s_lds[SplitLds<D, PREC>::kBytes];
    const uint32_t sweep = a.sweep[a.parity];
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t group = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (group >= a.total_blocks) return;
    const RepDesc &rep = a.reps[a.nrep == 1 ? 0 : find_replica(a.reps, a.nrep, group, kSplitBlocks)];
    const uint32_t first = (group - rep.split_group0) * kSplitLinks;
    SplitLds<D, PREC> lds(s_lds);
    if (wave == 1) {
        split_staples<D, PREC, true, kNormal>(a, rep, first, lds);
        __syncthreads();
        return;
    }
    if (wave == 2) {
        split_staples<D, PREC, false, kNormal>(a, rep, first, lds);
        __syncthreads();
        return;
    }
    const SplitSite<D> site(rep, first + (lane >> 2), a.parity);
    const uint32_t lid = split_lid<D>(rep, site, a.mu);
    if (wave == 3) {
        table[lane] = kLogTable[lane];
        table[lane + 64u] = kLogTable[lane + 64u];
        wave_lds_fence();
        if (a.nhit > 0) {
            s_proposal[0][lane] = draw_proposal(lid, sweep, split_word(0), rep.key0, rep.key1, table);
            if (a.nhit > 1)
                s_proposal[1][lane] = draw_proposal(lid, sweep, split_word(1), rep.key0, rep.key1, table);
        }
        __syncthreads();
        return;
    }
    const LinkRef uptr = link_ref<D, PREC>(a.links, rep, site.layer, a.mu, a.parity, site.x.s);
    const mat3<R> U = load_link<PREC>(uptr);
    Draw<R> draw[2] = {};
    if (a.nhit > 0) draw[0].d = draw_direction<R>(lid, sweep, split_word(0), rep.key0, rep.key1);
    if (a.nhit > 1) draw[1].d = draw_direction<R>(lid, sweep, split_word(1), rep.key0, rep.key1);
    __syncthreads();
    draw[0].p = s_proposal[0][lane];
    draw[1].p = s_proposal[1][lane];
    const SplitColumn<PREC, NC> col = split_sum<D, PREC, NC>(a, rep, lds);
    SplitSums<NC> sums;
    split_update<D, PREC, NC>(a, rep, site, sweep, col, U, draw, uptr, table, sums);
    split_flush<D, NC>(a, group, a.meas != nullptr ? a.sweep[3] : 0u, sums);
    advance_sweep(a, D, sweep);
}

// Wait until every group has done n slices; false past the limit.
__device__ __forceinline__ bool small_wait(const SmallArgs &s, uint32_t n, uint32_t lane)
{
    uint32_t spins = 0;
    while (__any(lane < s.u.total_blocks &&
                 __hip_atomic_load(s.work + kSmallDone + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n)) {
        if (++spins > s.spin_limit) {
            if (lane == 0) *s.failed = 1u;
            return false;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// The end of a launch of whole sweeps: the sweep counter, and the plaquettes
// of measured sweeps, a sweep per wave at a time.  The sums are those of
// measure_finalize_kernel, whose first wave holds all groups.
template <int D, int NC>
__device__ __forceinline__ void small_finish(const SmallArgs &s, uint32_t wave, uint32_t lane)
{
    if (!small_wait(s, 2u * D * s.sweeps, lane)) return;
    if (wave == 0 && lane == 0) s.u.sweep[0] = s.sweep0 + s.sweeps;
    if (s.u.meas == nullptr) return;
    for (uint32_t sw = wave; sw < s.sweeps; sw += 4u) {
        double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        UpdateArgs a = s.u;
        for (a.mu = 1; a.mu < D; ++a.mu)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (lane < a.total_blocks)
                    v[(a.mu == D - 1 ? 3 : 0) + c] += __hip_atomic_load(meas_of_block<D, NC>(a, sw, lane) + c,
                                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int i = 0; i < 6; ++i) v[i] += __shfl_xor(v[i], off);
        if (lane == 0) plaquette_row(v, D, s.V, s.nlat, a.beta0, a.beta1, s.series + size_t(sw) * 6);
    }
}

// Whole sweeps of a lattice so small that even its slices' launches cost more
// than their work: one launch for all of them.  The blocks of one XCD, whose
// L2 they share, take (slice, 16 links) items from a queue in order; the
// others leave at once.  An item waits until every item of the slices before
// is done.  Tickets rise, and a block works on its tickets in order, so the
// lowest unfinished item is always one that a running block works on: the
// wait ends however many blocks run, one would do.  A wave whose wait passes its
// limit tells the host (s.failed) and leaves; the others of its block end that
// item, whose links are then wrong, and leave with the next ticket, and the blocks
// that wait for its item give up in turn.
//
// A block is four waves.  Wave 0 updates; waves 1 and 2 make the forward and
// the backward staples; wave 3 takes the next ticket once the staples have been
// read (late enough that every block has taken its ticket of this slice).
// While wave 0 updates, waves 3, 1 and 2 draw for the next item: the proposals
// of hits 0 and 1, the direction of hit 0, that of hit 1.  Stores are complete
// in the shared L2 before an item counts as done (so plain stores serve for
// the links and the groups' words: one XCD, one L2); links are read past the
// L1, which an earlier slice may have filled (an invalidation of workgroup
// scope does not empty it).
//
// Bound by one chain per slice, in cycles: staples 3000, their sum 900, the
// update 4900, from the store to the others' sight of it 1500.  A slice took
// 13.7 us launched by itself one thread per link and takes 4.3 us here (4^4
// FP64-18, 128 links), 14.7 and 5.9 us for 8^3x4 (1024 links); sums of one word
// by all blocks instead of a word per group, or words written past the L2, made
// the latter 9 to 13 us.
//
// FP64 kernels spill registers from D = 5 on (8 at D = 5, 23 to 25 at D = 6) and
// where two layers are measured (18 to 28 at D = 4, up to 146 at D = 6).  They stay the
// faster form: a slice of D = 6 takes 5.5 to 7.0 us for 32 to 1024 links (13.6 to 17.2
// one thread per link, 7.6 shared by itself at 1536 links), measured on two layers
// 9.0 to 13.8 (16.5 to 21.8).
template <int D, int PREC, int NC>
__global__ void __launch_bounds__(256, 2) update_small_kernel(SmallArgs s)
{
    using R = typename Store<PREC>::real;
    __shared__ LogEntry table[128];
    // s_round: the item whose ticket has been taken; s_go: the item whose wait is
    // over; s_quit: a wave gave up a wait and left
    __shared__ uint32_t s_ticket, s_round, s_go, s_mine, s_quit;
    __shared__ Proposal s_proposal[2][64];
    __shared__ Direction<R> s_direction[2][64];
    __shared__ __align__(16) char s_lds[SplitLds<D, PREC>::kBytes];
    auto take = [&]() {
        return __hip_atomic_fetch_add(s.work + kSmallTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (threadIdx.x == 0) {
        const uint32_t team = small_team(xcc_id(), blockIdx.x);
        uint32_t old = 0;
        __hip_atomic_compare_exchange_strong(s.work + kSmallTeam, &old, team, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        s_mine = old == 0u || old == team;
        if (s_mine) s_ticket = take();
        s_round = 1;
        s_go = 0;
        s_quit = 0;
    }
    if (threadIdx.x < 128u) table[threadIdx.x] = kLogTable[threadIdx.x];
    __syncthreads();
    if (!s_mine) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    SplitLds<D, PREC> lds(s_lds);
    for (uint32_t round = 1;; ++round) {
        uint32_t spins = 0;
        while (__hip_atomic_load(&s_round, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != round)
            if (++spins > s.spin_limit * kSmallLdsPolls) {
                if (lane == 0) *s.failed = s_quit = 1u;
                return;
            }
        const uint32_t t = __builtin_amdgcn_readfirstlane(s_ticket);
        if (t >= s.items) {
            // one block, with the first ticket past the end, adds up the
            // plaquettes and steps the sweep counter
            if (t == s.items) small_finish<D, NC>(s, wave, lane);
            return;
        }
        const uint32_t n = div_by(t, s.per_slice), group = t - n * s.u.total_blocks;
        UpdateArgs a = s.u;
        const uint32_t sw = n / (2u * D), sl = n - sw * (2u * D), sweep = s.sweep0 + sw;
        a.parity = sl >= uint32_t(D) ? 1 : 0;
        a.mu = int(sl) - a.parity * D;
        const RepDesc &rep = a.reps[a.nrep == 1 ? 0 : find_replica(a.reps, a.nrep, group, kSplitBlocks)];
        const uint32_t first = (group - rep.split_group0) * kSplitLinks;
        const SplitSite<D> site(rep, first + (lane >> 2), a.parity);
        const uint32_t lid = split_lid<D>(rep, site, a.mu);
        if (wave == 0) {
            // only this slice of the sweep before wrote this link, and it is done
            // without a wait (small_team)
            const LinkRef uptr = link_ref<D, PREC>(a.links, rep, site.layer, a.mu, a.parity, site.x.s);
            const mat3<R> U = load_link<PREC, kFresh>(uptr);
            __syncthreads();  // the staples and the draws are there
            const SplitColumn<PREC, NC> col = split_sum<D, PREC, NC>(a, rep, lds);
            Draw<R> draw[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) draw[h] = Draw<R>{s_proposal[h][lane], s_direction[h][lane]};
            __syncthreads();  // and read
            SplitSums<NC> sums;
            split_update<D, PREC, NC>(a, rep, site, sweep, col, U, draw, uptr, table, sums);
            split_flush<D, NC>(a, group, sw, sums);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0)
                __hip_atomic_store(s.work + kSmallDone + group, n + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            continue;
        }
        if (wave == 3) {
            if (a.nhit > 0) {
                s_proposal[0][lane] = draw_proposal(lid, sweep, split_word(0), rep.key0, rep.key1, table);
                if (a.nhit > 1)
                    s_proposal[1][lane] = draw_proposal(lid, sweep, split_word(1), rep.key0, rep.key1, table);
            }
            __syncthreads();
            __syncthreads();
            if (lane == 0) {
                const uint32_t next = take();
                s_ticket = s_quit ? ~0u : next;
                __hip_atomic_store(&s_round, round + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            continue;
        }
        const uint32_t hit = wave - 1u;
        if (a.nhit > int(hit))
            s_direction[hit][lane] = draw_direction<R>(lid, sweep, split_word(hit), rep.key0, rep.key1);
        // every item of the slices before: wave 1 looks at the groups' words
        // (reads that pass the caches by: more of them would slow the links')
        // and tells wave 2 (also when it gives up: wave 2 need not wait longer)
        if (wave == 1) {
            if (!small_wait(s, n, lane)) {
                if (lane == 0) {
                    s_quit = 1u;
                    __hip_atomic_store(&s_go, round, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                return;
            }
            if (lane == 0) __hip_atomic_store(&s_go, round, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            while (__hip_atomic_load(&s_go, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != round)
                if (++spins > s.spin_limit * kSmallLdsPolls) {
                    if (lane == 0) *s.failed = s_quit = 1u;
                    return;
                }
        }
        asm volatile("" ::: "memory");
        if (wave == 1) split_staples<D, PREC, true, kFresh>(a, rep, first, lds);
        else split_staples<D, PREC, false, kFresh>(a, rep, first, lds);
        __syncthreads();
        __syncthreads();
    }
}

template <int D, int PREC>
static hipError_t launch_small_t(hipStream_t st, const SmallArgs &s)
{
    // a block for every group on whichever XCD begins first (small_team)
    const dim3 grid(8u * s.u.total_blocks), block(256);
    if (s.u.meas != nullptr && s.u.meas_classes == 3)
        return launch_kernel(update_small_kernel<D, PREC, 3>, grid, block, st, s);
    return launch_kernel(update_small_kernel<D, PREC, 1>, grid, block, st, s);
}

template <int D>
hipError_t launch_small_d(int prec, hipStream_t st, const SmallArgs &s)
{
    switch (prec) {
    case kFP64_18: return launch_small_t<D, kFP64_18>(st, s);
    case kFP32_18: return launch_small_t<D, kFP32_18>(st, s);
    case kFP32_12: return launch_small_t<D, kFP32_12>(st, s);
    case kFP64_12: return launch_small_t<D, kFP64_12>(st, s);
    default: return hipErrorInvalidValue;
    }
}

template <int D, int PREC>
static hipError_t launch_split_t(hipStream_t st, const UpdateArgs &a)
{
    const dim3 grid((a.total_blocks + 7) / 8 * 8), block(256);
    if (a.meas != nullptr && a.parity == 1 && a.meas_classes == 3)
        return launch_kernel(update_split_kernel<D, PREC, 3>, grid, block, st, a);
    return launch_kernel(update_split_kernel<D, PREC, 1>, grid, block, st, a);
}

template <int D>
hipError_t launch_split_d(int prec, hipStream_t st, const UpdateArgs &a)
{
    switch (prec) {
    case kFP64_18: return launch_split_t<D, kFP64_18>(st, a);
    case kFP32_18: return launch_split_t<D, kFP32_18>(st, a);
    case kFP32_12: return launch_split_t<D, kFP32_12>(st, a);
    case kFP64_12: return launch_split_t<D, kFP64_12>(st, a);
    default: return hipErrorInvalidValue;
    }
}

#ifdef SU3HB_DIM  // as in update.hip
template hipError_t launch_split_d<SU3HB_DIM>(int, hipStream_t, const UpdateArgs &);
template hipError_t launch_small_d<SU3HB_DIM>(int, hipStream_t, const SmallArgs &);
#else
extern template hipError_t launch_small_d<2>(int, hipStream_t, const SmallArgs &);
extern template hipError_t launch_small_d<3>(int, hipStream_t, const SmallArgs &);
extern template hipError_t launch_small_d<4>(int, hipStream_t, const SmallArgs &);
extern template hipError_t launch_small_d<5>(int, hipStream_t, const SmallArgs &);
extern template hipError_t launch_small_d<6>(int, hipStream_t, const SmallArgs &);
extern template hipError_t launch_split_d<2>(int, hipStream_t, const UpdateArgs &);
extern template hipError_t launch_split_d<3>(int, hipStream_t, const UpdateArgs &);
extern template hipError_t launch_split_d<4>(int, hipStream_t, const UpdateArgs &);
extern template hipError_t launch_split_d<5>(int, hipStream_t, const UpdateArgs &);
extern template hipError_t launch_split_d<6>(int, hipStream_t, const UpdateArgs &);

hipError_t launch_update_split(int D, int prec, hipStream_t st, const UpdateArgs &a)
{
    switch (D) {
    case 2: return launch_split_d<2>(prec, st, a);
    case 3: return launch_split_d<3>(prec, st, a);
    case 4: return launch_split_d<4>(prec, st, a);
    case 5: return launch_split_d<5>(prec, st, a);
    case 6: return launch_split_d<6>(prec, st, a);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_update_small(int D, int prec, hipStream_t st, const SmallArgs &s)
{
    switch (D) {
    case 2: return launch_small_d<2>(prec, st, s);
    case 3: return launch_small_d<3>(prec, st, s);
    case 4: return launch_small_d<4>(prec, st, s);
    case 5: return launch_small_d<5>(prec, st, s);
    case 6: return launch_small_d<6>(prec, st, s);
    default: return hipErrorInvalidValue;
    }
}
#endif

}  // namespace su3hb
