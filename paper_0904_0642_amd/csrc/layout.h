// layout.h -- descriptors shared by the host side and the kernels of the GPU
// library: storage modes, the per-replica descriptor and kernel arguments.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace su3hb {

constexpr int kFP64_18 = 0;
constexpr int kFP32_18 = 1;
constexpr int kFP32_12 = 2;
constexpr int kFP64_12 = 3;

constexpr int kMaxD = 6;          // kernels are instantiated for D = 2 .. 6
constexpr int kStatSlots = 256;   // spread of the per-block statistics atomics

inline constexpr int elems_per_link(int prec) { return (prec == kFP32_12 || prec == kFP64_12) ? 6 : 9; }
inline constexpr int bytes_per_elem(int prec) { return (prec == kFP64_18 || prec == kFP64_12) ? 16 : 8; }
inline constexpr bool is_fp32(int prec) { return prec == kFP32_18 || prec == kFP32_12; }
inline constexpr int bytes_per_link(int prec) { return elems_per_link(prec) * bytes_per_elem(prec); }

// Links are stored in tiles of kTile consecutive half-lattice sites (one
// wave); a slab of Vh links takes Vhp = Vh rounded up to whole tiles.
constexpr uint32_t kTile = 64;
inline constexpr uint32_t padded_half(uint32_t Vh) { return (Vh + kTile - 1) / kTile * kTile; }

// Division by an invariant integer (T. Granlund and P. L. Montgomery, PLDI
// 1994): for d >= 1 and 0 <= x < 2^31, x / d = (x m) >> s with
// l = ceil(log2 d), s = 31 + l and m = ceil(2^s / d), which is below 2^32
// (so m d - 2^s < d <= 2^l, the condition of their Theorem 4.2).
struct DivMagic {
    uint32_t m, s;
};

inline DivMagic div_magic(uint32_t d)
{
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    const uint32_t s = 31u + l;
    return DivMagic{uint32_t(((uint64_t(1) << s) + d - 1u) / d), s};
}

// One lattice ("replica").  A single lattice is a batch of one.  Its links
// start `elem_offset` complex elements into the batch's link buffer and are
// laid out as [layer][mu][parity][tile][packet][kTile].
struct RepDesc {
    uint64_t elem_offset;
    int32_t n[kMaxD];        // extents
    uint32_t stride[kMaxD];  // site-number strides: 1, n0, n0 n1, ...
    uint32_t V;              // sites per layer
    uint32_t Vh;             // V / 2
    uint32_t Vhp;            // Vh rounded up to a multiple of kTile (links per slab in memory)
    uint32_t nlat;           // 1 or 2
    uint32_t glued;          // dlt mask (only with nlat == 2)
    uint32_t lat2test;
    uint32_t key0, key1;     // Philox key (seed)
    double beta0, beta1;     // couplings used when the batch carries them
    uint32_t upd_block0;     // first block of this replica in an update launch
    uint32_t upd_blocks;     // blocks of this replica in an update launch
    uint32_t plq_block0;     // first block in a plaquette launch
    uint32_t plq_blocks;
    uint32_t plq_spt;        // plaquettes (or sites) per thread in the plaquette launch
    uint32_t pers_block0;    // first block in a persistent launch (kPersistentThreads links per block)
    uint32_t pers_blocks;
    uint32_t planes_block0;  // first block in a launch that gives planes to waves (kPlanesLinks links per block)
    uint32_t split_group0;   // first block in a launch that shares links between lanes (kSplitLinks links per block)
    DivMagic div[kMaxD - 1];  // division by n0 / 2 (entry 0) and by n_i (entry i, 0 < i < D - 1)
};

// Persistent batch launches: blocks of kPersistentThreads, as many per CU as
// the kernel's registers allow (2 waves per SIMD for FP64 links, 3 for
// FP32), slices separated by a grid barrier on a small array of counters
// (kBarrierWords words, each counter on its own 128-byte line): the start
// barrier's kBarrierLeaves leaf counters and top counter, an abort flag, and
// for the slice barriers per-XCD member counts, arrival counters and go
// words, a top counter of the XCDs and a release word.
constexpr int kPersistentThreads = 256;
inline constexpr int persistent_waves(int prec) { return (prec == kFP32_18 || prec == kFP32_12) ? 3 : 2; }
constexpr int kBarrierWords = 4096;
constexpr uint32_t kBarrierLeaves = 16;
constexpr uint32_t kBarrierTop = 1024;
constexpr uint32_t kBarrierFlag = 1536;
constexpr uint32_t kBarrierXcds = 16;            // XCC ids are 4 bits
constexpr uint32_t kBarrierXcdMembers = 2048;    // + 32 x: blocks on XCD x
constexpr uint32_t kBarrierXcdArrive = 2560;     // + 32 x
constexpr uint32_t kBarrierXcdGo = 3072;         // + 32 x
constexpr uint32_t kBarrierXcdTop = 3584;
constexpr uint32_t kBarrierXcdRelease = 3712;
constexpr uint32_t kBarrierSpinLimit = 1u << 22;

// The sweep counter on the device: word 0 is the index of the next sweep,
// which the parity-0 slices read; their last one copies it to word 1, which
// the parity-1 slices read, and the last of those writes word 0 of the sweep
// after.  No slice writes a word that it reads, so the counter needs no
// launch of its own: a launch of one wave between two slices cost 4.4 us, and
// so did adding up each sweep's plaquettes (5.7 us), now one launch for all
// sweeps of a call (4^4 FP64-18, 20 measured sweeps: 2.46 -> 2.13 ms;
// 16^4, 4 sweeps: 0.70 -> 0.64 ms).  Words 2 and 3 count the measured sweeps whose
// partial sums wait in `meas` in the same way (word 3 is read by the measured
// slices); adding them up sets word 2 back to 0.
constexpr int kSweepWords = 4;

// The three forms of a slice, and the lines between them.  One thread per link
// (update.hip) has the least work in all but leaves SIMDs idle where links are
// few; a link's update shared by lanes and waves (split.h, kSplitLinks links of
// a block) has the shortest chain and twice the work; planes of its staple on
// waves of their own (update_planes.hip, kPlanesLinks links of a block, D = 3 and
// 4) lie between.  Time of a slice, shared / planes / thread, us:
//   4D links   FP64-18           FP32-12
//    8192       8.2  9.9 15.1     7.2  8.5 13.2
//   20480      11.8 11.9 16.6     9.1  9.5 12.7
//   24576      13.8 12.3 17.0     9.8  9.8 12.7
//   32768      16.7 13.6 17.6    11.5  9.9 13.0
//   41472      20.3 20.2 18.4    13.0 11.1 13.0
//   49152      22.4 23.5 19.7    14.3 11.3 13.3
//   51840      23.6 24.4 20.0    14.9 13.6 13.2
//   3D: 24576  12.9 13.0 13.7    10.3 10.9 12.3
//       32000  15.6 13.4 14.8    12.0 11.2 12.4
//   2D: 18432  12.5    - 13.3    10.1    - 12.4;  25088  14.6    - 13.4    11.2    - 12.5
//   5D: 20480  14.8    - 18.9     9.5    - 14.0;  25600  19.4    - 19.6    11.2    - 14.1
// Planes stop where the device no longer holds all blocks at once: by the
// registers two (FP64) and three (FP32) on each of 256 CUs.
constexpr uint32_t kSplitLinks = 16;
constexpr uint32_t kPlanesLinks = 64;
inline constexpr bool fp32_links(int prec) { return prec == kFP32_18 || prec == kFP32_12; }
inline constexpr uint32_t shared_most(int D, int prec)  // links
{
    return D == 4 ? 20480 : D == 3 ? 24576 : fp32_links(prec) ? (D == 2 ? 28672 : 32768) : (D == 2 ? 20480 : 24576);
}
inline constexpr uint32_t planes_most(int D, int prec)  // blocks
{
    return D != 3 && D != 4 ? 0 : fp32_links(prec) ? 768 : 512;
}

// Statistics slot, padded to its own 128-byte line.
struct alignas(128) StatSlot {
    unsigned long long attempts[3];
    unsigned long long accepts[3];
    unsigned long long updates;
    double dtrace;
};

struct UpdateArgs {
    void *links;                 // base of the link buffer
    const RepDesc *reps;         // device array
    int nrep;
    int parity;                  // checkerboard colour being updated
    int mu;                      // direction being updated
    int nhit;                    // KP proposals per subgroup, at most; 0: overrelaxation
    int use_rep_beta;            // 1: couplings from RepDesc; 0: from beta0/beta1
    int order;                   // 0 hardware, 1 XCD-contiguous, 2 and 4 XCD slabs, 3, 5 and 6 XCD slabs of 3D blocks,
                                 // 7 XCD slabs of 4D wave tiles
    int reverse;                 // 1: each XCD walks its blocks last to first (alternate slices)
    uint32_t strip_row;          // order 1: the logical blocks go in strips (set_strips in capi.cpp): waves of a
    uint32_t strips, strip_last; // strip's row (0: no strips), strips, rows of a strip
    uint32_t slab;               // orders 2, 3: tiles of the last direction per XCD
    uint32_t cp;                 // orders 2, 3: blocks (order 3: waves) per (x_{D-2}, x_{D-1}) plane
    uint32_t n2;                 // orders 2, 3: extent of direction D-2
    uint32_t plane;              // order 3: half-sites of one (x_{D-2}, x_{D-1}) plane
    uint32_t tile2, tile3;       // order 3: waves of a block along x_{D-2} and x_{D-1}
    uint32_t n0h, n1;            // order 7: n_0 / 2 and n_1
    int stage;                   // 1: each wave stages the U_mu links its planes nu = 0, 1 read in LDS
    uint32_t stage_r;            // staging halo: n_0 / 2 half-sites before and after a wave's 64
    double beta0, beta1;
    uint32_t *sweep;             // device sweep counter, kSweepWords words
    StatSlot *stats;             // kStatSlots slots, or null: no counters are kept
    uint32_t total_blocks;       // real blocks (grid may be padded to 8)
    double *meas;                // fused plaquettes: [sweep][mu][total_blocks][meas_classes] partial sums, or null
    int meas_classes;            // 1: one lattice layer; 3: two layers (classes by base layer and tags)
    int persistent;              // 1: logical blocks of the persistent partition
    uint32_t *barrier;           // persistent launches: kBarrierWords counters, zeroed before the launch
};

// Whole sweeps in one launch (small lattices): the next ticket, the team of blocks
// that works (small_team) and, for every group of 16 links, the slices it has done;
// cleared before the launch.  Up to 64 groups an XCD gives each its block (two per
// compute unit in FP64); with two rounds of blocks a slice takes longer than
// launched by itself (2048 links, FP64-18: 9.9 us against 6.9 us).
constexpr uint32_t kSmallGroups = 64;
constexpr uint32_t kSmallTicket = 0, kSmallTeam = 32, kSmallDone = 64, kSmallWords = kSmallDone + kSmallGroups;
// The blocks of an XCD whose numbers leave the same remainder by 8: one block of a
// grid of 8 per group for every group at most, also where the grid has fewer than
// 8 XCDs (with 8, dealt round robin, all blocks of the XCD).  A block holds at most
// one ticket whose wait is not over, so that no ticket is given out two slices
// past an unfinished one, and a link may be loaded ahead of the wait: 2 D slices
// lie between two writes of it.
constexpr uint32_t small_team(uint32_t xcd, uint32_t block) { return (xcd << 3 | (block & 7u)) + 1u; }
constexpr uint32_t kSmallQueues = 64;             // queues cleared together; each launch takes the next one
// Polls until a wait for another block gives up, unless the host sets fewer.  A
// wait for another wave of the block, which such a wait can hold up, polls LDS
// (some 100 cycles against 1000) and has 64 times as many.
constexpr uint32_t kSmallSpinLimit = 1u << 24;
constexpr uint32_t kSmallLdsPolls = 64;

struct SmallArgs {
    UpdateArgs u;                // total_blocks: groups of a slice
    uint32_t items;              // 2 D n_sweeps total_blocks, below 2^31
    DivMagic per_slice;          // division by total_blocks
    uint32_t sweep0;             // index of the first sweep
    uint32_t sweeps;             // sweeps of the launch
    double V;                    // sites per layer
    int nlat;
    double *series;              // measured sweeps: 6 numbers each, in host memory
    uint32_t *work;              // kSmallWords words, zero
    uint32_t *failed;            // host memory: set to 1 by every wait past its limit
    uint32_t spin_limit;         // polls of a wait for other blocks, at most kSmallSpinLimit
};

struct PlaqArgs {
    const void *links;
    const RepDesc *reps;
    int nrep;
    double beta0, beta1;
    int use_rep_beta;
    double *partials;            // [block][5]
    uint32_t total_blocks;
    int by_site;                 // 1: one thread per site; 0: one per (site, plane)
};

constexpr int kDefaultWaves = 2;  // update kernels for D = 4 also exist for 3 (and, FP32, 4) waves/SIMD

}  // namespace su3hb
