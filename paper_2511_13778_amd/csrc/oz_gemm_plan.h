// Which workgroup of the slice GEMM takes which unit of C and which part of k: the split of a call into launches (host) and
// the walk of a workgroup over its units (device), kept apart from the kernel so that a host program can follow both.
#pragma once

#include <algorithm>

#include "oz_internal.h"

namespace oz {

constexpr int kDiag = 4;              // anti-diagonals accumulated side by side
constexpr int kRoundUnits = 32;       // workgroups an XCD runs at a time: 32 CUs, one workgroup each

// The streams of tiles run up to nine entries ahead of the multiplication: with at least this many per unit they never
// need to know more than the next unit.
constexpr int kMinUnitItems = 12;

// steps per 64 of k of a unit with S slices: S for the first group of anti-diagonals, kDiag fewer for each further one
__host__ __device__ inline int unit_items(int S) {
    const int groups = (S + kDiag - 1) / kDiag;
    return groups * S - kDiag * groups * (groups - 1) / 2;
}

// Position `slot` of an XCD's range -> unit of C.  Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; each XCD is given a
// contiguous range.  With a k split (zsplit > 1) a work item is (unit, part of the k range), ordered part by
// part, so the items an XCD runs together still are neighbours on the same k range.
// Plain order: the units themselves in the 4 x 8 order of lin_to_tile.  Per-block order (`order` maps a position
// to a kTile block): an XCD's blocks are taken in groups of 32, and a group in four rounds, one per quadrant, so a
// round touches one 128-row half of each panel: as many panel bytes as a 4 x 8 block of units.
// Returns false past the end of the range.
__host__ __device__ inline bool unit_of(int xcd, int slot, const GemmGrid& g, const int32_t* __restrict__ order, int& ui,
                                        int& uj, int& z, int& local, int& xcd_units) {
    z = 0;
    if (order && g.zsplit == 1) {
        const int per = g.count >> 3, rem = g.count & 7;
        const int blocks = per + (xcd < rem ? 1 : 0);
        xcd_units = 4 * blocks;
        local = 0;
        if (slot >= xcd_units) return false;
        const int grp = slot / (4 * kRoundUnits), in = slot - grp * 4 * kRoundUnits;
        const int gsz = blocks - grp * kRoundUnits < kRoundUnits ? blocks - grp * kRoundUnits : kRoundUnits;
        const int q = in / gsz;
        int ti, tj;
        lin_to_tile(order[g.begin + xcd * per + (xcd < rem ? xcd : rem) + grp * kRoundUnits + in - q * gsz], g.nti, g.ntj, ti, tj);
        ui = 2 * ti + (q & 1);
        uj = 2 * tj + (q >> 1);
        return true;
    }
    const int units = order ? 4 * g.count : g.count, total = units * g.zsplit;
    const int per = total >> 3, rem = total & 7;
    xcd_units = per + (xcd < rem ? 1 : 0);
    if (slot >= xcd_units) return false;
    const int item = xcd * per + (xcd < rem ? xcd : rem) + slot;
    z = item / units;
    local = item - z * units;
    if (order) {
        const int q = local / g.count;
        int ti, tj;
        lin_to_tile(order[g.begin + local - q * g.count], g.nti, g.ntj, ti, tj);
        ui = 2 * ti + (q & 1);
        uj = 2 * tj + (q >> 1);
    } else {
        lin_to_tile(g.begin + local, g.um, g.un, ui, uj);
    }
    return true;
}

// A unit that is a padding-only quadrant of an edge block is passed over: `owed` is called for it (what its round still
// expects of it), and a persistent workgroup moves on to the next unit of its share.  One that is not persistent has no
// next one: every other position belongs to another workgroup, also where the range of its XCD is one longer than
// gridDim.x / 8.  Returns false when nothing is left.
template <class Owed>
__host__ __device__ inline bool skip_padding(int xcd, int stride, int& slot, const GemmGrid& g, const int32_t* __restrict__ order,
                                             int& ui, int& uj, int& z, int& local, int& xcd_units, Owed&& owed) {
    while (ui >= g.um || uj >= g.un) {
        owed();
        if (!g.persistent) return false;
        slot += stride;
        if (!unit_of(xcd, slot, g, order, ui, uj, z, local, xcd_units)) return false;
    }
    return true;
}

// Tiles of C a workgroup of gemm_small_kernel owns.
constexpr int kSmallTile = 32;
constexpr int kSmallLdsMax = 160 * 1024;         // all of a CU's LDS

// The same of gemm_mid_kernel, the most slices it holds, and the most with which two workgroups share a CU.
constexpr int kMidTile = 64;
constexpr int kMidMaxSlices = 16;
constexpr int kMidPairSlices = 8;

struct Split { int z; bool atomic; };

// How a call's units are dealt to launches.
struct LaunchPlan {
    GemmGrid g;
    int per_pos;           // units per position of the launch order
    int positions;
    int kt;                // 64s of k
    int raw_units;         // 128 x 128 slots per plane of the raw buffer
    int min_entries;       // stream entries per 64 of k of a unit with the fewest slices the call can come out with
    int full, rest;        // positions in full rounds, and left over
    Split last;            // of the rest (of everything, if there is no full round)
    bool two;              // the rest in a launch of its own
    bool few;              // at most two slices, on 256 x 256 blocks (gemm_i8_few_kernel) instead of all that
    // slice GEMM and recomposition in one launch instead of all that:
    bool small;            // on 32 x 32 tiles (gemm_small_kernel)
    bool mid, mid_pair;    // on 64 x 64 tiles (gemm_mid_kernel), two workgroups to a CU

    explicit LaunchPlan(const Problem& p) : g() {
        g.nti = int(p.mp / kTile);
        g.ntj = int(p.np / kTile);
        g.um = int((p.m + kUnit - 1) / kUnit);
        g.un = int((p.n + kUnit - 1) / kUnit);
        // the workgroup-to-XCD reasoning behind the in-step waits holds for the whole chip only
        // (8 XCDs of 32 CUs); a partitioned device runs the same kernel without them
        g.full_chip = p.num_cu == 8 * kRoundUnits ? 1 : 0;
        per_pos = p.tile_mode ? 4 : 1;
        positions = p.tile_mode ? g.nti * g.ntj : g.um * g.un;
        kt = int((p.k + kBK - 1) / kBK);
        g.kt_total = kt;
        raw_units = 4 * p.raw_slots;
        min_entries = unit_items(p.s_min);
        // Units are dealt in rounds of one per CU.  A call with less than a round may be split along k as a whole;
        // otherwise the full rounds run unsplit and what is left may be split along k in a launch of its own.
        // (Per-block order: a full round of the order table is one block per CU.)
        // Problems that share a launch (p.batch) are counted together; they share one only with less than a round in all.
        const int round = p.num_cu / p.batch.count;
        full = round != 0 ? positions / round * round : positions;
        rest = positions - full;
        int64_t last_ns = 0;
        last = rest != 0 && rest * per_pos < round ? split(p, rest * per_pos, last_ns) : Split{1, false};
        two = full != 0 && last.z > 1;
        few = few_slices(p);
        fuse(p, last_ns);
    }

    // whether the problems of p.batch can share the launches
    bool can_batch(const Problem& p) const {
        return small || mid || (!few && int64_t(positions) * per_pos * p.batch.count <= p.num_cu);
    }

    // tiles of one problem
    int64_t small_tiles(const Problem& p) const {
        return ((p.m + kSmallTile - 1) / kSmallTile) * ((p.n + kSmallTile - 1) / kSmallTile);
    }

    // Whether slice GEMM and recomposition take longer in their two launches than in one, and in which: estimated in ns for S
    // slices (one more than the fewest where the device decides).  What a tile costs beside its products is its start and
    // its end, its sums and the digits it writes: with many slices and a long k the 128 x 128 units, which read fewer bytes
    // per product, win; otherwise the larger of the small tiles that still gives every CU one.
    //   units       10 us, and for seven slices 14 us, 5.5 us per million elements of C, 0.5 us per part of a k split, and what
    //               split() estimates or 4.2 us per 64 of k and 5 us per round of units; (S+1)/8 of that for S; 0.925 of it
    //               all, and 0.32 us per slice and million elements
    //   64 x 64     a workgroup per CU: per round 1.07 us + 0.60 per slice, and per 64 of k 0.36 us + 37 ns per pair of slices; 2.8 us
    //               per million elements.  Two to a CU (a stage of one 64 of k each; the slice count must be known): 0.81, 0.85, 0.45
    //               and 66, per round of twice as many, one alone 0.95, 0.52 and 54; 2.6 us per million elements
    //   32 x 32     a workgroup per CU at most: 2.5 us, and per 64 of k 0.42 us + 19 ns per slice + 12 per pair; beyond that, per
    //               round of two to a CU: 2.8 us + 0.28 per slice, and per 64 of k 0.55 us + 4 ns per slice + 16 per pair
    // Rounds are whole up to four, beyond that workgroups end at different times.
    // Fitted to 1770 timings of 499 calls of 1 to 16 slices (60 to 8000, k to 6000, one to four problems): the choice is 1 % off the
    // best on average, and against the better of units and 32 x 32 tiles 7 % faster on average (29 % slower at most).  The 64 x 64
    // tiles have to be 12 % better than the others: on a full chip and a long k, at a lower clock, they are worse than estimated (2048^3
    // and 4224 x 3008 x 1792, seven slices, 4 %).
    // Whole calls, units / 32 x 32 / 64 x 64: 200x300x260 nine slices 69 / 36 / 44 us, 512^3 nine 84 / 45 / 58, 1000^3 seven 95 / 86 /
    // 71, 1500x1700x1000 seven 142 / - / 130, 2048^3 seven 246 / 435 / 257, 7936x7936 seven: k = 64 573 / - / 378, k = 256 850 / - / 740,
    // k = 1024 1660 / - / 1730.
    void fuse(const Problem& p, int64_t last_ns) {
        small = mid = mid_pair = false;
        if (p.nkb != 1) return;
        const int64_t S = p.s_min == p.s_cap ? p.s_cap : p.s_min + 1, pairs = S * (S + 1) / 2, cus = p.num_cu;
        const int64_t area = p.m * p.n * p.batch.count;
        // workgroups, per round, ns of a round
        auto rounds_ns = [](int64_t all, int64_t per, int64_t ns) { return all < 4 * per ? (all + per - 1) / per * ns : all * ns / per; };
        const int64_t whole = (int64_t(full) * per_pos * p.batch.count + cus - 1) / cus, unit_ns = int64_t(4200) * kt + 5000;
        int64_t gemm = whole * unit_ns;
        if (rest != 0) gemm += last.z > 1 ? last_ns + int64_t(500) * last.z : (int64_t(rest) * per_pos * p.batch.count + cus - 1) / cus * unit_ns;
        int64_t best = (10000 + (14000 + area * 55 / 10000 + gemm) * (S + 1) / 8) * 925 / 1000 + area * S * 32 / 100000;
        const int64_t small_all = small_tiles(p) * p.batch.count;
        const int64_t small_ns = small_all <= cus ? 2540 + kt * (416 + 19 * S + 12 * pairs)
                                                  : rounds_ns(small_all, 2 * cus, 2770 + 278 * S + kt * (550 + 4 * S + 16 * pairs));
        if (small_ns < best && small_tiles(p) * 512 <= kMaxGridThreads) {
            best = small_ns;
            small = true;
        }
        best = best * 88 / 100;
        if (p.s_cap > kMidMaxSlices || p.m * p.n / (kMidTile * kMidTile) > kMaxGridThreads / 1024) return;
        const int64_t mid_all = ((p.m + kMidTile - 1) / kMidTile) * ((p.n + kMidTile - 1) / kMidTile) * p.batch.count;
        const int64_t mid_ns = rounds_ns(mid_all, cus, 1070 + 600 * S + kt * (357 + 37 * pairs)) + area * 279 / 100000;
        if (mid_ns < best) {
            best = mid_ns;
            small = false;
            mid = true;
        }
        if (p.s_min != p.s_cap || p.s_cap > kMidPairSlices) return;
        const int64_t pair_ns = 810 + 850 * S + kt * (449 + 66 * pairs), alone_ns = 952 * S + kt * (519 + 54 * pairs);
        const int64_t on_cu = (mid_all + cus - 1) / cus;          // workgroups of the fullest CU
        const int64_t two_ns = (mid_all < 8 * cus ? on_cu / 2 * pair_ns + on_cu % 2 * alone_ns : mid_all * pair_ns / (2 * cus)) + area * 262 / 100000;
        if (two_ns < best) {
            small = false;
            mid = mid_pair = true;
        }
    }

    // At most two slices, whatever the device finds: 256 x 256 blocks, where their estimated time is the shorter one.  In us:
    // T and L written at 4.5 TB/s, 12 to finish the first of two anti-diagonals, and per round of all CUs 8 and 0.75 per
    // pair and 64 of k; 128 x 128 units take, per round and all in all, 5.3 and 0.425 per 64 of k with one slice, 8.1 and
    // 0.67 with two.  (Blocks / units measured: one slice 3000^3 43 / 91, 8192^3 462 / 955; two slices 4096 x 4096 x 512 60 / 54,
    // 5000 x 5000 x 1000 116 / 134, 8192^3 1236 / 1493.)
    bool few_slices(const Problem& p) const {
        if (p.s_cap > 2 || p.tile_mode) return false;
        const int64_t blocks = int64_t(g.nti) * g.ntj, pairs = p.s_cap * (p.s_cap + 1) / 2;
        const int64_t blocks_ns = blocks * kTile * kTile * (3 + p.s_cap) / 4500 + 12000 * (p.s_cap - 1) +
                                  (blocks + p.num_cu - 1) / p.num_cu * (8000 + 750 * pairs * kt);
        const int64_t units_ns = (int64_t(g.um) * g.un + p.num_cu - 1) / p.num_cu *
                                 (p.s_cap == 1 ? 5300 + int64_t(425) * kt : 8100 + int64_t(670) * kt);
        return blocks_ns < units_ns;
    }

    // k-blocks a part can touch, whatever the slice count turns out to be (fewer slices: longer k-blocks)
    int nkb_part(const Problem& p, int z) const {
        const int64_t len = (int64_t(kt) + z - 1) / z * kBK;
        return p.nkb == 1 ? 1 : int(std::min<int64_t>(p.nkb, (len - 1) / p.kblk + 2));
    }

    // k split of a launch that cannot fill the chip.  Estimated time in ns for `units` units, seven slices assumed
    // (the slice count is decided on the device): a 64 of k costs a unit about 4.2 us, a workgroup about 5 us to
    // start and to write its sums.  Parts with slots of their own move 10 bytes per element and part (60 ns per part and
    // unit) and, for the rest of a larger product, need a launch to be added (6 us); atomics add 28 bytes per element
    // and part (170 ns) and need the slots zeroed (8 us), but no more memory for more parts.
    Split split(const Problem& p, int units, int64_t& best_ns) const {
        const bool whole = units == positions * per_pos;     // the recomposition puts it together
        const int64_t all = int64_t(units) * p.batch.count;
        const int64_t raw_bytes = int64_t(p.nkb) * p.s_cap * raw_units * (kUnit * kUnit * 4);
        Split best{1, false};
        best_ns = (int64_t(kt) * 4200 + 5000) * 95 / 100;     // a split has to gain 5 %
        for (int z = 2; z <= kt && all * z <= p.num_cu; ++z) {
            const int64_t steps = (kt + z - 1) / z;
            if (int64_t(z - 1) * units * nkb_part(p, z) * part_slot_bytes(p.s_cap) <= raw_bytes) {
                const int64_t ns = steps * 4200 + 5000 + (whole ? 1000 : 6000) + int64_t(60) * all * z;
                if (ns < best_ns) { best_ns = ns; best = Split{z, false}; }
            }
            if (whole && p.batch.count == 1) {
                const int64_t ns = steps * 4800 + 5000 + 8000 + int64_t(170) * units * z;
                if (ns < best_ns) { best_ns = ns; best = Split{z, true}; }
            }
        }
        return best;
    }

    // geometry of the launch of positions [begin, begin + count), and its workgroups
    GemmGrid launch(const Problem& p, int begin, int count, Split sp, unsigned& workgroups) const {
        GemmGrid l = g;
        const int units = count * per_pos;
        l.begin = begin;
        l.count = count;
        l.zsplit = sp.z;
        l.nkb_part = nkb_part(p, sp.z);
        l.persistent = 0;
        // unsplit launches in per-block order give every XCD whole blocks: the ranges differ by up to four units
        workgroups = (p.tile_mode && sp.z == 1) ? unsigned(8 * 4 * ((count + 7) / 8)) : unsigned(units) * unsigned(sp.z);
        // more units than CUs: one workgroup per CU that walks its share (eight equal ranges, one per XCD), if
        // the units are long enough for the streams.  Parts of k never: a workgroup keeps its part (a split fills at most one
        // round of all CUs, which is more than `cus` where their number is no multiple of eight).
        const unsigned cus = unsigned(p.num_cu) & ~7u;
        if (sp.z == 1 && workgroups > cus && cus != 0 && kt * min_entries >= kMinUnitItems) {
            workgroups = cus;
            l.persistent = 1;
        }
        return l;
    }
};

// the slice GEMM of a plan with `few` set, and what it needs before its first launch on a device
bool prepare_gemm_i8_few();
// the slice GEMM and the recomposition of a plan with `small` set
bool prepare_gemm_small();
void launch_gemm_small(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp, double alpha, double beta,
                       double* C, int64_t ldc, const Fallback& fb);
void launch_gemm_i8_few(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp);
// the same of a plan with `mid` set
bool prepare_gemm_mid();
void launch_gemm_mid(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp, double alpha, double beta,
                     double* C, int64_t ldc, const Fallback& fb);

}  // namespace oz
