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
constexpr int kSmallPairSlices = 17;             // most slices with which two of them share a CU
constexpr int kSmallLdsMax = 160 * 1024;         // all of a CU's LDS

// The same of gemm_mid_kernel, the most slices it holds, and the most with which two workgroups share a CU.
constexpr int kMidTile = 64;
constexpr int kMidMaxSlices = 16;
constexpr int kMidPairSlices = 8;
constexpr int kMidDoubleSlices = 10;             // most slices of which all of the LDS holds two stages

constexpr int64_t kCallStagesNs = 16000;         // stages that problems in launches of their own run once each, over the shared ones

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
    bool small, small_pair;    // on 32 x 32 tiles (gemm_small_kernel), two workgroups to a CU
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
        last = rest != 0 && rest * per_pos < round ? split(p, rest * per_pos) : Split{1, false};
        two = full != 0 && last.z > 1;
        few = few_slices(p);
        fuse(p);
    }

    // whether the problems of p.batch can share the launches
    bool can_batch(const Problem& p) const { return small || mid || units_batch(p); }
    bool units_batch(const Problem& p) const {
        return !few && int64_t(positions) * per_pos * p.batch.count <= p.num_cu;
    }

    // tiles of one problem
    int64_t small_tiles(const Problem& p) const {
        return ((p.m + kSmallTile - 1) / kSmallTile) * ((p.n + kSmallTile - 1) / kSmallTile);
    }

    // Whether slice GEMM and recomposition take longer in their two launches than in one, and in which: estimated in ns for S
    // slices (two more than the fewest where the device decides).  What a tile costs beside its products is its start and
    // its end, its sums and the digits it writes: with many slices and a long k the 128 x 128 units, which read fewer bytes
    // per product, win; otherwise the larger of the small tiles that still gives every CU one.  The times below are those of a whole
    // call but for what all routes share, in us; el: million elements of C.
    //   units       1.0, 3.5 el, and per round of all CUs 0.46 per 64 of k and step of a unit and 9.3 per group of anti-diagonals; a split
    //               of k adds, with slots, 0.7 and per part 1.57 and 7 ns per unit and byte of a sum, with atomics per part 0.16 and 28 ns
    //               per unit and slice.  256 x 256 blocks (few): per round 9.9 and per 64 of k 0.70 with one slice, 2.07 with two; 2.8 el,
    //               1 el S
    //   64 x 64     a workgroup per CU: 1.9, per round 0.37 per slice (and 0.51 per slice short of four), and per 64 of k 0.107 and 42 ns per
    //               pair of slices, where the LDS holds one stage only 40 ns per slice besides, no less than 0.243 and 26 ns per slice for the
    //               transfers; 4.7 el less 0.31 el S.  Two to a CU (the slice count must be known): per round of twice as many and per 64 of k
    //               0.086 and 79 ns per pair, no less than 0.08 and 204 ns per slice, one alone 0.238 and 23 per pair; 5 el less 1.5 el S, 0.4 el
    //               at least.  The products take longer on a chip full of tiles, up to 17 and 20 %, and with a long k, up to 10 and 12 %: the
    //               clock is lower and fewer slices come from L2
    //   32 x 32     alone on a CU (no more tiles than CUs, or more slices than half the LDS holds): per round 0.148 per slice, and per 64
    //               of k 0.53 and 14 ns per pair; two to a CU: per round of twice as many 1.67 and 0.088 per slice, and per 64 of k 0.72
    //               and 17 ns per pair; 5.2 el.  No less than the slices at 9 TB/s and 1.5 el
    // Rounds are whole up to four, beyond that workgroups end at different times.
    // Units are fitted to 5100 calls, tiles to 3240 (1 to 26 slices, 40 to 8192, k 16 to 16000, one to four problems, counts known and decided by
    // the device), each timed on every route for 10 to 150 ms on end: of 2150 others the choice is 0.3 % off the best on average, 66 are more
    // than 3 % off and seven more than 10 %.  (Constants of calls of 5 to 16 slices, and a margin of 14 to 28 % for two to a CU from four tiles
    // to a CU on, were 0.8 % off, 195 and 41: 1061 x 4496 x 1016 with eight slices 241 us on units, 175 on tiles; 2417 x 1677 x 1383 with seven
    // 219 and 195; 249 x 3425 x 2858 with twelve 303 and 265; 93 x 1321 x 378 with two 17.3 on 64 x 64 tiles, 15.9 on 32 x 32.)
    // 32 x 32 tiles have to be 7 % better from four rounds of two to a CU on.
    // Units share launches only while a round holds all problems' (units_batch); otherwise each problem pays its rounds and stages.  Of 735
    // complex products and 734 batches of 200 to 3500, about 200 take tiles for it, 11 % faster on average (1556 x 939 x 331 complex 317 us on
    // units, now 192; 2006 x 1146 x 1529 967, now 617), and fifteen more than 3 % slower (1666 x 2989 x 1234 1171, now 1478).
    // (A rule that took two workgroups of 32 x 32 to a CU for any slice count, with no bound on the bytes, was 1.9 % off; 4010 x 2372 x 137 at
    // up to 26 slices took 287 us, now 205, 46 x 119 x 4154 with five 76, now 53, and 2270 x 944 x 2390 with seven 281, now 234.)
    void fuse(const Problem& p) {
        small = small_pair = mid = mid_pair = false;
        if (p.nkb != 1) return;
        const int64_t S = p.s_min == p.s_cap ? p.s_cap : std::min(p.s_cap, p.s_min + 2), pairs = S * (S + 1) / 2, cus = p.num_cu, count = p.batch.count;
        const int64_t area = p.m * p.n * count;
        auto el = [&](int64_t ns) { return area * ns / 1000000; };
        // workgroups, per round, ns of a round
        auto rounds_ns = [](int64_t all, int64_t per, int64_t ns) { return all < 4 * per ? (all + per - 1) / per * ns : all * ns / per; };
        auto units_ns = [&](int64_t problems) -> int64_t {
            const int64_t own = p.m * p.n * problems;
            auto el_own = [&](int64_t ns) { return own * ns / 1000000; };
            if (few) return (int64_t(g.nti) * g.ntj + cus - 1) / cus * (9900 + (S == 1 ? 695 : 2065) * kt) + el_own(2770 + 1010 * S);
            const int64_t step = unit_items(int(S)) * 460, ends = (S + kDiag - 1) / kDiag * 9260, per_cu = int64_t(per_pos) * problems;
            int64_t ns = 975 + el_own(3506 + 13 * S) + ((last.z > 1 ? full : positions) * per_cu + cus - 1) / cus * (kt * step + ends);
            if (last.z > 1) {
                const int64_t parts = last.z * rest * per_cu;
                ns += (kt + last.z - 1) / last.z * step + ends +
                      (last.atomic ? 155 * last.z + 28 * parts * S : 708 + 1565 * last.z + 7 * parts * (4 + S));
            }
            return ns;
        };
        int64_t best = count == 1 || units_batch(p) ? units_ns(count) : count * units_ns(1) + (count - 1) * kCallStagesNs;
        const int64_t small_all = small_tiles(p) * count;
        const bool pair = small_all > cus && p.s_cap <= kSmallPairSlices;
        const int64_t small_products = pair ? rounds_ns(small_all, 2 * cus, 1673 + 88 * S + kt * (720 + 17 * pairs))
                                            : rounds_ns(small_all, cus, 148 * S + kt * (530 + 14 * pairs));
        const int64_t small_ns = std::max(small_products + el(5236), small_all * (2 * kSmallTile * kBK) * kt * S / 9000 + el(1500));
        if (small_ns < best * (small_all >= 8 * cus ? 93 : 100) / 100 && small_tiles(p) * 512 <= kMaxGridThreads) {
            best = small_ns;
            small = true;
            small_pair = pair;
        }
        if (p.s_cap > kMidMaxSlices || p.m * p.n / (kMidTile * kMidTile) > kMaxGridThreads / 1024) return;
        const int64_t mid_all = ((p.m + kMidTile - 1) / kMidTile) * ((p.n + kMidTile - 1) / kMidTile) * count;
        // thousandths by which the products take longer: on a chip full of tiles (from `first` rounds on, all of it four later) and for a long k (all
        // of it from 128 64s on)
        auto slower = [&](int64_t most, int64_t first, int64_t most_long) {
            return 1000 + most * std::clamp<int64_t>(mid_all - first * cus, 0, 4 * cus) / (4 * cus) + most_long * std::min(kt, 128) / 128;
        };
        const int64_t alone_kt = std::max<int64_t>(107 + 42 * pairs + (S > kMidDoubleSlices ? 40 * S : 0), 243 + 26 * S);
        const int64_t alone_ns = 1905 + el(std::max<int64_t>(4663 - 310 * S, 0)) +
                                 rounds_ns(mid_all, cus, 367 * S + std::max<int64_t>(512 * (4 - S), 0) + kt * alone_kt * slower(169, 1, 103) / 1000);
        if (alone_ns < best) {
            best = alone_ns;
            mid = true;
        }
        if (p.s_min == p.s_cap && p.s_cap <= kMidPairSlices && mid_all > cus) {
            const int64_t two = kt * std::max<int64_t>(86 + 79 * pairs, 80 + 204 * S), one = kt * (238 + 23 * pairs);
            const int64_t on_cu = (mid_all + cus - 1) / cus;          // workgroups of the fullest CU
            const int64_t products = mid_all < 8 * cus ? on_cu / 2 * two + on_cu % 2 * one : mid_all * two / (2 * cus);
            if (products * slower(203, 2, 123) / 1000 + el(std::max<int64_t>(435, 5000 - 1500 * S)) < best) mid = mid_pair = true;
        }
        if (mid) small = small_pair = false;
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
    Split split(const Problem& p, int units) const {
        const bool whole = units == positions * per_pos;     // the recomposition puts it together
        const int64_t all = int64_t(units) * p.batch.count;
        const int64_t raw_bytes = int64_t(p.nkb) * p.s_cap * raw_units * (kUnit * kUnit * 4);
        Split best{1, false};
        int64_t best_ns = (int64_t(kt) * 4200 + 5000) * 95 / 100;     // a split has to gain 5 %
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
