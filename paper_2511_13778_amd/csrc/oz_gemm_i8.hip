// Slice-pair INT8 GEMMs with exact int32 accumulation: the one dense contraction of the method.
// (paper: section "FP64 Emulation on Low-Precision Units": products are computed slice by slice;
//  section "ESC": cost is quadratic in the slice count; the kept pairs are s + t <= S - 1, the
//  count behind "seven slices rather than eight: 22 % less compute"; section "Pre-processing
//  and Safety Checks": partial results are aggregated so that accumulators cannot overflow.)
//
//   P_d[j][i] = sum_{s+t=d} sum_{l in k-block kb} As[s][i][l] * Bs[t][j][l],   d = 0..S-1
//
// One launch covers all S(S+1)/2 pairs.  A workgroup owns a 128x128 unit of C and takes the
// anti-diagonals in groups of up to four, from the least significant (S-1) to the most significant
// (0): four sets of int32 accumulators grow side by side while k is walked once per group.  When a
// group is complete, its sums are split exactly, least significant first, into a balanced digit
// (T mod 256 in [-128,127], one byte per element, written out) and a carry (T - digit)/256 added to
// the next anti-diagonal's sum; the carry out of a group is the start value of the next one, and
// d = 0 is written as an int32 word.  So a k-block leaves the exact integer sum_d P_d 256^(S-1-d) in
// 4 + (S-1) bytes per element instead of 4S, already aggregated.
//
// What bounds it: the power limit and idle issue slots together.  At 8192^3 with seven slices it reaches 2.99 POP/s, the matrix
// unit busy 76 % of the cycles at 1.88 GHz; an MFMA-only loop on the same register tile and random digits reaches 4.2 POP/s, busy
// 99 % at 2.0 GHz (4.9 with constant operands at 2.35 GHz; 32x32x32 tiles on random digits 3.5 at 1.67 GHz).  The clock is
// below its 2.4 GHz in all of them, so what the idle quarter is worth is open: schedules between 71 and 76 % busy differed by
// 1.5 % in time.  Ends of groups, where sums are written and reloads of spilled registers wait for the transfers in flight,
// are about 2 % at this size.  Every byte moved takes its share of the power: one LDS read of 1 KB per two 32x32x32 MFMAs 8 %,
// one direct-to-LDS transfer of 1 KB per four another 10 % (loops of the same shape as the one below).
// Hence the order of the loops.  Four anti-diagonals at a time means that an A fragment read from LDS
// meets four B slices, and a B fragment that has been read stays in registers for four steps:
//  * A step is one slice s of A for 64 of k.  With d_hi the group's first anti-diagonal, step s multiplies
//    A_s with B_t, t = d_hi-s-j, j = 0..3 (as far as t >= 0), accumulator set j.  From one step to
//    the next the window of B slices moves by one: it lives in four register slots.
//  * For seven slices a 64 of k thus costs 10 tiles of A and of B for 28 pairs (7 + 3 in the groups
//    6..3 and 2..0) instead of 28: 29 % fewer bytes through L2, LDS and the fabric than 256x256 tiles that
//    walk the pairs one by one, at the same 256 accumulator registers per lane.
//  * v_mfma_i32_16x16x64_i8: per operation it moves a fifth less through the register file than
//    32x32x32 (16x16 sums are read and written for 64 of k instead of 32).
// Measured with seven slices, against one pair at a time on 256x256 tiles of 32x32x32: 8192^3 11.2 -> 10.3 ms
// (2.75 -> 2.99 POP/s), 1024x1024x65536 1.85 -> 1.27 ms, and
// where the quarter of the size lets more CUs work without a k split, 2048^3 0.53 -> 0.17 ms.  Calls of one or two slices that
// fill the chip are better off on 256x256 blocks, pair by pair (oz_gemm_few.hip).
//
// Mapping to gfx950:
//  * 4 waves per workgroup, each 64x64 x four anti-diagonals (256 accumulator registers per lane); one
//    workgroup per CU.
//  * 10 LDS stages of 16 KB (all 160 KB), one per step.  Tiles go from L2 straight into LDS
//    with global_load_lds_dwordx4 (no staging registers, no LDS store instructions), issued seven
//    steps ahead; one workgroup barrier per step.  The slice panels are stored [k/16][row][16], so a
//    tile is four contiguous 2 KB runs per operand and the LDS image [k chunk][row][16 B] is what
//    the MFMA operand loads read (ds_read_b128 per lane: row = lane%16, k chunk = lane/16).
//  * The B-slices feed the MFMA's row operand and the A-slices its column operand, so the lane
//    index of the result runs along i and the four registers of a lane are four consecutive j: one
//    dword of the digit planes.
//  * Workgroup ids are remapped so that the units resident on one XCD form a compact block and
//    share their A and B panels in that XCD's L2; the workgroups of such a round wait for each
//    other (bounded) so that they stay within what L2 holds.
//  * One wave per SIMD, so nothing hides an instruction that delays the next MFMA: LDS reads, transfers and scalar
//    work are spread over the gaps between a step's MFMAs, and the loops are laid out for few branches.
#include <type_traits>

#include "oz_f64_direct.h"
#include "oz_gemm_device.h"

namespace oz {

constexpr int kDiagAtomic = 3;                   // the same in the atomic variant (its 32x32 tiles need more registers in flight)
constexpr int kStages = 10;                      // LDS stages; the pipeline below counts on ten
constexpr int kOperandBytes = kUnit * kBK;       // 8 KB: one operand's tile
constexpr int kStageBytes = 2 * kOperandBytes;   // A tile, then B tile
constexpr int kRingBytes = kStages * kStageBytes;
constexpr int kGemmLds = kRingBytes;             // 160 KB: all of the CU's LDS
static_assert(kKPad % kBK == 0, "k padding must cover whole steps");
static_assert(kTile == 2 * kUnit, "a block of C with its own slice count is two by two units");

constexpr int kSyncMinK = 2048;       // units of a shorter k run without the in-step waits
constexpr int kSyncMinItems = 320;    // nor one of fewer steps than seven slices have there (8192 x 8192 x 2048: one slice
                                      // 681 -> 630 us, two 845 -> 807, three 1055 -> 1005, four 1388 -> 1350)

// 16 bytes per lane to a wave-uniform base (scalar register pair) plus a 32-bit per-lane byte offset.
// Written as assembly so that the address stays in this form: left to itself the compiler builds a
// 64-bit per-lane address for each of the stores of an epilogue, hoists them out of the loop over the groups
// and spills them.
// The s_nop covers the five wait states the hardware needs between a vector-ALU write of a scalar
// register (a register-allocator reload with v_readlane, say) and a memory instruction that reads
// it as its base: inside an asm block the compiler does not insert them itself, and a store issued
// too early takes the stale register value as its address.  The one behind it keeps the next instruction from
// overwriting the data before the store has read all four registers.
// Streamed past L2, where the slices are (four 900 x 1000 x 1500 234 -> 230 us, 6144 x 6144 x 1024 1040 -> 1031; level where k is long).
__device__ __forceinline__ void store_lane_16(void* uniform_base, uint32_t lane_byte_off, v4i data) {
    asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1"
                 :: "v"(lane_byte_off), "v"(data), "s"(uniform_base) : "memory");
}

template <int N>
struct Int { static constexpr int v = N; };

// The order of a step's work between its MFMAs: 0..3 fragments of the next A tile (first: the next step starts with
// them), 10.. the step's NB further LDS reads, 20..23 transfers, 30..33 the streams move on, 34 and 35 the ring.
constexpr int kOwnPieces = 14;
template <int NB>
constexpr int kPieces[kOwnPieces + NB] = {0, 1, 2, 20, 3, 21, 34, 22, 35, 23, 30, 31, 32, 33};
template <>
constexpr int kPieces<4>[kOwnPieces + 4] = {0, 1, 2, 20, 3, 10, 21, 11, 12, 22, 13, 34, 23, 35, 30, 31, 32, 33};
template <>
constexpr int kPieces<8>[kOwnPieces + 8] = {0, 1, 2, 20, 3, 10, 11, 21, 12, 13, 22, 14, 15, 23, 16, 17, 34, 35, 30, 31, 32, 33};

// ATOMIC = false: 16x16x64 MFMAs; the sums are aggregated in registers and written as T / L, to the matrix planes
// (part 0) or to the part's slot of the raw buffer (parts z > 0 of a k split).
// ATOMIC = true: unaggregated sums are added into the unit's raw slot with integer atomics (exact and order-free; the
// host zeroes the slots before and aggregates them after): as many parts as one likes in the same memory, for
// outputs of few units.  32x32x32 MFMAs there: a half-wave then adds to 128 contiguous bytes instead of 64, and
// such launches are bound by the atomics.
//
// A workgroup takes units slot, slot + stride, ... of its XCD's range (one only where the launch has a workgroup per
// unit); the stream of tiles runs on into the next unit, so neither the first tiles' latency nor the drain
// of the last sums is waited for.
template <bool ATOMIC>
__device__ __forceinline__ void gemm_i8_body(const int8_t* __restrict__ As, const int8_t* __restrict__ Bs, int32_t* __restrict__ T,
                                             int8_t* __restrict__ L, int32_t* __restrict__ raw, int raw_units, int64_t mp,
                                             int64_t np, int64_t kp, int s_cap, Record* rec, const GemmGrid& g,
                                             const int32_t* __restrict__ tile_S) {
    constexpr int D = ATOMIC ? kDiagAtomic : kDiag;
    constexpr int TAIL = D - 1;          // last steps of a 64 of k: D-1 .. 1 accumulator sets
    extern __shared__ __align__(16) uint8_t lds[];
    if (rec->res.fallback) return;
    const int S_all = rec->res.slices_used;
    // k-range one int32 accumulator can take with S slices (S*kblk digit products of at most 2^14);
    // the k-blocks are those of the call's largest slice count, whatever this block's own count is
    const int64_t kblk = k_block_length(S_all);
    // per-block mode: the table of slice counts is followed by the order the blocks are dealt in
    const int32_t* order = tile_S ? tile_S + g.nti * g.ntj : nullptr;

    const int xcd = int(blockIdx.x) & 7, stride = int(gridDim.x) >> 3;
    int slot = int(blockIdx.x) >> 3;
    int ui, uj, z, local, xcd_units;
    if (!unit_of(xcd, slot, g, order, ui, uj, z, local, xcd_units)) return;

    // Keep the workgroups that share panels in step.  An XCD runs 32 workgroups at a time (one
    // per CU) and its units are ordered so that each such round is one 4x8 block.  Where a unit is long, the
    // workgroups of a round wait for each other at its start and, when k is very long, after every
    // group of anti-diagonals, because workgroups that have drifted apart never fall back into step by
    // themselves and then miss in L2 what their neighbours loaded (measured: 2 % at 8192^3, 6 % at 16384^3).
    // Arrival number q of a workgroup of round r waits for 32*r*steps + (q+1)*members arrivals on the XCD's
    // counter (earlier rounds are full).  The wait also drains the wave's stores, so short units go without.
    const int sync_steps = kp >= kMidSyncMinK ? int((kp + kblk - 1) / kblk) * ((S_all + D - 1) / D) : 1;
    const bool sync_on = !ATOMIC && g.full_chip && g.zsplit == 1 && xcd_units > kRoundUnits && kp >= kSyncMinK && g.kt_total * unit_items(S_all) >= kSyncMinItems &&
                         (stride == kRoundUnits || stride >= xcd_units);
    int sync_q = 0;
    bool sync_wait = true;               // thread 0: stop waiting once the others were not met in time
    auto arrive = [&]() {
        const int round = slot / kRoundUnits;
        const int members = min(kRoundUnits, xcd_units - round * kRoundUnits);
        ++sync_q;
        round_sync(&rec->tile_sync[xcd], round * kRoundUnits * sync_steps + sync_q * members, sync_wait);
    };
    // a quadrant of an edge block that holds padding only: nothing to do but the arrivals it owes its round
    auto pass_padding = [&]() -> bool {
        return skip_padding(xcd, stride, slot, g, order, ui, uj, z, local, xcd_units, [&]() {
            if (sync_on && threadIdx.x == 0) atomicAdd(&rec->tile_sync[xcd], sync_steps);
        });
    };
    if (!pass_padding()) return;
    // slice count of a unit: its block's own (per-block mode: the first S digit planes of the operands
    // and the pairs s + t <= S - 1) or the call's
    auto slices_of = [&](int i, int j) -> int { return tile_S ? min(tile_S[(j >> 1) * g.nti + (i >> 1)], S_all) : S_all; };
    int S = slices_of(ui, uj);

    // this workgroup's share of k, in steps of 64: part z of zsplit equal parts of the whole range
    const int kt_total = g.kt_total;
    const int kt_first = int(int64_t(kt_total) * z / g.zsplit);
    const int kt_end = int(int64_t(kt_total) * (z + 1) / g.zsplit);
    const int kt_per_block = int(kblk / kBK);
    const int kb_first = kt_first / kt_per_block, kb_last = (kt_end - 1) / kt_per_block;
    // 64s of k [kt_lo(kb), kt_lo(kb) + kt_count(kb)) of k-block kb belong to this workgroup
    auto kt_lo = [&](int kb) -> int { return max(kb * kt_per_block, kt_first); };
    auto kt_count = [&](int kb) -> int { return min((kb + 1) * kt_per_block, kt_end) - kt_lo(kb); };

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = wave & 1, wj = wave >> 1;

    // ---- the streams of tiles -----------------------------------------------------------------
    // Entry e of the A (B) stream: for each unit, k-block, group and 64 of k, slice s = 0..d_hi of A (t = d_hi..0 of B).
    // Item x is entry x of A and entry x+2 of B; it goes to LDS stage x mod 10.  Wave w fetches k chunk w of both
    // tiles: four transfers of 1 KB.
    struct Stream {
        const uint8_t* p;                // next entry
        int64_t wrap;                    // from the last slice of a 64 of k to the first of the next
        int r, n;                        // entries left of this 64 of k; entries per 64 of k
        int c;                           // 64s of k left in this group of this k-block
        int kb;
        bool ahead;                      // already on the next unit
    };
    const int64_t planeA = kp * mp, planeB = kp * np;                     // bytes per slice plane
    const int64_t stepA = int64_t(kBK) * mp, stepB = int64_t(kBK) * np;   // bytes per 64 of k
    auto base_of = [&](const int8_t* X, int64_t rows, int unit) -> const uint8_t* {
        return reinterpret_cast<const uint8_t*>(X) + (int64_t(wave) * rows + int64_t(unit) * kUnit) * 16;
    };
    bool has_next = false;               // the unit after this one, for the streams to run on into
    int nui = 0, nuj = 0, nS = 0, nslot = 0;
    auto find_next = [&]() {
        const int cui = ui, cuj = uj, cslot = slot;
        slot += stride;
        has_next = unit_of(xcd, slot, g, order, ui, uj, z, local, xcd_units) && pass_padding();
        nui = ui; nuj = uj; nslot = slot;
        if (has_next) nS = slices_of(nui, nuj);
        ui = cui; uj = cuj; slot = cslot;
    };
    auto group_start = [&](Stream& s, bool is_b) {       // s.n and s.kb are set
        s.r = s.n;
        s.c = kt_count(s.kb);
        const int64_t kt = kt_lo(s.kb);
        if (is_b) {
            s.p = base_of(Bs, np, s.ahead ? nuj : uj) + int64_t(s.n - 1) * planeB + kt * stepB;
            s.wrap = stepB + int64_t(s.n - 1) * planeB;
        } else {
            s.p = base_of(As, mp, s.ahead ? nui : ui) + kt * stepA;
            s.wrap = stepA - int64_t(s.n - 1) * planeA;
        }
    };
    // past the last entry of a group: the next group, k-block or unit; at the very end the last group
    // once more (surplus entries that land in stages nobody reads)
    auto group_end = [&](Stream& s, bool is_b) {
        if (s.n > D) {
            s.n -= D;
        } else if (s.kb < kb_last) {
            ++s.kb;
            s.n = s.ahead ? nS : S;
        } else if (has_next && !s.ahead) {
            s.ahead = true;
            s.kb = kb_first;
            s.n = nS;
        } else {
            s.n = (s.ahead ? nS : S) % D == 0 ? D : (s.ahead ? nS : S) % D;
        }
        group_start(s, is_b);
    };
    Stream sa, sb;
    const int64_t downB = -planeB;
    // The next entry: `wrap` bytes on after the last slice of a 64 of k, else a plane on (A) or back (B).  Without a
    // branch but for the end of a group, and in assembly so that it stays at eight scalar instructions: they fit the
    // gaps between the matrix instructions, while a taken branch leaves the matrix unit idle for tens of cycles.
    // r is written before the other operands are read, hence its '&': without it the compiler may put n in the same register,
    // being the same number whenever a 64 of k begins.
    int64_t by = 0;
    auto next_by = [&](Stream& s, bool is_b) {
        asm volatile("s_sub_u32 %[r], %[r], 1\n\ts_cmp_eq_u32 %[r], 0\n\ts_cselect_b64 %[by], %[wrap], %[plane]\n\t"
                     "s_cselect_b32 %[r], %[n], %[r]\n\ts_subb_u32 %[c], %[c], 0"
                     : [r] "+&s"(s.r), [c] "+s"(s.c), [by] "=&s"(by)
                     : [wrap] "s"(s.wrap), [plane] "s"(is_b ? downB : planeA), [n] "s"(s.n) : "scc");
    };
    auto next_check = [&]() {            // one branch for both streams
        if (__builtin_expect(min(uint32_t(sa.c), uint32_t(sb.c)) == 0, 0)) {
            if (sa.c == 0) group_end(sa, false);
            if (sb.c == 0) group_end(sb, true);
        }
    };
    const uint32_t lane_off = uint32_t(lane) * 16;
    const uint32_t lds_wave = uint32_t(uintptr_t((__attribute__((address_space(3))) uint8_t*)lds)) + uint32_t(wave) * (kUnit * 16);
    // transfer x of an item into the stage at byte `stage` of the ring
    auto dma = [&](uint32_t stage, int x) {
        const uint32_t la = lds_wave + stage;
        if (x == 0) dma16<0>(sa.p, lane_off, la);
        else if (x == 1) dma16<kOperandBytes>(sb.p, lane_off, la);
        else if (x == 2) dma16<1024>(sa.p, lane_off + 1024, la);
        else dma16<kOperandBytes + 1024>(sb.p, lane_off + 1024, la);
    };

    // ---- fragments ------------------------------------------------------------------------------
    // 16x16x64: fragment f = rows 16f..16f+15, all 64 of k.  32x32x32: f = 2 * (rows 32(f/2)..) + (half of k).
    const uint32_t rd_lane = ATOMIC ? uint32_t(lane >> 5) * (kUnit * 16) + uint32_t(lane & 31) * 16
                                    : uint32_t(lane >> 4) * (kUnit * 16) + uint32_t(lane & 15) * 16;
    const uint32_t rdA = rd_lane + uint32_t(wi) * 1024, rdB = rd_lane + uint32_t(wj) * 1024 + kOperandBytes;
    constexpr int kFragImm[4] = {0, ATOMIC ? 4096 : 256, 512, ATOMIC ? 4608 : 768};
    auto frag = [&](uint32_t off) -> v4i { return *reinterpret_cast<const v4i*>(lds + off); };

    v4i fa[3][4], fb[4][4];              // A: two in turn and one for the last step of a 64 of k; B: [slot][f]
    constexpr int NT = ATOMIC ? 2 : 4;   // MFMA tiles per wave and direction
    typedef typename std::conditional<ATOMIC, v16i, v4i>::type acc_t;
    acc_t acc[D][NT][NT];                // [j][tj][ti]
    // Cleared by matrix instructions with zero operands: written by the vector ALU, an accumulator would be kept in an
    // ordinary vector register by the register allocator and moved in and out in every step.
    const v4i zero4 = {0, 0, 0, 0};
    auto clear = [&](int from) {
#pragma unroll
        for (int j = 0; j < D; ++j)
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    if (j < from) continue;
                    if constexpr (ATOMIC) {
                        const v16i none = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                        acc[j][a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(zero4, zero4, none, 0, 0, 0);
                    } else {
                        acc[j][a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(zero4, zero4, zero4, 0, 0, 0);
                    }
                }
    };
    clear(0);
    constexpr int kSetMfma = ATOMIC ? 8 : 16;
    // MFMA number q of accumulator set j; consecutive ones share an operand
    auto mfma = [&](int j, const v4i (&xb)[4], const v4i (&xa)[4], int q) {
        if constexpr (ATOMIC) {
            const int ks = q >> 2, tj = (q >> 1) & 1, ti = tj ? 1 - (q & 1) : (q & 1);
            acc[j][tj][ti] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xb[2 * tj + ks], xa[2 * ti + ks], acc[j][tj][ti], 0, 0, 0);
        } else {
            const int tj = q >> 2, ti = (tj & 1) ? 3 - (q & 3) : (q & 3);
            acc[j][tj][ti] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xb[tj], xa[ti], acc[j][tj][ti], 0, 0, 0);
        }
    };

    // ---- one step ---------------------------------------------------------------------------------
    // Step a multiplies entry a of A with entries a .. a+sets-1 of B.  Before it, items up to a+2 have landed, and no wave
    // reads item a-3 any more, so item a+7 may overwrite that stage.
    //
    // Register slots.  Within a 64 of k with n entries, entry s of B lies in slot (s + o) mod 4 with o such that the
    // last TAIL steps always start at slot 0: o = (TAIL - n) mod 4.  So the tail is straight code, and the steps
    // before it (all with D sets, step u serving slots u, u+1, .. mod 4) are a loop unrolled by four behind up to
    // three single ones: a few branches per 64 of k.  (With a test per accumulator set, seven branches a step kept
    // the matrix unit idle a quarter of the time: 16x16x64 leaves 16 cycles to fetch what comes next.)
    //   step u        reads entry a+3 of B into slot u+3, which step u-1 gave up
    //   tail 0        reads no B
    //   tail TAIL-2   reads what the next 64 of k starts with in the two slots that are free by then
    //   tail TAIL-1   the same for the slot that tail TAIL-2 gave up
    //   next step     the same for the last one
    // Which entries those are depends on the next o: entry j of the next 64 of k goes to slot (j + o) mod 4, it lies in
    // item c1 + j - 2 when c1 is the first step of that 64 (j = 3 is read again by that step itself: harmless).
    //
    // The memory work is spread over the MFMAs: four waves' LDS reads take 32 cycles, their transfers 64.
    uint32_t cur = 0, nxt = 0, put = 0;  // ring offsets of the stages of items a, a+1 and a+7
    uint32_t oa = 0, ob = 0;             // where this lane reads A and B of item a+1 (computed in the step before)
    auto ring = [&](uint32_t off) -> uint32_t { return off >= uint32_t(kRingBytes) ? off - kRingBytes : off; };
    uint32_t pre_base = 0;               // ring offset of item c1 - 2
    int o_next = 0;
    auto preload = [&](int sl, int f) {  // fragment f of what slot `sl` starts the next 64 of k with
        const uint32_t st = ring(pre_base + uint32_t((sl - o_next) & 3) * kStageBytes);
        fb[sl][f] = frag(rdB + st + kFragImm[f]);
    };
    // SETS accumulator sets, first B slot SLOT, A in fa[AR], next A into fa[AW]; B(x) = x-th of NB further pieces
    auto step = [&](auto SETS, auto SLOT, auto AR, auto AW, auto NB, auto WAITLDS, auto&& more) {
        constexpr int sets = decltype(SETS)::v, first = decltype(SLOT)::v, ar = decltype(AR)::v, aw = decltype(AW)::v;
        uint32_t oa_next = 0, ob_next = 0;
        constexpr int nb = decltype(NB)::v, pieces = kOwnPieces + nb, gaps = sets * kSetMfma;
#pragma unroll
        for (int j = 0; j < sets; ++j)
#pragma unroll
            for (int q = 0; q < kSetMfma; ++q) {
                mfma(j, fb[(first + j) & 3], fa[ar], q);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int x = 0; x < pieces; ++x)
                    if (x * gaps / pieces == j * kSetMfma + q) {
                        const int w = kPieces<nb>[x];
                        if (w < 10) fa[aw][w] = frag(oa + kFragImm[w]);
                        else if (w < 20) more(w - 10);
                        else if (w < 30) dma(put, w - 20);
                        else if (w == 30) next_by(sa, false);
                        else if (w == 31) sa.p += by;
                        else if (w == 32) next_by(sb, true);
                        else if (w == 33) { sb.p += by; next_check(); }
                        else if (w == 34) { asm volatile("" : "+s"(cur)); cur = ring(cur + kStageBytes); nxt = ring(cur + kStageBytes); }
                        else { asm volatile("" : "+s"(nxt)); oa_next = rdA + nxt; ob_next = rdB + nxt; }
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
        put = ring(put + kStageBytes);
        oa = oa_next;
        ob = ob_next;
        // The wait as a builtin: the compiler then knows which LDS reads have returned.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x4070 | (decltype(WAITLDS)::v ? 0x0000 : 0x0F00));       // vmcnt(16), lgkmcnt(0) or none
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto none = [](int) {};
    auto head = [&](auto UU) {           // step u: all D sets
        constexpr int u = decltype(UU)::v;
        step(Int<D>{}, Int<u>{}, Int<(u & 1)>{}, Int<((u + 1) & 1)>{}, Int<4>{}, Int<1>{},
             [&](int x) { fb[(u + 3) & 3][x] = frag(ob + kFragImm[x]); });
    };

    // prologue: the first two entries of B, seven items; what the first step starts with; then on
    sa = Stream{nullptr, 0, 0, S, 0, kb_first, false};
    sb = sa;
    if (g.persistent) find_next();
    group_start(sa, false);
    group_start(sb, true);
    if (sync_on) arrive();
#pragma unroll
    for (int e = 0; e < 2; ++e) {        // into stages 8 and 9, where items -2 and -1 would lie
        dma(uint32_t(8 + e) * kStageBytes, 1);
        dma(uint32_t(8 + e) * kStageBytes, 3);
        next_by(sb, true);
        sb.p += by;
        next_check();
    }
    for (int x = 0; x < 7; ++x) {
        const uint32_t st = uint32_t(x) * kStageBytes;
        dma(st, 0); dma(st, 1); dma(st, 2); dma(st, 3);
        next_by(sa, false);
        sa.p += by;
        next_by(sb, true);
        sb.p += by;
        next_check();
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x4070);          // vmcnt(16): items up to 2 have landed
    asm volatile("s_barrier" ::: "memory");
    pre_base = uint32_t(8) * kStageBytes;
    o_next = (TAIL - S) & 3;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        fa[0][x] = frag(rdA + kFragImm[x]);
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) preload(sl, x);
    }
    nxt = kStageBytes;
    put = 7 * kStageBytes;
    oa = rdA + nxt;
    ob = rdB + nxt;

    int kb = kb_first, d_hi = S - 1;
    for (;;) {
        // ---- group d_hi of k-block kb of unit (ui, uj) ----
        const int n = d_hi + 1, nd = min(D, n), heads = n - TAIL;
        const int o = (TAIL - n) & 3;
        const bool last = d_hi < D && kb == kb_last;             // of the unit
        const int n_after = d_hi >= D ? n - D : (kb < kb_last ? S : nS);      // entries of the next group's 64s of k
        const int o_after = (TAIL - n_after) & 3;
        for (int c = kt_count(kb); c > 0; --c) {
            // the slot that the last tail step gave up, and the A tile where a first step that is not step 0 expects it
#pragma unroll
            for (int x = 0; x < 4; ++x) preload((D - 2) & 3, x);
            if (o != 0) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    fa[1][x] = fa[0][x];
                    fa[2][x] = fa[0][x];
                }
            }
            // a first round of the loop that starts at step o
            for (int h = -o; h < heads; h += 4) {
                if (__builtin_expect(h >= 0, 1)) head(Int<0>{});
                if (__builtin_expect(h >= -1, 1)) head(Int<1>{});
                if (__builtin_expect(h >= -2, 1)) head(Int<2>{});
                head(Int<3>{});
            }
            o_next = c == 1 ? o_after : o;
            if constexpr (D > 3) {
                if (__builtin_expect(n > 2, 1)) step(Int<3>{}, Int<0>{}, Int<0>{}, Int<1>{}, Int<0>{}, Int<1>{}, none);
            }
            if (__builtin_expect(n > 1, 1)) {
                pre_base = cur;          // this is step c1 - 2
                step(Int<2>{}, Int<D - 3>{}, Int<(D - 3)>{}, Int<2>{}, Int<8>{}, Int<0>{},
                     [&](int x) { preload(x < 4 ? (D & 3) : ((D - 1) & 3), x & 3); });
            } else {
                pre_base = cur >= uint32_t(kStageBytes) ? cur - kStageBytes : cur + (kRingBytes - kStageBytes);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    preload(D & 3, x);
                    preload((D - 1) & 3, x);
                }
            }
            step(Int<1>{}, Int<D - 2>{}, Int<2>{}, Int<0>{}, Int<4>{}, Int<0>{}, [&](int x) { preload((D - 3) & 3, x); });
        }

        // anti-diagonals d_hi .. d_hi-nd+1 of k-block kb are complete in acc[0 .. nd-1].
        // Every address below is a wave-uniform pointer (scalar arithmetic) plus one per-lane 32-bit offset that
        // is the same for all stores of a kind.
        if constexpr (ATOMIC) {
            // result register r of MFMA tile (tj, ti): j = tj*32 + 8*(r/4) + 4*(lane/32) + r%4, i = ti*32 + lane%32
            const uint32_t lane_raw = uint32_t(wj * 64 + 4 * (lane >> 5)) * kUnit + uint32_t(wi * 64 + (lane & 31));
#pragma unroll
            for (int j = 0; j < D; ++j) {
                if (j < nd) {
                    int32_t* dst = raw + ((int64_t(kb) * s_cap + (d_hi - j)) * raw_units + local) * (kUnit * kUnit) + lane_raw;
#pragma unroll
                    for (int tj = 0; tj < NT; ++tj)
#pragma unroll
                        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                            for (int q = 0; q < 16; ++q)
                                atomicAdd(dst + (tj * 32 + 8 * (q >> 2) + (q & 3)) * kUnit + ti * 32, acc[j][tj][ti][q]);
                }
            }
            clear(0);
        } else {
            // where T / L go: the matrix planes, or (parts z > 0) the unit's own slots in the raw buffer.
            // row: elements between neighbouring j of T, j/4 of L
            int64_t row = mp, planeL = np * mp;
            uint8_t* wT = reinterpret_cast<uint8_t*>(T) + ((int64_t(kb) * np + int64_t(uj) * kUnit) * mp + int64_t(ui) * kUnit) * 4;
            uint8_t* wL = reinterpret_cast<uint8_t*>(L) + int64_t(kb) * (s_cap - 1) * planeL +
                          (int64_t(uj) * (kUnit / 4) * mp + int64_t(ui) * kUnit) * 4;
            if (z > 0) {
                const int units = order ? 4 * g.count : g.count;
                row = kUnit;
                planeL = kUnit * kUnit;
                wT = reinterpret_cast<uint8_t*>(raw) +
                     ((int64_t(z - 1) * units + local) * g.nkb_part + (kb - kb_first)) * part_slot_bytes(s_cap);
                wL = wT + kUnit * kUnit * 4;
            }
            wT += (int64_t(wj) * 64 * row + wi * 64) * 4;
            wL += (int64_t(wj) * 16 * row + wi * 64) * 4;
            // Result register r of MFMA tile (tj, ti): j = tj*16 + 4*(lane/16) + r, i = ti*16 + lane%16.  A lane's dwords
            // for four ti are 16 apart in i; they change places through LDS (in the part of the stage that this
            // wave alone fills next, free until then), so that a lane stores 16 bytes and 16 lanes 256 in a row.
            const uint32_t lq = uint32_t(lane >> 4), lx = uint32_t(lane & 15);
            const uint32_t lane_L = (lq * uint32_t(row) + lx * 4) * 4u, lane_T = (4 * lq * uint32_t(row) + lx * 4) * 4u;
            constexpr uint32_t kScratchRow = 320;        // 64 dwords, and 64 bytes that move the next row to other banks
            uint8_t* const scratch = lds + put + wave * (kUnit * 16) + lq * kScratchRow;
            auto regroup = [&](int half, const uint32_t (&w)[NT]) -> v4i {
                uint8_t* const sc = scratch + half * kOperandBytes;
#pragma unroll
                for (int ti = 0; ti < NT; ++ti) *reinterpret_cast<uint32_t*>(sc + (ti * 16 + lx) * 4) = w[ti];
                asm volatile("" ::: "memory");
                const v4i out = *reinterpret_cast<const v4i*>(sc + lx * 16);
                asm volatile("" ::: "memory");
                return out;
            };
            v4i carry[NT][NT];
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b) carry[a][b] = zero4;
            // A row is stored after the next one's arithmetic, which covers its way through LDS (four digits of a lone
            // workgroup 5.0 -> 4.2 us, the leading word 2.0 -> 1.5; 7936 x 7936 x 256 852 -> 833 us for the call).
            auto put = [&](auto JJ) {
                constexpr int j = decltype(JJ)::v;
                const int d = d_hi - j;
                int64_t row_here = row;
                asm volatile("" : "+s"(row_here));
                if (d > 0) {
                    // balanced digit out (two's complement: the low byte of the sum), carry stays.  The 128 that rounds the
                    // carry is added before the bytes are taken and comes out of them with one XOR for four.
                    uint8_t* dst = wL + int64_t(d - 1) * planeL;
                    v4i before = zero4;
#pragma unroll
                    for (int tj = 0; tj < NT; ++tj) {
                        uint32_t w[NT];
#pragma unroll
                        for (int ti = 0; ti < NT; ++ti) {
                            const v4i t = acc[j][tj][ti] + carry[tj][ti] + 128;
                            const uint32_t lo = __builtin_amdgcn_perm(uint32_t(t[1]), uint32_t(t[0]), 0x00000400u);
                            const uint32_t hi = __builtin_amdgcn_perm(uint32_t(t[3]), uint32_t(t[2]), 0x00000400u);
                            w[ti] = __builtin_amdgcn_perm(hi, lo, 0x05040100u) ^ 0x80808080u;
                            carry[tj][ti] = t >> 8;
                        }
                        const v4i out = regroup(tj & 1, w);
                        if (tj > 0) store_lane_16(dst + int64_t((tj - 1) * 4) * row_here * 4, lane_L, before);
                        before = out;
                    }
                    store_lane_16(dst + int64_t((NT - 1) * 4) * row_here * 4, lane_L, before);
                } else {
                    // the leading word; the next k-block starts from zero
                    v4i before = zero4;
#pragma unroll
                    for (int tj = 0; tj < NT; ++tj)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            uint32_t w[NT];
#pragma unroll
                            for (int ti = 0; ti < NT; ++ti) w[ti] = uint32_t(acc[j][tj][ti][q] + carry[tj][ti][q]);
                            const v4i out = regroup(q & 1, w);
                            if (tj > 0 || q > 0)
                                store_lane_16(wT + int64_t(q > 0 ? tj * 16 + q - 1 : tj * 16 - 13) * row_here * 4, lane_T, before);
                            before = out;
                        }
                    store_lane_16(wT + int64_t(NT * 16 - 13) * row_here * 4, lane_T, before);
#pragma unroll
                    for (int tj = 0; tj < NT; ++tj)
#pragma unroll
                        for (int ti = 0; ti < NT; ++ti) carry[tj][ti] = zero4;
                }
            };
            put(Int<0>{});
            if (nd > 1) {
                put(Int<1>{});
                if (nd > 2) {
                    put(Int<2>{});
                    if (nd > 3) put(Int<3>{});
                }
            }
            clear(1);
            // The carries enter the next group's first accumulator set as the result of a matrix instruction
            // with zero operands (0*0 + carry), for the same reason as in clear().
#pragma unroll
            for (int tj = 0; tj < NT; ++tj)
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
                    acc[0][tj][ti] = __builtin_amdgcn_mfma_i32_16x16x64_i8(zero4, zero4, carry[tj][ti], 0, 0, 0);
        }

        if (!last) {
            if (d_hi >= D) {
                d_hi -= D;
            } else {
                ++kb;
                d_hi = S - 1;
            }
            if (sync_on && sync_q < sync_steps) arrive();
        } else {
            // a unit with fewer groups than the call's largest count still owes the round its
            // remaining arrivals: the workgroups that walk more of them count on every member
            if (sync_on && sync_q < sync_steps && threadIdx.x == 0) atomicAdd(&rec->tile_sync[xcd], sync_steps - sync_q);
            if (!has_next) break;
            ui = nui; uj = nuj; S = nS; slot = nslot;
            kb = kb_first;
            d_hi = S - 1;
            sa.ahead = sb.ahead = false;
            find_next();
            sync_q = 0;
            if (sync_on) arrive();
        }
    }
    // drain the surplus transfers before the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <bool ATOMIC>
__global__ __launch_bounds__(256) void gemm_i8_kernel(const int8_t* __restrict__ As, const int8_t* __restrict__ Bs,
                                                      int32_t* __restrict__ T, int8_t* __restrict__ L,
                                                      int32_t* __restrict__ raw, int raw_units, int64_t mp, int64_t np,
                                                      int64_t kp, int s_cap, Record* rec, GemmGrid g,
                                                      const int32_t* __restrict__ tile_S) {
    gemm_i8_body<ATOMIC>(As, Bs, T, L, raw, raw_units, mp, np, kp, s_cap, rec, g, tile_S);
}

// Several problems in one launch.  A kernel of its own: pointers that are computed take scalar registers from the other's steps.
__global__ __launch_bounds__(256) void gemm_i8_batch_kernel(const int8_t* __restrict__ As, const int8_t* __restrict__ Bs,
                                                            int32_t* __restrict__ T, int8_t* __restrict__ L,
                                                            int32_t* __restrict__ raw, int raw_units, int64_t mp, int64_t np,
                                                            int64_t kp, int s_cap, Record* rec, GemmGrid g,
                                                            const int32_t* __restrict__ tile_S, Batch bt) {
    const int64_t ws = bt.ws_at(blockIdx.z);
    gemm_i8_body<false>(at_bytes(As, ws), at_bytes(Bs, ws), at_bytes(T, ws), at_bytes(L, ws), at_bytes(raw, ws), raw_units, mp, np, kp,
                        s_cap, at_bytes(rec, ws), g, tile_S ? at_bytes(tile_S, ws) : nullptr);
}

// raw = 0 on the slots of a launch whose workgroups add their parts of the k range into them.
// grid (units of the launch, planes); a workgroup clears one 128 x 128 slot of one plane.
__global__ __launch_bounds__(256) void zero_raw_kernel(int32_t* __restrict__ raw, int raw_units, int s_cap, const Record* rec) {
    if (rec->res.fallback || int(blockIdx.y) % s_cap >= rec->res.slices_used) return;
    int4* base = reinterpret_cast<int4*>(raw + (int64_t(blockIdx.y) * raw_units + blockIdx.x) * (kUnit * kUnit));
#pragma unroll 4
    for (int v = threadIdx.x; v < kUnit * kUnit / 4; v += 256) base[v] = make_int4(0, 0, 0, 0);
}

// Unit `local` of a launch, and its slice count, for the kernels that follow a split launch.
__device__ __forceinline__ int split_unit(const GemmGrid& g, int local, const int32_t* __restrict__ tile_S, int S_all, int& ui,
                                          int& uj) {
    if (tile_S) {
        int ti, tj;
        const int q = local / g.count;
        lin_to_tile(tile_S[g.nti * g.ntj + g.begin + local - q * g.count], g.nti, g.ntj, ti, tj);
        ui = 2 * ti + (q & 1);
        uj = 2 * tj + (q >> 1);
        return min(tile_S[tj * g.nti + ti], S_all);
    }
    lin_to_tile(g.begin + local, g.um, g.un, ui, uj);
    return S_all;
}

// Adds the parts of a launch that covers the last units of a product only (a product that is split as a whole is put
// together by the recomposition): part 0 lies in the matrix planes, the others in their slots, every one as
// leading word and balanced digits of its own exact integer.  Digits are added plane by plane with the carry chain
// of the slice GEMM (at most zsplit * 128 per digit), which gives the digits of the whole integer.  Only the parts that
// have k in k-block kb count (the planes of the others hold nothing).
// Bound by latency: the loads of eight digits of a part are in flight together (one by one, a call of 7936 x 7936 x 256
// spent 31 us here on four units).  grid (units of the launch, k-blocks, 16); thread = one i and one row j/4 of the unit.
__global__ __launch_bounds__(256) void add_parts_kernel(const int32_t* __restrict__ raw, int32_t* __restrict__ T,
                                                        int8_t* __restrict__ L, int64_t mp, int64_t np, int64_t kp, int s_cap,
                                                        GemmGrid g, const Record* rec, const int32_t* __restrict__ tile_S) {
    if (rec->res.fallback) return;
    const int S_all = rec->res.slices_used;
    const int64_t kblk = k_block_length(S_all);
    const int nkb = int((kp + kblk - 1) / kblk);
    const int kb = blockIdx.y, local = blockIdx.x;
    if (kb >= nkb) return;
    int ui, uj;
    const int S = split_unit(g, local, tile_S, S_all, ui, uj);
    if (ui >= g.um || uj >= g.un) return;
    const int units = tile_S ? 4 * g.count : g.count;
    const int kt_total = g.kt_total, kt_per_block = int(kblk / kBK);
    const int64_t slot_words = part_slot_bytes(s_cap) / 4;
    int z_lo, z_hi;
    parts_of_block(kt_total, kt_per_block, g.zsplit, kb, z_lo, z_hi);
    if (z_hi == 0) return;                  // all of it came from part 0: already in place
    const int il = threadIdx.x & (kUnit - 1), jl4 = int(blockIdx.z) * 2 + (threadIdx.x >> 7);
    const int64_t i = int64_t(ui) * kUnit + il, j0 = int64_t(uj) * kUnit;
    uint32_t* const lw = reinterpret_cast<uint32_t*>(L) + (int64_t(kb) * (s_cap - 1) * (np / 4) + j0 / 4 + jl4) * mp + i;
    const int64_t plane = (np / 4) * mp;    // dwords between digit planes
    int32_t* const tw = T + (int64_t(kb) * np + j0 + jl4 * 4) * mp + i;
    auto slot_of = [&](int z) -> const int32_t* {
        return raw + ((int64_t(z - 1) * units + local) * g.nkb_part + (kb - part_first(kt_total, g.zsplit, z) / kt_per_block)) * slot_words;
    };
    int carry[4] = {0, 0, 0, 0};
    constexpr int kBatch = 8;
    for (int d_hi = S - 1; d_hi >= 1; d_hi -= kBatch) {
        int t[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) t[u][q] = 0;
        for (int z = z_lo; z <= z_hi; ++z) {
            const uint32_t* src = z == 0 ? lw : reinterpret_cast<const uint32_t*>(slot_of(z) + kUnit * kUnit) + jl4 * kUnit + il;
            const int64_t step = z == 0 ? plane : int64_t(kUnit / 4) * kUnit;
            uint32_t w[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) w[u] = d_hi - u >= 1 ? src[(d_hi - u - 1) * step] : 0u;
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) t[u][q] += int(w[u] << (24 - 8 * q)) >> 24;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (d_hi - u < 1) continue;
            uint32_t w = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int v = t[u][q] + carry[q];
                w |= (uint32_t(v) & 255u) << (8 * q);
                carry[q] = (v + 128) >> 8;
            }
            lw[(d_hi - u - 1) * plane] = w;
        }
    }
    for (int z = z_lo; z <= z_hi; ++z) {
#pragma unroll
        for (int q = 0; q < 4; ++q) carry[q] += z == 0 ? tw[q * mp] : slot_of(z)[(jl4 * 4 + q) * kUnit + il];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) tw[q * mp] = carry[q];
}

void tile_order_shape(const Problem& p, int& first, int& deal) {
    const LaunchPlan lp(p);
    first = lp.two ? lp.full : lp.positions;
    deal = (lp.g.full_chip && lp.full != 0 && lp.positions <= (1 << 16)) ? 1 : 0;
}

bool can_batch(const Problem& p) { return LaunchPlan(p).can_batch(p); }

bool prepare_gemm_i8() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_kernel<false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_batch_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds) == hipSuccess &&
           prepare_gemm_i8_few() && prepare_gemm_small() && prepare_gemm_mid();
}

SplitPlan launch_gemm_i8(hipStream_t st, const Workspace& w, const Problem& p, double alpha, double beta, double* C, int64_t ldc,
                         const Fallback& fallback, bool& fell_back) {
    const LaunchPlan lp(p);
    Fallback fb = fallback;
    if (fb.A && (lp.small || lp.mid)) {
        const int64_t lda = std::max(fb.a_sr, fb.a_sl), ldb = std::max(fb.b_sr, fb.b_sl);       // one of either is 1
        const F64Size size = f64_size(p.m, p.n, p.k, p.batch.count, true, beta != 0.0, fb.a_rows, lda, fb.b_rows, ldb);
        const size_t scratch = size_t(reinterpret_cast<uint8_t*>(w.tile_span) - reinterpret_cast<uint8_t*>(w.As));
        fell_back = !wide_offsets(p.m, p.n, p.k, std::max(lda, ldb)) &&
                    f64_folds(size, p.num_cu, scratch, lp.small ? kSmallTile : kMidTile, lp.small && !lp.small_pair);
    }
    if (!fell_back) fb.A = nullptr;
    if (lp.small) {
        launch_gemm_small(st, w, p, lp, alpha, beta, C, ldc, fb);
        return SplitPlan{KSplit::kDone, lp.g, lp.raw_units};
    }
    if (lp.mid) {
        launch_gemm_mid(st, w, p, lp, alpha, beta, C, ldc, fb);
        return SplitPlan{KSplit::kDone, lp.g, lp.raw_units};
    }
    if (lp.few) {
        launch_gemm_i8_few(st, w, p, lp);
        return SplitPlan{KSplit::kNone, lp.g, lp.raw_units};
    }
    const int32_t* tile_S = p.tile_mode ? w.tile_S : nullptr;
    auto launch = [&](int begin, int count, Split sp) -> GemmGrid {
        unsigned grid;
        const GemmGrid g = lp.launch(p, begin, count, sp, grid);
        const int units = count * lp.per_pos;
        if (sp.atomic) {
            hipLaunchKernelGGL(zero_raw_kernel, dim3(unsigned(units), unsigned(p.nkb * p.s_cap)), dim3(256), 0, st, w.raw,
                               lp.raw_units, p.s_cap, w.rec);
            hipLaunchKernelGGL(gemm_i8_kernel<true>, dim3(grid), dim3(256), kGemmLds, st, w.As, w.Bs, w.T, w.L, w.raw,
                               lp.raw_units, p.mp, p.np, p.kp, p.s_cap, w.rec, g, tile_S);
        } else {
            hipLaunchKernelGGL(gemm_i8_kernel<false>, dim3(grid), dim3(256), kGemmLds, st, w.As, w.Bs, w.T, w.L, w.raw,
                               lp.raw_units, p.mp, p.np, p.kp, p.s_cap, w.rec, g, tile_S);
            if (sp.z > 1 && count < lp.positions)
                hipLaunchKernelGGL(add_parts_kernel, dim3(unsigned(units), unsigned(p.nkb), kUnit / 4 / 2), dim3(256), 0, st,
                                   w.raw, w.T, w.L, p.mp, p.np, p.kp, p.s_cap, g, w.rec, tile_S);
        }
        return g;
    };
    if (lp.two) {
        launch(0, lp.full, Split{1, false});
        return SplitPlan{KSplit::kNone, launch(lp.full, lp.rest, lp.last), lp.raw_units};
    }
    if (p.batch.count > 1) {             // can_batch: one launch, no more units than CUs
        unsigned grid;
        const GemmGrid g = lp.launch(p, 0, lp.positions, lp.last, grid);
        hipLaunchKernelGGL(gemm_i8_batch_kernel, dim3(grid, 1, unsigned(p.batch.count)), dim3(256), kGemmLds, st, w.As, w.Bs, w.T, w.L,
                           w.raw, lp.raw_units, p.mp, p.np, p.kp, p.s_cap, w.rec, g, tile_S, p.batch);
        return SplitPlan{lp.last.z == 1 ? KSplit::kNone : KSplit::kParts, g, lp.raw_units};
    }
    const GemmGrid g = launch(0, lp.positions, lp.last);
    return SplitPlan{lp.last.z == 1 ? KSplit::kNone : (lp.last.atomic ? KSplit::kAtomic : KSplit::kParts), g, lp.raw_units};
}

}  // namespace oz
