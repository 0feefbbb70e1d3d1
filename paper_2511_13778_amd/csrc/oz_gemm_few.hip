// Slice GEMM of calls that get at most two slices, on 256 x 256 blocks of C: the same sums and the same T / L planes as
// gemm_i8_kernel leaves, pair by pair.
//
// With one or two slices the 128 x 128 units of gemm_i8_kernel have one or three products per 64 of k in which to use
// what they load, and a unit is over before its start and the writing of its sums are paid for.  Here a tile of A and
// one of B meet in four times as many products.  0.67-0.75 of the MFMA-only loop on 32x32x32 (3.5 POP/s); bound by the
// writing of T where k is short.
// 128 x 128 units -> here, this kernel alone: one slice at 8192^3 955 -> 466 us (2.36 POP/s), 8192 x 8192 x 2048 303 -> 179,
// 8192 x 8192 x 256 156 -> 101; two slices 1493 -> 1262 (2.61 POP/s), 470 -> 392, 195 -> 153.
//
// A workgroup owns one block of C: 4 waves of 128 x 128 on v_mfma_i32_32x32x32_i8 (256 accumulator registers per lane), one
// workgroup per CU.  Anti-diagonals from the least significant up; inside one, its pairs, and inside a pair the steps of 64
// of k.  Four LDS stages of 32 KB, tiles loaded straight into LDS three steps ahead across pairs and anti-diagonals.
#include "oz_gemm_device.h"

namespace oz {

namespace {

constexpr int kFewStages = 4;
constexpr int kFewOperand = kTile * kBK;             // 16 KB
constexpr int kFewStage = 2 * kFewOperand;           // A tile, then B tile
constexpr int kFewLds = kFewStages * kFewStage;      // 128 KB
static_assert((kFewStages & (kFewStages - 1)) == 0, "stages are counted modulo a power of two");

}  // namespace

// One dword per lane to a wave-uniform base plus a 32-bit per-lane byte offset; as assembly, with the five wait states
// between a vector-ALU write of a scalar register and its use as a base, so that no 64-bit per-lane address is built per
// store.
template <bool STREAM>
__device__ __forceinline__ void store_lane_dword(void* uniform_base, uint32_t lane_byte_off, uint32_t data) {
    if (STREAM) asm volatile("s_nop 4\n\tglobal_store_dword %0, %1, %2 nt" :: "v"(lane_byte_off), "v"(data), "s"(uniform_base) : "memory");
    else asm volatile("s_nop 4\n\tglobal_store_dword %0, %1, %2" :: "v"(lane_byte_off), "v"(data), "s"(uniform_base) : "memory");
}

__device__ __forceinline__ v4i as_v4i(const uint4& v) { return v4i{int(v.x), int(v.y), int(v.z), int(v.w)}; }

// grid: one workgroup per block of C
template <bool STREAM>
__global__ __launch_bounds__(256) void gemm_i8_few_kernel(const int8_t* __restrict__ As, const int8_t* __restrict__ Bs,
                                                          int32_t* __restrict__ T, int8_t* __restrict__ L, int64_t mp, int64_t np,
                                                          int64_t kp, int s_cap, Record* rec, int kt_total, int full_chip) {
    extern __shared__ __align__(16) uint8_t lds[];
    if (rec->res.fallback) return;
    const int S = rec->res.slices_used;
    // k-range one int32 accumulator can take
    const int64_t kblk = k_block_length(S);
    const int nkb = int((kp + kblk - 1) / kblk);
    // Workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets a contiguous range of the block order, in which 32
    // consecutive blocks are 4 x 8.
    const int nti = int(mp / kTile), tiles = nti * int(np / kTile);
    const int xcd = int(blockIdx.x) & 7, slot = int(blockIdx.x) >> 3;
    const int per = tiles >> 3, rem = tiles & 7, xcd_tiles = per + (xcd < rem ? 1 : 0);
    int ti, tj;
    lin_to_tile(xcd * per + min(xcd, rem) + slot, nti, int(np / kTile), ti, tj);
    const int kt_per_block = int(kblk / kBK);
    const int kb_last = nkb - 1;
    // The workgroups that share panels start together and, where k is long, every anti-diagonal (see gemm_i8_kernel).
    // Arrival number q of a workgroup of round r waits for 32*r*steps + (q+1)*members arrivals on the XCD's counter
    // (earlier rounds are full).
    const int sync_steps = kp >= kMidSyncMinK ? nkb * S : 1;
    const int sync_round = slot / kRoundUnits;
    const int sync_members = min(kRoundUnits, xcd_tiles - sync_round * kRoundUnits);
    const int sync_base = sync_round * kRoundUnits * sync_steps;
    const bool sync_on = full_chip && xcd_tiles > kRoundUnits && sync_members > 1;
    int sync_q = 0;
    bool sync_wait = true;
    if (sync_on) round_sync(&rec->tile_sync[xcd], sync_base + (++sync_q) * sync_members, sync_wait);

    const int64_t i0 = int64_t(ti) * kTile, j0 = int64_t(tj) * kTile;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = wave & 1, wj = wave >> 1;

    v16i acc[4][4];   // [fj][fi]
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = zero;

    // K steps [kt_lo(kb), kt_lo(kb) + kt_count(kb)) make k-block kb
    auto kt_lo = [&](int kb) -> int { return kb * kt_per_block; };
    auto kt_count = [&](int kb) -> int { return min((kb + 1) * kt_per_block, kt_total) - kt_lo(kb); };

    // (nkb_, nd, ns, nkt) walks the (k-block, anti-diagonal, pair, K step) sequence ahead of the
    // compute, so the prefetch runs across pair and anti-diagonal boundaries without a bubble.
    // After the last tile it stays put: the surplus transfers land in stages nobody reads again.
    int nkb_ = 0, nd = S - 1, ns = 0, nkt = 0;
    int nxt_ktc = kt_count(0);
    int issue_stage = 0;
    const uint32_t lds_base = uint32_t(uintptr_t((__attribute__((address_space(3))) uint8_t*)lds));
    const uint8_t* gA = reinterpret_cast<const uint8_t*>(As) + (i0 + wave * 64) * 16;   // wave-uniform
    const uint8_t* gB = reinterpret_cast<const uint8_t*>(Bs) + (j0 + wave * 64) * 16;
    const uint32_t lane_off = uint32_t(lane) * 16;
    // per-lane byte offsets of the four k chunks of a tile (chunk q is q*rows*16 bytes further on)
    uint32_t offA[4], offB[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        offA[q] = lane_off + uint32_t(q) * uint32_t(mp) * 16u;
        offB[q] = lane_off + uint32_t(q) * uint32_t(np) * 16u;
    }
    const int64_t planeA = kp * mp, planeB = kp * np;   // bytes per slice plane

    // addresses of the next tile to fetch (8 transfers per wave: 4 k chunks of A, 4 of B).  The
    // pointers advance by one K step per tile; only when the pair changes are they recomputed from
    // the iterator (once per k-block length, outside the common path).
    const uint8_t* pa = gA;
    const uint8_t* pb = gB + int64_t(S - 1) * (kp * np);   // pair (0, S-1)
    const int64_t stepA = int64_t(kBK) * mp, stepB = int64_t(kBK) * np;   // bytes per K step
    uint32_t la;
#define OZ_TILE_ADDR()                                                                           \
    { la = lds_base + issue_stage * kFewStage + wave * 1024; }
// transfer number x (0..7) of the tile addressed by pa / pb / la
#define OZ_DMA(x)                                                                                \
    {                                                                                            \
        switch (x) {                                                                             \
            case 0: dma16<0 * (kTile * 16)>(pa, offA[0], la); break;                             \
            case 1: dma16<kFewOperand + 0 * (kTile * 16)>(pb, offB[0], la); break;               \
            case 2: dma16<1 * (kTile * 16)>(pa, offA[1], la); break;                             \
            case 3: dma16<kFewOperand + 1 * (kTile * 16)>(pb, offB[1], la); break;               \
            case 4: dma16<2 * (kTile * 16)>(pa, offA[2], la); break;                             \
            case 5: dma16<kFewOperand + 2 * (kTile * 16)>(pb, offB[2], la); break;               \
            case 6: dma16<3 * (kTile * 16)>(pa, offA[3], la); break;                             \
            default: dma16<kFewOperand + 3 * (kTile * 16)>(pb, offB[3], la); break;              \
        }                                                                                        \
    }
#define OZ_TILE_ADVANCE()                                                                        \
    {                                                                                            \
        issue_stage = (issue_stage + 1) & (kFewStages - 1);                                      \
        if (++nkt == nxt_ktc) {                                                                  \
            nkt = 0;                                                                             \
            if (++ns > nd) {                                                                     \
                ns = 0;                                                                          \
                if (--nd < 0) {                                                                  \
                    nd = S - 1;                                                                  \
                    if (++nkb_ > kb_last) nkb_ = kb_last;                                        \
                    nxt_ktc = kt_count(nkb_);                                                    \
                }                                                                                \
            }                                                                                    \
            const int64_t kc = int64_t(kt_lo(nkb_)) * (kBK / 16);                                \
            pa = gA + int64_t(ns) * planeA + kc * mp * 16;                                       \
            pb = gB + int64_t(nd - ns) * planeB + kc * np * 16;                                  \
        } else {                                                                                 \
            pa += stepA;                                                                         \
            pb += stepB;                                                                         \
        }                                                                                        \
    }
#define OZ_ISSUE_TILE()                                                                          \
    {                                                                                            \
        OZ_TILE_ADDR();                                                                          \
        _Pragma("unroll") for (int x = 0; x < 8; ++x) OZ_DMA(x);                                 \
        OZ_TILE_ADVANCE();                                                                       \
    }
// operand fragment f of K sub-step kk (0 or 1) of the tile in LDS stage `stage`
#define OZ_READ_A(dst, stage, kk, f)                                                             \
    dst[f] = as_v4i((reinterpret_cast<const uint4*>(lds + (stage) * kFewStage) + wi * 128 +      \
                     (lane & 31) + ((kk) * 2 + (lane >> 5)) * kTile)[(f) * 32])
#define OZ_READ_B(dst, stage, kk, f)                                                             \
    dst[f] = as_v4i((reinterpret_cast<const uint4*>(lds + (stage) * kFewStage + kFewOperand) +   \
                     wj * 128 + (lane & 31) + ((kk) * 2 + (lane >> 5)) * kTile)[(f) * 32])
#define OZ_READ_FRAGS(dstA, dstB, stage, kk)                                                     \
    _Pragma("unroll") for (int f = 0; f < 4; ++f) {                                              \
        OZ_READ_A(dstA, stage, kk, f);                                                           \
        OZ_READ_B(dstB, stage, kk, f);                                                           \
    }
#define OZ_MFMA(srcA, srcB, fj, fi)                                                              \
    acc[fj][fi] = __builtin_amdgcn_mfma_i32_32x32x32_i8(srcB[fj], srcA[fi], acc[fj][fi], 0, 0, 0)

    // prologue: three tiles in flight, then wait for the first, publish it, issue the fourth
    OZ_ISSUE_TILE();
    OZ_ISSUE_TILE();
    OZ_ISSUE_TILE();
    asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");
    OZ_TILE_ADDR();
#pragma unroll
    for (int x = 0; x < 8; ++x) OZ_DMA(x);   // the iterator moves on in the first half of the loop body
    v4i fa0[4], fb0[4], fa1[4], fb1[4];
    int stage = 0;
    OZ_READ_FRAGS(fa0, fb0, stage, 0);

    for (int kb = 0; kb <= kb_last; ++kb) {
        const int ktc = kt_count(kb);
        for (int d = S - 1; d >= 0; --d) {
            const int n_iter = (d + 1) * ktc;
            for (int it = 0; it < n_iter; ++it) {
                // invariant here: transfers of the next three tiles are in flight (24 per wave);
                // fragments of sub-step 0 of the current tile are in fa0/fb0
                // first half: MFMAs of sub-step 0 (16); one LDS read of sub-step 1 after each of the
                // first eight, so that all have returned well before the barrier
#pragma unroll
                for (int q = 0; q < 12; ++q) {
                    OZ_MFMA(fa0, fb0, q >> 2, q & 3);
                    __builtin_amdgcn_sched_barrier(0);
                    if (q < 8) {
                        if (q & 1) { OZ_READ_B(fb1, stage, 1, q >> 1); } else { OZ_READ_A(fa1, stage, 1, q >> 1); }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (q == 9) {   // a gap without memory work: move the iterator past the tile issued last
                        OZ_TILE_ADVANCE();
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // next tile landed (own transfers), every LDS read of this tile returned; after the
                // barrier that holds for all waves, so this stage may be overwritten.  The last four
                // MFMAs of the first half cover the barrier.
                asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                const int next_stage = (stage + 1) & (kFewStages - 1);
                OZ_TILE_ADDR();
#pragma unroll
                for (int q = 12; q < 16; ++q) {
                    OZ_MFMA(fa0, fb0, q >> 2, q & 3);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // second half: MFMAs of sub-step 1; after each one either an LDS read of the next
                // tile's sub-step 0 or a transfer of the tile three stages ahead
#pragma unroll
                for (int g = 0; g < 8; ++g) {
                    OZ_MFMA(fa1, fb1, g >> 1, (g & 1) * 2);
                    __builtin_amdgcn_sched_barrier(0);
                    if (g & 1) { OZ_READ_B(fb0, next_stage, 0, g >> 1); } else { OZ_READ_A(fa0, next_stage, 0, g >> 1); }
                    __builtin_amdgcn_sched_barrier(0);
                    OZ_MFMA(fa1, fb1, g >> 1, (g & 1) * 2 + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    OZ_DMA(g);
                    __builtin_amdgcn_sched_barrier(0);
                }
                stage = next_stage;
            }

            // anti-diagonal d of k-block kb is complete.
            // result register r of MFMA tile (fj, fi): j = fj*32 + 8*(r/4) + 4*(lane/32) + r%4,
            // i = fi*32 + lane%32.  Every address below is a wave-uniform pointer (scalar arithmetic)
            // plus one per-lane 32-bit element offset that is the same for all stores of a kind.
            // the row stride as a value the compiler cannot trace out of this iteration: otherwise the row
            // addresses of all stores (loop-invariant offsets) are hoisted out of the anti-diagonal loop
            // and kept alive, several hundred registers' worth, across the MFMA loop
            int64_t mp_here = mp;
            asm volatile("" : "+s"(mp_here));
            if (d > 0) {
                // balanced digit out (the low byte of T is its two's-complement form), carry stays: four
                // consecutive j of one i make a dword, so the lanes of a half-wave write 128 contiguous bytes
                uint32_t* dst = reinterpret_cast<uint32_t*>(L) +
                                ((int64_t(kb) * (s_cap - 1) + (d - 1)) * (np / 4) + (j0 + wj * 128) / 4) * mp + i0 + wi * 128;
                const uint32_t lane_L = (uint32_t(lane >> 5) * uint32_t(mp) + uint32_t(lane & 31)) * 4u;   // bytes
                const v4i zero4 = {0, 0, 0, 0};
#pragma unroll
                for (int fj = 0; fj < 4; ++fj)
#pragma unroll
                    for (int fi = 0; fi < 4; ++fi) {
                        const v16i t = acc[fj][fi];
                        v16i carry;
#pragma unroll
                        for (int rq = 0; rq < 4; ++rq) {
                            const uint32_t w = (uint32_t(t[4 * rq]) & 255u) | ((uint32_t(t[4 * rq + 1]) & 255u) << 8) |
                                               ((uint32_t(t[4 * rq + 2]) & 255u) << 16) | (uint32_t(t[4 * rq + 3]) << 24);
                            store_lane_dword<STREAM>(dst + (int64_t(fj * 8 + 2 * rq) * mp_here + fi * 32), lane_L, w);
                        }
#pragma unroll
                        for (int r = 0; r < 16; ++r) carry[r] = (t[r] + 128) >> 8;
                        // The carries go back into the accumulator tile as the result of a matrix instruction
                        // with zero operands (0*0 + carry).  Written by the vector ALU instead, the tile
                        // would be kept in the ordinary vector registers by the register allocator, and
                        // sixteen such tiles do not fit there beside the loop's own registers.
                        acc[fj][fi] = __builtin_amdgcn_mfma_i32_32x32x32_i8(zero4, zero4, carry, 0, 0, 0);
                    }
            } else {
                // the leading word; the next k-block starts from zero
                int32_t* dst = T + (int64_t(kb) * np + j0 + wj * 128) * mp + i0 + wi * 128;
                const uint32_t lane_T = (uint32_t(4 * (lane >> 5)) * uint32_t(mp) + uint32_t(lane & 31)) * 4u;   // bytes
#pragma unroll
                for (int fj = 0; fj < 4; ++fj)
#pragma unroll
                    for (int fi = 0; fi < 4; ++fi) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            store_lane_dword<STREAM>(dst + (int64_t(fj * 32 + 8 * (r >> 2) + (r & 3)) * mp_here + fi * 32), lane_T,
                                                     uint32_t(acc[fj][fi][r]));
                        }
                        acc[fj][fi] = zero;
                    }
            }
            if (sync_on && sync_q < sync_steps)
                round_sync(&rec->tile_sync[xcd], sync_base + (++sync_q) * sync_members, sync_wait);
            // The operand fragments of the next K step were read during the last one, as in every K
            // step; reading them again here (eight LDS reads per anti-diagonal) ends their lifetime
            // before the epilogue above, which needs the registers to pass the accumulators through.
            OZ_READ_FRAGS(fa0, fb0, stage, 0);
        }
    }
    // drain the surplus transfers before the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

#undef OZ_ISSUE_TILE
#undef OZ_READ_FRAGS
#undef OZ_MFMA
#undef OZ_DMA
#undef OZ_TILE_ADDR
#undef OZ_TILE_ADVANCE
#undef OZ_READ_A
#undef OZ_READ_B

bool prepare_gemm_i8_few() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_few_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kFewLds) == hipSuccess &&
           hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_few_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kFewLds) == hipSuccess;
}

void launch_gemm_i8_few(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp) {
    const auto kernel = results_stream(p) ? gemm_i8_few_kernel<true> : gemm_i8_few_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(lp.g.nti) * unsigned(lp.g.ntj)), dim3(256), kFewLds, st, w.As, w.Bs, w.T, w.L,
                       p.mp, p.np, p.kp, p.s_cap, w.rec, lp.kt, lp.g.full_chip);
}

}  // namespace oz
