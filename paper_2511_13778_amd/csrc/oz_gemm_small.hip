// Slice-pair GEMMs and FP64 recomposition of a small call in one kernel: what gemm_i8_kernel and recompose_kernel compute,
// for outputs of few 128 x 128 units and a short k.
// (paper: section "FP64 Emulation on Low-Precision Units".)
//
// What bounds such a call is not arithmetic but the chain of dependent steps: with 128 x 128 units a workgroup walks k once per
// four anti-diagonals, writes sums after each, and a k split leaves parts that a second launch puts together.  Here a
// workgroup owns 32 x 32 elements of C and keeps all S slices of both operands of a 64 of k in LDS (4 KB per slice), so k
// is walked once and every anti-diagonal grows at the same time, in the registers of the wave it is dealt to; the carry
// chain, the powers of two and alpha / beta follow from LDS in the same launch.  Up to 16 times as many workgroups as units.
// The price is LDS bandwidth: four MFMAs per four fragments read, twice what the matrix unit's rate allows.  So
// it is the shorter way only while the units would leave the chip idle (LaunchPlan::fuse).
// 200 x 300 x 260 with nine slices: slice GEMM and recomposition 33 + 14 us, now 10 (the call 72 -> 31 us, with the
// fallback in the same launch and one launch less before it).
#include "oz_f64_direct.h"
#include "oz_gemm_device.h"

namespace oz {

constexpr int kSmallWaves = 8;
constexpr int kSliceBytes = kSmallTile * kBK;               // one slice of one operand for a 64 of k: [k chunk][row][16 B]
constexpr int kSumRow = kSmallTile + 4;                     // words between rows of the sums: the four rows a wave writes at a
                                                            // time are then 16 banks apart
constexpr int kSumPlane = kSmallTile * kSumRow * 4;         // bytes per anti-diagonal
constexpr int kSmallDiags = (kMaxSlices + kSmallWaves - 1) / kSmallWaves;     // anti-diagonals per wave
static_assert(kSmallTile == 32 && kBK == 64, "the transfers below move 2 x 32 rows of 16 bytes, the waves 2 x 2 MFMA tiles");
static_assert(kSmallPairSlices * kSumPlane <= kSmallLdsMax / 2 && kSmallPairSlices * 2 * kSliceBytes <= kSmallLdsMax / 2, "one of two workgroups");
static_assert(f64_direct_lds(2, 2, kSmallWaves) <= kSmallLdsMax / 2, "the fallback shares the LDS");
static_assert(kMaxSlices * kSumPlane <= kSmallLdsMax && kMaxSlices * 2 * kSliceBytes <= kSmallLdsMax, "one stage must fit");

template <int N>
struct Count { static constexpr int v = N; };

// grid (32 x 32 tiles of C, i fastest); one k-block.
__global__ __launch_bounds__(64 * kSmallWaves, 4) void gemm_small_kernel(
    const int8_t* __restrict__ As, const int8_t* __restrict__ Bs, int32_t* __restrict__ T, int8_t* __restrict__ L,
    const int32_t* __restrict__ eA, const int32_t* __restrict__ eB, int64_t m, int64_t n, int64_t mp, int64_t np, int64_t kp,
    int kt_total, int lds_bytes, double alpha, double beta, double* __restrict__ C, int64_t ldc, const Record* rec,
    const int32_t* __restrict__ tile_S, Batch bt, Fallback fb) {
    extern __shared__ __align__(16) uint8_t lds[];
    {
        const int64_t ws = bt.ws_at(blockIdx.z);
        As = at_bytes(As, ws); Bs = at_bytes(Bs, ws);
        T = at_bytes(T, ws); L = at_bytes(L, ws);
        eA = at_bytes(eA, ws); eB = at_bytes(eB, ws);
        rec = at_bytes(rec, ws);
        if (tile_S) tile_S = at_bytes(tile_S, ws);
        C += int64_t(blockIdx.z) * bt.c;
    }
    const int fallback = rec->res.fallback, S_all = rec->res.slices_used;
    const int ntm = int((m + kSmallTile - 1) / kSmallTile);
    const int tj = int(blockIdx.x) / ntm, ti = int(blockIdx.x) - tj * ntm;
    const int64_t i0 = int64_t(ti) * kSmallTile, j0 = int64_t(tj) * kSmallTile;
    if (fallback) {
        if (fb.A) fall_back<2, 2, kSmallWaves>(fb, bt, int(blockIdx.z), reinterpret_cast<double*>(lds), m, n, i0, j0, alpha, beta, C, ldc);
        return;
    }
    const int S = tile_S ? min(tile_S[(j0 / kTile) * (mp / kTile) + i0 / kTile], S_all) : S_all;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // The elements of C this thread finishes: column i, rows j and j+1.  Requested without conditions, at clamped addresses: a
    // wait for them here would put a round trip before the first transfer.
    const int ei = threadIdx.x & 31, ej = (int(threadIdx.x) >> 5) * 2;
    const int64_t i = i0 + ei, j = j0 + ej;
    const int ea = eA[i];
    const int2 eb2 = *reinterpret_cast<const int2*>(eB + j);
    double cin[2] = {0.0, 0.0};
    if (beta != 0.0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) cin[q] = C[min(j + q, n - 1) * ldc + min(i, m - 1)];
    }

    // ---- transfers: slice q of both operands (A's, then B's) is two pieces of 1 KB, k chunks 0 and 1, 2 and 3 of the 64 of
    // k; a wave takes one half of every fourth slice
    const int half = wave & 1;
    const uint32_t lane_a = (uint32_t(lane >> 5) * uint32_t(mp) + uint32_t(lane & 31)) * 16u;
    const uint32_t lane_b = (uint32_t(lane >> 5) * uint32_t(np) + uint32_t(lane & 31)) * 16u;
    const uint32_t lds_base = uint32_t(uintptr_t((__attribute__((address_space(3))) uint8_t*)lds));
    const uint32_t stage_bytes = uint32_t(2 * kSliceBytes) * uint32_t(S);
    const int stages = min(kt_total, lds_bytes / int(stage_bytes));
    const int pieces = (2 * S - (wave >> 1) + 3) >> 2;      // of this wave per 64 of k
    auto issue = [&](int kt, int stage) {
        const int64_t chunk = int64_t(kt) * (kBK / 16) + half * 2;
        const uint8_t* a = reinterpret_cast<const uint8_t*>(As) + (chunk * mp + i0) * 16;
        const uint8_t* b = reinterpret_cast<const uint8_t*>(Bs) + (chunk * np + j0) * 16;
        const uint32_t to = lds_base + uint32_t(stage) * stage_bytes + uint32_t(half) * 1024u;
        for (int q = wave >> 1; q < 2 * S; q += 4) {
            if (q < S) dma16<0>(a + q * (kp * mp), lane_a, to + uint32_t(q) * kSliceBytes);
            else dma16<0>(b + (q - S) * (kp * np), lane_b, to + uint32_t(q) * kSliceBytes);
        }
    };
    // Two 64s of k are requested at the start, further ones while an earlier one is multiplied: the transfers of a 64 of k
    // keep the CU's path to the L2 busy for 100 cycles per slice, and all that fit at once would only put off the first.
    int issued = 0, put = 0;             // 64s of k requested, and the stage of the next
    auto issue_next = [&](int limit) {
        if (issued >= limit) return;
        issue(issued, put);
        ++issued;
        put = put + 1 == stages ? 0 : put + 1;
    };
    issue_next(1);
    issue_next(min(2, stages));

    // ---- anti-diagonals: number x from the longest down goes to a wave so that the four SIMDs (waves w and w + 4) get equal
    // shares of the pairs
    const int place = wave < 4 ? wave : 11 - wave;
    int d_of[kSmallDiags];
#pragma unroll
    for (int u = 0; u < kSmallDiags; ++u) d_of[u] = S - 1 - (u * kSmallWaves + ((u & 1) ? kSmallWaves - 1 - place : place));
    v4i acc[kSmallDiags][2][2];
#pragma unroll
    for (int u = 0; u < kSmallDiags; ++u)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[u][a][b] = v4i{0, 0, 0, 0};
    const uint32_t rd = uint32_t(lane >> 4) * (kSmallTile * 16) + uint32_t(lane & 15) * 16;
    int stage = 0;
    for (int kt = 0; kt < kt_total; ++kt) {
        wait_transfers((issued - 1 - kt) * pieces);
        // every wave's part of this stage has landed, and every wave is done with the stage before: its reads have returned
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
        asm volatile("s_barrier" ::: "memory");
        // up to two more, into stages that are free by now; one wave of a SIMD before its products, the other behind them
        const int limit = min(min(kt + stages, issued + 2), kt_total);
        if (wave < kSmallWaves / 2) {
            issue_next(limit);
            issue_next(limit);
        }
        const uint8_t* at = lds + uint32_t(stage) * stage_bytes + rd;
#pragma unroll
        for (int u = 0; u < kSmallDiags; ++u) {
            const int d = d_of[u];
            if (d < 0) continue;
            const uint8_t* pa = at;                                          // slice s of A, s = 0 .. d
            const uint8_t* pb = at + uint32_t(S + d) * kSliceBytes;          // slice d - s of B
            auto multiply = [&](auto N) {
                constexpr int count = decltype(N)::v;
                v4i fa[count][2], fb[count][2];
#pragma unroll
                for (int x = 0; x < count; ++x)
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        fa[x][f] = *reinterpret_cast<const v4i*>(pa + x * kSliceBytes + f * 256);
                        fb[x][f] = *reinterpret_cast<const v4i*>(pb - x * kSliceBytes + f * 256);
                    }
#pragma unroll
                for (int x = 0; x < count; ++x)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int a = 0; a < 2; ++a)
                            acc[u][b][a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[x][b], fa[x][a], acc[u][b][a], 0, 0, 0);
                pa += count * kSliceBytes;
                pb -= count * kSliceBytes;
            };
            for (int left = d + 1; left >= 2; left -= 2) multiply(Count<2>{});
            if ((d & 1) == 0) multiply(Count<1>{});
        }
        if (wave >= kSmallWaves / 2) {
            issue_next(limit);
            issue_next(limit);
        }
        if (stages == 1) {               // 21 slices and more (11 in half the LDS): the one stage is free when all are done with it
            __builtin_amdgcn_s_waitcnt(0xC07F);
            asm volatile("s_barrier" ::: "memory");
            issue_next(kt_total);
        }
        stage = stage + 1 == stages ? 0 : stage + 1;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("s_barrier" ::: "memory");

    // ---- the sums meet in LDS; result register r of tile (b, a): j = 16b + 4*(lane/16) + r, i = 16a + lane%16
    int32_t* const sums = reinterpret_cast<int32_t*>(lds);
#pragma unroll
    for (int u = 0; u < kSmallDiags; ++u) {
        if (d_of[u] < 0) continue;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    sums[d_of[u] * (kSumPlane / 4) + (b * 16 + 4 * (lane >> 4) + r) * kSumRow + a * 16 + (lane & 15)] = acc[u][b][a][r];
    }
    __syncthreads();

    // carry chain from the least significant anti-diagonal, digits and leading word out, FP64 in recompose_kernel's order
    const int32_t* mine = sums + ej * kSumRow + ei;
    uint16_t* const lw = reinterpret_cast<uint16_t*>(L + ((j >> 2) * mp + i) * 4 + (ej & 2));
    const int64_t planeL = np * mp / 2;          // in 16-bit units
    const int eb[2] = {eb2.x, eb2.y};
    int carry[2] = {0, 0};
    double Rb[2] = {0.0, 0.0};
    constexpr int kAhead = 4;                    // anti-diagonals read from LDS together
    for (int d_hi = S - 1; d_hi >= 1; d_hi -= kAhead) {
        int p[kAhead][2];
#pragma unroll
        for (int x = 0; x < kAhead; ++x)
#pragma unroll
            for (int q = 0; q < 2; ++q) p[x][q] = mine[max(d_hi - x, 0) * (kSumPlane / 4) + q * kSumRow];
#pragma unroll
        for (int x = 0; x < kAhead; ++x) {
            const int d = d_hi - x;
            if (d < 1) break;
            uint32_t w = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int v = p[x][q] + carry[q];
                carry[q] = (v + 128) >> 8;
                w |= (uint32_t(v) & 255u) << (8 * q);
                Rb[q] = double((v << 24) >> 24) + Rb[q] * 0x1p-8;
            }
            lw[(d - 1) * planeL] = uint16_t(w);
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int t = mine[q * kSumRow] + carry[q];
        T[(j + q) * mp + i] = t;
        const double R = 0.0 + (double(t) + Rb[q] * 0x1p-8);
        const int sc = (ea > kExpAllZero ? ea : 0) + (eb[q] > kExpAllZero ? eb[q] : 0) + (2 * kHeadroomBits - 12);
        double out = __dmul_rn(alpha, ldexp(R, sc));
        if (beta != 0.0) out = __dadd_rn(out, __dmul_rn(beta, cin[q]));
        if (i < m && j + q < n) C[(j + q) * ldc + i] = out;
    }
}

bool prepare_gemm_small() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_small_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kSmallLdsMax) == hipSuccess;
}

void launch_gemm_small(hipStream_t st, const Workspace& w, const Problem& p, const LaunchPlan& lp, double alpha, double beta,
                       double* C, int64_t ldc, const Fallback& fb) {
    const int64_t tiles = lp.small_tiles(p);
    const int lds = lp.small_pair ? kSmallLdsMax / 2 : kSmallLdsMax;
    hipLaunchKernelGGL(gemm_small_kernel, dim3(unsigned(tiles), 1, unsigned(p.batch.count)), dim3(64 * kSmallWaves), lds, st, w.As, w.Bs, w.T, w.L, w.eA,
                       w.eB, p.m, p.n, p.mp, p.np, p.kp, lp.kt, lds, alpha, beta, C, ldc, w.rec, p.tile_mode ? w.tile_S : nullptr, p.batch, fb);
}

}  // namespace oz
