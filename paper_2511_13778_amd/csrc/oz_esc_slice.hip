// ESC, verdict and slicing of a small call in one launch.
// (paper: sections "ESC", "Heuristic run time Selection", "Unsigned Slice Encoding".)
//
// A small call waits for its chain of dependent launches, not for what they compute, and the ESC kernel is a chain of its own: load
// the tables, leave the span, arrive, read everybody's, decide, write the record, which the slicing loads first.  Here every
// workgroup of the slicing holds the encoded tables of the whole call in LDS, finds the largest span and the verdict for itself, and
// cuts its part of the operands, loaded meanwhile; one of them leaves the record.  No workgroup waits for another.
// The ESC is the one of oz_esc.hip: max-plus product on the BF16 matrix unit, and on packed int16 for the 64 x 64 blocks of pairs
// whose spans that cannot hold.
#include "oz_slice_device.h"
#include "oz_verdict.h"

namespace oz {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x16_t __attribute__((ext_vector_type(16)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef uint16_t ushort2_t __attribute__((ext_vector_type(2)));

constexpr int kDecideThreads = 512, kDecideWaves = kDecideThreads / 64;
constexpr int kDecideTiles = 32;             // most blocks of C that can take their own slice count

struct DecideSide {
    Operand o;
    const uint4* enc;        // encoded table [chunks][rows_p], rows of eight h
    const int16_t* tab;      // [2G][rows_p]
    const int32_t* e;
    int8_t* out;
    int32_t rows64;          // rows of the tables that count, a multiple of 64
    int32_t row_blocks, blocks;      // workgroups along the rows, in all
};

struct DecideShared {
    int tile_span[kDecideTiles];
    uint32_t open;                       // blocks of 64 x 64 pairs, a bit each
    int span;
    oz_result_t res;
};

// Smallest of a lane's chunk-maximum sums of a 32 x 32 tile, as FP32 bit patterns.  Rows and columns of padding are encoded as
// infinity: their sums are infinite or no numbers, larger than any other as bit patterns.
__device__ __forceinline__ uint32_t tile_least(const uint4* eu, const uint4* ev, int ru, int rv, int steps, int i0, int j0) {
    const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
    const f32x16_t zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t run[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) run[r] = 0;
    for (int c = 0; c < steps; ++c) {                // 16 h each
        const u32x16_t d = __builtin_bit_cast(u32x16_t, __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                               __builtin_bit_cast(bf16x8_t, eu[(2 * c + lh) * ru + i0 + lr]),
                               __builtin_bit_cast(bf16x8_t, ev[(2 * c + lh) * rv + j0 + lr]), zero, 0, 0, 0));
#pragma unroll
        for (int r = 0; r < 16; ++r) run[r] = max(run[r], d[r]);
    }
    uint32_t least = run[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) least = min(least, run[r]);
    return least;
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x = min(x, uint32_t(__shfl_xor(int(x), off)));
    return x;
}
// the span of a sum; more than kEncRange: of no meaning
__device__ __forceinline__ int span_of(uint32_t sum) {
    return 64 - (int(sum >> 23) - 127 - 2 * kEncBias + kEncScale * 64) / kEncScale;
}

// Rows of padding in the unencoded tables: sums that no span comes from, whatever they are added to.
constexpr int kDecidePad = 16000;
constexpr int kDecideLowest = -2000;         // stands for the exponent of a row of zeros, none of whose sums counts

// Largest span of a 64 x 64 block the exact way, 8 x 8 pairs a lane; of one wave.  eA, eB: no less than kDecideLowest.
__device__ __forceinline__ int block_exact(const int16_t* u, const int16_t* v, int ru, int rv, int H2, const int32_t* eA, const int32_t* eB,
                                           int i0, int j0) {
    const int lane = threadIdx.x & 63, i = i0 + (lane >> 3) * 8, j = j0 + (lane & 7) * 8;
    short2_t acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = short2_t{-32768, -32768};
#pragma unroll 1
    for (int h = 0; h < H2; ++h) {
        const short8_t x = *reinterpret_cast<const short8_t*>(u + h * ru + i);
        const short8_t y = *reinterpret_cast<const short8_t*>(v + h * rv + j);
        const short2_t y2[4] = {short2_t{y[0], y[1]}, short2_t{y[2], y[3]}, short2_t{y[4], y[5]}, short2_t{y[6], y[7]}};
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = __builtin_elementwise_max(acc[a][c], short2_t{x[a], x[a]} + y2[c]);
    }
    // Moved up by -kSumDeadBelow, sums "that contribute nothing" are the largest as unsigned numbers, and leave no span by a difference that
    // stops at zero; those "without information" are the smallest, and one of them is the cap.
    ushort2_t lowest = {0xFFFF, 0xFFFF}, most = {0, 0}, eb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) eb[c] = ushort2_t{uint16_t(eB[j + 2 * c]), uint16_t(eB[j + 2 * c + 1])};
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const uint16_t ea = uint16_t(eA[i + a] - kSumDeadBelow);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const ushort2_t z = __builtin_bit_cast(ushort2_t, acc[a][c]) + uint16_t(-kSumDeadBelow);
            lowest = __builtin_elementwise_min(lowest, z);
            most = __builtin_elementwise_max(most, __builtin_elementwise_sub_sat(eb[c] + ea, z));
        }
    }
    int best = min(int(lowest[0]), int(lowest[1])) < kSumRealFloor - kSumDeadBelow ? kEscCap : max(int(most[0]), int(most[1]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) best = max(best, __shfl_xor(best, off));
    return best;
}

// workgroups [0, a.blocks) cut a, the others b: 32 k of 64 rows, four k a thread
template <int MAXS>
__global__ __launch_bounds__(kDecideThreads, 2) void esc_slice_kernel(DecideSide a, DecideSide b, int m, int n, int64_t k, int64_t kp, int H2,
                                                                      int steps, Record* rec, VerdictArgs v, Batch bt) {
    extern __shared__ __align__(16) uint4 tables[];
    __shared__ DecideShared sh;
    round_down_fp64();
    const int lane = threadIdx.x & 63, tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t ws = bt.ws_at(blockIdx.z);
    rec = at_bytes(rec, ws);
    const bool second = int(blockIdx.x) >= a.blocks;
    DecideSide s = second ? b : a;
    s.o.X += second ? bt.b_at(blockIdx.z) : bt.a_at(blockIdx.z);
    s.out = at_bytes(s.out, ws);
    const int id = int(blockIdx.x) - (second ? a.blocks : 0);
    const int cb = id / s.row_blocks, rb = id - cb * s.row_blocks;

    // everything that comes from memory is requested before the first of it is waited for
    const int infnan = any_infnan(rec, v.infnan_parts);
    const bool rows = s.o.stride_r == 1;
    // rows contiguous: a wave takes 64 rows and part (wave & 3) of a chunk of 16 k; k contiguous: 16 rows and a chunk
    const int64_t c = int64_t(cb) * 2 + (wave >> 2), r0 = int64_t(rb) * 64 + (rows ? 0 : (wave & 3) * 16);
    const int er = at_bytes(s.e, ws)[r0 + (rows ? lane : lane >> 2)];
    uint64_t bits[4];
    if (rows) load_rows4(s.o, r0, uint32_t(lane), c, wave & 3, k, bits);
    else load_k(s.o, r0, c, k, bits);
    // ---- tables of both operands: a's, then b's; 64 rows at a time, all loads in flight together
    const int chunks = 2 * steps;
    uint4* const eu = tables;
    uint4* const ev = tables + chunks * a.rows64;
    {
        const int per_a = a.rows64 / 64, per_b = b.rows64 / 64, of_a = chunks * per_a, pieces = of_a + chunks * per_b;
        constexpr int kMost = kDecideLds / 1024 / kDecideWaves;
        uint4 x[kMost];
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
            const int p = wave + i * kDecideWaves;
            if (p >= pieces) continue;
            const bool in_b = p >= of_a;
            const int q = in_b ? p - of_a : p, per = in_b ? per_b : per_a, h = q / per, r = (q - h * per) * 64 + lane;
            const uint4* const src = at_bytes(in_b ? b.enc : a.enc, ws);
            const bool there = r < (in_b ? b.o.rows : a.o.rows);
            x[i] = src[h * (in_b ? b.o.rows_p : a.o.rows_p) + r];
            if (!there) x[i] = make_uint4(0x7F807F80u, 0x7F807F80u, 0x7F807F80u, 0x7F807F80u);
        }
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
            const int p = wave + i * kDecideWaves;
            if (p < pieces) tables[p * 64 + lane] = x[i];
        }
    }
    if (tid < kDecideTiles) sh.tile_span[tid] = 0;
    if (tid == 0) {
        sh.span = 0;
        sh.open = 0;
    }
    __syncthreads();

    // ---- the widest span: of all of C, or block by block where it is to be known or where some are beyond the encoding
    const int nbi = a.rows64 / kDecidePairs, blocks = nbi * (b.rows64 / kDecidePairs);
    auto leave = [&](int bi, int bj, int span) {
        if (lane == 0) {
            atomicMax(&sh.span, span);
            if (v.tile_mode) atomicMax(&sh.tile_span[(bj >> 2) * v.nti + (bi >> 2)], span);
        }
    };
    // in the forced mode only the record needs the span
    const bool whole = blockIdx.x == 0 || v.o.mode != OZ_FORCED_GUARDED;
    const int nti = (m + 31) / 32, tiles = infnan || !whole ? 0 : nti * ((n + 31) / 32);
    bool open = false;
    if (!v.tile_mode) {
        uint32_t least = 0xFFFFFFFFu;
        for (int x = wave; x < tiles; x += kDecideWaves) {
            const int tj = x / nti, ti = x - tj * nti;
            least = min(least, tile_least(eu, ev, a.rows64, b.rows64, steps, ti * 32, tj * 32));
        }
        if (wave < tiles) {
            const int span = span_of(wave_min(least));
            open = span > kEncRange;
            if (!open) leave(0, 0, span);
        }
        open = __syncthreads_or(open);
        if (open && tid == 0) sh.open = ~0u;
    } else {
        open = false;
        for (int x = wave; x < tiles; x += kDecideWaves) {
            const int tj = x / nti, ti = x - tj * nti;
            const int span = span_of(wave_min(tile_least(eu, ev, a.rows64, b.rows64, steps, ti * 32, tj * 32)));
            if (span <= kEncRange) {
                leave(ti >> 1, tj >> 1, span);
            } else {
                if (lane == 0) atomicOr(&sh.open, 1u << ((tj >> 1) * nbi + (ti >> 1)));
                open = true;
            }
        }
        open = __syncthreads_or(open);
    }
    if (open) {
        // below the encodable range, or no candidate at all: the unencoded tables, in the same place
        auto stage_table = [&](const DecideSide& d, uint4* to) {
            const int16_t* const src = at_bytes(d.tab, ws);
            const int per = d.rows64 / 8;
#pragma unroll 4
            for (int p = tid; p < H2 * per; p += kDecideThreads) {
                const int h = p / per, r = p - h * per;
                short8_t x = reinterpret_cast<const short8_t*>(src)[h * (d.o.rows_p / 8) + r];
#pragma unroll
                for (int q = 0; q < 8; ++q) x[q] = r * 8 + q < d.o.rows ? x[q] : short(kDecidePad);
                to[p] = __builtin_bit_cast(uint4, x);
            }
        };
        stage_table(a, eu);
        stage_table(b, ev);
        int32_t* const ea = reinterpret_cast<int32_t*>(tables + chunks * (a.rows64 + b.rows64));
        int32_t* const eb = ea + a.rows64;
        for (int x = tid; x < a.rows64; x += kDecideThreads) ea[x] = x < m ? max(at_bytes(a.e, ws)[x], kDecideLowest) : 0;
        for (int x = tid; x < b.rows64; x += kDecideThreads) eb[x] = x < n ? max(at_bytes(b.e, ws)[x], kDecideLowest) : 0;
        __syncthreads();
        for (int x = wave; x < blocks; x += kDecideWaves) {
            if (!(sh.open >> x & 1)) continue;
            const int bj = x / nbi, bi = x - bj * nbi;
            leave(bi, bj, block_exact(reinterpret_cast<const int16_t*>(eu), reinterpret_cast<const int16_t*>(ev), a.rows64, b.rows64, H2, ea, eb,
                                      bi * kDecidePairs, bj * kDecidePairs));
        }
        __syncthreads();
    }

    // ---- verdict
    if (tid == 0) {
        unsigned long long pairs = 0;
        int smin = kMaxSlices;
        if (v.tile_mode) {
            for (int t = 0; t < v.nti * v.ntj; ++t) {
                const int S = span_slices(v.o, sh.tile_span[t]);
                pairs += (unsigned long long)(S) * (S + 1) / 2;
                smin = min(smin, S);
            }
        }
        const oz_result_t r = verdict(v, infnan, sh.span, pairs, smin, m, n, k);
        sh.res = r;
        if (blockIdx.x == 0) {
            rec->res = r;
            if (v.user) v.user[blockIdx.z] = r;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && v.tile_mode && !infnan && tid < v.nti * v.ntj) {
        int32_t* const tile_S = at_bytes(v.tile_S, ws);
        tile_S[tid] = span_slices(v.o, sh.tile_span[tid]);
        if (!sh.res.fallback) tile_S[v.nti * v.ntj + tid] = tid;         // dealt as they come (decide_in_slice)
    }
    if (sh.res.fallback) return;
    const int S = sh.res.slices_used;
    emit<MAXS, 4>(bits, er, S, s.out + (c * s.o.rows_p + r0) * 16, rows ? uint32_t(lane) * 16u + uint32_t(wave & 3) * 4u : uint32_t(lane) * 4u,
                  kp * s.o.rows_p);
}

bool decide_in_slice(const Problem& p) {
    if (!decide_fits(p)) return false;
    if (!p.tile_mode) return true;
    int first, deal;
    tile_order_shape(p, first, deal);
    return deal == 0 && (p.mp / kTile) * (p.np / kTile) <= kDecideTiles;
}

void launch_esc_slice(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p, const oz_opts_t& o,
                      const oz_heuristic_t& hm, oz_result_t* user_result) {
    const int H2 = 2 * p.G, steps = (H2 + kEncChunk - 1) / kEncChunk;
    auto side = [&](const Operand& x, const uint16_t* enc, const int16_t* tab, const int32_t* e, int8_t* out) {
        const int rbs = int(x.rows_p / 64);
        return DecideSide{x, reinterpret_cast<const uint4*>(enc), tab, e, out, int32_t(round_up(x.rows, 64)), rbs, rbs * int(p.kp / 32)};
    };
    const DecideSide sa = side(a, w.EU, w.U, w.eA, w.As), sb = side(b, w.EV, w.V, w.eB, w.Bs);
    const auto kernel = p.s_cap <= 8 ? esc_slice_kernel<8> : p.s_cap <= 16 ? esc_slice_kernel<16> : esc_slice_kernel<kMaxSlices>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(sa.blocks + sb.blocks), 1, unsigned(p.batch.count)), dim3(kDecideThreads),
                       size_t(decide_table_bytes(p)), st, sa, sb, int(p.m), int(p.n), p.k, p.kp, H2, steps, w.rec,
                       verdict_args(w, p, o, hm, user_result), p.batch);
}

}  // namespace oz
