// Exponent-aligned slicing of op(A) (per row) and op(B) (per column) into 8-bit two's-complement
// digits with the unsigned-slice encoding.
// (paper: section "ESC" on the per-row shift space; section "Unsigned Slice Encoding": the
//  leading slice is rounded toward -infinity so that the remainder is non-negative, and every
//  sub-leading u8 digit >= 128 is stored as digit-256 with a carry into the next higher digit.)
//
// Output layout (what the INT8 GEMM's tiles load with contiguous 16-byte pieces):
//   slices[s][l/16][r][l%16]  for row r (padded to rows_p), k index l (padded to kp); padding = 0.
// HBM-bound: 8 B read and S bytes written per element; 8192^3 with seven slices 360 to 410 us by storage order, 4.9 to 5.6 TB/s (a copy
// reaches 5.6).  Operands and slices are touched once per call here, so loads and stores carry the streaming (non-temporal) hint.
#include "oz_slice_device.h"

namespace oz {

struct SliceSide {
    Operand o;
    const int32_t* e_row;
    int8_t* out;
    int64_t row_blocks, blocks;      // workgroups along the rows, in all
};

// workgroups [0, a.blocks) cut a, the others b
// MAXS: the most slices the call can come out with.  The widest form has the registers of the next, 115, and four workgroups to a CU: most
// calls that may need more than 16 slices need fewer (with 137 and three 1024 x 1024 x 16000 with nine slices 106 to 115 us, now 93 to 97).
template <int MAXS>
__global__ __launch_bounds__(256, MAXS <= 8 ? 6 : 4) void slice_kernel(SliceSide a, SliceSide b, int64_t k, int64_t kp, const Record* rec, Batch bt) {
    round_down_fp64();
    const bool second = int64_t(blockIdx.x) >= a.blocks;
    const int64_t ws = bt.ws_at(blockIdx.z);
    SliceSide s = second ? b : a;
    s.o.X += second ? bt.b_at(blockIdx.z) : bt.a_at(blockIdx.z);
    s.e_row = at_bytes(s.e_row, ws);
    s.out = at_bytes(s.out, ws);
    rec = at_bytes(rec, ws);
    const int64_t id = int64_t(blockIdx.x) - (second ? a.blocks : 0);
    const int64_t rb = id % s.row_blocks, cb = id / s.row_blocks;
    const bool rows = s.o.stride_r == 1;
    // the row's exponent is requested together with the record: two loads in a row before the operand's is what a small
    // call waits for
    const int er = s.e_row[rows ? rb * 256 + threadIdx.x : rb * 64 + (threadIdx.x >> 2)];
    const int fallback = rec->res.fallback, S = rec->res.slices_used;
    if (fallback) return;
    if (rows) {                          // 256 rows x 16 k
        uint64_t bits[16];
        load_rows(s.o, rb, threadIdx.x, cb, k, bits);
        put_rows<MAXS>(bits, s.o, rb, threadIdx.x, cb, kp, er, s.out, S);
        return;
    }
    // 64 rows x 64 k, all four chunks requested before the first is cut (one in work and one on its way, for wider words: 8192 x 8192
    // twice at up to 26 slices, nine used, 507 to 528 us, now 423 to 485; 3000 x 3000 twice 81, now 75)
    const int64_t r0 = rb * 64 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 16, c0 = cb * 4;
    uint64_t bits[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) load_k(s.o, r0, c0 + c, k, bits[c]);
    if constexpr (MAXS <= 8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) put_k<MAXS>(bits[c], s.o, r0, c0 + c, kp, er, s.out, S);
    } else {                             // one copy of the longer code
#pragma unroll 1
        for (int c = 0; c < 4; ++c) {
            put_k<MAXS>(bits[0], s.o, r0, c0 + c, kp, er, s.out, S);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bits[0][e] = bits[1][e];
                bits[1][e] = bits[2][e];
                bits[2][e] = bits[3][e];
            }
        }
    }
}

void launch_slice(hipStream_t st, const Operand& a, const Operand& b, const Workspace& w, const Problem& p) {
    auto side = [&](const Operand& o, const int32_t* e, int8_t* out) {
        const bool rows = o.stride_r == 1;
        const int64_t rbs = o.rows_p / (rows ? 256 : 64);
        return SliceSide{o, e, out, rbs, rbs * (p.kp / (rows ? 16 : 64))};
    };
    const SliceSide sa = side(a, w.eA, w.As), sb = side(b, w.eB, w.Bs);
    // a kernel for up to 8 slices, one for up to 16 and one for all: what the wider words need in registers would halve the
    // waves in flight of the others
    const auto kernel = p.s_cap <= 8 ? slice_kernel<8> : p.s_cap <= 16 ? slice_kernel<16> : slice_kernel<kMaxSlices>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(sa.blocks + sb.blocks), 1, unsigned(p.batch.count)), dim3(256), 0, st, sa, sb, p.k, p.kp, w.rec,
                       p.batch);
}

}  // namespace oz
