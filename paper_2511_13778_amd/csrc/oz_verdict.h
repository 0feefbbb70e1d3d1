// The verdict of a guarded call, for the two kernels that give it (oz_esc.hip, oz_esc_slice.hip).
// (paper: sections "Heuristic run time Selection" and "GPU-Resident Integration".)
#pragma once

#include "oz_internal.h"

namespace oz {

// What the host knows of the decision.
struct VerdictArgs {
    oz_opts_t o;
    oz_heuristic_t hm;
    int32_t s_cap, tile_mode;
    int32_t nti, ntj, first, deal;       // per-block mode: the blocks, and how they are dealt (tile_order)
    int32_t infnan_parts;                // workgroups of a scan in one launch, 0: otherwise
    int32_t* tile_S;
    oz_result_t* user;
};

// slice count of the fixed and forced modes
__host__ __device__ inline int fixed_slices(const oz_opts_t& o) {
    const int s = o.slices > 0 ? o.slices : (o.max_bits + 1 + 7) / 8;
    return s < 1 ? 1 : (s > kMaxSlices ? kMaxSlices : s);
}

// Slice count and fallback decision of a guarded call from the scan's flag and the ESC.  pairs, smin: per-block mode,
// pair products over all blocks and the smallest count.
__device__ inline oz_result_t verdict(const VerdictArgs& v, int infnan, int span_max, unsigned long long pairs_all, int smin, int64_t m,
                               int64_t n, int64_t k) {
    const oz_opts_t& o = v.o;
    oz_result_t r;
    r.fallback = 0; r.reason = 0; r.slices_used = 0; r.esc = -1; r.required_bits = 0; r.infnan = 0;
    r.slices_min = 0; r.reserved_ = 0; r.pair_tiles = 0;
    const int64_t tiles = ((m + kTile - 1) / kTile) * ((n + kTile - 1) / kTile);
    bool per_tile = false;    // the blocks of C carry their own counts
    const int s_fixed = fixed_slices(o);
    if (infnan) {
        r.fallback = 1; r.reason = 1; r.infnan = 1;
    } else {
        const int esc = min(span_max + 1, kEscCap);
        r.esc = esc;
        r.required_bits = o.target_bits + esc;
        // slices that hold required_bits, the sign and the headroom bit
        int S = (o.target_bits + esc + 1 + kHeadroomBits + 7) / 8;
        if (o.mode == OZ_FORCED_GUARDED) {
            r.slices_used = s_fixed;
        } else if (r.required_bits > o.max_bits) {
            r.fallback = 1; r.reason = 2;
        } else if (o.mode == OZ_FIXED_GUARDED) {
            // the fixed slices must really carry the bits (S slices carry 8S - 2: "55 bits" is 54)
            if (S > s_fixed) { r.fallback = 1; r.reason = 2; }
            else r.slices_used = s_fixed;
        } else {
            S = max(1, min(S, kMaxSlices));
            per_tile = v.tile_mode != 0;
            bool slower = false;
            if (o.heuristic) {
                const int64_t flops = 2 * m * n * k;
                // pair products per block of C: S(S+1)/2, or the mean over the blocks, rounded up
                const int64_t pairs = per_tile ? int64_t((pairs_all + (unsigned long long)(tiles) - 1) /
                                                         (unsigned long long)(tiles))
                                               : int64_t(S) * (S + 1) / 2;
                const int64_t stream = (16 + S) * (m * k + k * n) + (2 * int64_t(S) + 22) * m * n;
                const int64_t t_emu = v.hm.fixed_ns + (flops / v.hm.int8_ops_per_ns) * pairs + stream / v.hm.bytes_per_ns;
                const int64_t t_f64 = flops / v.hm.fp64_flops_per_ns;
                slower = t_emu > t_f64;
            }
            if (slower) { r.fallback = 1; r.reason = 3; }
            else r.slices_used = S;
        }
    }
    // The workspace holds s_cap slice planes and the host sized it for the largest count these options
    // can select, so this never binds; if it ever did, running with fewer slices would lose bits
    // silently, so the call goes native and says why.
    if (!r.fallback && r.slices_used > v.s_cap) { r.fallback = 1; r.reason = 2; r.slices_used = 0; }
    if (!r.fallback && r.slices_used > 0) {
        r.slices_min = per_tile ? smin : r.slices_used;
        r.pair_tiles = per_tile ? int64_t(pairs_all) : tiles * (int64_t(r.slices_used) * (r.slices_used + 1) / 2);
    }
    return r;
}

inline VerdictArgs verdict_args(const Workspace& w, const Problem& p, const oz_opts_t& o, const oz_heuristic_t& hm, oz_result_t* user) {
    VerdictArgs v = {o, hm, p.s_cap, p.tile_mode, int(p.mp / kTile), int(p.np / kTile), 0, 0, scan_once(p) ? int((p.mp + p.np) / kOnceRows) : 0, w.tile_S, user};
    if (p.tile_mode) tile_order_shape(p, v.first, v.deal);
    return v;
}

// Inf or NaN in the operands: of all lanes of a wave
__device__ __forceinline__ int any_infnan(const Record* rec, int parts) {
    static_assert(kScanOnceParts == 2 * 64, "two flags a lane");
    const int lane = threadIdx.x & 63;
    return parts == 0 ? rec->infnan
                      : __any((lane < parts && rec->infnan_part[lane] != 0) || (lane + 64 < parts && rec->infnan_part[lane + 64] != 0));
}

// slice count that carries the target and a span
__device__ __forceinline__ int span_slices(const oz_opts_t& o, int span) {
    return max(1, min((o.target_bits + min(span + 1, kEscCap) + 1 + kHeadroomBits + 7) / 8, kMaxSlices));
}

}  // namespace oz
