// Follows every workgroup of the slice GEMM's launches on the host, with the library's own launch plan and walk, and
// counts how often each (unit of C, part of k) is taken.  Reads lines "m n k s_cap tile_mode num_cu"; prints per line
// "kind zsplit missed repeated mixed few" with kind 0 whole, 1 parts, 2 atomics (of the launch that may be split), mixed =
// workgroups that take units of different parts, few = the call goes to the 256 x 256 blocks instead.
#include <cstdio>
#include <vector>

#include "oz_gemm_plan.h"

using namespace oz;

static Problem problem(int64_t m, int64_t n, int64_t k, int s_cap, int tile_mode, int num_cu) {
    Problem p{};
    p.m = m; p.n = n; p.k = k;
    p.mp = round_up(m, kRowPad); p.np = round_up(n, kRowPad); p.kp = round_up(k, kKPad);
    p.s_cap = s_cap;
    p.s_min = tile_mode ? 1 : s_cap;
    p.kblk = k_block_length(s_cap);
    p.nkb = int((p.kp + p.kblk - 1) / p.kblk);
    p.num_cu = num_cu;
    p.tile_mode = tile_mode;
    p.raw_slots = int(std::min<int64_t>((p.mp / kTile) * (p.np / kTile), num_cu));
    return p;
}

int main() {
    long long m, n, k;
    int s_cap, tile_mode, num_cu;
    while (std::scanf("%lld %lld %lld %d %d %d", &m, &n, &k, &s_cap, &tile_mode, &num_cu) == 6) {
        const Problem p = problem(m, n, k, s_cap, tile_mode, num_cu);
        const LaunchPlan lp(p);
        std::vector<int32_t> order(size_t(lp.g.nti) * lp.g.ntj);      // any permutation will do
        for (size_t i = 0; i < order.size(); ++i) order[i] = int32_t(order.size() - 1 - i);
        const int32_t* ord = tile_mode ? order.data() : nullptr;
        struct Launch { int begin, count; Split split; };
        std::vector<Launch> launches;
        if (lp.two) launches = {{0, lp.full, Split{1, false}}, {lp.full, lp.rest, lp.last}};
        else launches = {{0, lp.positions, lp.last}};
        // taken[unit][64 of k]
        std::vector<std::vector<int>> taken(size_t(lp.g.um) * lp.g.un, std::vector<int>(lp.kt, 0));
        long long mixed = 0;
        for (const Launch& l : launches) {
            unsigned workgroups;
            const GemmGrid g = lp.launch(p, l.begin, l.count, l.split, workgroups);
            const int stride = int(workgroups) >> 3;
            for (unsigned b = 0; b < workgroups; ++b) {
                const int xcd = int(b & 7);
                int slot = int(b >> 3), ui, uj, z, local, xcd_units, first_z = -1;
                bool more = unit_of(xcd, slot, g, ord, ui, uj, z, local, xcd_units);
                while (more && skip_padding(xcd, stride, slot, g, ord, ui, uj, z, local, xcd_units, [] {})) {
                    if (first_z < 0) first_z = z;
                    if (z != first_z) ++mixed;
                    for (int t = part_first(g.kt_total, g.zsplit, z); t < part_first(g.kt_total, g.zsplit, z + 1); ++t)
                        ++taken[size_t(uj) * lp.g.um + ui][t];
                    if (!g.persistent) break;
                    slot += stride;
                    more = unit_of(xcd, slot, g, ord, ui, uj, z, local, xcd_units);
                }
            }
        }
        long long missed = 0, repeated = 0;
        for (auto& unit : taken)
            for (int c : unit) {
                missed += c == 0;
                repeated += c > 1;
            }
        std::printf("%d %d %lld %lld %lld %d\n", lp.last.z == 1 ? 0 : (lp.last.atomic ? 2 : 1), lp.last.z, missed, repeated, mixed, int(lp.few));
    }
    return 0;
}
