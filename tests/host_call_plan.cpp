// Which kernels an emulated call takes, on the host.  Reads lines "m n k most_slices fewest_slices per_block problems"; prints per line the
// column of tests/golden/route_times.txt: 0 units (or blocks of 256 x 256), 1 tiles of 32, 2 tiles of 64, 3 tiles of 64 two to a CU.
#include <cstdio>

#include "oz_gemm_plan.h"

using namespace oz;

int main() {
    long long m, n, k;
    int s_cap, s_min, tile_mode, problems;
    while (std::scanf("%lld %lld %lld %d %d %d %d", &m, &n, &k, &s_cap, &s_min, &tile_mode, &problems) == 7) {
        Problem p{};
        p.m = m; p.n = n; p.k = k;
        p.mp = round_up(m, kRowPad); p.np = round_up(n, kRowPad); p.kp = round_up(k, kKPad);
        p.s_cap = s_cap;
        p.s_min = s_min;
        p.kblk = k_block_length(s_cap);
        p.nkb = int((p.kp + p.kblk - 1) / p.kblk);
        p.num_cu = 256;
        p.tile_mode = tile_mode;
        p.batch.count = problems;
        p.raw_slots = int(std::min<int64_t>((p.mp / kTile) * (p.np / kTile), p.num_cu));
        const LaunchPlan lp(p);
        std::printf("%d\n", lp.small ? 1 : (lp.mid ? (lp.mid_pair ? 3 : 2) : 0));
    }
    return 0;
}
