// The scan's launches on the host.  Reads lines "m n k esc_block a_rows_contig b_rows_contig"; prints per line
// "launches most_threads groups_covered groups_needed".
#include <algorithm>
#include <cstdio>

#include "oz_internal.h"

using namespace oz;

int main() {
    long long m, n, k;
    int b, ar, br;
    while (std::scanf("%lld %lld %lld %d %d %d", &m, &n, &k, &b, &ar, &br) == 6) {
        Problem p{};
        p.m = m; p.n = n; p.k = k;
        p.mp = round_up(m, kRowPad); p.np = round_up(n, kRowPad);
        p.esc_block = b;
        p.G = int((k + b - 1) / b);
        p.num_cu = 256;
        const ScanGrid g = scan_grid(p, ar != 0, br != 0);
        long long launches = 0, most = 0, covered = 0;
        for (int64_t y = 0; y < g.groups; y += g.slab) {
            const int64_t gy = std::min(g.groups - y, g.slab);
            most = std::max<long long>(most, (g.row_blocks_a + g.row_blocks_b) * gy * 256);
            covered += gy * g.per;
            ++launches;
        }
        std::printf("%lld %lld %lld %d\n", launches, most, covered, p.G);
    }
    return 0;
}
