// The ESC kernel's walk over its blocks on the host.  Reads lines "nbi nbj workgroups"; prints per line "missed_or_repeated
// most_of_a_row most_of_a_column": how many blocks of one block row (column) the busiest workgroup meets.
#include <algorithm>
#include <cstdio>
#include <map>
#include <utility>
#include <vector>

#include "oz_internal.h"

using namespace oz;

int main() {
    long long nbi, nbj, grid;
    while (std::scanf("%lld %lld %lld", &nbi, &nbj, &grid) == 3) {
        std::vector<int> taken(size_t(nbi * nbj));
        std::map<std::pair<long long, long long>, int> row, col;
        long long wrong = 0;
        int most_row = 0, most_col = 0;
        for (int64_t p = 0; p < nbi * nbj; ++p) {
            int64_t bi, bj;
            esc_block_at(p, nbi, nbj, grid, bi, bj);
            if (bi < 0 || bi >= nbi || bj < 0 || bj >= nbj) { ++wrong; continue; }
            ++taken[size_t(bj * nbi + bi)];
            most_row = std::max(most_row, ++row[{p % grid, bi}]);
            most_col = std::max(most_col, ++col[{p % grid, bj}]);
        }
        for (int c : taken) wrong += c != 1;
        std::printf("%lld %d %d\n", wrong, most_row, most_col);
    }
    return 0;
}
