// LDS of the small calls that decide in the slicing's launch, on the host.  Reads lines "m n k esc_block num_cu"; prints per line whether the call's
// sizes fit, the bytes of its tables, and the most a workgroup may have in all.
#include <cstdio>

#include "oz_internal.h"

using namespace oz;

int main() {
    long long m, n, k;
    int b, cus;
    while (std::scanf("%lld %lld %lld %d %d", &m, &n, &k, &b, &cus) == 5) {
        Problem p{};
        p.m = m; p.n = n; p.k = k;
        p.mp = round_up(m, kRowPad); p.np = round_up(n, kRowPad); p.kp = round_up(k, kKPad);
        p.esc_block = b;
        p.G = int((k + b - 1) / b);
        p.num_cu = cus;
        std::printf("%d %lld %d\n", decide_fits(p) ? 1 : 0, static_cast<long long>(decide_table_bytes(p)), kDecideLds);
    }
    return 0;
}
