// Whether native products of one shape share one launch, on the host.  Reads lines "m n k a_rows b_rows problems at_once scratch_bytes";
// prints per line "together".
#include <cstdio>

#include "oz_f64_plan.h"

using namespace oz;

int main() {
    long long m, n, k, scratch;
    int ar, br, problems, at_once;
    while (std::scanf("%lld %lld %lld %d %d %d %d %lld", &m, &n, &k, &ar, &br, &problems, &at_once, &scratch) == 8) {
        const F64Size c = f64_size(m, n, k, 1, false, false, ar, ar ? m : k, br, br ? n : k);
        std::printf("%d\n", int(f64_together(c, problems, at_once, 256, size_t(scratch))));
    }
    return 0;
}
