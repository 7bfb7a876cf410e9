// Host unit test of the weight-ordered loop's index range (gr_order.h): on the
// largest graph it takes, no step past a row's end leaves int32.  Exits non-zero
// on failure.
#include <climits>
#include <cstdio>

#include "gr_order.h"

int main() {
    int32_t lo = 1, hi = INT_MAX;  // the largest m that is taken
    while (lo < hi) {
        const int32_t mid = lo + (int32_t)(((int64_t)hi - lo + 1) / 2);
        if (gr::order_indexes(mid)) lo = mid;
        else hi = mid - 1;
    }
    // the last row's last entry starts at m - 1 at most; a lane adds less than a run
    const int64_t end = (int64_t)lo - 1 + gr::kOrderRun;
    if (end > INT32_MAX || gr::order_indexes(0) || !gr::order_indexes(1 << 30)) {
        std::printf("FAIL m = %d, end = %lld\n", lo, (long long)end);
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
