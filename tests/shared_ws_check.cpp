// CPU check of shared_pend_doubles (host_plan.hpp): it covers every launch of
// the call and never shrinks the workspace's need when the constraint set or
// the number of objectives grows.
#include "host_plan.hpp"

using namespace blp;

int main() {
    const PendLimits tiles[] = {{64, 128, 12}, {128, 256, 6}, {256, 512, 3}, {512, 1024, 1}};
    const int nt = 4, cus = 256;
    int failures = 0;
    long checks = 0;
    auto bound = [&](int from, int m, int n, int64_t c) { return shared_pend_doubles(tiles, nt, from, cus, m, n, c); };
    const int64_t counts[] = {1, 2, 255, 256, 700, 1535, 1536, 2500, 2559, 2560, 2600, 3073, 50000};
    const int edges[] = {1, 2, 3, 4, 5, 13, 14, 15, 16, 17, 30, 31, 32, 33, 60, 62, 63, 64, 65, 66, 96, 100, 110, 111, 112, 113,
                         126, 127, 128, 129, 130, 200, 255, 256, 257, 300, 383, 384, 385, 500, 511, 512, 513, 600, 1023, 1024};
    for (int from = 0; from < nt; ++from)
        for (int m : edges)
            for (int n : edges) {
                int t = from;
                while (t < nt && (m > tiles[t].rows || n + m > tiles[t].slots)) ++t;
                int64_t last = 0;
                for (int64_t c : counts) {
                    const int64_t b = bound(from, m, n, c);
                    ++checks;
                    if (b < last) ++failures, std::printf("count: %d x %d x %lld\n", m, n, (long long)c);
                    last = b;
                    // any number of workgroups that the tile may run
                    if (t < nt && b < std::min<int64_t>((int64_t)cus * tiles[t].per_cu, c) * pend_slot(m, n + m))
                        ++failures, std::printf("need: %d x %d x %lld\n", m, n, (long long)c);
                    for (int dm : {1, 2, 16, 64})
                        for (int dn : {0, 1, 4, 64})
                            if ((m > dm && bound(from, m - dm, n, c) > b) || (n > dn && bound(from, m, n - dn, c) > b) ||
                                (m > dm && n > dn && bound(from, m - dm, n - dn, c) > b))
                                ++failures, std::printf("shape: %d x %d x %lld\n", m, n, (long long)c);
                }
            }
    std::printf("%ld checks, %d failures\n", checks, failures);
    return failures != 0;
}
