// CPU check of plan_forks (host_plan.hpp).
#include <cstdlib>

#include "host_plan.hpp"

using namespace blp;

static int failures = 0;
static void expect(bool ok, const char* what) {
    if (!ok) ++failures, std::printf("%s\n", what);
}

int main() {
    std::vector<int> on;
    // classes without LPs, by size before the others, take no stream from them
    expect(plan_forks({0, 0, 555, 0, 490, 96}, 3, 250, on) == 3, "three streams");
    expect(on[2] != on[4] && on[2] != on[5] && on[4] != on[5], "the classes with LPs share no stream");
    expect(on[0] == on[5] && on[1] == on[5] && on[3] == on[5], "empty launches go where there is least work");
    // short launches are not worth a fork
    expect(plan_forks({24, 24, 9, 0, 0}, 3, 250, on) == 0, "tiny LPs");
    expect(plan_forks({5000, 100, 80}, 3, 250, on) == 0, "one long launch");
    expect(plan_forks({5000, 300}, 3, 250, on) == 2, "two launches");
    expect(plan_forks({}, 3, 250, on) == 0 && on.empty(), "no launch");
    // no stream holds more than the longest launch and a fair share
    for (int r = 0; r < 2000; ++r) {
        std::vector<double> us((size_t)(1 + std::rand() % 16));
        double sum = 0, most = 0, load[3] = {};
        for (double& u : us) {
            u = std::rand() % 3 ? std::rand() % 5000 : 0;
            sum += std::max(u, 10.0), most = std::max(most, std::max(u, 10.0));
        }
        const int nf = plan_forks(us, 3, 0, on);
        expect(nf >= 1 && nf <= 3 && on.size() == us.size(), "streams in range");
        for (size_t i = 0; i < us.size(); ++i) {
            expect(on[i] >= 0 && on[i] < nf, "stream of a launch");
            load[on[i]] += std::max(us[i], 10.0);
        }
        for (double l : load) expect(l <= most + sum / 3 + 1e-6, "balance");
    }
    std::printf("%d failures\n", failures);
    return failures != 0;
}
