// Host-only test of three_way_runs_fit: three-way tiles close early only where
// the padded panels keep to 32-bit indices, so no class that fits full tiles is
// refused for them.  Built and run by tests/test_three_way_runs.py.
#include <cstdio>

#include "../../paper_2202_04110_amd/csrc/compile.h"

using namespace lbp;

int main() {
    int failures = 0;
    auto expect = [&](bool ok, const char *what, long long f, int n) {
        if (ok) return;
        std::printf("FAIL: %s (%lld factors, %d states)\n", what, f, n);
        ++failures;
    };
    for (int n = 2; n <= 4; ++n) {
        // the most factors that fit in full tiles
        const int64_t most = (kPanelFloatsMax - 1) / (kLanes * n * n * n) * kLanes;
        expect(!three_way_runs_fit(most, n, 0, 0), "the largest class keeps full tiles", most, n);
        const int64_t padded = (kPanelFloatsMax - 1) / (kLanes * n * n * n) * 48;
        expect(three_way_runs_fit(padded, n, 0, 0), "fits at 48 a tile", padded, n);
        expect(!three_way_runs_fit(padded + 1, n, 0, 0), "one past that", padded + 1, n);
        expect(!three_way_runs_fit(padded, n, 0, kLanes * n * n * n), "behind other potentials", padded, n);
        expect(!three_way_runs_fit(480, n, kPanelFloatsMax - 10 * kLanes * 3 * n, 0), "behind other messages", 480, n);
        expect(three_way_runs_fit(480, n, kPanelFloatsMax - 10 * kLanes * 3 * n - 1, 0), "just before", 480, n);
        // the worst padding of the accepted class stays in range
        expect((padded + 47) / 48 * kLanes * n * n * n < kPanelFloatsMax, "in range", padded, n);
    }
    if (!failures) std::printf("three-way runs ok\n");
    return failures != 0;
}
