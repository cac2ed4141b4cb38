// GPU test: the launch shapes of a relay graph's variable launches are the
// ones set by lbp_graph_set_launch and chosen by lbp_autotune, in two-phase
// and in relay iterations alike, and change no result.  Built and run by
// tests/test_gpu_relay_shapes.py.
#include <cstdio>
#include <string>
#include <vector>

#include "../../paper_2202_04110_amd/csrc/runtime.h"
#include "desc_builder.h"

using lbp_test::Builder;

namespace {
int failures = 0;
void expect(bool ok, const std::string &what) {
    if (ok) return;
    std::printf("FAIL: %s\n", what.c_str());
    ++failures;
}

std::vector<float> solve(lbp_graph *g) {
    std::vector<float> m(g->ES);
    expect(lbp_reset_messages(g) == LBP_OK && lbp_run_bp(g, 6, 0.5f, 0.0f) == LBP_OK &&
               lbp_get_messages(g, m.data(), 0) == LBP_OK,
           "solve");
    return m;
}

bool same_shapes(const lbp_graph *g) {
    bool ok = g->relay_vl.size() == g->vl.size();
    for (size_t i = 0; ok && i < g->vl.size(); ++i)
        ok = g->relay_vl[i].shape.wpb == g->vl[i].shape.wpb && g->relay_vl[i].shape.swizzle == g->vl[i].shape.swizzle;
    return ok;
}
}  // namespace

int main() {
    lbp_ctx *ctx = nullptr;
    if (lbp_ctx_create(0, nullptr, &ctx) != LBP_OK) {
        std::printf("FAIL: no context: %s\n", lbp_last_error());
        return 1;
    }
    // 64 inputs of AND factors (four of them wide enough for the block path),
    // 256 products, one OR over them
    Builder b;
    for (int i = 0; i < 64 + 256 + 1; ++i) b.var(2);
    std::vector<int> ors;
    for (int j = 0; j < 256; ++j) {
        b.logical({j % 4, 4 + j % 60, 64 + j}, LBP_FACTOR_AND);
        ors.push_back(64 + j);
    }
    ors.push_back(64 + 256);
    b.logical(ors, LBP_FACTOR_OR);
    lbp_graph *g = nullptr;
    expect(lbp_graph_upload(ctx, b.desc(), &g) == LBP_OK && g && g->relay, "upload with relay views");
    if (!failures) {
        const std::vector<float> want = solve(g);
        expect(same_shapes(g), "shapes at upload");
        for (int z : {1, 0, 1}) {
            for (int32_t i = 0; i < (int32_t)g->vl.size(); ++i)
                expect(lbp_graph_set_launch(g, i, 4, z) == LBP_OK, "set_launch");
            expect(same_shapes(g) && g->vl[0].shape.swizzle == z, "shapes after set_launch " + std::to_string(z));
            expect(solve(g) == want, "messages at swizzle " + std::to_string(z));
        }
        expect(lbp_autotune(g, 0.5f, 0.0f, 3, nullptr) == LBP_OK, "autotune");
        expect(same_shapes(g), "shapes after autotune");
        expect(solve(g) == want, "messages after autotune");
    }
    if (g) lbp_graph_free(g);
    lbp_ctx_destroy(ctx);
    if (!failures) std::printf("relay shapes ok\n");
    return failures != 0;
}
