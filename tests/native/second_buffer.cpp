// GPU test of graphs whose second message buffer is optional: device
// allocations above a limit are refused here (this program's hipMalloc stands
// in front of the runtime's), and an upload that no longer fits with the
// buffer goes through without it, with the same results.  Built and run by
// tests/test_gpu_second_buffer.py.
#include <dlfcn.h>

#include <cstdio>
#include <string>
#include <vector>

#include "../../paper_2202_04110_amd/csrc/runtime.h"
#include "desc_builder.h"

using lbp_test::Builder;

namespace {
size_t alloc_limit = SIZE_MAX;
int refused = 0, failures = 0;

void expect(bool ok, const std::string &what) {
    if (ok) return;
    std::printf("FAIL: %s\n", what.c_str());
    ++failures;
}

// dense three-way factors along the rows of an L x L grid
void triples(Builder &b, int L) {
    for (int i = 0; i < L * L; ++i) b.var(3);
    const int t = b.table(3);
    for (int r = 0; r < L; ++r)
        for (int c = 0; c + 2 < L; ++c) b.enumf({r * L + c, r * L + c + 1, r * L + c + 2}, t);
}

// OR factors over products that are each the child of one AND; the products
// fill variable tiles of their own
void layered(Builder &b, int inputs, int outputs, int fan) {
    for (int i = 0; i < inputs; ++i) b.var(2);
    const int prod = inputs;
    for (int i = 0; i < outputs * (fan + 1); ++i) b.var(2);
    for (int o = 0; o < outputs; ++o) {
        std::vector<int> ors;
        for (int j = 0; j < fan; ++j) {
            const int x = (7 * o + 3 * j) % inputs;
            ors.push_back(prod + o * fan + j);
            b.logical({x, (x + 1 + j % (inputs - 1)) % inputs, ors[j]}, LBP_FACTOR_AND);
        }
        ors.push_back(prod + outputs * fan + o);
        b.logical(ors, LBP_FACTOR_OR);
    }
}

std::vector<float> solve(lbp_graph *g) {
    std::vector<float> m(g->ES);
    expect(lbp_run_bp(g, 7, 0.5f, 1.0f) == LBP_OK, "run");
    expect(lbp_get_messages(g, m.data(), 0) == LBP_OK, "messages");
    return m;
}

void check(lbp_ctx *ctx, const char *name, Builder &b) {
    std::printf("%s\n", name);
    std::fflush(stdout);
    const std::string at = std::string(name) + ": ";
    lbp_graph *full = nullptr, *tight = nullptr;
    expect(lbp_graph_upload(ctx, b.desc(), &full) == LBP_OK, at + "upload");
    if (!full) return;
    expect(full->m2 && (full->relay || full->tri), at + "has a second buffer");
    const std::vector<float> want = solve(full);
    alloc_limit = full->dbytes - 1;
    refused = 0;
    const int rc = lbp_graph_upload(ctx, b.desc(), &tight);
    alloc_limit = SIZE_MAX;
    expect(refused == 1, at + "the first allocation was refused");
    expect(rc == LBP_OK, at + "upload without the second buffer gave " + std::to_string(rc));
    if (rc == LBP_OK) {
        expect(!tight->m2 && !tight->relay && !tight->tri && tight->dbytes < full->dbytes, at + "no second buffer");
        expect(solve(tight) == want, at + "same messages");
        lbp_graph_free(tight);
    }
    alloc_limit = 64;  // nothing fits: still an error
    tight = nullptr;
    expect(lbp_graph_upload(ctx, b.desc(), &tight) == LBP_E_OOM && !tight, at + "out of memory reported");
    alloc_limit = SIZE_MAX;
    lbp_graph_free(full);
}
}  // namespace

extern "C" hipError_t hipMalloc(void **p, size_t n) {
    using fn = hipError_t (*)(void **, size_t);
    static const fn real = (fn)dlsym(RTLD_NEXT, "hipMalloc");
    if (n > alloc_limit) {
        ++refused;
        return hipErrorOutOfMemory;
    }
    return real(p, n);
}

int main() {
    lbp_ctx *ctx = nullptr;
    if (lbp_ctx_create(0, nullptr, &ctx) != LBP_OK) {
        std::printf("FAIL: no context: %s\n", lbp_last_error());
        return 1;
    }
    {
        Builder b;
        triples(b, 30);
        check(ctx, "three-way", b);
    }
    {
        Builder b;
        layered(b, 30, 12, 40);
        check(ctx, "logical", b);
    }
    lbp_ctx_destroy(ctx);
    if (!failures) std::printf("second buffer ok\n");
    return failures != 0;
}
