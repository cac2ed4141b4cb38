// Host-only test of the layout check on what the fused three-way, relay and
// one-workgroup kernels and the widened gathers follow: clean layouts pass,
// each single corruption is rejected with the matching message.  Built and
// run by tests/test_layout_forms.py.
#include <cstdio>
#include <functional>
#include <string>
#include <utility>
#include <vector>

#include "../../paper_2202_04110_amd/csrc/compile.h"
#include "desc_builder.h"

using namespace lbp;
using lbp_test::Builder;

namespace {
int failures = 0;

void expect(bool ok, const std::string &what) {
    if (ok) return;
    std::printf("FAIL: %s\n", what.c_str());
    ++failures;
}

HostLayout run(const char *name, Builder &b,
               const std::vector<std::pair<std::string, std::function<void(HostLayout &)>>> &cases) {
    HostLayout L;
    std::string err;
    const int rc = compile_desc(b.desc(), &L, &err);
    expect(rc == LBP_OK, std::string(name) + ": compile: " + err);
    expect(check_layout(L, &err) == LBP_OK, std::string(name) + ": clean layout rejected: " + err);
    for (const auto &c : cases) {
        HostLayout bad = L;
        c.second(bad);
        std::string e;
        const int r = check_layout(bad, &e);
        expect(r != LBP_OK && e.find(c.first) != std::string::npos,
               std::string(name) + ": corruption '" + c.first + "' gave rc " + std::to_string(r) + " '" + e + "'");
    }
    return L;
}

// the first frelay entry of a lane (wide = false) or wavefront tile
int32_t &entry(HostLayout &L, bool wide) {
    for (const FTile &t : L.ftile)
        if (t.kind == (wide ? TK_LOGW : TK_LOGL))
            for (int32_t i = 0; i < t.a * (wide ? 1 : kLanes); ++i)
                if (L.frelay[t.vb_off + i] >= 0) return L.frelay[t.vb_off + i];
    std::printf("FAIL: no relay entry\n");
    ++failures;
    return L.frelay[0];
}
}  // namespace

int main() {
    {
        Builder b;  // dense three-way factors along rows; 81 variables: idle lanes in the second tile
        for (int i = 0; i < 81; ++i) b.var(3);
        const int t = b.table(3);
        for (int r = 0; r < 9; ++r)
            for (int c = 0; c + 2 < 9; ++c) b.enumf({9 * r + c, 9 * r + c + 1, 9 * r + c + 2}, t);
        const HostLayout L =
            run("three-way", b,
                {{"fused slot variable", [](HostLayout &L) { L.fvar[2 * kLanes + 1] = (int32_t)L.V; }},
                 {"fused slot states", [](HostLayout &L) { L.vns[L.fvar[2 * kLanes]] = 2; }},
                 {"fused edge rows", [](HostLayout &L) { L.vtile[0].kmax = 0; }},
                 {"belief-low message", [](HostLayout &L) { L.vedge[L.vtile[1].e_off + 40] = (int32_t)L.M - 64; }},
                 {"belief-low B/theta", [](HostLayout &L) { L.vtile[1].b_off = (int32_t)L.VB - 2 * kLanes; }}});
        expect(L.tri_fusable && !L.fusable, "three-way: fused form");
    }
    {
        Builder b;  // a chain: square pairwise factors, idle lanes in the last tiles
        for (int i = 0; i < 70; ++i) b.var(4);
        const int t = b.table(2);
        for (int i = 0; i + 1 < 70; ++i) b.enumf({i, i + 1}, t);
        run("chain", b,
            {{"pair slot in the spare panel", [](HostLayout &L) { L.fvb[3] = (int32_t)L.VB - 4 * kLanes; }},
             {"fused edge rows", [](HostLayout &L) { L.vtile[0].kmax = 0; }}});
    }
    {
        // relay: products of two inputs each, ORs over 100 and over 5 of them
        // (wavefront and lane tiles), the outputs after the products
        Builder b;
        const int in = 64, wide = 2, fan = 100, small = 20, sfan = 5;
        for (int i = 0; i < in + wide * fan + small * sfan + wide + small; ++i) b.var(2);
        int prod = in;
        const int out0 = in + wide * fan + small * sfan;
        std::vector<std::vector<int>> ors;
        for (int o = 0; o < wide + small; ++o) {
            std::vector<int> vs;
            for (int j = 0; j < (o < wide ? fan : sfan); ++j, ++prod) {
                b.logical({prod % in, (prod * 5 + 1) % in, prod}, LBP_FACTOR_AND);
                vs.push_back(prod);
            }
            vs.push_back(out0 + o);
            ors.push_back(vs);
        }
        for (const auto &vs : ors) b.logical(vs, LBP_FACTOR_OR);
        const HostLayout L =
            run("relay", b,
                {{"relay address", [](HostLayout &L) { entry(L, false) = 2 * (int32_t)L.M; }},
                 {"relay entry", [](HostLayout &L) { entry(L, false) = -1; }},
                 {"relay entry", [](HostLayout &L) { entry(L, true) = -1; }},
                 {"relay pair", [](HostLayout &L) { entry(L, false) ^= 1; }},
                 {"relay pair", [](HostLayout &L) { entry(L, true) += 2; }},
                 {"relay row", [](HostLayout &L) {
                      for (FTile &t : L.ftile) t.relay = 0;
                  }},
                 {"relay entry", [](HostLayout &L) { L.relay_vgroups[0].tiles.clear(); }},
                 {"wave logical beliefs", [](HostLayout &L) {
                      for (FTile &t : L.ftile)
                          if (t.kind == TK_LOGW) L.fvb[t.vb_off + 2 * kLanes - 1] = (int32_t)L.VB - kLanes;
                  }}});
        expect(!L.frelay.empty(), "relay: views");
    }
    if (!failures) std::printf("layout forms ok\n");
    return failures != 0;
}
