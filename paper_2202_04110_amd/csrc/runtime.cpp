// Internal runtime shared by the C-ABI and the serving loop (see runtime.h).
#include "runtime.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

namespace lbp {

namespace {
thread_local std::string t_err;
}

int set_error(int code, const std::string &msg) {
    t_err = msg;
    return code;
}

int hip_error(hipError_t e, const char *what) {
    return set_error(LBP_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

const char *last_error() { return t_err.c_str(); }

bool valid_params(int32_t iters, float d, float T, std::string *why) {
    if (iters < 0) {
        *why = "iters < 0";
        return false;
    }
    if (!(d >= 0.0f && d <= 1.0f)) {
        *why = "damping outside [0, 1]";
        return false;
    }
    if (!(T >= 0.0f) || !std::isfinite(T)) {
        *why = "temperature must be finite and >= 0";
        return false;
    }
    return true;
}

// ------------------------------------------------------------ launch lists
void add_to_lists(LaunchLists &ll, int32_t gi, const GraphShape &s, std::vector<WorkItem> *mids,
                  std::vector<WorkItem> *highs, std::vector<WorkItem> *cols) {
    for (const VGroup &vg : s.vgroups) {
        size_t i = 0;
        while (i < ll.vbucket.size() && ll.vbucket[i] != vg.bucket) ++i;
        if (i == ll.vbucket.size()) {
            ll.vbucket.push_back(vg.bucket);
            ll.vitems.emplace_back();
        }
        for (int32_t t : vg.tiles) ll.vitems[i].push_back(WorkItem{gi, t});
    }
    for (int32_t h : s.mids) mids->push_back(WorkItem{gi, h});
    for (int32_t h : s.highs) highs->push_back(WorkItem{gi, h});
    for (int32_t h : s.cols) cols->push_back(WorkItem{gi, h});
    for (const FGroup &fg : s.fgroups) {
        size_t i = 0;
        while (i < ll.fshape.size() &&
               !(ll.fshape[i].kind == fg.kind && ll.fshape[i].a == fg.a && ll.fshape[i].b == fg.b))
            ++i;
        if (i == ll.fshape.size()) {
            FGroup sh;
            sh.kind = fg.kind;
            sh.a = fg.a;
            sh.b = fg.b;
            ll.fshape.push_back(sh);
            ll.fitems.emplace_back();
        }
        for (int32_t t : fg.tiles) ll.fitems[i].push_back(WorkItem{gi, t});
    }
}

GraphShape relay_shape(const GraphShape &s) {
    GraphShape r = s;
    r.vgroups = s.relay_vgroups;
    return r;
}

namespace {
void merge_lists(LaunchLists &ll) {
    std::vector<size_t> sq;
    for (size_t i = 0; i < ll.fshape.size(); ++i) {
        const FGroup &f = ll.fshape[i];
        if (f.kind == TK_PAIR && f.a == f.b && f.a >= 2 && f.a <= kPairStatesMax) sq.push_back(i);
    }
    if (sq.size() > 1) {
        std::vector<FGroup> shape;
        std::vector<std::vector<WorkItem>> items;
        FGroup mixed;
        mixed.kind = TK_PAIR;
        mixed.a = mixed.b = 0;
        shape.push_back(mixed);
        items.emplace_back();
        size_t k = 0;
        for (size_t i = 0; i < ll.fshape.size(); ++i) {
            if (k < sq.size() && sq[k] == i) {
                items[0].insert(items[0].end(), ll.fitems[i].begin(), ll.fitems[i].end());
                ++k;
            } else {
                shape.push_back(ll.fshape[i]);
                items.push_back(std::move(ll.fitems[i]));
            }
        }
        ll.fshape = std::move(shape);
        ll.fitems = std::move(items);
    }
    bool small = ll.vbucket.size() > 1;
    int32_t top = 0;
    for (int32_t b : ll.vbucket) {
        small = small && b <= 8;
        top = std::max(top, b);
    }
    if (small) {
        std::vector<WorkItem> all;
        for (const auto &v : ll.vitems) all.insert(all.end(), v.begin(), v.end());
        ll.vbucket.assign(1, top);
        ll.vitems.assign(1, std::move(all));
    }
}
}  // namespace

void finish_lists(LaunchLists &ll, std::vector<WorkItem> &mids, std::vector<WorkItem> &highs,
                  std::vector<WorkItem> &cols, bool merge) {
    if (merge) merge_lists(ll);
    if (mids.empty() && highs.empty() && cols.empty()) return;
    if (ll.vbucket.empty()) {
        ll.vbucket.push_back(2);
        ll.vitems.emplace_back();
    }
    ll.n_mid = (int32_t)mids.size();
    ll.n_high = (int32_t)(cols.size() + highs.size());
    std::vector<WorkItem> &v = ll.vitems[0];
    v.insert(v.end(), mids.begin(), mids.end());
    // Block b of the variable launch takes block-path item b and runs on XCD
    // b mod 8 (workgroups go to the XCDs in turn).  Column group position p
    // holds group (p mod 8) * q + p / 8 (q = n / 8; the last n mod 8 keep
    // their place), so each XCD runs a run of consecutive groups: the groups
    // that read one cache line of edge rows then share that XCD's L2.
    const int64_t n = (int64_t)cols.size(), q = n / 8;
    for (int64_t p = 0; p < n; ++p) v.push_back(cols[p < 8 * q ? (p % 8) * q + p / 8 : p]);
    v.insert(v.end(), highs.begin(), highs.end());
}

size_t lists_bytes(const LaunchLists &ll) {
    size_t b = 0;
    for (const auto &v : ll.vitems) b += align256(std::max<size_t>(1, v.size()) * sizeof(WorkItem));
    for (const auto &v : ll.fitems) b += align256(std::max<size_t>(1, v.size()) * sizeof(WorkItem));
    return b;
}

// The lists' work items sit one 256-aligned run per launch: variable
// launches, then factor launches.
void describe_lists(const LaunchLists &ll, char *mem, std::vector<Launch> *vl, std::vector<Launch> *fl) {
    vl->clear();
    fl->clear();
    size_t off = 0;
    for (size_t i = 0; i < ll.vitems.size(); ++i) {
        const auto &v = ll.vitems[i];
        Launch L{-1, ll.vbucket[i], 0, 0, (WorkItem *)(mem + off)};
        L.n_mid = i == 0 ? ll.n_mid : 0;
        L.n_high = i == 0 ? ll.n_high : 0;
        L.n = (int32_t)v.size() - L.n_mid - L.n_high;
        vl->push_back(L);
        off += align256(std::max<size_t>(1, v.size()) * sizeof(WorkItem));
    }
    for (size_t i = 0; i < ll.fitems.size(); ++i) {
        const auto &v = ll.fitems[i];
        fl->push_back(Launch{ll.fshape[i].kind, ll.fshape[i].a, ll.fshape[i].b, (int32_t)v.size(),
                             (WorkItem *)(mem + off)});
        off += align256(std::max<size_t>(1, v.size()) * sizeof(WorkItem));
    }
}

void pack_lists(const LaunchLists &ll, char *host) {
    size_t off = 0;
    for (const auto *lists : {&ll.vitems, &ll.fitems})
        for (const auto &v : *lists) {
            if (!v.empty()) std::memcpy(host + off, v.data(), sizeof(WorkItem) * v.size());
            off += align256(std::max<size_t>(1, v.size()) * sizeof(WorkItem));
        }
}

hipError_t upload_lists(const LaunchLists &ll, char *mem, hipStream_t st, std::vector<Launch> *vl,
                        std::vector<Launch> *fl) {
    describe_lists(ll, mem, vl, fl);
    hipError_t e = hipSuccess;
    for (const auto *ls : {vl, fl})
        for (size_t i = 0; i < ls->size() && e == hipSuccess; ++i) {
            const Launch &L = (*ls)[i];
            const auto &v = ls == vl ? ll.vitems[i] : ll.fitems[i];
            if (!v.empty())
                e = hipMemcpyAsync(L.items, v.data(), sizeof(WorkItem) * v.size(), hipMemcpyHostToDevice, st);
        }
    return e;
}

hipError_t launch_iteration(const DevGraph *gs, const std::vector<Launch> &vl, const std::vector<Launch> &fl,
                            const TParams &P, bool maxp, hipStream_t st, int phases, bool relay) {
    hipError_t e = hipSuccess;
    if (phases & 1)
        for (const Launch &L : vl) {
            e = launch_belief(gs, L.items, L.n, L.n_mid, L.n_high, L.a, L.shape, st);
            if (e != hipSuccess) return e;
        }
    if (phases & 2)
        for (const Launch &L : fl) {
            switch (L.kind) {
            case TK_PAIR: e = launch_pair(gs, L.items, L.n, L.a, L.b, maxp, P, L.shape, st); break;
            case TK_LOGL: e = launch_logical(gs, L.items, L.n, false, maxp, P, L.shape, st, relay); break;
            case TK_LOGW: e = launch_logical(gs, L.items, L.n, true, maxp, P, L.shape, st, relay); break;
            default: e = launch_gen(gs, L.items, L.n, maxp, P, L.a, st); break;
            }
            if (e != hipSuccess) return e;
        }
    return e;
}

hipError_t launch_fused(const DevGraph *view, const std::vector<Launch> &fl, const TParams &P, bool maxp,
                        hipStream_t st) {
    hipError_t e = hipSuccess;
    // no launch before every one is known to have a fused form
    for (const Launch &L : fl)
        if (L.kind != TK_PAIR && (L.kind != TK_GEN || L.a >= 0)) return hipErrorInvalidValue;
    for (const Launch &L : fl) {
        e = L.kind == TK_PAIR ? launch_pair(view, L.items, L.n, L.a, L.b, maxp, P, L.fshape, st, true, L.halves())
                              : launch_gen(view, L.items, L.n, maxp, P, L.a, st, true);
        if (e != hipSuccess) break;
    }
    return e;
}

hipError_t launch_loop(const DevGraph *gs, const DevGraph *fused, const std::vector<Launch> &vl,
                       const std::vector<Launch> &fl, int32_t iters, const TParams &P, bool maxp, hipStream_t st,
                       int32_t fused_stride, const std::vector<Launch> *relay) {
    hipError_t e = hipSuccess;
    int32_t it = 0;
    if (fused && relay)
        for (; it + 1 < iters && e == hipSuccess; it += 2)
            for (int h = 0; h < 2 && e == hipSuccess; ++h)
                e = launch_iteration(fused + h * fused_stride, *relay, fl, P, maxp, st, 3, true);
    else if (fused)
        for (; it + 1 < iters && e == hipSuccess; it += 2)
            for (int h = 0; h < 2 && e == hipSuccess; ++h)
                e = launch_fused(fused + h * fused_stride, fl, P, maxp, st);
    for (; it < iters && e == hipSuccess; ++it) e = launch_iteration(gs, vl, fl, P, maxp, st);
    return e;
}

// ------------------------------------------------------------ captured loops
namespace {
constexpr size_t kMaxCachedLoops = 4;
}

void destroy_loops(std::vector<CachedLoop> &v) {
    for (CachedLoop &c : v) (void)hipGraphExecDestroy(c.exec);
    v.clear();
}

hipError_t run_loop(lbp_ctx *ctx, std::vector<CachedLoop> &cache, const DevGraph *gs, const DevGraph *fused,
                    const std::vector<Launch> &vl, const std::vector<Launch> &fl, int32_t iters, float d, float T,
                    int32_t fused_stride, const std::vector<Launch> *relay) {
    const TParams P = make_params(d, T);
    const bool maxp = T == 0.0f;
    const size_t per_iter = vl.size() + fl.size();
    if (!ctx->use_graphs || iters < 2 || per_iter == 0)
        return launch_loop(gs, fused, vl, fl, iters, P, maxp, ctx->stream, fused_stride, relay);
    for (const CachedLoop &c : cache)
        if (c.iters == iters && c.d == d && c.T == T) return hipGraphLaunch(c.exec, ctx->stream);
    if (!ctx->capture) {
        hipError_t e = hipStreamCreateWithFlags(&ctx->capture, hipStreamNonBlocking);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return e;
    hipError_t le = launch_loop(gs, fused, vl, fl, iters, P, maxp, ctx->capture, fused_stride, relay);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(ctx->capture, &graph);
    if (le != hipSuccess || e != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return le != hipSuccess ? le : e;
    }
    hipGraphExec_t exec = nullptr;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return e;
    if (cache.size() >= kMaxCachedLoops) {
        (void)hipGraphExecDestroy(cache.front().exec);
        cache.erase(cache.begin());
    }
    cache.push_back(CachedLoop{iters, d, T, exec});
    return hipGraphLaunch(exec, ctx->stream);
}

// ------------------------------------------------------------ graph memory
namespace {

struct Piece {
    const void *src;
    size_t bytes;
    size_t off;
};

// The pieces of one graph's allocation in a fixed order (shared by the size
// query, the host image and the upload): the pieces with host data first,
// then the pieces that start as zeros.
struct GraphPieces {
    std::vector<Piece> p;
    size_t total = 0;
    size_t faff;
    bool raw = false;       // the image holds the raw evidence and tables; panels are scattered on the device
    size_t rev = 0, rlp = 0;
    size_t base = 0;        // device offset where the host image starts (after the raw potentials)
    size_t m, B, th, phi, ft, fvb, fvar, vt, ve, vns, hv, he, gc, gr, em, es, vs, vn, vx, fp, lp, fl, dg, q, map, items;
    size_t m2 = 0, fdg = 0, fr = 0, ritems = 0;
    size_t data_end = 0;
    bool fused;
    bool relay;          // with the second message buffer and views of relay iterations
    LaunchLists ll, rll;  // the launches, and relay iterations'

    GraphPieces(const HostLayout &L, bool with_fused)
        : fused(with_fused && (L.fusable || L.tri_fusable)), relay(with_fused && !L.frelay.empty()) {
        auto add = [&](const void *src, size_t bytes) {
            p.push_back(Piece{src, bytes, total});
            total += align256(std::max<size_t>(bytes, 4));
            return p.size() - 1;
        };
        // A layout compiled with its panels carries them in the image.  One
        // compiled without them (the server's preparation threads) carries the
        // evidence as given instead, the tables as given come from a buffer
        // of their own, and graph_create scatters both into panels that
        // start as zeros: the device does the transpose.
        raw = L.theta_panel.size() != (size_t)L.VB || L.phi_panel.size() != (size_t)L.P;
        if (raw) {
            rlp = add(nullptr, sizeof(float) * L.Tn);  // copied from the caller's buffer, not the image
            base = total;
            rev = add(nullptr, sizeof(float) * L.VS);  // written by graph_fill_image
        } else {
            th = add(L.theta_panel.data(), sizeof(float) * L.VB);
            phi = add(L.phi_panel.data(), sizeof(float) * L.P);
        }
        ft = add(L.ftile.data(), sizeof(FTile) * L.ftile.size());
        fvb = add(L.fvb.data(), sizeof(int32_t) * L.fvb.size());
        fvar = add(L.fvar.data(), sizeof(int32_t) * L.fvar.size());
        faff = add(L.faff.data(), sizeof(int32_t) * L.faff.size());
        vt = add(L.vtile.data(), sizeof(VTile) * L.vtile.size());
        ve = add(L.vedge.data(), sizeof(int32_t) * L.vedge.size());
        vns = add(L.vns.data(), sizeof(int32_t) * L.vns.size());
        hv = add(L.hvar.data(), sizeof(HVar) * L.hvar.size());
        he = add(L.hedge.data(), sizeof(int32_t) * L.hedge.size());
        gc = add(L.gcls.data(), sizeof(GenClass) * L.gcls.size());
        gr = add(L.grows.data(), L.grows.size());
        em = add(L.edge_maddr.data(), sizeof(int32_t) * L.edge_maddr.size());
        es = add(L.es_off.data(), sizeof(int64_t) * L.es_off.size());
        vs = add(L.vs_off.data(), sizeof(int64_t) * L.vs_off.size());
        vn = add(L.vn.data(), sizeof(int32_t) * L.vn.size());
        vx = add(L.vext.data(), sizeof(int32_t) * L.vext.size());
        fp = add(L.fac_phi.data(), sizeof(int32_t) * L.fac_phi.size());
        lp = add(L.lp_off.data(), sizeof(int64_t) * L.lp_off.size());
        fr = add(L.frelay.data(), sizeof(int32_t) * L.frelay.size());
        const GraphShape s{L.fgroups, L.vgroups, L.mids, L.highs, L.cols, L.relay_vgroups};
        auto lists = [](const GraphShape &shape, LaunchLists *out) {
            std::vector<WorkItem> mids, highs, cols;
            add_to_lists(*out, 0, shape, &mids, &highs, &cols);
            finish_lists(*out, mids, highs, cols);
        };
        lists(s, &ll);
        items = add(nullptr, lists_bytes(ll));  // packed by pack_lists
        if (!L.frelay.empty()) {
            lists(relay_shape(s), &rll);
            ritems = add(nullptr, lists_bytes(rll));
        }
        dg = add(nullptr, sizeof(DevGraph));    // written into the image by graph_create
        data_end = total;  // everything above is copied from the host image, everything below starts zero
        m = add(nullptr, sizeof(float) * L.M);
        B = add(nullptr, sizeof(float) * L.VB);
        fl = add(nullptr, sizeof(int32_t) * 4);
        if (raw) {
            th = add(nullptr, sizeof(float) * L.VB);
            phi = add(nullptr, sizeof(float) * L.P);
        }
        q = add(nullptr, sizeof(float) * L.VS);
        map = add(nullptr, sizeof(int32_t) * L.V);
        if (fused || relay) {
            m2 = add(nullptr, sizeof(float) * L.M);
            fdg = add(nullptr, sizeof(DevGraph) * 2);
        }
    }
};

}  // namespace

size_t graph_device_bytes(const HostLayout &L, bool with_fused) { return GraphPieces(L, with_fused).total; }

size_t graph_image_bytes(const HostLayout &L) {
    GraphPieces gp(L, false);
    return gp.data_end - gp.base;
}

int graph_fill_image(const HostLayout &L, char *image, const lbp_graph_desc *d) {
    GraphPieces gp(L, false);
    // pieces are placed by device offset; the image starts at gp.base (every
    // piece written here lies at or above it)
    auto at = [&](size_t off) { return image + (off - gp.base); };
    for (const Piece &p : gp.p)
        if (p.src && p.bytes) std::memcpy(at(p.off), p.src, p.bytes);
    pack_lists(gp.ll, at(gp.p[gp.items].off));
    if (!L.frelay.empty()) pack_lists(gp.rll, at(gp.p[gp.ritems].off));
    if (!gp.raw) return LBP_OK;
    // the evidence as given (graph_create scatters it into its panel)
    if (!d) return set_error(LBP_E_INVALID, "graph image: the layout has no panels and no description was given");
    float *ev = (float *)at(gp.p[gp.rev].off);
    if (d->evidence) std::memcpy(ev, d->evidence, sizeof(float) * L.VS);
    else std::memset(ev, 0, sizeof(float) * L.VS);
    return LBP_OK;
}

int graph_create(lbp_ctx *ctx, const HostLayout &L, bool with_fused, char *mem, hipStream_t st, lbp_graph **out,
                 char *image, bool wait, const float *raw_lp) {
    lbp_graph *g = nullptr;
    char *own_image = nullptr;  // built here when the caller brings none
    try {
        GraphPieces gp(L, with_fused);
        g = new lbp_graph;
        g->ctx = ctx;
        if (mem) {
            g->dmem = mem;
            g->owns_memory = false;
        } else {
            hipError_t e = hipMalloc((void **)&g->dmem, gp.total);
            if (e != hipSuccess && (gp.relay || (gp.fused && !L.fusable))) {
                // no room for the second message buffer, which these forms can do without
                (void)hipGetLastError();
                gp = GraphPieces(L, false);
                e = hipMalloc((void **)&g->dmem, gp.total);
            }
            if (e != hipSuccess) {
                delete g;
                (void)hipGetLastError();
                return set_error(LBP_E_OOM, "device allocation of " + std::to_string(gp.total) + " bytes failed");
            }
        }
        g->dbytes = gp.total;
        auto ptr = [&](size_t i) { return (void *)(g->dmem + gp.p[i].off); };
        if (gp.raw && (!image || (L.Tn > 0 && !raw_lp))) {
            if (g->owns_memory) (void)hipFree(g->dmem);
            delete g;
            return set_error(LBP_E_INVALID, "graph_create: a layout without panels needs its image and potentials");
        }
        if (!image) {
            wait = true;  // the image built here is freed before returning
            own_image = (char *)panel_alloc(gp.data_end);
            if (!own_image) throw std::bad_alloc();
            graph_fill_image(L, own_image, nullptr);  // compiled with its panels: cannot fail
            image = own_image;
        }
        DevGraph &h = g->host;
        h.m = (float *)ptr(gp.m);
        h.mo = h.m;
        h.B = (float *)ptr(gp.B);
        h.theta = (float *)ptr(gp.th);
        h.phi = (float *)ptr(gp.phi);
        h.ftile = (const FTile *)ptr(gp.ft);
        h.fvb = (const int32_t *)ptr(gp.fvb);
        h.fvar = (const int32_t *)ptr(gp.fvar);
        h.faff = (const int32_t *)ptr(gp.faff);
        h.vtile = (const VTile *)ptr(gp.vt);
        h.vedge = (const int32_t *)ptr(gp.ve);
        h.vns = (const int32_t *)ptr(gp.vns);
        h.hvar = (const HVar *)ptr(gp.hv);
        h.hedge = (const int32_t *)ptr(gp.he);
        h.gcls = (const GenClass *)ptr(gp.gc);
        h.grows = (const uint8_t *)ptr(gp.gr);
        h.edge_maddr = (const int32_t *)ptr(gp.em);
        h.es_off = (const int64_t *)ptr(gp.es);
        h.vs_off = (const int64_t *)ptr(gp.vs);
        h.vn = (const int32_t *)ptr(gp.vn);
        h.vext = L.vext.empty() ? nullptr : (const int32_t *)ptr(gp.vx);
        h.fac_phi = (const int32_t *)ptr(gp.fp);
        h.lp_off = (const int64_t *)ptr(gp.lp);
        h.flag = (int32_t *)ptr(gp.fl);
        h.frelay = L.frelay.empty() ? nullptr : (const int32_t *)ptr(gp.fr);
        h.V = (int32_t)L.V;
        h.E = (int32_t)L.E;
        h.F = (int32_t)L.F;
        h.zero_addr = L.zero_addr;
        h.raw_msgs = 0;
        g->dgraph = (DevGraph *)ptr(gp.dg);
        g->q_tmp = (float *)ptr(gp.q);
        g->map_tmp = (int32_t *)ptr(gp.map);
        // the descriptor travels in the image: one copy of every host piece
        // (a single DMA when the image is page-locked), one fill for
        // messages, beliefs, flag and scratch
        std::memcpy(image + (gp.p[gp.dg].off - gp.base), &g->host, sizeof(DevGraph));
        hipError_t e = hipSuccess;
        if (gp.raw && L.Tn > 0)
            e = hipMemcpyAsync(ptr(gp.rlp), raw_lp, sizeof(float) * L.Tn, hipMemcpyHostToDevice, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(g->dmem + gp.base, image, gp.data_end - gp.base, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipMemsetAsync(g->dmem + gp.data_end, 0, gp.total - gp.data_end, st);
        if (gp.raw && e == hipSuccess) {  // panels from the raw evidence and tables of the image
            e = launch_evidence_in(g->dgraph, (int)L.V, (const float *)ptr(gp.rev), st);
            if (e == hipSuccess) e = launch_logpot_in(g->dgraph, (int)L.F, (const float *)ptr(gp.rlp), st);
        }
        DevGraph fv[2];
        if (gp.fused || gp.relay) {
            float *m2 = (float *)ptr(gp.m2);
            fv[0] = g->host;
            fv[0].mo = m2;
            fv[1] = g->host;
            fv[1].m = m2;
            fv[1].mo = g->host.m;
            DevGraph *views = (DevGraph *)ptr(gp.fdg);
            (gp.relay ? g->relay : L.fusable ? g->fused : g->tri) = views;
            g->m2 = m2;
            if (e == hipSuccess) e = hipMemcpyAsync(views, fv, sizeof(fv), hipMemcpyHostToDevice, st);
        }
        describe_lists(gp.ll, (char *)ptr(gp.items), &g->vl, &g->fl);
        bool four = L.fusable;
        for (const VTile &vt : L.vtile) four = four && vt.kmax <= 4;
        for (Launch &x : g->fl) x.half = four;
        if (gp.relay) {
            std::vector<Launch> fl;  // the factor launches are the same
            describe_lists(gp.rll, (char *)ptr(gp.ritems), &g->relay_vl, &fl);
        }
        // the host image and the descriptors must outlive the copies (the
        // descriptors live in g; without wait, the caller keeps the image)
        if (e == hipSuccess && (wait || gp.fused || gp.relay)) e = hipStreamSynchronize(st);
        if (e != hipSuccess) (void)hipStreamSynchronize(st);  // no copy may still read an image
        panel_free(own_image);
        own_image = nullptr;
        if (e != hipSuccess) {
            if (g->owns_memory) (void)hipFree(g->dmem);
            delete g;
            return hip_error(e, "graph upload");
        }
        g->shape = GraphShape{L.fgroups, L.vgroups, L.mids, L.highs, L.cols, L.relay_vgroups};
        for (const FGroup &fg : L.fgroups)
            if (fg.kind == TK_LOGL || fg.kind == TK_LOGW) g->has_logical = true;
        g->fusable = L.fusable;
        g->V = L.V; g->VS = L.VS; g->F = L.F; g->E = L.E; g->ES = L.ES; g->Tn = L.Tn;
        g->M = L.M; g->VB = L.VB; g->P = L.P;
        g->nvt = (int32_t)L.vtile.size();
        make_pair_solve(L, solve_lds_limit(ctx->device) / 4, &g->small);
        g->resident_ok = make_solve_plan(g->vl, g->fl, L, solve_lds_limit(ctx->device) / 4, &g->plan);
        *out = g;
        return LBP_OK;
    } catch (const std::bad_alloc &) {
        panel_free(own_image);
        if (g) {
            if (g->dmem && g->owns_memory) (void)hipFree(g->dmem);
            delete g;
        }
        return set_error(LBP_E_OOM, "host allocation failed");
    }
}

bool make_solve_plan(const std::vector<Launch> &vl, const std::vector<Launch> &fl, const HostLayout &L,
                     int64_t limit_words, SolvePlan *plan) {
    static_assert(sizeof(VTile) == 16 && sizeof(FTile) == 32 && sizeof(HVar) == 16, "4-byte-word structs");
    const int64_t w[SA_COUNT] = {L.M, L.VB, (int64_t)L.vedge.size(), (int64_t)L.fvb.size(), (int64_t)L.hedge.size(),
                                 (int64_t)L.vns.size(), 4 * (int64_t)L.vtile.size(), 8 * (int64_t)L.ftile.size(),
                                 4 * (int64_t)L.hvar.size(), L.VB, L.P};
    if (L.M <= 0 || L.VB <= 0 || solve_words_aligned(w[SA_M]) + solve_words_aligned(w[SA_B]) > limit_words ||
        vl.size() + fl.size() > (size_t)kSolveLaunchesMax)
        return false;
    SolvePlan p;
    int64_t used = 0;
    for (int a = 0; a < SA_COUNT; ++a) {
        p.words[a] = (int32_t)w[a];
        if (used + solve_words_aligned(w[a]) <= limit_words) {
            p.lds_mask |= 1u << a;
            used += solve_words_aligned(w[a]);
        }
    }
    p.lds_words = (int32_t)used;
    for (const Launch &x : vl) {
        if (x.n_high != 0) return false;
        p.l[p.nv++] = SolveLaunch{-1, x.a, 0, x.n, x.n_mid, 0, x.items};
    }
    for (const Launch &x : fl) {
        if (x.kind != TK_PAIR && x.kind != TK_LOGL) return false;
        p.l[p.nv + p.nf++] = SolveLaunch{x.kind, x.a, x.b, x.n, 0, 0, x.items};
    }
    *plan = p;
    return true;
}

bool make_pair_solve(const HostLayout &L, int64_t limit_words, PairSolve *plan) {
    *plan = PairSolve{};
    if (L.fgroups.size() != 1 || L.fgroups[0].kind != TK_PAIR || L.fgroups[0].a != L.fgroups[0].b ||
        L.fgroups[0].a > kPairStatesMax || !L.highs.empty() || !L.cols.empty() ||
        L.mids.size() != L.hvar.size() || L.fgroups[0].tiles.size() != L.ftile.size())
        return false;
    PairSolve S;
    S.n = L.fgroups[0].a;
    const int64_t nt = (int64_t)L.ftile.size(), nvt = (int64_t)L.vtile.size(), nmid = (int64_t)L.hvar.size();
    const int64_t maxw = kPairSolveThreads / 64, B = L.VB - (int64_t)kLanes * kMaxStates;  // without the spare panel
    if (nt > maxw * pair_solve_tiles_per_wave(S.n) || nvt > 2 * maxw || nmid > 4096 || L.M >= 65536) return false;
    S.ntiles = (int32_t)nt;
    S.nvt = (int32_t)nvt;
    S.nmid = (int32_t)nmid;
    // a wavefront per tile while there are that many
    const int64_t w = std::max({(nt + pair_solve_tiles_per_wave(S.n) - 1) / pair_solve_tiles_per_wave(S.n),
                                std::min(maxw, nt), (nvt + 1) / 2, std::min(maxw, (nmid + 3) / 4), int64_t(1)});
    S.waves = (int32_t)std::min(maxw, w);
    S.M = (int32_t)L.M;
    S.B = (int32_t)B;
    S.zero = L.zero_addr;
    S.maxdeg = 0;
    for (const VTile &vt : L.vtile) S.maxdeg = std::max(S.maxdeg, vt.kmax);
    S.vedge = S.maxdeg > 4 ? (int32_t)L.vedge.size() : 0;
    S.lds = pair_solve_lds(S);
    S.lds_limit = (int32_t)limit_words;
    if (S.lds > S.lds_limit) return false;
    *plan = S;
    return true;
}

// Where one workgroup beats launched iterations.  Max-product: wherever the
// graph fits (slowest seen: a 64 x 64 bipartite layer, 4.2 against 4.5 us per
// iteration; Potts 22 x 22, 8 states 2.3 against 5.4).  Sums: the workgroup's
// cycles, estimated from the busiest SIMD's factor tiles (per table entry an
// add, a subtraction, a multiplication, an exponential and an add, exponentials
// at a quarter of the rate; the rows' damping) and variable sums, 3400 of them
// a us as measured, against what the graph's launched iterations take whatever
// the size of a small graph: 4.4 us and 0.35 more per state above two in two
// launches, 2.5 and 0.32 where fused ones are in use (variables of at most
// four edges, the lane's serial chain; of two, 0.23; fused iterations of more
// edges take 7 us and up).  Near a tie with fused ones the workgroup is taken
// (2.8 and 0.27 or 0.16 in the rule): a replay starts 2 us later than one
// launch, and a new graph's first run captures its loop (24 recorded iterations
// of a 32 x 32 grid of three states in three segments, with the reverse sweep:
// 459 us on a new graph in one workgroup, 615 in captured loops).  Measured at
// T = 1, two-phase / fused / this (- no such form): Ising 42 x 42 4.6 / 2.6 / 2.4, 45 x 45 4.8 / 2.4 / 2.7; Potts
// 32 x 32, 3 states 4.9 / 2.7 / 2.8; 23 x 23, 4 states 5.2 / 3.1 / 2.8,
// 26 x 26 5.1 / 3.1 / 3.4; 22 x 22, 5 states 5.7 / 3.4 / 3.3; 18 x 18, 6 states
// 6.0 / 3.7 / 3.5, 20 x 20 6.1 / 3.7 / 4.4; 16 x 16, 7 states 6.6 / 4.0 / 3.3,
// 18 x 18 6.6 / 4.1 / 4.6; 16 x 16, 8 states 7.2 / 4.4 / 4.1; chains of 500
// variables, 6 states 5.3 / 3.3 / 2.5, of 700 5.3 / 3.3 / 3.5; bipartite
// 56 x 56 4.4 / - / 3.5.
static bool pair_solve_wins(const PairSolve &S, bool maxp, bool fused) {
    if (maxp) return true;
    constexpr int64_t kCyclesPerUs = 3400;
    const int64_t n = S.n, tiles = (S.ntiles + 3) / 4, vts = (S.nvt + 3) / 4, mids = (S.nmid + 15) / 16;
    const int64_t tile = 4 * (2 * n * n * 5 + 24 * n) + 16 * (2 * n * n + 2 * n);
    const int64_t cycles = tiles * tile + vts * 4 * n * (6 + 2 * S.maxdeg) + mids * 4 * (60 + 60 * n) + 1000;
    const int64_t launched_ns = fused && S.maxdeg <= 4 ? 2800 + (S.maxdeg <= 2 ? 160 : 270) * (n - 2)
                                                      : 4400 + 350 * (n - 2);
    return cycles * 1000 < kCyclesPerUs * launched_ns;
}

// Fused iterations of three-way graphs gather each variable's messages once
// per factor that touches it, which pays while they sit in L2 and the second
// launch is a good part of an iteration.  Two-phase / fused, us per iteration
// at T = 1 and T = 0 (tiles in brackets): three states, 256 x 256 (2080)
// 10.3 / 9.3 and 8.9 / 8.1, 300 x 300 (2900) 13.0 / 12.1 and 11.0 / 11.1,
// 350 x 350 (3900) 15.8 / 15.1 and 13.7 / 14.1, 400 x 400 17.6 / 18.3; four
// states, 256 x 256 16.3 / 15.5 and 13.5 / 12.5, 200 x 200 (1290) 9.8 / 10.1 at
// T = 0; two states, 500 x 500 (8050) 12.9 / 12.7 and 12.4 / 12.0.
static bool tri_fused_wins(const std::vector<Launch> &fl, bool maxp) {
    for (const Launch &L : fl) {
        const int32_t most = L.a == -2 ? 8192 : L.a == -3 ? (maxp ? 2500 : 4000) : (maxp ? 1000 : 2500);
        if (L.n > most) return false;
    }
    return true;
}

bool runs_small(const lbp_graph *g, int32_t iters, float T) {
    if (!g->automatic || !g->small.n || iters < 2) return false;
    const int8_t timed = g->small_timed[T == 0.0f];
    return timed >= 0 ? timed != 0 : pair_solve_wins(g->small, T == 0.0f, g->use_fused);
}

const DevGraph *loop_views(const lbp_graph *g, float T) {
    if (g->use_fused) return g->fused;
    if (!g->automatic) return nullptr;
    if (g->relay) return g->relay;
    return g->tri && tri_fused_wins(g->fl, T == 0.0f) ? g->tri : nullptr;
}

static const std::vector<Launch> *loop_relay(const lbp_graph *g) {
    return g->relay && g->automatic ? &g->relay_vl : nullptr;
}

hipError_t run_graph(lbp_graph *g, int32_t iters, float d, float T) {
    if (runs_small(g, iters, T)) {
        const hipError_t e =
            launch_solve_pair(g->dgraph, g->small, iters, T == 0.0f, make_params(d, T), g->ctx->stream);
        if (e == hipSuccess) return e;
        (void)hipGetLastError();  // refused (LDS size): launched iterations from here on
        g->small.n = 0;
    }
    return run_loop(g->ctx, g->loops, g->dgraph, loop_views(g, T), g->vl, g->fl, iters, d, T, 1, loop_relay(g));
}

// A check on a two-phase path costs a copy of the messages, two launches, the
// residual's two and a copy back to the host; with fused views the last
// iteration is fused too and the second buffer is the copy, and the result is
// written where the host reads it: Potts 128 x 128 with 5 states, checked every
// 10 iterations until settled, 374 -> 273 us a solve.
hipError_t run_graph_residual(lbp_graph *g, int32_t iters, float d, float T, float *mprev, float *partial, float *out) {
    hipStream_t st = g->ctx->stream;
    const DevGraph *views = loop_views(g, T);
    const std::vector<Launch> *relay = loop_relay(g);
    // (below two iterations a small graph is not in one workgroup anyway)
    if (views && !runs_small(g, iters, T)) {
        if (iters % 2 == 0) {
            // pairs of fused iterations: the last wrote the messages from the
            // second buffer, which still holds the iterate before
            hipError_t e = run_loop(g->ctx, g->loops, g->dgraph, views, g->vl, g->fl, iters, d, T, 1, relay);
            return e == hipSuccess ? launch_residual(g->dgraph, (int)g->E, g->m2, partial, out, st) : e;
        }
        hipError_t e = hipSuccess;
        if (iters > 1) e = run_loop(g->ctx, g->loops, g->dgraph, views, g->vl, g->fl, iters - 1, d, T, 1, relay);
        const TParams P = make_params(d, T);
        if (e == hipSuccess)  // one more, into the second buffer, and from there back
            e = relay ? launch_iteration(views, *relay, g->fl, P, T == 0.0f, st, 3, true)
                      : launch_fused(views, g->fl, P, T == 0.0f, st);
        if (e == hipSuccess) e = launch_residual(g->dgraph, (int)g->E, g->m2, partial, out, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(g->host.m, g->m2, sizeof(float) * g->M, hipMemcpyDeviceToDevice, st);
        return e;
    }
    hipError_t e = iters > 1 ? run_graph(g, iters - 1, d, T) : hipSuccess;
    if (e == hipSuccess) e = hipMemcpyAsync(mprev, g->host.m, sizeof(float) * g->M, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = run_loop(g->ctx, g->loops, g->dgraph, nullptr, g->vl, g->fl, 1, d, T);
    return e == hipSuccess ? launch_residual(g->dgraph, (int)g->E, mprev, partial, out, st) : e;
}

void graph_destroy(lbp_graph *g) {
    if (!g) return;
    destroy_loops(g->loops);
    if (g->conv) (void)hipFree(g->conv);
    if (g->residual) (void)hipHostFree(g->residual);
    if (g->adj.dmem && g->adj.owns_memory) (void)hipFree(g->adj.dmem);
    if (g->owns_memory) (void)hipFree(g->dmem);
    delete g;
}

int graph_readout(lbp_graph *g, float *q, int normalized, int32_t *map, bool on_device, hipStream_t st) {
    const TParams P = make_params(0.5f, g->last_T);
    const bool maxp = g->last_T == 0.0f;
    hipError_t e = launch_iteration(g->dgraph, g->vl, g->fl, P, maxp, st, 1);
    if (e != hipSuccess) return hip_error(e, "belief launch");
    float *qd = q ? (on_device ? q : g->q_tmp) : nullptr;
    int32_t *md = map ? (on_device ? map : g->map_tmp) : nullptr;
    HIP_TRY(launch_readout(g->dgraph, g->nvt, maxp, P, qd, normalized, md, st));
    if (on_device) return LBP_OK;
    if (q) HIP_TRY(hipMemcpyAsync(q, g->q_tmp, sizeof(float) * g->VS, hipMemcpyDeviceToHost, st));
    if (map) HIP_TRY(hipMemcpyAsync(map, g->map_tmp, sizeof(int32_t) * g->V, hipMemcpyDeviceToHost, st));
    return LBP_OK;
}

// ------------------------------------------------------------ reverse sweep
namespace {

struct AdjLayout {
    size_t ck, seg, A, nb, Bb, Bt, z, tb, pb, v, total;
    AdjLayout(size_t M, size_t VB, size_t P, int32_t nseg, int32_t k) {
        size_t off = 0;
        auto take = [&](size_t bytes) {
            size_t o = off;
            off += align256(std::max<size_t>(bytes, 4));
            return o;
        };
        ck = take(sizeof(float) * M * std::max(nseg, 1));
        seg = take(sizeof(float) * M * k);
        A = take(sizeof(float) * M);
        nb = take(sizeof(float) * M);
        Bb = take(sizeof(float) * VB);
        Bt = take(sizeof(float) * VB);
        z = take(sizeof(float) * VB);
        tb = take(sizeof(float) * VB);
        pb = take(sizeof(float) * P);
        v = take(sizeof(DevGraph) * (k + 2));
        total = off;
    }
};

void record_shape(int32_t iters, int32_t ckpt_every, int32_t *k, int32_t *nseg) {
    *k = std::min<int32_t>(ckpt_every, std::max<int32_t>(iters, 1));
    *nseg = (iters + *k - 1) / *k;
}

}  // namespace

size_t adjoint_bytes(int64_t M, int64_t VB, int64_t P, int32_t iters, int32_t ckpt_every) {
    int32_t k, nseg;
    record_shape(iters, ckpt_every, &k, &nseg);
    return AdjLayout((size_t)M, (size_t)VB, (size_t)P, nseg, k).total;
}

int adjoint_prepare(lbp_graph *g, int32_t iters, float d, float T, int32_t ckpt_every, char *mem, hipStream_t st,
                    std::vector<DevGraph> *staging) {
    auto &J = g->adj;
    J.valid = false;
    int32_t k, nseg;
    record_shape(iters, ckpt_every, &k, &nseg);
    const AdjLayout al((size_t)g->M, (size_t)g->VB, (size_t)g->P, nseg, k);
    if (mem) {
        if (J.dmem && J.owns_memory) {
            HIP_TRY(hipStreamSynchronize(st));
            (void)hipFree(J.dmem);
        }
        J.dmem = mem;
        J.bytes = al.total;
        J.owns_memory = false;
    } else if (!J.owns_memory || al.total > J.bytes) {
        if (J.dmem && J.owns_memory) {
            HIP_TRY(hipStreamSynchronize(st));
            (void)hipFree(J.dmem);
        }
        J.dmem = nullptr;
        J.bytes = 0;
        J.owns_memory = true;
        hipError_t e = hipMalloc((void **)&J.dmem, al.total);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            J.dmem = nullptr;
            return set_error(LBP_E_OOM, "adjoint workspace of " + std::to_string(al.total) + " bytes");
        }
        J.bytes = al.total;
    }
    const size_t M = (size_t)g->M, VB = (size_t)g->VB;
    J.ckpt = (float *)(J.dmem + al.ck);
    J.seg = (float *)(J.dmem + al.seg);
    J.A = (float *)(J.dmem + al.A);
    J.nbar = (float *)(J.dmem + al.nb);
    J.Bbar = (float *)(J.dmem + al.Bb);
    J.Bt = (float *)(J.dmem + al.Bt);
    J.zeros = (float *)(J.dmem + al.z);
    J.thetabar = (float *)(J.dmem + al.tb);
    J.phibar = (float *)(J.dmem + al.pb);
    J.views = (DevGraph *)(J.dmem + al.v);
    // zero panels of the iterate buffers and of nbar must read as zero
    HIP_TRY(hipMemsetAsync(J.seg, 0, sizeof(float) * M * k, st));
    HIP_TRY(hipMemsetAsync(J.nbar, 0, sizeof(float) * M, st));
    HIP_TRY(hipMemsetAsync(J.zeros, 0, sizeof(float) * VB, st));
    std::vector<DevGraph> local;
    std::vector<DevGraph> &views = staging ? *staging : local;
    views.assign(k + 2, g->host);
    for (int32_t j = 0; j < k; ++j) {
        views[j].m = J.seg + M * j;
        views[j].mo = J.seg + M * std::min(j + 1, k - 1);
        views[j].B = J.Bt;
    }
    views[k].B = J.Bt;
    views[k + 1].m = J.nbar;
    views[k + 1].mo = J.nbar;
    views[k + 1].raw_msgs = 1;  // adjoint sums, one state per panel row
    views[k + 1].theta = J.zeros;
    views[k + 1].B = J.Bbar;
    HIP_TRY(hipMemcpyAsync(J.views, views.data(), sizeof(DevGraph) * (k + 2), hipMemcpyHostToDevice, st));
    if (!staging) HIP_TRY(hipStreamSynchronize(st));  // the local staging must outlive its copy
    J.iters = iters;
    J.k = k;
    J.nseg = nseg;
    J.d = d;
    J.T = T;
    return LBP_OK;
}

int adjoint_checkpoint(lbp_graph *g, int32_t seg, hipStream_t st) {
    auto &J = g->adj;
    HIP_TRY(hipMemcpyAsync(J.ckpt + (size_t)g->M * seg, g->host.m, sizeof(float) * g->M, hipMemcpyDeviceToDevice, st));
    return LBP_OK;
}

void adjoint_finish_record(lbp_graph *g) {
    g->adj.valid = true;
    g->adj.version = g->version;
}

int adjoint_backward(lbp_graph *g, const float *grad_q, float *grad_logpot, float *grad_evidence, hipStream_t st) {
    auto &J = g->adj;
    const TParams P = make_params(J.d, J.T);
    const int64_t M = g->M;
    const int k = J.k;
    // Fused form: one launch per recomputed iteration and per reverse step.  A
    // segment's first iterate is its checkpoint itself, which leaves the first
    // iterate buffer to the second nbar.
    // (Eight states, past a wavefront per compute unit: the gathers of 256
    // messages a lane cost more than the launches. Start / fused, 20 iterations:
    // 80 x 80 742 / 644 us, 110 x 110 789 / 799, 160 x 160 over 30 iterations
    // 1264 / 1307; 250 x 250 with seven states 1159 / 1106.)
    bool fused = g->fusable && J.iters > 0;
    for (const Launch &L : g->fl)
        if (L.a >= 8 && L.n > 256) fused = false;
    float *nbar[2] = {J.nbar, J.seg};
    int cur = 0;  // the nbar written last
    AdjBufs B{J.A, J.nbar, J.Bbar, J.phibar, nullptr, J.thetabar};
    if (!fused) {
        HIP_TRY(hipMemsetAsync(J.A, 0, sizeof(float) * M, st));
        HIP_TRY(hipMemsetAsync(J.phibar, 0, sizeof(float) * g->P, st));
    }
    // read-out adjoint at the recorded final iterate (the graph's messages)
    hipError_t e = launch_iteration(J.views + k, g->vl, g->fl, P, false, st, 1);
    if (e == hipSuccess) e = launch_readout_adj(J.views + k, g->nvt, P, grad_q, J.Bbar, J.thetabar, st);
    for (int32_t sidx = J.nseg - 1; sidx >= 0 && e == hipSuccess; --sidx) {
        const int32_t len = std::min(k, J.iters - sidx * k);
        if (fused) {
            e = launch_set_messages(J.views, J.ckpt + M * sidx, st);
            for (int32_t j = 0; j + 1 < len && e == hipSuccess; ++j)
                for (const Launch &L : g->fl)
                    if (e == hipSuccess)
                        e = launch_pair(J.views + j, L.items, L.n, L.a, L.b, false, P, L.fshape, st, true, L.halves());
            for (int32_t j = len - 1; j >= 0 && e == hipSuccess; --j) {
                B.nbar = nbar[cur ^ 1];
                for (const Launch &L : g->fl)
                    if (e == hipSuccess) e = launch_pair_adj(J.views + j, L.items, L.n, L.a, L.b, P, B, st, true);
                cur ^= 1;
                B.nbar_in = nbar[cur];
            }
            continue;
        }
        e = hipMemcpyAsync(J.seg, J.ckpt + M * sidx, sizeof(float) * M, hipMemcpyDeviceToDevice, st);
        for (int32_t j = 0; j + 1 < len && e == hipSuccess; ++j)
            e = launch_iteration(J.views + j, g->vl, g->fl, P, false, st, 3);
        for (int32_t j = len - 1; j >= 0 && e == hipSuccess; --j) {
            e = launch_iteration(J.views + j, g->vl, g->fl, P, false, st, 1);  // B_t
            for (const Launch &L : g->fl) {
                if (e != hipSuccess) break;
                if (L.kind == TK_PAIR) e = launch_pair_adj(J.views + j, L.items, L.n, L.a, L.b, P, B, st);
                else e = launch_gen_adj(J.views + j, L.items, L.n, P, B, st);
            }
            if (e == hipSuccess) e = launch_iteration(J.views + k + 1, g->vl, g->fl, P, false, st, 1);  // Bbar_t
            if (e == hipSuccess) e = launch_accumulate(J.thetabar, J.Bbar, g->VB, st);
        }
    }
    if (fused && e == hipSuccess) {  // Bbar_0, from the view that sums J.nbar or its sibling over J.seg
        if (cur == 1) e = launch_set_messages(J.views + k + 1, J.seg, st);
        if (e == hipSuccess) e = launch_iteration(J.views + k + 1, g->vl, g->fl, P, false, st, 1);
        if (cur == 1 && e == hipSuccess) e = launch_set_messages(J.views + k + 1, J.nbar, st);
        if (e == hipSuccess) e = launch_accumulate(J.thetabar, J.Bbar, g->VB, st);
    }
    if (e == hipSuccess) e = launch_logpot_out(g->dgraph, (int)g->F, J.phibar, grad_logpot, st);
    if (e == hipSuccess && grad_evidence) e = launch_evidence_out(g->dgraph, (int)g->V, J.thetabar, grad_evidence, st);
    if (e != hipSuccess) return hip_error(e, "backward launch");
    return LBP_OK;
}

}  // namespace lbp
