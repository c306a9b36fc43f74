// The host runtime (bfs_host.cpp) against a HIP runtime and kernels of its own
// that only keep count: level loops, group sizes and refusals without a GPU.
// Usage: host_runtime CASE; prints what differs from what is wanted.
#include "../paper_1906_03113_amd/csrc/bfs_host.cpp"

#include <cstdlib>
#include <random>

static struct {
    uint32_t levels = 1;                    // levels the search has
    uint32_t steps = 0, past = 0;           // step launches; those after the first that reported the end
    bool restart = false;                   // a search's first launch is number 0 again
    uint32_t deep_wanted = 1;               // deep launches until the list is empty
    uint32_t deep = 0, deep_past = 0, wide = 0, narrow = 0, cw_inits = 0, ms = 0, decided = 0, conversions = 0;
    uint64_t most_vertices = 0;
} fake;

static uint32_t *slot;                      // the progress slot

// ---- the HIP runtime ------------------------------------------------------------------------
extern "C" {
hipError_t hipMalloc(void **p, size_t b) { *p = aligned_alloc(256, (b + 511) & ~size_t(255)); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t b, unsigned) { slot = (uint32_t *)(*p = calloc(1, b)); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t b) { memset(p, v, b); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t b, hipMemcpyKind) { memcpy(d, s, b); return hipSuccess; }
// workspaces are addresses nobody looks at; what comes back is a claim-word state
hipError_t hipMemcpyAsync(void *d, const void *, size_t b, hipMemcpyKind kind, hipStream_t) {
    if (kind != hipMemcpyDeviceToHost) return hipSuccess;
    memset(d, 0, b);
    if (b == sizeof(CwState))
        for (auto &c : ((CwState *)d)->cnt) c[0] = fake.deep < fake.deep_wanted ? 1u : 0u;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipGetLastError() { return hipSuccess; }
}

// ---- the kernels ----------------------------------------------------------------------------
namespace bfsi {
hipError_t launch_init(const LevelParams &, int32_t, const int32_t *, int32_t, hipStream_t) {
    if (fake.restart) fake.steps = 0;
    return hipSuccess;
}
hipError_t launch_level(const LevelParams &, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_step(const LevelParams &p, uint32_t, uint32_t, hipStream_t) {
    const uint32_t j = fake.steps++;
    if (j > fake.levels) {
        ++fake.past;
        return hipSuccess;
    }
    p.host_status[0] = j + 1;
    p.host_status[1] = j < fake.levels ? 1u : 0u;
    p.host_status[2] = j;
    return hipSuccess;
}
hipError_t launch_step_fold(const LevelParams &, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_parents(const LevelParams &, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_persistent(const LevelParams &, uint32_t, hipStream_t) { return hipErrorNotSupported; }
uint32_t persistent_max_grid(int) { return 0; }
hipError_t launch_sl_init(const SlParams &, int32_t, const int32_t *, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_sl_level(const SlParams &p, uint32_t, hipStream_t) {
    p.host_status[0] = 1;
    p.host_status[1] = 0;
    return hipSuccess;
}
SlLayout sl_layout(uint32_t) { return SlLayout{}; }
hipError_t static_scratch(void **) { return hipErrorNotSupported; }
hipError_t launch_ms(const MsLevel &p, MsPhase phase, uint32_t k, uint32_t, hipStream_t) {
    ++fake.ms;
    if (phase == kMsSettle || phase == kMsClose || phase == kMsRoots) {
        const uint32_t at = phase == kMsRoots ? 0u : k + 1;
        if (p.mlp != nullptr) ++fake.decided;
        if (at <= fake.levels) {
            p.host_status[0] = at;
            p.host_status[1] = at < fake.levels ? 1u : 0u;
        }
    }
    return hipSuccess;
}
hipError_t launch_ms_zero(unsigned long long *, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_ms_levels(const MsLevel &p, uint32_t planes, unsigned long long *, uint32_t, hipStream_t) {
    ++fake.conversions;
    return ms_levels_fit(p.n, planes) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_ms_out(const MsLevel &, uint32_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_ms_rpull(const MsLevel &, uint32_t, uint32_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_cw_init(const CwParams &p, hipStream_t) {
    ++fake.cw_inits;
    fake.deep = 0;
    fake.most_vertices = std::max<uint64_t>(fake.most_vertices, p.V);
    return hipSuccess;
}
hipError_t launch_cw_wide(const CwParams &, uint32_t, uint32_t, hipStream_t) { ++fake.wide; ++fake.deep; return hipSuccess; }
hipError_t launch_cw_narrow(const CwParams &, uint32_t, uint32_t, uint32_t, uint32_t, hipStream_t) { ++fake.narrow; ++fake.deep; return hipSuccess; }
hipError_t launch_cw_rows(const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_cw_deep(const CwParams &, uint32_t, uint32_t, uint32_t, bool, hipStream_t) {
    if (fake.deep >= fake.deep_wanted && ++fake.deep_past > 1u << 20) return hipErrorUnknown;   // (ends a runaway loop)
    ++fake.deep;
    return hipSuccess;
}
hipError_t launch_cw_out(const CwParams &, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_pack(const PackParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_unpack(const PackParams &, hipStream_t) { return hipSuccess; }
CmpLayout cmp_layout(int32_t) { return CmpLayout{}; }
SpLayout sp_layout(int32_t, int32_t) { return SpLayout{}; }
hipError_t launch_spmspv(const SpParams &, uint32_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_cmp_init(const CmpParams &, int32_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_cmp_step(const CmpParams &, uint32_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_mlp_forward(const float *, const float *, float *, int32_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_mlp_grad(const float *, const float *, const float *, const float *, int32_t, float, float *, float *,
                           hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_mlp_adam(float *, float *, float *, float *, int32_t, float, hipStream_t) { return hipErrorNotSupported; }
}  // namespace bfsi

// ---- the cases ------------------------------------------------------------------------------
static int bad = 0;
#define WANT(cond, ...) do { if (!(cond)) { ++bad; printf("%s: ", #cond); printf(__VA_ARGS__); printf("\n"); } } while (0)

static void *address(size_t i = 1) { return (void *)(i << 40); }      // of device memory: aligned, never read

// The step launches' host loop ends whatever levels_per_sync is, and issues no
// more than two launches past the one that finds the end.
static void steps() {
    for (uint32_t levels : {1u, 2u, 5u, 17u, 200u})
        for (int32_t n : {(int32_t)levels, 300})
            for (uint32_t per : {0u, 1u, 2u, 8u, 64u, 4096u}) {
                if (n < (int32_t)levels) continue;
                bfs_graph g;
                g.n = n;
                g.max_deg = 20;                 // not a thin graph
                fake.levels = levels;
                fake.steps = fake.past = 0;
                bfs_run_options opt{};
                opt.levels_per_sync = per;
                const bfs_status st = bfs_run(&g, 0, (int32_t *)address(2), (int32_t *)address(3), &opt, address(), size_t(1) << 40, nullptr);
                WANT(st == BFS_OK, "n %d, %u levels, levels_per_sync %u: %s", n, levels, per, bfs_last_error_detail());
                WANT(opt.levels == levels, "n %d, levels_per_sync %u: %u levels, not %u", n, per, opt.levels, levels);
                WANT(fake.past <= 2, "n %d, levels_per_sync %u: %u launches past the end", n, per, fake.past);
            }
}

static void thin(bfs_graph &g, int32_t n, uint32_t depth) {            // a road-like graph of n vertices
    g.n = n;
    g.nnz = 3u * (uint32_t)std::min(n, 1 << 29);
    g.max_deg = 4;
    g.thin_rows = (int32_t *)address(9);
    g.thin_width = 4;
    g.deep_levels = depth;
}

// A batch on a slowly growing graph runs claim-word searches side by side, as
// many as their 32-bit counts and the workspace allow, never refused for their
// number and never by the forms that launch a level at a time.
static void deep_groups() {
    for (int32_t n : {1000, 4000000, 33000000, 33554432, 40000000, 67108863, 67200000, 1 << 30, 2147480000, 2147483647})
        for (int32_t nq : {2, 64, 65, 200}) {
            bfs_graph g;
            thin(g, n, 1u << 30);
            std::vector<bfs_graph *> gs((size_t)nq, &g);
            std::vector<int32_t> src((size_t)nq, 0);
            std::vector<int32_t *> out((size_t)nq, (int32_t *)address(5));
            for (size_t bytes : {bfs_workspace_size(&g, nq, 0), size_t(1) << 50}) {
                for (uint32_t variant : {kHeuristic, kLearned}) {
                    fake.levels = fake.deep_wanted = 3;
                    fake.cw_inits = fake.wide = fake.narrow = 0;
                    fake.most_vertices = 0;
                    bfs_run_options opt{};
                    opt.variant = variant;
                    const bfs_status st = bfs_run_batch(nq, gs.data(), src.data(), out.data(), out.data(), &opt, address(), bytes, nullptr);
                    WANT(st == BFS_OK, "n %d, %d sources, %zu bytes: %s", n, nq, bytes, bfs_last_error_detail());
                    WANT(fake.wide + fake.narrow == 0, "n %d, %d sources: %u wide and %u narrow launches", n, nq, fake.wide, fake.narrow);
                    WANT(2 * fake.most_vertices + 4096 * 64 < 1ull << 32, "n %d, %d sources: %llu vertices side by side", n, nq,
                         (unsigned long long)fake.most_vertices);
                }
            }
        }
}

// The deep form's launches past the end of a search: no more than the eight
// between two reads of the count, whatever levels_per_sync is, and no more than
// by default where it asks for fewer.
static void deep_syncs() {
    for (uint32_t launches : {1u, 2u, 3u, 7u, 40u})
        for (uint32_t per : {0u, 1u, 2u, 8u, 64u, 4096u, 0xFFFFFFFFu})
            for (int32_t nq : {1, 3}) {
                if (nq == 1 && per > 4096) continue;           // refused
                bfs_graph g;
                thin(g, 1000, 500);
                std::vector<bfs_graph *> gs((size_t)nq, &g);
                std::vector<int32_t> src((size_t)nq, 0);
                std::vector<int32_t *> out((size_t)nq, (int32_t *)address(5));
                fake.deep_wanted = launches;
                fake.deep_past = 0;
                bfs_run_options opt{};
                opt.levels_per_sync = per;
                const bfs_status st = bfs_run_batch(nq, gs.data(), src.data(), out.data(), out.data(), &opt, address(), size_t(1) << 40, nullptr);
                const uint32_t most = launches <= 2 ? 1u : (launches <= 6 ? 3u : 7u);
                WANT(st == BFS_OK, "%u launches, levels_per_sync %u, %d sources: %s", launches, per, nq, bfs_last_error_detail());
                WANT(fake.deep_past <= most && (per != 1 || fake.deep_past == 0), "%u launches, levels_per_sync %u, %d sources: %u past the end", launches, per, nq,
                     fake.deep_past);
            }
}

// The planes become levels only where the words in the way fit one mask buffer,
// whatever the vertices and the levels, launches past the end among them.
static void levels_fit() {
    for (uint32_t planes = 1; planes <= kMsPlanes; ++planes)
        for (int32_t n = (1 << (planes - 1)) + 1; n < 5000; ++n)
            WANT(ms_levels_fit(n, planes), "%d vertices, %u planes", n, planes);
    WANT(!ms_levels_fit(2, 3) && !ms_levels_fit(8, 5), "too few vertices for the planes");
    for (int32_t n = 1; n <= 120; ++n)
        for (uint32_t levels = 1; levels <= (uint32_t)n; ++levels)
            for (uint32_t variant : {kPush, kPull}) {
                bfs_graph g;
                g.n = n;
                const int32_t src[2] = {0, 0};
                fake.levels = levels;
                fake.conversions = 0;
                bfs_run_options opt{};
                opt.variant = variant;
                const bfs_status st = bfs_run_batch_vm(&g, 2, src, (int32_t *)address(2), (int32_t *)address(3), &opt, address(), size_t(1) << 40, nullptr);
                WANT(st == BFS_OK && opt.levels == levels, "%d vertices, %u levels: %s", n, levels, bfs_last_error_detail());
                WANT(fake.conversions == 1, "%d vertices, %u levels: %u conversions", n, levels, fake.conversions);
            }
}

// The automatic form of a push on graphs with hubs: by the vertices and the
// entries, the list form on small ones and on medium ones of few entries.
static void sliced_choice() {
    struct Case { int32_t n; uint32_t nnz, hub; uint32_t form; };
    const Case cases[] = {
        {49151, 1400000, 9000, BFS_PUSH_LIST},   {50000, 1410000, 8000, BFS_PUSH_SLICED},   // R-MAT, 28 a vertex
        {50000, 400000, 3300, BFS_PUSH_SLICED},  {50000, 290000, 2500, BFS_PUSH_LIST},      // 8 and 6 a vertex
        {131071, 520000, 4000, BFS_PUSH_LIST},   {131071, 700000, 4000, BFS_PUSH_SLICED},
        {50000, 99998, 49999, BFS_PUSH_LIST},    {130000, 259998, 129999, BFS_PUSH_LIST},   // stars
        {60000, 119998, 30000, BFS_PUSH_LIST},                                               // a hub with a long tail
        {108900, 393000, 1000, BFS_PUSH_LIST},                                               // a grid with a hub
        {131072, 262142, 131071, BFS_PUSH_SLICED}, {1 << 20, 30000000, 30000, BFS_PUSH_SLICED},
    };
    for (const Case &c : cases) {
        bfs_graph g;
        g.n = c.n;
        g.nnz = c.nnz;
        g.max_deg = c.hub;
        g.sl_S = 1;
        g.sl_sw = 32768;
        fake.levels = 1;
        fake.steps = 0;
        bfs_run_options opt{};
        const bfs_status st = bfs_run(&g, 0, (int32_t *)address(2), (int32_t *)address(3), &opt, address(), size_t(1) << 40, nullptr);
        WANT(st == BFS_OK && opt.push_used == c.form, "%d vertices, %u entries, hub of %u: form %u, %s", c.n, c.nnz, c.hub, opt.push_used,
             bfs_last_error_detail());
    }
}

// The network is asked for the levels that the host decides on alone: from level
// 16 on a push decision covers eight levels, whose first seven closing launches
// leave no direction behind.
static void ms_decisions() {
    for (uint32_t levels : {1u, 3u, 16u, 17u, 24u, 100u}) {
        bfs_graph g;
        g.n = 5000;
        g.nnz = 100000;
        g.max_deg = 20;                         // not a thin graph
        std::vector<bfs_graph *> gs(3, &g);
        std::vector<int32_t> src(3, 0);
        std::vector<int32_t *> out(3, (int32_t *)address(5));
        fake.levels = levels;
        fake.ms = fake.decided = 0;
        bfs_run_options opt{};
        opt.variant = kLearned;
        opt.selector = (const float *)address(7);
        const bfs_status st = bfs_run_batch(3, gs.data(), src.data(), out.data(), out.data(), &opt, address(), size_t(1) << 40, nullptr);
        WANT(st == BFS_OK && opt.levels == levels, "%u levels: %u, %s", levels, opt.levels, bfs_last_error_detail());
        const uint32_t alone = std::min(levels, 16u), groups = (levels - alone + 7) / 8;
        WANT(fake.decided == 1 + alone + groups, "%u levels: the network asked %u times, not %u", levels, fake.decided, 1 + alone + groups);
    }
}

// ---- graphs for the choice of a batch's form ----
typedef std::vector<std::pair<int32_t, int32_t>> Edges;

static bfs_graph *undirected(int32_t n, const Edges &edges) {
    std::vector<int32_t> ptr((size_t)n + 1, 0), idx(2 * edges.size() + 1);
    for (auto &e : edges) ++ptr[(size_t)e.first + 1], ++ptr[(size_t)e.second + 1];
    for (int32_t v = 0; v < n; ++v) ptr[(size_t)v + 1] += ptr[(size_t)v];
    std::vector<int32_t> at(ptr.begin(), ptr.end() - 1);
    for (auto &e : edges) {
        idx[(size_t)at[(size_t)e.first]++] = e.second;
        idx[(size_t)at[(size_t)e.second]++] = e.first;
    }
    bfs_graph *g = nullptr;
    const bfs_status st = bfs_graph_create(n, ptr.data(), idx.data(), nullptr, nullptr, 0, nullptr, &g);
    WANT(st == BFS_OK, "create: %s", bfs_last_error_detail());
    return g;
}

// k random perfect matchings, each edge kept with probability p, none at the
// vertices n t / 4 when `apart`.
static bfs_graph *matchings(int32_t n, int k, double p, bool apart = false) {
    std::mt19937 r(5);
    std::uniform_real_distribution<double> u(0, 1);
    std::vector<int32_t> perm((size_t)n);
    Edges e;
    const auto alone = [&](int32_t v) { return apart && v % (n / 4) == 0; };
    for (int m = 0; m < k; ++m) {
        for (int32_t v = 0; v < n; ++v) perm[(size_t)v] = v;
        std::shuffle(perm.begin(), perm.end(), r);
        for (int32_t v = 0; v + 1 < n; v += 2)
            if (u(r) < p && !alone(perm[(size_t)v]) && !alone(perm[(size_t)v + 1])) e.push_back({perm[(size_t)v], perm[(size_t)v + 1]});
    }
    return undirected(n, e);
}

static bfs_graph *grid(int32_t a, int32_t b, int32_t c) {                // a x b x c, each vertex with its neighbours
    Edges e;
    for (int32_t x = 0; x < a; ++x)
        for (int32_t y = 0; y < b; ++y)
            for (int32_t z = 0; z < c; ++z) {
                const int32_t v = (x * b + y) * c + z;
                if (x + 1 < a) e.push_back({v, v + b * c});
                if (y + 1 < b) e.push_back({v, v + c});
                if (z + 1 < c) e.push_back({v, v + 1});
            }
    return undirected(a * b * c, e);
}

// Even degrees that fan out take the sliced push where a search is through in a
// few levels: two searches at the graph's creation tell.
static void even_choice() {
    for (uint32_t levels : {7u, 11u, 12u, 40u}) {
        fake.levels = levels;
        fake.steps = 0;
        fake.restart = true;
        bfs_graph *g = matchings(1 << 18, 14, 1.0);
        fake.restart = false;
        fake.steps = 0;
        bfs_run_options opt{};
        const bfs_status st = bfs_run(g, 0, (int32_t *)address(2), (int32_t *)address(3), &opt, address(), size_t(1) << 40, nullptr);
        WANT(st == BFS_OK && opt.push_used == (levels <= 11 ? BFS_PUSH_SLICED : BFS_PUSH_LIST), "%u levels: form %u, %s", levels, opt.push_used,
             bfs_last_error_detail());
        bfs_graph_destroy(g);
    }
}

// A learned batch takes the claim-word searches where its levels are many and
// thin for its vertices and sources, and the multi-source levels elsewhere.
static void deep_choice() {
    struct Case {
        const char *name;
        bfs_graph *g;
        std::vector<int32_t> deep, shared;          // numbers of sources for either form
    };
    Case cases[] = {
        {"grid 400 x 400", grid(400, 400, 1), {2, 16, 64, 256}, {}},
        {"grid 45 x 44", grid(45, 44, 1), {2, 64, 256, 1024}, {}},
        {"path of 3,000", grid(3000, 1, 1), {2, 64, 256}, {}},
        {"grid 58^3", grid(58, 58, 58), {2, 16, 64}, {256, 1024}},
        {"3 matchings, 0.6", matchings(200000, 3, 0.6), {2, 16}, {256, 1024}},
        {"3 matchings, 0.7", matchings(200000, 3, 0.7), {2, 16}, {128, 256, 1024}},
        {"8 matchings, the probed vertices apart", matchings(200000, 8, 1.0, true), {}, {2, 16, 64, 256}},
        {"one vertex", grid(1, 1, 1), {}, {2, 64, 130}},
        {"path of 5", grid(5, 1, 1), {}, {70, 130}},
    };
    for (const Case &c : cases)
        for (int kind = 0; kind < 2; ++kind)
            for (int32_t nq : kind ? c.shared : c.deep)
                for (uint32_t variant : {kPush, kHeuristic, kLearned}) {
                    std::vector<bfs_graph *> gs((size_t)nq, c.g);
                    std::vector<int32_t> src((size_t)nq, 0);
                    std::vector<int32_t *> out((size_t)nq, (int32_t *)address(5));
                    fake.levels = fake.deep_wanted = 3;
                    fake.cw_inits = fake.ms = 0;
                    bfs_run_options opt{};
                    opt.variant = variant;
                    const bfs_status st = bfs_run_batch(nq, gs.data(), src.data(), out.data(), out.data(), &opt, address(),
                                                        bfs_workspace_size(c.g, nq, 0), nullptr);
                    WANT(st == BFS_OK, "%s, %d sources: %s", c.name, nq, bfs_last_error_detail());
                    WANT((kind == 0) == (fake.cw_inits > 0) && (kind == 1) == (fake.ms > 0), "%s, %d sources, variant %u: %s", c.name, nq, variant,
                         fake.cw_inits ? "claim-word" : "multi-source");
                }
    for (Case &c : cases) bfs_graph_destroy(c.g);
}

int main(int argc, char **argv) {
    const std::string which = argc > 1 ? argv[1] : "";
    if (which == "steps") steps();
    else if (which == "deep_groups") deep_groups();
    else if (which == "deep_syncs") deep_syncs();
    else if (which == "deep_choice") deep_choice();
    else if (which == "ms_decisions") ms_decisions();
    else if (which == "sliced_choice") sliced_choice();
    else if (which == "even_choice") even_choice();
    else if (which == "levels_fit") levels_fit();
    else return 2;
    printf("%d wrong\n", bad);
    return bad != 0;
}
