// Scenarios about the routes that the runtime picks for a call, on the
// host-only build with the launchers of routes_sim.cpp:
//
//   driver replay     calls of one shape and one set of buffers whose instances
//                     change their bias kinds: a captured launch sequence
//                     serves only calls of the kernels that it holds
//   driver retry      frontier builds that give up their chain: the call runs
//                     again in order, pooled and in caller memory, and leaves a
//                     clean workspace
//   driver tables     the guides, the hop table and the rank index appear under
//                     calls of four threads, and are left out where memory is
//                     short; every call gives the same results
//   driver room       a server on a device with room for one walk guide, or none
//   driver give_back  calls, graphs and servers that need the memory of such tables
//                     get it, also while other threads' calls read them
//   driver refused    tables that do not fit are asked for ever more seldom, all
//                     those that calls build by themselves take half of the free
//                     memory at most, and none is built or used when turned off
//   driver autotune   the autotuner's calls: one setting for each list length that
//                     lanes scan, no guide on their account
//   driver scratch    a call that fills the library's own scratch without room for
//                     a dirty list
#define main other_scenarios
#include "driver.cpp"
#undef main

namespace hipsim_hooks {
extern std::atomic<int64_t> misrouted, selects, in_order, queries, guides, hops, ranks, with_guide, with_hops, with_rank;
extern std::atomic<size_t> device_limit;
extern std::atomic<int32_t> stuck_layer;
extern std::atomic<bool> stuck_list;
}  // namespace hipsim_hooks

namespace {

// Sampling calls of one shape into one set of device buffers.
struct Call {
    std::vector<int64_t> soff;
    std::vector<int32_t> seeds, fan;
    int32_t L = 2;
    int32_t* dseeds = nullptr;
    csaw_sample_out out{};

    Call(const Host& h, csaw_graph g, int32_t ni, int32_t per, const std::vector<int32_t>& row) : soff(1, 0) {
        L = (int32_t)row.size();
        for (int32_t i = 0; i < ni; ++i) {
            const auto sd = pick_seeds(h, per, 300 + i);
            seeds.insert(seeds.end(), sd.begin(), sd.end());
            soff.push_back((int64_t)seeds.size());
            fan.insert(fan.end(), row.begin(), row.end());
        }
        dseeds = dev_copy(seeds);
        std::vector<int32_t> bias(ni, CSAW_BIAS_UNIFORM);
        csaw_sample_args a = args(bias);
        OK(csaw_sample_bound(g, &a, &out.edge_capacity));
        out.src = dev_copy(std::vector<int32_t>((size_t)out.edge_capacity, -9));
        out.dst = dev_copy(std::vector<int32_t>((size_t)out.edge_capacity, -9));
        out.offsets = dev_copy(std::vector<int64_t>((size_t)L * ni + 1, -9));
    }
    ~Call() {
        for (void* p : {(void*)dseeds, (void*)out.src, (void*)out.dst, (void*)out.offsets}) (void)hipFree(p);
    }
    csaw_sample_args args(const std::vector<int32_t>& bias) const {
        csaw_sample_args a{};
        a.num_instances = (int32_t)soff.size() - 1;
        a.seed_offsets = soff.data();
        a.seeds = dseeds;
        a.num_layers = L;
        a.fanouts = fan.data();
        a.fanout_stride = L;
        a.bias_kinds = bias.data();
        a.rng_seed = 7;
        return a;
    }
    void check(const Host& h, csaw_graph g, const std::vector<int32_t>& bias, hipStream_t s, bool noalloc = false) {
        csaw_sample_args a = args(bias);
        OK(noalloc ? csaw_sample_noalloc(g, &a, &out, s) : csaw_sample(g, &a, &out, s));
        check_edges(h, bias);
    }
    void check_edges(const Host& h, const std::vector<int32_t>& bias) {
        Edges e;
        e.src.assign(out.src, out.src + out.num_edges);
        e.dst.assign(out.dst, out.dst + out.num_edges);
        e.offsets.assign(out.offsets, out.offsets + (size_t)L * (soff.size() - 1) + 1);
        expect_equal(e, reference_sample(h, soff, seeds, L, fan, bias));
    }
};

void scenario_replay() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_graph(1 << 12, 16 << 12, 31);
    for (int32_t kind : {CSAW_BIAS_EDGE_WEIGHT, CSAW_BIAS_NEIGHBOR_DEGREE}) {
        Dev d = upload(h, s);
        const csaw_tuning off{};
        OK(csaw_set_tuning(d.g, &off));
        Call c(h, d.g, 6, 20, {5, 3});
        std::vector<int32_t> weighted(6, kind), mixed = weighted;
        for (size_t i = 0; i < mixed.size(); i += 2) mixed[i] = CSAW_BIAS_UNIFORM;
        for (int rep = 0; rep < 3; ++rep) {
            c.check(h, d.g, weighted, s);
            c.check(h, d.g, mixed, s);
        }
        OK(csaw_graph_destroy(d.g));
    }
    CHECK(hipsim_hooks::misrouted.load() == 0);
    (void)hipStreamDestroy(s);
}

void scenario_retry() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_graph(1 << 12, 16 << 12, 33);
    Dev d = upload(h, s);
    Call c(h, d.g, 6, 20, {5, 3, 2}), other(h, d.g, 2, 30, {4, 4, 3});
    for (int32_t kind : {CSAW_BIAS_UNIFORM, CSAW_BIAS_EDGE_WEIGHT}) {
        const std::vector<int32_t> bias(6, kind);
        c.check(h, d.g, bias, s, true);
        for (int32_t layer = 0; layer < 3; ++layer)
            for (bool list : {false, true})
                for (bool noalloc : {false, true}) {
                    hipsim_hooks::stuck_list = list;
                    hipsim_hooks::stuck_layer = layer;
                    hipsim_hooks::in_order = 0;
                    c.check(h, d.g, bias, s, noalloc);
                    CHECK(hipsim_hooks::in_order.load() == 3);
                    hipsim_hooks::stuck_layer = -1;
                    other.check(h, d.g, std::vector<int32_t>(2, kind), s, noalloc);  // the same workspace
                    CHECK(hipsim_hooks::in_order.load() == 3);
                }
    }
    OK(csaw_graph_destroy(d.g));
    (void)hipStreamDestroy(s);
}

// An undirected graph (lists sorted, weights out-degrees) with lists of more than 64 entries.
Host make_symmetric(int64_t n, int64_t draws, uint64_t seed) {
    Host h = make_graph(n, draws, seed);
    std::vector<std::set<int32_t>> adj(n);
    for (int64_t u = 0; u < n; ++u)
        for (int64_t e = h.rp[u]; e < h.rp[u + 1]; ++e) {
            adj[u].insert(h.col[e]);
            adj[h.col[e]].insert((int32_t)u);
        }
    h.col.clear();
    for (int64_t u = 0; u < n; ++u) {
        h.rp[u + 1] = h.rp[u] + (int64_t)adj[u].size();
        h.col.insert(h.col.end(), adj[u].begin(), adj[u].end());
    }
    h.ew.assign(h.col.size(), 0);
    for (size_t e = 0; e < h.col.size(); ++e) h.ew[e] = (uint32_t)(h.rp[h.col[e] + 1] - h.rp[h.col[e]]);
    return h;
}

// A device limit that hipMalloc and the library's own query agree on (0: none).
void limit_device(size_t bytes) {
    hipsim::set_device_limit(bytes);
    hipsim_hooks::device_limit = bytes;
}

struct Walks {
    std::vector<int32_t> starts;
    int32_t* dstarts = nullptr;
    int32_t* paths = nullptr;
    int32_t length;

    Walks(const Host& h, int64_t walkers, int32_t len, uint64_t seed) : starts(pick_seeds(h, walkers, seed)), length(len) {
        dstarts = dev_copy(starts);
        paths = dev_copy(std::vector<int32_t>(starts.size() * (length + 1), -1));
    }
    ~Walks() {
        (void)hipFree(dstarts);
        (void)hipFree(paths);
    }
    void check(const Host& h, csaw_graph g, int32_t kind, hipStream_t s) {
        csaw_walk_args w{};
        w.bias_kind = kind;
        w.num_walkers = (int64_t)starts.size();
        w.starts = dstarts;
        w.length = length;
        w.rng_seed = 5;
        w.w_return = 1;
        w.w_common = 2;
        w.w_outward = 4;
        int64_t steps = 0, count = 0;
        OK(csaw_walk(g, &w, paths, &steps, s));
        for (size_t k = 0; k < starts.size(); ++k)
            for (int32_t t = 0; t < length; ++t) {
                const int32_t u = paths[k * (length + 1) + t], v = paths[k * (length + 1) + t + 1];
                if (v < 0) break;
                CHECK(std::binary_search(h.col.begin() + h.rp[u], h.col.begin() + h.rp[u + 1], v));
                ++count;
            }
        CHECK(count == steps);
    }
};

// One call of every kind that may build or use a table.
struct Client {
    const Host& h;
    csaw_graph g;
    hipStream_t s = nullptr;
    Call call;
    Walks walks;
    std::vector<int64_t> offs{0, 40, 80};
    int32_t* pool;
    int32_t* out[3];

    Client(const Host& hh, csaw_graph gg, uint64_t seed) : h(hh), g(gg), call(hh, gg, 4, 40, {10, 5}), walks(hh, 200, 30, seed) {
        CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
        const std::vector<int32_t> one = pick_seeds(h, 40, seed + 1);
        std::vector<int32_t> two = one;
        two.insert(two.end(), one.begin(), one.end());
        pool = dev_copy(two);
        for (auto& o : out) o = dev_copy(std::vector<int32_t>(2 * 64, 0));
    }
    ~Client() {
        (void)hipFree(pool);
        for (auto* o : out) (void)hipFree(o);
        (void)hipStreamDestroy(s);
    }
    void round() {
        for (int32_t kind : {CSAW_BIAS_EDGE_WEIGHT, CSAW_BIAS_NEIGHBOR_DEGREE}) {
            call.check(h, g, std::vector<int32_t>(4, kind), s);
            csaw_layer_args a{};
            a.num_instances = 2;
            a.seed_offsets = offs.data();
            a.seeds = pool;
            a.num_layers = 1;
            const int32_t fan = 64;
            a.fanouts = &fan;
            a.bias_kind = kind;
            OK(csaw_layer_sample(g, &a, out[0], out[1], out[2], s));
        }
        for (int32_t kind : {CSAW_BIAS_UNIFORM, CSAW_BIAS_NODE2VEC, CSAW_BIAS_EDGE_WEIGHT}) walks.check(h, g, kind, s);
        csaw_mdrw_args a{};
        a.num_instances = 2;
        a.pool_offsets = offs.data();
        a.pool = pool;
        a.budget = 64;
        int64_t total = 0;
        OK(csaw_mdrw(g, &a, out[0], out[1], nullptr, &total, s));
    }
};

void scenario_tables() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_symmetric(1 << 10, 6 << 10, 35);
    {
        Dev d = upload(h, s);
        std::vector<std::thread> threads;
        for (int t = 0; t < 4; ++t)
            threads.emplace_back([&, t] {
                Client c(h, d.g, 40 + t);
                for (int rep = 0; rep < 12; ++rep) c.round();
            });
        for (auto& t : threads) t.join();
        CHECK(hipsim_hooks::guides.load() == 2 && hipsim_hooks::hops.load() == 1 && hipsim_hooks::ranks.load() == 1);
        CHECK(hipsim_hooks::with_guide.load() > 0 && hipsim_hooks::with_hops.load() > 0 && hipsim_hooks::with_rank.load() > 0);
        OK(csaw_graph_destroy(d.g));
    }
    {
        Dev d = upload(h, s);
        OK(csaw_set_walk_guides(d.g, 0));  // weighted walks through the chunk tables
        Client c(h, d.g, 50);
        c.round();
        hipsim_hooks::guides = hipsim_hooks::hops = hipsim_hooks::ranks = 0;
        limit_device(hipsim::device_bytes_in_use() + (size_t(4) << 10));
        for (int rep = 0; rep < 12; ++rep) c.round();
        CHECK(hipsim_hooks::guides.load() == 0 && hipsim_hooks::hops.load() == 0 && hipsim_hooks::ranks.load() == 0);
        limit_device(0);
        OK(csaw_graph_destroy(d.g));
    }
    (void)hipStreamDestroy(s);
}

// A server needs its executors' memory and the degree tables; the walk guides are built where they fit.
void scenario_room() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_symmetric(1 << 12, 16 << 12, 36);
    const size_t n = (size_t)h.n, m = h.col.size();
    const size_t degree = 4 * m + 12 * n + (m / 512 + 1) * (64 + 1) * 8;  // weights, counts, totals, chunk tables
    const size_t guide = 16 * m + 16 * n + 16 * (2 * m + n);              // two buckets per edge
    for (const int fit : {1, 2, 0}) {
        Dev d = upload(h, s);
        auto trace = make_trace(h, 12, 60, 300, 12, 37);
        csaw_server_config cfg{};
        cfg.memory_budget_bytes = int64_t(8) << 20;
        cfg.num_streams = 2;
        hipsim_hooks::guides = 0;
        limit_device(hipsim::device_bytes_in_use() + (size_t)cfg.memory_budget_bytes + degree + fit * guide + guide / 2);
        csaw_server srv = nullptr;
        OK(csaw_server_create(d.g, &cfg, &srv));
        CHECK(hipsim_hooks::guides.load() == fit);
        limit_device(0);  // (the checks below make calls of their own)
        run_trace(d, srv, trace, 1, s);
        OK(csaw_server_destroy(srv));
        OK(csaw_graph_destroy(d.g));
    }
    (void)hipStreamDestroy(s);
}

// An allocator that fails once in the thread that asks for it.
thread_local int fail_allocs = 0;
void* picky_alloc(size_t bytes, void*) {
    if (fail_allocs > 0 && fail_allocs--) return nullptr;
    void* p = nullptr;
    return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void picky_free(void* p, void*) { (void)hipFree(p); }

void scenario_give_back() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_symmetric(1 << 12, 6 << 12, 38);
    const size_t slack = size_t(16) << 10;
    // what needs the memory: a sampling call with a larger workspace, a weight
    // array's tables, a second graph, a partitioned graph, a server
    for (int what = 0; what < 5; ++what) {
        Dev d = upload(h, s);
        Client c(h, d.g, 60);
        Call large(h, d.g, 60, 10, {6, 4});
        Walks degree(h, 50, 8, 64);
        const int32_t kinds[3] = {CSAW_BIAS_EDGE_WEIGHT, CSAW_BIAS_UNIFORM, CSAW_BIAS_NODE2VEC};
        for (int rep = 0; rep < 30; ++rep) {
            c.call.check(h, d.g, std::vector<int32_t>(4, CSAW_BIAS_EDGE_WEIGHT), s);
            for (int32_t k : kinds) c.walks.check(h, d.g, k, s);
        }
        const size_t with = hipsim::device_bytes_in_use();
        limit_device(with + slack);
        if (what == 0) large.check(h, d.g, std::vector<int32_t>(60, CSAW_BIAS_EDGE_WEIGHT), s);
        if (what == 1) degree.check(h, d.g, CSAW_BIAS_NEIGHBOR_DEGREE, s);
        Dev other;
        if (what == 2) other = upload(h, s);
        csaw_pgraph pg = nullptr;
        if (what == 3)
            OK(csaw_pgraph_create(h.n, (int64_t)h.col.size(), h.rp.data(), h.col.data(), h.ew.data(), 4, 1, s, &pg));
        csaw_server srv = nullptr;
        csaw_server_config cfg{};
        cfg.memory_budget_bytes = int64_t(1) << 20;
        cfg.num_streams = 1;
        if (what == 4) OK(csaw_server_create(d.g, &cfg, &srv));
        limit_device(0);
        hipsim_hooks::with_hops = hipsim_hooks::with_rank = 0;
        c.round();  // without them
        CHECK(hipsim_hooks::with_hops.load() == 0 && hipsim_hooks::with_rank.load() == 0);
        if (srv) OK(csaw_server_destroy(srv));
        if (pg) OK(csaw_pgraph_destroy(pg));
        if (other.g) OK(csaw_graph_destroy(other.g));
        OK(csaw_graph_destroy(d.g));
    }
    {  // weighted walks without room for a guide
        Dev d = upload(h, s);
        Walks w(h, 50, 8, 65);
        w.check(h, d.g, CSAW_BIAS_UNIFORM, s);  // (its workspace)
        limit_device(hipsim::device_bytes_in_use() + slack);
        w.check(h, d.g, CSAW_BIAS_EDGE_WEIGHT, s);
        limit_device(0);
        OK(csaw_graph_destroy(d.g));
    }
    OK(csaw_set_allocator(picky_alloc, picky_free, nullptr));
    const Host small = make_graph(1 << 8, 4 << 8, 39);
    int given = 0;
    for (int rep = 0; rep < 3; ++rep) {
        Dev d = upload(h, s);
        std::atomic<int> running{3};
        std::vector<std::thread> threads;
        for (int t = 0; t < 3; ++t)
            threads.emplace_back([&, t] {
                Client c(h, d.g, 70 + t);
                for (int k = 0; k < 4; ++k) c.round();
                --running;
            });
        while (running.load()) {  // a new graph's first workspace
            Dev mine = upload(small, s);
            Call c(small, mine.g, 4, 10, {4, 3});
            const std::vector<int32_t> bias(4, CSAW_BIAS_EDGE_WEIGHT);
            csaw_sample_args a = c.args(bias);
            fail_allocs = 1;
            const csaw_status st = csaw_sample(mine.g, &a, &c.out, s);
            CHECK(fail_allocs == 0 && (st == CSAW_OK || st == CSAW_ERR_OUT_OF_MEMORY));  // (no tables at that moment)
            if (st == CSAW_OK) {
                c.check_edges(small, bias);
                ++given;
            }
            OK(csaw_graph_destroy(mine.g));
        }
        for (auto& t : threads) t.join();
        OK(csaw_graph_destroy(d.g));
    }
    CHECK(given > 0);
    OK(csaw_set_allocator(nullptr, nullptr, nullptr));
    (void)hipStreamDestroy(s);
}

void scenario_refused() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_symmetric(1 << 10, 6 << 10, 41);
    const size_t n = (size_t)h.n, m = h.col.size();
    {
        Dev d = upload(h, s);
        Client c(h, d.g, 80);
        c.call.check(h, d.g, std::vector<int32_t>(4, CSAW_BIAS_NEIGHBOR_DEGREE), s);
        limit_device(hipsim::device_bytes_in_use() + 8 * m);
        hipsim_hooks::queries = hipsim_hooks::guides = hipsim_hooks::hops = 0;
        for (int rep = 0; rep < 200; ++rep) c.round();
        CHECK(hipsim_hooks::guides.load() == 0 && hipsim_hooks::hops.load() == 0);
        CHECK(hipsim_hooks::queries.load() < 100);
        limit_device(0);  // there is room again: they come in the end
        for (int rep = 0; rep < 1000 && (hipsim_hooks::guides.load() < 2 || hipsim_hooks::hops.load() < 1); ++rep) c.round();
        CHECK(hipsim_hooks::guides.load() == 2 && hipsim_hooks::hops.load() == 1);
        OK(csaw_graph_destroy(d.g));
    }
    {
        Dev d = upload(h, s);
        Client c(h, d.g, 81);
        CHECK(m % 4 == 2);  // (the last quad of column ids is not full)
        const size_t guide = 16 * m + 16 * n + 16 * (4 * m + n);
        c.call.check(h, d.g, std::vector<int32_t>(4, CSAW_BIAS_NEIGHBOR_DEGREE), s);
        const size_t before = hipsim::device_bytes_in_use(), room = 2 * guide + 2 * 16 * m;
        limit_device(before + room);  // the guide would fit half of what the hop table and the rank index leave
        hipsim_hooks::guides = hipsim_hooks::hops = hipsim_hooks::ranks = 0;
        for (int rep = 0; rep < 60; ++rep) {
            c.call.check(h, d.g, std::vector<int32_t>(4, CSAW_BIAS_EDGE_WEIGHT), s);
            c.walks.check(h, d.g, CSAW_BIAS_UNIFORM, s);
            c.walks.check(h, d.g, CSAW_BIAS_NODE2VEC, s);
        }
        CHECK(hipsim_hooks::guides.load() == 0 && hipsim_hooks::hops.load() == 1 && hipsim_hooks::ranks.load() == 1);
        CHECK(hipsim::device_bytes_in_use() - before <= room / 2);
        limit_device(0);
        OK(csaw_graph_destroy(d.g));
    }
    {
        Dev d = upload(h, s);
        OK(csaw_set_walk_guides(d.g, 0));
        Client c(h, d.g, 82);
        hipsim_hooks::guides = hipsim_hooks::hops = hipsim_hooks::ranks = 0;
        for (int rep = 0; rep < 20; ++rep) c.round();
        CHECK(hipsim_hooks::guides.load() == 0 && hipsim_hooks::hops.load() == 0 && hipsim_hooks::ranks.load() == 0);
        OK(csaw_set_walk_guides(d.g, 1));
        for (int rep = 0; rep < 20; ++rep) c.round();
        CHECK(hipsim_hooks::guides.load() == 2 && hipsim_hooks::hops.load() == 1 && hipsim_hooks::ranks.load() == 1);
        OK(csaw_set_walk_guides(d.g, 0));
        hipsim_hooks::with_guide = hipsim_hooks::with_hops = hipsim_hooks::with_rank = 0;
        c.round();
        CHECK(hipsim_hooks::with_guide.load() == 0 && hipsim_hooks::with_hops.load() == 0 &&
              hipsim_hooks::with_rank.load() == 0);
        OK(csaw_graph_destroy(d.g));
    }
    (void)hipStreamDestroy(s);
}

void scenario_autotune() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_symmetric(1 << 10, 6 << 10, 43);
    Dev d = upload(h, s);
    Call c(h, d.g, 30, 40, {20});
    const std::vector<int32_t> bias(30, CSAW_BIAS_NEIGHBOR_DEGREE);
    csaw_sample_args a = c.args(bias);
    csaw_tuning t{};
    const int32_t reps = 20;
    OK(csaw_autotune_sample(d.g, &a, &c.out, reps, s, &t));
    c.check_edges(h, bias);
    CHECK(c.out.num_edges * reps > (int64_t)h.col.size());
    CHECK(hipsim_hooks::selects.load() == 4 * (reps + 1) && hipsim_hooks::guides.load() == 0);
    c.check(h, d.g, bias, s);  // they paid for nothing
    CHECK(hipsim_hooks::guides.load() == 0);
    while (hipsim_hooks::guides.load() == 0) c.check(h, d.g, bias, s);
    const csaw_tuning mine{5, 7};  // with the guide no list is scanned: one call, the setting stays
    OK(csaw_set_tuning(d.g, &mine));
    hipsim_hooks::selects = 0;
    OK(csaw_autotune_sample(d.g, &a, &c.out, reps, s, &t));
    c.check_edges(h, bias);
    CHECK(hipsim_hooks::selects.load() == 1 && t.bound16 == 5 && t.bound32 == 7);
    OK(csaw_get_tuning(d.g, &t));
    CHECK(t.bound16 == 5 && t.bound32 == 7);
    OK(csaw_graph_destroy(d.g));
    (void)hipStreamDestroy(s);
}

// 9 instances of 5,035 seeds on 2^22 vertices: 1.2M bitmap words; at most 2.9M picks of layer 0 at
// 40 bytes each in the scratch of 128 MiB, not at 48.
void scenario_scratch() {
    hipStream_t s;
    CHECK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess);
    const Host h = make_graph(1 << 22, 500000, 45);
    Dev d = upload(h, s);
    Call c(h, d.g, 9, 5035, {64, 1});
    c.check(h, d.g, std::vector<int32_t>(9, CSAW_BIAS_UNIFORM), s, true);
    c.check(h, d.g, std::vector<int32_t>(9, CSAW_BIAS_EDGE_WEIGHT), s, true);
    OK(csaw_graph_destroy(d.g));
    (void)hipStreamDestroy(s);
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "replay") scenario_replay();
    else if (what == "retry") scenario_retry();
    else if (what == "tables") scenario_tables();
    else if (what == "room") scenario_room();
    else if (what == "give_back") scenario_give_back();
    else if (what == "refused") scenario_refused();
    else if (what == "autotune") scenario_autotune();
    else if (what == "scratch") scenario_scratch();
    else return other_scenarios(argc, argv);
    std::printf("ok %s\n", what.c_str());
    return 0;
}
