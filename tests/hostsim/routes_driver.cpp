// Scenarios about the routes that the runtime picks for a call, on the
// host-only build with the launchers of routes_sim.cpp:
//
//   driver replay     calls of one shape and one set of buffers whose instances
//                     change their bias kinds: a captured launch sequence
//                     serves only calls of the kernels that it holds
//   driver retry      frontier builds that give up their chain: the call runs
//                     again in order, pooled and in caller memory, and leaves a
//                     clean workspace
#define main other_scenarios
#include "driver.cpp"
#undef main

namespace hipsim_hooks {
extern std::atomic<int64_t> misrouted, in_order;
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

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "replay") scenario_replay();
    else if (what == "retry") scenario_retry();
    else return other_scenarios(argc, argv);
    std::printf("ok %s\n", what.c_str());
    return 0;
}
