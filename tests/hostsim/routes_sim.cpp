// Stand-in launchers of kernels_sim.cpp with what the route tests add: they
// note launches whose kernel cannot serve the entries that it is given, and
// build and read the tables that speed calls up (walk guides, hop table, rank
// index). Test infrastructure only.
#include "../../paper_2009_09103_amd/csrc/kernels.h"

#define launch_select placeholder_select
#define launch_frontier_build placeholder_build
#define launch_walk placeholder_walk
#define launch_layer_sample placeholder_layer
#define launch_mdrw placeholder_mdrw
#define launch_walk_guides placeholder_guides
#include "kernels_sim.cpp"
#undef launch_select
#undef launch_frontier_build
#undef launch_walk
#undef launch_layer_sample
#undef launch_mdrw
#undef launch_walk_guides

namespace hipsim_hooks {
std::atomic<int64_t> misrouted{0};  // unbiased draws given to the kernel that draws by weight alone
std::atomic<int64_t> selects{0};    // selection launches that ran
std::atomic<int32_t> stuck_layer{-1};  // builds of this layer give up their chain by block index ...
std::atomic<bool> stuck_list{false};   // ... in the compaction
std::atomic<int64_t> in_order{0};      // builds whose blocks take tickets
std::atomic<size_t> device_limit{0};   // what free_device_bytes counts down from (0: plenty)
std::atomic<int64_t> queries{0};       // ... and how often it was asked
std::atomic<int64_t> guides{0}, hops{0}, ranks{0};  // tables built
std::atomic<int64_t> with_guide{0}, with_hops{0}, with_rank{0};  // launches that were given one
}  // namespace hipsim_hooks

namespace csaw {

namespace {

// Reads every table that a launch is given, whole: a table that goes while a
// call uses it is an access that the sanitizers see.
void read_tables(const GraphDev& g) {
    for (int k = 0; k < 2; ++k) {
        const WalkBucket* gd = k ? g.wgd_deg : g.wgd_ew;
        if (!gd) continue;
        ++hipsim_hooks::with_guide;
        const WalkEdge* rec = k ? g.wrec_deg : g.wrec_ew;
        const WalkVertex* vtx = k ? g.wvtx_deg : g.wvtx_ew;
        const uint64_t* tot = k ? g.wtot_deg : g.wtot_ew;
        const int per = k ? g.gper_deg : g.gper_ew;
        for (int64_t v = 0; v < g.n; ++v) {
            const int64_t b = g.rowptr[v], d = g.rowptr[v + 1] - b;
            if (vtx[v].W != tot[v] || vtx[v].beg != b || vtx[v].d != d) abort();
            if (tot[v] == 0) continue;
            if (rec[b + d - 1].S != tot[v] || rec[b].col != g.col[b]) abort();
            const uint64_t last = (tot[v] - 1) >> guide_shift(tot[v], d, per);
            if (gd[guide_base(b, v, per) + (int64_t)last].pos >= d) abort();
        }
    }
    if (g.hops) {
        ++hipsim_hooks::with_hops;
        for (int64_t e = 0; e < g.m; ++e)
            if (g.hops[e].col != g.col[e] || g.hops[e].beg != g.rowptr[g.col[e]]) abort();
    }
    if (g.rank) {
        ++hipsim_hooks::with_rank;
        volatile int32_t last = 0;  // lookups read whole quads of the column ids
        for (int64_t e = g.m / 4 * 4; e < (g.m + 3) / 4 * 4; ++e) last = g.col[e];
        (void)last;
        for (int64_t v = 0; v < g.n; ++v) {
            const int64_t b = g.rowptr[v], d = g.rowptr[v + 1] - b;
            if (d >= kRankMinD && g.rank[rank_base(b, v) + (1 << rank_log(d))] != d) abort();
        }
    }
}

}  // namespace

size_t free_device_bytes() {
    ++hipsim_hooks::queries;
    const size_t limit = hipsim_hooks::device_limit.load(), used = hipsim::device_bytes_in_use();
    return limit == 0 ? size_t(1) << 40 : limit > used ? limit - used : 0;
}

void launch_walk_guides(RowPtr rowptr, const int32_t* col, const uint32_t* w, const uint64_t* wtot, int64_t n,
                        WalkEdge* rec, WalkVertex* vtx, WalkBucket* gd, int per, hipStream_t s) {
    ++hipsim_hooks::guides;
    hipsim::enqueue(s, [=] {
        for (int64_t v = 0; v < n; ++v) {
            const int64_t b = rowptr[v], d = rowptr[v + 1] - b;
            const uint64_t W = wtot[v];
            if (vtx) vtx[v] = WalkVertex{W, (uint32_t)b, (uint32_t)d};
            if (W == 0) continue;
            const int sh = guide_shift(W, d, per);
            const uint64_t K = ((W - 1) >> sh) + 1;
            if (K > (uint64_t)(per * d)) abort();  // the list's slots hold its buckets
            WalkBucket* G = gd + guide_base(b, v, per);
            uint64_t run = 0, k = 0;
            for (int64_t i = 0; i < d; ++i) {
                run += w[b + i];
                rec[b + i] = WalkEdge{run, col[b + i], w[b + i]};
                for (; k < K && (k << sh) < run; ++k) G[k] = WalkBucket{run, (uint32_t)i, col[b + i]};
            }
        }
    });
}

void launch_walk_guides(RowPtr rowptr, const int32_t* col, const uint32_t* w, const uint64_t* wtot, int64_t n,
                        WalkEdge* rec, WalkVertex* vtx, WalkBucket* gd, hipStream_t s) {
    launch_walk_guides(rowptr, col, w, wtot, n, rec, vtx, gd, kGuideBucketsPerEdge, s);
}

void launch_walk_hops(RowPtr rowptr, const int32_t* col, int64_t m, WalkHop* hops, hipStream_t s) {
    ++hipsim_hooks::hops;
    hipsim::enqueue(s, [=] {
        for (int64_t e = 0; e < m; ++e)
            hops[e] = WalkHop{col[e], (uint32_t)rowptr[col[e]], (uint32_t)(rowptr[col[e] + 1] - rowptr[col[e]]), 0u};
    });
}

void launch_walk_ranks(RowPtr rowptr, const int32_t* col, int64_t n, uint32_t* rank, int32_t* repeats, hipStream_t s) {
    ++hipsim_hooks::ranks;
    hipsim::enqueue(s, [=] {
        for (int64_t v = 0; v < n; ++v) {
            const int64_t b = rowptr[v], d = rowptr[v + 1] - b;
            for (int64_t i = 1; i < d; ++i)
                if (col[b + i] == col[b + i - 1]) *repeats = 1;
            if (d < kRankMinD) continue;
            uint32_t* R = rank + rank_base(b, v);
            for (int64_t k = 0, i = 0; k <= 1 << rank_log(d); ++k) {
                while (i < d && (int64_t)col[b + i] < k << rank_shift(n, d)) ++i;
                R[k] = (uint32_t)i;
            }
        }
    });
}

void launch_walk(const WalkParams& p, int grid, hipStream_t s, LaunchEvents ev) {
    hipsim::enqueue(s, [p] { read_tables(p.g); });
    placeholder_walk(p, grid, s, ev);
}

void launch_layer_sample(const LayerParams& p, hipStream_t s, LaunchEvents ev) {
    hipsim::enqueue(s, [p] { read_tables(p.g); });
    placeholder_layer(p, s, ev);
}

void launch_mdrw(const MdrwParams& p, hipStream_t s, LaunchEvents ev) {
    hipsim::enqueue(s, [p] { read_tables(p.g); });
    placeholder_mdrw(p, s, ev);
}

// Checked when the launch runs, so that a replayed launch is checked against
// the tables of the call that it serves.
void launch_select(const SampleLayer& p, int grid, hipStream_t s, LaunchEvents ev) {
    hipsim::enqueue(s, [p] {
        read_tables(p.g);
        ++hipsim_hooks::selects;
        for (int64_t e = 0; p.wave_only && e < p.ctl->fcount[p.layer]; ++e) {
            const int32_t P = p.fpos[e] & ~kWideList;
            if (p.bias[p.fi[e]] == kUniform && p.cnt[e] > 0 && p.cnt[e] < P) ++hipsim_hooks::misrouted;
        }
    });
    placeholder_select(p, grid, s, ev);
}

// A build that gives up leaves bits behind that the second try must not see.
void launch_frontier_build(const FrontierBuild& fb, hipStream_t s, LaunchEvents ev) {
    placeholder_build(fb, s, ev);
    hipsim::enqueue(s, [fb] {
        if (fb.ordered) {
            ++hipsim_hooks::in_order;
        } else if (fb.layer == hipsim_hooks::stuck_layer.load()) {
            (hipsim_hooks::stuck_list.load() ? fb.ctl->list_stuck : fb.ctl->lookback_stuck) = 1;
            std::fill(fb.visited, fb.visited + fb.nwords, 0x55555555u);
        }
    });
}

}  // namespace csaw
