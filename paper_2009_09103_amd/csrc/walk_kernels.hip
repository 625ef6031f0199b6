// walk_kernels.hip -- gfx950 kernels of random walks (DeepWalk, biased
// DeepWalk, node2vec; Section II-A of the paper).
//
// A walk is a chain of one-draw selections (NeighborSize 1, with
// replacement). The step loop runs inside the kernel: walkers are
// independent, so no host round trip is needed between steps.
//   - unbiased walks: one lane per walker (a step is one Philox draw and one
//     load of the picked edge's record, its neighbor and that one's list, or
//     without the hop table a neighbor load and two row-offset loads);
//   - edge-weight and degree-biased walks through the graph's walk guide
//     (exact per-edge prefixes and a bucket table per list; a step is two
//     rounds of loads, now and then three): one lane per walker in launches of at
//     least kLaneWalkMin walkers, else one wavefront per walker; with the guide
//     off, one wavefront per walker through the chunk tables;
//   - other biased walks: one wavefront per walker; pass 1 streams the
//     biases of N(v) into a coarse prefix table in LDS, r is drawn in [0, W),
//     and pass 2 rescans only the group of the table that holds r.
//   - node2vec: the bias of x in N(v) needs "is x adjacent to the previous
//     vertex t"; adjacency lists are sorted, so the shorter of N(v) and N(t)
//     is looked up in the longer one through the graph's rank index, or, where
//     the graph has none, N(v) is merged with N(t) (or, for a much longer N(t), each
//     candidate binary-searches it).
#include "device_common.h"
#include "kernels.h"

namespace csaw {

namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

// Restart / jump rule of a step: draws x in [0, 2^32) with counter (walker,
// step, v, 2); below restart the walker returns to its start, below
// restart + jump it moves to a vertex drawn in [0, n) with counter (walker,
// step, v, 3). Returns whether the step is such a move.
__device__ __forceinline__ bool walk_move(const WalkParams& p, Key key, uint32_t c0, int32_t s, int32_t v,
                                         int32_t start, int32_t& to) {
    if ((p.restart | p.jump) == 0) return false;
    const uint64_t x = draw(key, c0, (uint32_t)s, (uint32_t)v, 2u, 1ull << 32);
    if (x < (uint64_t)p.restart) {
        to = start;
        return true;
    }
    if (x < (uint64_t)p.restart + p.jump) {
        to = (int32_t)draw(key, c0, (uint32_t)s, (uint32_t)v, 3u, (uint64_t)p.g.n);
        return true;
    }
    return false;
}

// Walker w's Philox key, length, walker id (counter word 0), path row and
// step counter: from the call, or from its request's entries in a batch.
struct WalkerCtx {
    Key key;
    int32_t length;
    uint32_t c0;
    int32_t* path;
    unsigned long long* steps;
};

__device__ __forceinline__ WalkerCtx walker_ctx(const WalkParams& p, int64_t w) {
    WalkerCtx c;
    if (p.batch.req) {
        const int32_t q = p.batch.req[w];
        const uint64_t k = p.batch.key[q];
        c.key = Key{(uint32_t)k, (uint32_t)(k >> 32)};
        c.length = p.batch.length[q];
        const int64_t i = w - p.batch.first[q];
        c.c0 = (uint32_t)(p.batch.base[q] + (uint64_t)i);
        c.path = p.paths + p.batch.path[q] + i * ((int64_t)c.length + 1);
        c.steps = p.batch.steps + q;
    } else {
        c.key = Key{p.k0, p.k1};
        c.length = p.length;
        c.c0 = (uint32_t)(p.walker_ids ? p.walker_ids[w] : p.walker_base + (uint64_t)w);
        c.path = p.paths + w * ((int64_t)p.length + 1);
        c.steps = p.steps;
    }
    return c;
}

// Adds each lane's steps to its request's counter (every lane of the wavefront calls
// it; its lanes may belong to several requests): one atomic per request, since
// atomics to one address pass one after the other, some 13 ns apart. With one per lane
// seven walk requests of 188,672 walkers took 2.45 ms, 0.46 with these.
__device__ __forceinline__ void count_steps(int64_t steps, unsigned long long* counter) {
    for (uint64_t todo = ballot(steps != 0); todo;) {
        const int lead = __ffsll((unsigned long long)todo) - 1;
        const uint64_t to = readlane_u64((uint64_t)(uintptr_t)counter, lead);
        const bool mine = steps != 0 && (uint64_t)(uintptr_t)counter == to;
        const int64_t sum = wave_sum_i64(mine ? steps : 0);
        if (lane_id() == lead) atomicAdd(counter, (unsigned long long)sum);
        todo &= ~ballot(mine);
    }
}

// A lane's path entries, written kPathRun at a time in 16-byte stores: a 4-byte
// store into a row of its own per step leaves each line part written in the L2
// when it is evicted, over and over; a run of a line's length reaches its line
// (or two) at once. 2^20 unbiased walkers x 80: 2.63 ms with runs of 8, 2.53
// with 16, 2.37 with 32 and 2.25 with 64, although the registers cost
// occupancy; 262,144 weighted walkers: 1.05 ms with 8 to 32, 1.12 with 64. A
// launch whose lines stay in the L2 until they are full only pays for the run, in
// registers and in each step's chain, and stores every entry at once (runs of 1).
// R-MAT 22, length 80, as it is (most walkers end early) / symmetrised (all walk on),
// runs of 1 against the long ones: unbiased 92 against 126 us / 116 against 131 for 16,384
// walkers, 98 against 132 / 126 against 136 for 32,768, 123 against 149 / 184 against 168
// for 65,536; weighted, by lanes, 252 against 270 / 271 against 290 for 16,384, 256 against
// 275 / 279 against 294 for 32,768, 302 against 287 / 335 against 309 for 65,536. The lines
// lie where the symmetrised graph's figures cross.
constexpr int64_t kUniformRunMin = 49152, kLaneRunMin = 45056;
typedef int32_t PathQuad __attribute__((ext_vector_type(4), aligned(4)));
template <int kPathRun>
struct PathRun {
    int32_t e[kPathRun] = {};
    int n = 0;
    int64_t at = 1;  // path index of e[0]
    __device__ __forceinline__ void flush(int32_t* path) {
#pragma unroll
        for (int j = 0; j < kPathRun; ++j)
            if (j < n) path[at + j] = e[j];
        at += n;
        n = 0;
    }
    __device__ __forceinline__ void push(int32_t* path, int32_t x) {
#pragma unroll
        for (int j = 0; j < kPathRun; ++j) e[j] = n == j ? x : e[j];
        if (++n == kPathRun) {
#pragma unroll
            for (int j = 0; j < kPathRun; j += 4)
                *(PathQuad*)(path + at + j) = PathQuad{e[j], e[j + 1], e[j + 2], e[j + 3]};
            at += kPathRun;
            n = 0;
        }
    }
};

template <>
struct PathRun<1> {
    int64_t at = 1;
    __device__ __forceinline__ void flush(int32_t*) {}
    __device__ __forceinline__ void push(int32_t* path, int32_t x) { path[at++] = x; }
};

// v's list.
__device__ __forceinline__ void list_of(const GraphDev& g, int32_t v, int64_t& beg, int64_t& d) {
    beg = g.rowptr[v];
    d = g.rowptr[v + 1] - beg;
}

// Unbiased walks, one lane per walker. kHops: the graph has its hop table, and a
// step is one scattered 16-byte read, the picked edge's record (neighbor and
// its list), plus its share of a path run; without the table, the neighbor id
// and then its row offsets. Scattered lines bound it (41e9 a second on this
// chip): 2^20 walkers x 80 on 500M edges took 4.96 ms with two reads a step and
// a 4-byte path store each, 2.23 ms with one read and runs.
// kMoves: the call restarts or jumps. Lanes that move wait for their list with the
// others (in a step of their own, 1,000 walkers x 80 with restarts took 189 us on
// R-MAT 22, 144 now); walks without moves do without the test, and its registers
// (262,144 unbiased walkers x 80: 389 us with it, 346 without).
// kRun: see PathRun. Metropolis-Hastings walkers stay where they are for many steps
// and find the list's line again in the L2 of their die: with long runs three
// wavefronts per SIMD hold as many lists as fit it (symmetrised R-MAT 22, 2^20
// walkers x 80: 1.03 ms with three, 1.20 with four, 1.08 with two; R-MAT 22 as it
// is 0.91, 0.89, 1.03). Unbiased walkers leave and take four (2.03, 2.06 with three).
// kMH: Metropolis-Hastings (Section II-A): the uniform pick u is a proposal,
// accepted iff x * deg(u) < deg(v) * 2^32 for x in [0, 2^32) drawn with
// counter (walker id, step, v, 4); a rejected proposal is a step that stays.
template <bool kMH, bool kHops, bool kMoves, int kRun>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, kMH && kRun > 1 ? 3 : 8)))
k_walk_uniform(WalkParams p) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t w0 = blockIdx.x * (int64_t)blockDim.x; w0 < p.num_walkers; w0 += stride) {
        const int64_t w = w0 + threadIdx.x;
        int64_t my_steps = 0;
        unsigned long long* my_counter = p.steps;
        if (w < p.num_walkers) {
            const WalkerCtx wc = walker_ctx(p, w);
            const Key key = wc.key;
            const int64_t L1 = (int64_t)wc.length + 1;
            int32_t* path = wc.path;
            my_counter = wc.steps;
            int32_t v = p.starts[w];
            int32_t s = 0;
            if (v < 0 || (int64_t)v >= p.g.n) {
                *p.bad_start = 1;
                for (int64_t q = 0; q < L1; ++q) path[q] = -1;
            } else {
                path[0] = v;
                const int32_t start = v;
                const uint32_t c0 = wc.c0;
                PathRun<kRun> run;
                int64_t beg, d;
                list_of(p.g, v, beg, d);
                for (; s < wc.length; ++s) {
                    int32_t u;
                    int64_t ub, ud;
                    bool move = true;
                    const bool moved = kMoves && walk_move(p, key, c0, s, v, start, u);
                    if (moved) {
                        if (kHops) list_of(p.g, u, ub, ud);
                    } else {
                        if (d == 0) break;
                        const uint64_t r = draw(key, c0, (uint32_t)s, (uint32_t)v, 0u, (uint64_t)d);
                        if (kHops) {
                            const uint4 h = *(const uint4*)(p.g.hops + beg + (int64_t)r);
                            u = (int32_t)h.x;
                            ub = h.y;
                            ud = h.z;
                        } else {
                            u = p.g.col[beg + (int64_t)r];
                        }
                    }
                    if (!kHops) list_of(p.g, u, ub, ud);  // one wait for the lanes that moved and the others
                    if (kMH && !moved) {
                        const uint64_t x = draw(key, c0, (uint32_t)s, (uint32_t)v, 4u, uint64_t(1) << 32);
                        move = x * (uint64_t)ud < ((uint64_t)d << 32);
                    }
                    if (move) {
                        v = u;
                        beg = ub;
                        d = ud;
                    }
                    run.push(path, v);
                }
                run.flush(path);
                for (int64_t q = s + 1; q < L1; ++q) path[q] = -1;
            }
            my_steps = s;
        }
        if (p.batch.req) {
            count_steps(my_steps, my_counter);
        } else {
            const int64_t ws = wave_sum_i64(my_steps);
            if (lane_id() == 0 && ws) atomicAdd(p.steps, (unsigned long long)ws);
        }
    }
}

__global__ void k_walk_hops(RowPtr rowptr, const int32_t* __restrict__ col, int64_t m, WalkHop* __restrict__ hops) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = col[e];
        const int64_t b = rowptr[x];
        *(uint4*)(hops + e) = make_uint4((uint32_t)x, (uint32_t)b, (uint32_t)(rowptr[x + 1] - b), 0u);
    }
}

// is x in the sorted list col[b, e)?
__device__ __forceinline__ bool in_sorted(const int32_t* __restrict__ col, int64_t b, int64_t e, int32_t x) {
    int64_t lo = b, hi = e;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const int32_t y = col[mid];
        if (y < x) lo = mid + 1;
        else hi = mid;
    }
    return lo < e && col[lo] == x;
}

// Weighted and node2vec steps: one wavefront per walker. Pass 1 streams
// N(v) in tiles of kWalkTile candidates (kWalkPer coalesced loads per lane,
// the next tile's loads in flight while the current one is processed),
// evaluates the biases and records the inclusive prefix at the end of every
// group of 2^shift tiles in an LDS table (at most kWalkTab groups). After the
// draw, a binary search in the table finds the group and pass 2 rescans only
// that group, 64 candidates at a time (scan + ballot).
// node2vec: x in N(t) is found by merging N(v) with N(t) -- both sorted --
// through an LDS window of kWalkWin entries of N(t) (the following window is
// prefetched into registers), or, when N(t) is much longer than N(v), by a
// binary search per candidate; membership of the first kWalkBits candidates
// is kept as bits for pass 2.
constexpr int kWalkPer = 4;
constexpr int kWalkTile = kWalkPer * kWave;   // 256
constexpr int kWalkTileLog = 8;
constexpr int kWalkTab = 256;
constexpr int kWalkWin = 256;
constexpr int kWinPer = kWalkWin / kWave;
constexpr int kWalkBits = 16384;
constexpr int64_t kMergeRatio = 8;              // merge while d_t <= 8 d_v + kWalkWin

template <bool kN2v>
struct WalkLds {
    uint64_t tab[kWalkTab + 1];
    uint32_t bits[kN2v ? kWalkBits / 32 : 1];
    int32_t win[kN2v ? kWalkWin : 1];
};

// Entries of win[0, kWalkWin) below each of x[0..kWalkPer): four branch-free
// binary searches stepped together, so their LDS reads overlap. The window
// is padded with INT32_MAX; callers use a rank only for x no larger than the
// window's last real entry, where it is the lower bound among the real ones.
__device__ __forceinline__ void win_rank4(const int32_t* win, const int32_t (&x)[kWalkPer], int32_t (&r)[kWalkPer]) {
#pragma unroll
    for (int q = 0; q < kWalkPer; ++q) r[q] = 0;
#pragma unroll
    for (int step = kWalkWin / 2; step >= 1; step >>= 1) {
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) r[q] += win[r[q] + step - 1] < x[q] ? step : 0;
    }
}

// N(t) window loads: entries [at, at + kWalkWin) of col, clipped to te
__device__ __forceinline__ void load_window(const int32_t* __restrict__ col, int64_t at, int64_t te,
                                            int32_t (&y)[kWinPer]) {
    const int lane = lane_id();
#pragma unroll
    for (int q = 0; q < kWinPer; ++q) {
        const int64_t i = at + q * kWave + lane;
        y[q] = i < te ? col[i] : INT32_MAX;
    }
}

template <bool kN2v>
__device__ __forceinline__ int64_t walk_step_biased(const WalkParams& p, WalkLds<kN2v>& lds, Key key, uint32_t c0,
                                                    int32_t s, int32_t v, int64_t beg, int64_t d, int32_t t,
                                                    int64_t tb, int64_t te, bool& stop) {
    const int lane = lane_id();
    const int32_t* col = p.g.col;
    const uint32_t* wts = p.bias == kEdgeWeight ? p.g.ew : p.g.degw;
    // pass 1 reads weights (first-order) or neighbor ids (node2vec)
    const uint32_t* src = kN2v ? (const uint32_t*)col + beg : wts + beg;
    stop = false;
    int shift = 0;
    while (((d + ((int64_t)kWalkTile << shift) - 1) >> (kWalkTileLog + shift)) > kWalkTab) ++shift;
    const int64_t g = (int64_t)kWalkTile << shift;
    const int64_t ng = (d + g - 1) / g;
    const bool merge = kN2v && (te - tb) <= kMergeRatio * d + kWalkWin;
    int64_t jw = tb;  // N(t) window: win[0, wn) = col[jw, jw + wn)
    int32_t wn = 0;
    int32_t ynext[kWinPer];
    if (merge) load_window(col, jw, te, ynext);
    uint32_t cur[kWalkPer], nxt[kWalkPer];
#pragma unroll
    for (int q = 0; q < kWalkPer; ++q) {
        const int64_t idx = q * kWave + lane;
        cur[q] = idx < d ? src[idx] : 0u;
    }
    uint64_t run = 0;
    for (int64_t base = 0; base < d; base += kWalkTile) {
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {  // next tile in flight
            const int64_t idx = base + kWalkTile + q * kWave + lane;
            nxt[q] = idx < d ? src[idx] : 0u;
        }
        uint32_t x[kWalkPer];
        if (!kN2v) {
#pragma unroll
            for (int q = 0; q < kWalkPer; ++q) x[q] = cur[q];
        } else {
            int32_t a[kWalkPer];
            bool open[kWalkPer], found[kWalkPer];
#pragma unroll
            for (int q = 0; q < kWalkPer; ++q) {
                open[q] = base + q * kWave + lane < d;
                a[q] = (int32_t)cur[q];
                found[q] = false;
            }
            if (merge) {
                while (true) {
                    const int32_t wmax = wn > 0 ? lds.win[wn - 1] : INT32_MIN;
                    bool take[kWalkPer], any = false;
#pragma unroll
                    for (int q = 0; q < kWalkPer; ++q) {
                        take[q] = open[q] && a[q] <= wmax;
                        any |= take[q];
                    }
                    if (ballot(any)) {
                        int32_t r[kWalkPer];
                        win_rank4(lds.win, a, r);
#pragma unroll
                        for (int q = 0; q < kWalkPer; ++q) {
                            if (take[q]) {
                                found[q] = lds.win[r[q]] == a[q];
                                open[q] = false;
                            }
                        }
                    }
                    bool pending = false;
#pragma unroll
                    for (int q = 0; q < kWalkPer; ++q) pending |= open[q];
                    if (ballot(pending) == 0) break;
                    jw += wn;  // every entry of this window is below the open candidates
                    if (jw >= te) break;
                    wn = (int32_t)(te - jw < kWalkWin ? te - jw : kWalkWin);
                    wave_lds_sync();
#pragma unroll
                    for (int q = 0; q < kWinPer; ++q) lds.win[q * kWave + lane] = ynext[q];
                    wave_lds_sync();
                    load_window(col, jw + wn, te, ynext);  // the window after it, in flight
                }
            } else {
#pragma unroll
                for (int q = 0; q < kWalkPer; ++q)
                    if (open[q]) found[q] = in_sorted(col, tb, te, a[q]);
            }
#pragma unroll
            for (int q = 0; q < kWalkPer; ++q) {
                const int64_t idx = base + q * kWave + lane;
                const bool valid = idx < d;
                x[q] = !valid ? 0u : (a[q] == t ? p.w_return : (found[q] ? p.w_common : p.w_outward));
                const uint64_t fm = ballot(valid && found[q]);
                const int64_t i0 = base + q * kWave;
                if (i0 < kWalkBits && lane < 2) lds.bits[i0 / 32 + lane] = (uint32_t)(fm >> (32 * lane));
            }
        }
        uint64_t ls = 0;
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) ls += x[q];
        run += wave_sum_u64(ls);
        const int64_t tile = base >> kWalkTileLog;
        if (((tile + 1) & ((1ll << shift) - 1)) == 0 || base + kWalkTile >= d)
            if (lane == 0) lds.tab[(tile >> shift) + 1] = run;
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) cur[q] = nxt[q];
    }
    const uint64_t W = run;
    if (W == 0) {
        stop = true;
        return 0;
    }
    if (lane == 0) lds.tab[0] = 0;
    wave_lds_sync();
    const uint64_t r = draw(key, c0, (uint32_t)s, (uint32_t)v, 0u, W);
    int64_t lo = 0, hi = ng;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (lds.tab[mid] <= r) lo = mid;
        else hi = mid;
    }
    uint64_t acc = lds.tab[lo];
    const int64_t end = (lo + 1) * g < d ? (lo + 1) * g : d;
    int64_t m = end - 1;
    for (int64_t base = lo * g; base < end; base += kWave) {
        const int64_t idx = base + lane;
        uint32_t x = 0;
        if (idx < end) {
            if (!kN2v) {
                x = wts[beg + idx];
            } else {
                const int32_t a = col[beg + idx];
                const bool found = idx < kWalkBits ? ((lds.bits[idx >> 5] >> (idx & 31)) & 1u) != 0
                                                   : in_sorted(col, tb, te, a);
                x = a == t ? p.w_return : (found ? p.w_common : p.w_outward);
            }
        }
        const uint64_t incl = wave_incl_scan_u64(x);
        const uint64_t tot = readlane_u64(incl, kWave - 1);
        if (acc + tot > r) {
            m = base + __popcll(ballot(acc + incl <= r));
            break;
        }
        acc += tot;
    }
    wave_lds_sync();  // the table and bits are rewritten by the next step
    return m;
}

// node2vec step for lists of at most kWalkBits candidates. The bias of x is
// w_return (x = t), w_common (x in N(t)) or w_outward, so the prefix is fixed
// by the membership bits and the position of t: pass 1 only finds membership
// (merge of sorted N(v) with N(t) through the LDS window, a branch-free
// search per candidate), keeping one bit per candidate and their count;
// W = w_out (d - c - [t in N(v)]) + w_common c + w_return [t in N(v)]. Pass 2
// finds the 32-candidate word holding r from word popcounts (64 words per
// ballot) and the candidate inside it.
__device__ __forceinline__ int64_t walk_step_n2v(const WalkParams& p, WalkLds<true>& lds, Key key, uint32_t c0,
                                                 int32_t s, int32_t v, int64_t beg, int64_t d, int32_t t,
                                                 int64_t tb, int64_t te, bool& stop) {
    const int lane = lane_id();
    const int32_t* col = p.g.col;
    stop = false;
    const bool merge = (te - tb) <= kMergeRatio * d + kWalkWin;
    int64_t jw = tb;
    int32_t wn = 0;
    int32_t ynext[kWinPer];
    if (merge) load_window(col, jw, te, ynext);
    int32_t cur[kWalkPer], nxt[kWalkPer];
#pragma unroll
    for (int q = 0; q < kWalkPer; ++q) {
        const int64_t idx = q * kWave + lane;
        cur[q] = idx < d ? col[beg + idx] : 0;
    }
    uint64_t members = 0, nt = 0;  // candidates in N(t) other than t; copies of t
    int64_t pos_t = -1;            // first copy of t (sorted lists keep copies together)
    for (int64_t base = 0; base < d; base += kWalkTile) {
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {  // next tile in flight
            const int64_t idx = base + kWalkTile + q * kWave + lane;
            nxt[q] = idx < d ? col[beg + idx] : 0;
        }
        bool open[kWalkPer], found[kWalkPer];
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {
            open[q] = base + q * kWave + lane < d;
            found[q] = false;
        }
        if (merge) {
            while (true) {
                const int32_t wmax = wn > 0 ? lds.win[wn - 1] : INT32_MIN;
                bool take[kWalkPer], any = false;
#pragma unroll
                for (int q = 0; q < kWalkPer; ++q) {
                    take[q] = open[q] && cur[q] <= wmax;
                    any |= take[q];
                }
                if (ballot(any)) {
                    int32_t r[kWalkPer];
                    win_rank4(lds.win, cur, r);
#pragma unroll
                    for (int q = 0; q < kWalkPer; ++q) {
                        if (take[q]) {
                            found[q] = lds.win[r[q]] == cur[q];
                            open[q] = false;
                        }
                    }
                }
                bool pending = false;
#pragma unroll
                for (int q = 0; q < kWalkPer; ++q) pending |= open[q];
                if (ballot(pending) == 0) break;
                jw += wn;
                if (jw >= te) break;
                wn = (int32_t)(te - jw < kWalkWin ? te - jw : kWalkWin);
                wave_lds_sync();
#pragma unroll
                for (int q = 0; q < kWinPer; ++q) lds.win[q * kWave + lane] = ynext[q];
                wave_lds_sync();
                load_window(col, jw + wn, te, ynext);
            }
        } else {
#pragma unroll
            for (int q = 0; q < kWalkPer; ++q)
                if (open[q]) found[q] = in_sorted(col, tb, te, cur[q]);
        }
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {
            const bool valid = base + q * kWave + lane < d;
            const uint64_t fm = ballot(valid && found[q] && cur[q] != t);
            const uint64_t tm = ballot(valid && cur[q] == t);
            const int64_t i0 = base + q * kWave;
            if (lane < 2) lds.bits[i0 / 32 + lane] = (uint32_t)(fm >> (32 * lane));
            members += __popcll(fm);
            if (tm && pos_t < 0) pos_t = i0 + __ffsll((unsigned long long)tm) - 1;
            nt += __popcll(tm);
            cur[q] = nxt[q];
        }
    }
    const uint64_t wo = p.w_outward, wc = p.w_common, wr = p.w_return;
    const uint64_t W = wo * ((uint64_t)d - members - nt) + wc * members + wr * nt;
    if (W == 0) {
        stop = true;
        return 0;
    }
    wave_lds_sync();
    const uint64_t r = draw(key, c0, (uint32_t)s, (uint32_t)v, 0u, W);
    // S(i) = total bias of candidates [0, i) = wo (i - C - T) + wc C + wr T with
    // C members and T copies of t before i: find the word holding r
    const auto copies_before = [&](int64_t i) -> uint64_t {
        if (pos_t < 0 || i <= pos_t) return 0;
        return (uint64_t)(i - pos_t) < nt ? (uint64_t)(i - pos_t) : nt;
    };
    const int64_t nwords = (d + 31) / 32;
    int64_t wstar = 0;
    uint64_t Cw = 0, prevC = 0;  // members before the chosen word / before the last word of the previous run
    uint32_t carry = 0;
    for (int64_t w0 = 0; w0 < nwords; w0 += kWave) {
        const int64_t w = w0 + lane;
        const bool valid = w < nwords;
        const uint32_t pc = valid ? (uint32_t)__popc(lds.bits[w]) : 0u;
        const uint32_t incl = wave_incl_scan_u32(pc);
        const uint64_t C = (uint64_t)carry + (incl - pc);
        const int64_t i = w * 32;
        const uint64_t T = copies_before(i);
        const uint64_t S = wo * ((uint64_t)i - C - T) + wc * C + wr * T;
        const int nle = __popcll(ballot(valid && S <= r));
        const int nvalid = (int)(nwords - w0 < kWave ? nwords - w0 : kWave);
        if (nle < nvalid || w0 + kWave >= nwords) {  // the word holding r ends here
            if (nle == 0) {  // r starts this run: it is in the last word of the previous one
                wstar = w0 - 1;
                Cw = prevC;
            } else {
                wstar = w0 + nle - 1;
                Cw = readlane_u64(C, nle - 1);
            }
            break;
        }
        prevC = readlane_u64(C, kWave - 1);
        carry += readlane_u32(incl, kWave - 1);
    }
    const int64_t e0 = wstar * 32;
    const uint64_t Tw = copies_before(e0);
    const uint64_t Sw = wo * ((uint64_t)e0 - Cw - Tw) + wc * Cw + wr * Tw;
    const uint32_t word = lds.bits[wstar];
    const int64_t j = e0 + lane;
    uint64_t b = 0;
    if (lane < 32 && j < d)
        b = (pos_t >= 0 && j >= pos_t && (uint64_t)(j - pos_t) < nt) ? wr : (((word >> lane) & 1u) ? wc : wo);
    const uint64_t incl = wave_incl_scan_u64(b);
    const int64_t m = e0 + __popcll(ballot(lane < 32 && j < d && Sw + incl <= r));
    wave_lds_sync();  // bits are rewritten by the next step
    return m;
}

// First-order weighted step on a list of at most kWaveMaxD candidates, in one
// memory round trip: lane i loads candidates i, i + 64, ... of the list,
// weights and neighbor ids together (coalesced). The weights pass through LDS
// so that lane i holds the run [8i, 8i + 8); the lanes' totals are scanned,
// r is drawn in [0, W) and m = #{i : S_(i+1) <= r} (the candidate whose
// interval [S_i, S_(i+1)) holds r) is the number of whole runs below r plus
// the count inside the run that holds it. Returns the neighbor id.
// The step's Philox word on the vector unit. A walk step is wave-uniform, so
// its Philox rounds would otherwise run on the scalar unit (one per compute
// unit), which the step's other uniform work (addresses, loop control)
// already keeps busy; the vector unit forms each 32 x 32 -> 64-bit product in
// one instruction. The same rounds as philox_u64: the empty asm only places
// the counter words in vector registers. The caller takes it at the top of
// the step (the counter is known before any list data arrives) and reduces it
// to [0, W) with range_reduce once W is known.
__device__ __forceinline__ uint64_t philox_vec(Key key, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
    uint32_t k0 = key.k0, k1 = key.k1;
    asm volatile("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3), "+v"(k0), "+v"(k1));
    return (uint64_t)uniform_i64((int64_t)philox_u64(k0, k1, c0, c1, c2, c3));
}

constexpr int kShortPer = kWaveMaxD / kWave;  // 8
static_assert(sizeof(WalkLds<false>::tab) >= kWaveMaxD * sizeof(uint32_t), "short-list staging fits the LDS table");
__device__ __forceinline__ int32_t walk_step_short(const uint32_t* __restrict__ w, const int32_t* __restrict__ col,
                                                   uint32_t* sh, uint64_t u, int64_t beg, int32_t d, bool& stop) {
    const int lane = lane_id();
    uint32_t x[kShortPer];
    int32_t y[kShortPer];
#pragma unroll
    for (int q = 0; q < kShortPer; ++q) {
        const int32_t i = q * kWave + lane;
        const bool in = i < d;
        x[q] = in ? w[beg + i] : 0u;
        y[q] = in ? col[beg + i] : 0;
    }
#pragma unroll
    for (int q = 0; q < kShortPer; ++q) sh[q * kWave + lane] = x[q];
    wave_lds_sync();
    uint32_t a[kShortPer];
#pragma unroll
    for (int k = 0; k < kShortPer; ++k) a[k] = sh[lane * kShortPer + k];
    wave_lds_sync();  // the next step rewrites sh
    uint64_t t = 0;
#pragma unroll
    for (int k = 0; k < kShortPer; ++k) t += a[k];
    const uint64_t incl = wave_incl_scan_u64(t);
    const uint64_t W = readlane_u64(incl, kWave - 1);
    stop = W == 0;
    if (stop) return -1;
    const uint64_t r = range_reduce(u, W);
    const int L = __popcll(ballot(incl <= r));  // whole runs below r: lane L's run holds it
    uint64_t acc = incl - t;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kShortPer; ++k) {
        acc += a[k];
        c += acc <= r ? 1u : 0u;
    }
    const int32_t m = L * kShortPer + (int32_t)readlane_u32(c, L);
    const int qm = m / kWave;
    int32_t nb = y[0];
#pragma unroll
    for (int q = 1; q < kShortPer; ++q) nb = q == qm ? y[q] : nb;
    return readlane_i32(nb, m % kWave);
}

// First-order weighted step on a list longer than kWaveMaxD, through the
// graph's tables instead of a pass over the list: ctab holds the list's
// running total at the end of each 1024-weight chunk (so W is its last
// entry), gtab each chunk's inclusive 16-weight group prefixes. The chunk
// holding r is found by ballot over up to 64 running totals (lists of more
// than 64 chunks first narrow the range with 64 evenly spaced totals), the
// group by ballot over the chunk's 64 group prefixes, and the candidate from
// the group's 16 weights, loaded with their neighbor ids. Every sum is exact,
// so the pick is the one a scan of the whole list gives. Returns the neighbor.
constexpr int kWalkTotLoads = 4;  // lists of up to 4 * 64 chunks read every running total at once
__device__ __forceinline__ int32_t walk_step_long(const uint32_t* __restrict__ w, const int32_t* __restrict__ col,
                                                  const uint64_t* __restrict__ gtab,
                                                  const uint64_t* __restrict__ ctab, uint64_t u, int64_t beg, int64_t d,
                                                  bool& stop) {
    const int lane = lane_id();
    const int64_t row0 = beg >> kTabShift;
    const uint64_t* C = ctab + row0;
    const int64_t nch = (d + kChunk - 1) / kChunk;
    int64_t lo = 0, hi = nch;  // r lies in chunks [lo, hi)
    uint64_t acc = 0;          // running total before chunk lo
    uint64_t r = 0;
    bool drawn = false;
    int64_t j = 0;
    if (nch <= (int64_t)kWave * kWalkTotLoads) {
        // every running total at once: lane L holds totals q * 64 + L, all
        // loads issued before any is used (one memory round trip); j is the
        // number of totals at or below r (they never decrease)
        uint64_t e[kWalkTotLoads];
#pragma unroll
        for (int q = 0; q < kWalkTotLoads; ++q) {
            const int64_t i = (int64_t)q * kWave + lane;
            e[q] = ~0ull;
            if ((int64_t)q * kWave < nch && i < nch) e[q] = C[i];
        }
        const int64_t last = nch - 1;
        uint64_t el = e[0];
#pragma unroll
        for (int q = 1; q < kWalkTotLoads; ++q) el = q == (int)(last / kWave) ? e[q] : el;
        const uint64_t W = readlane_u64(el, (int)(last % kWave));  // total of the whole list
        stop = W == 0;
        if (stop) return -1;
        r = range_reduce(u, W);
        int64_t c = 0;
#pragma unroll
        for (int q = 0; q < kWalkTotLoads; ++q) c += __popcll(ballot(e[q] <= r));
        j = c;
        if (c > 0) {
            uint64_t ec = e[0];
#pragma unroll
            for (int q = 1; q < kWalkTotLoads; ++q) ec = q == (int)((c - 1) / kWave) ? e[q] : ec;
            acc = readlane_u64(ec, (int)((c - 1) % kWave));
        }
        lo = hi;  // done: skip the sampled search below
    }
    while (lo < hi) {
        const int64_t len = hi - lo;
        const int64_t stride = (len + kWave - 1) / kWave;
        const int64_t nb = (len + stride - 1) / stride;  // sampled totals (lanes in use)
        const bool in = lane < nb;
        int64_t idx = lo + (int64_t)(lane + 1) * stride - 1;
        idx = idx < hi ? idx : hi - 1;
        const uint64_t e = in ? C[idx] : ~0ull;
        if (!drawn) {
            const uint64_t W = readlane_u64(e, (int)nb - 1);  // total of the whole list
            stop = W == 0;
            if (stop) return -1;
            r = range_reduce(u, W);
            drawn = true;
        }
        const int c = __popcll(ballot(in && e <= r));  // sampled ranges ending at or below r
        if (c > 0) acc = readlane_u64(e, c - 1);
        if (stride == 1) {
            j = lo + c;
            break;
        }
        lo += (int64_t)c * stride;
        hi = lo + stride < hi ? lo + stride : hi;
    }
    const uint64_t gp = gtab[(row0 + j) * kChunkGroups + lane];  // inclusive prefix of groups 0..lane of chunk j
    const int gi = __popcll(ballot(acc + gp <= r));              // the group holding r
    const uint64_t before = acc + (gi > 0 ? readlane_u64(gp, gi - 1) : 0ull);
    const int64_t i0 = j * kChunk + (int64_t)gi * 16;
    const bool in = lane < 16 && i0 + lane < d;
    // the group's weights and ids at clamped positions, lanes past it zeroed
    const int64_t ii = beg + (in ? i0 + lane : i0);
    uint64_t x = (uint64_t)w[ii];
    const int32_t y = col[ii];
    x = in ? x : 0ull;
    const uint64_t incl = wave_incl_scan_u64(x);
    const int k = __popcll(ballot(in && before + incl <= r));
    return readlane_i32(y, k);
}

// First-order weighted step on a list longer than kWaveMaxD through its walk
// guide, one wavefront per walker: r's bucket names the pick (one load after
// the row offsets and the list's total) or the first position that can be it;
// then the edge records from there on, 64 at a time, exact prefixes beside
// neighbor ids. Returns the neighbor.
__device__ __forceinline__ int32_t walk_step_guide(const WalkEdge* __restrict__ er, const WalkBucket* __restrict__ gd,
                                                   int per, uint64_t r, uint64_t W, int64_t beg, int64_t d, int64_t v) {
    const int lane = lane_id();
    const int sh = guide_shift(W, d, per);
    const uint64_t k = r >> sh;
    const WalkBucket* q = gd + guide_base(beg, v, per) + k;
    const WalkBucket b{ld_uniform(&q->S), ld_uniform(&q->pos), ld_uniform(&q->col)};
    if ((uint32_t)(b.S >> 32) != ~0u)
        return (uint32_t)(r - (k << sh)) >= (uint32_t)b.S ? (int32_t)(b.S >> 32) : b.col;
    for (int64_t lo = b.pos;; lo += kWave) {
        // both loads issued at clamped positions (the list's last prefix
        // exceeds r): guarded loads were waited for one after the other
        const int64_t j = beg + (lo + lane < d ? lo + lane : d - 1);
        const uint64_t S = er[j].S;
        const int32_t y = er[j].col;
        __builtin_amdgcn_sched_barrier(0);  // both loads in flight before either is used
        const int c = __popcll(ballot(S <= r));
        if (c < kWave) return readlane_i32(y, c);
    }
}

// node2vec step from v when the previous vertex t has a short list (fewer
// than 64 entries) and N(v) a long one: instead of merging all of N(v) with
// N(t), lane k takes the k-th entry x of N(t) and binary-searches both ends
// of x's run in N(v) (lane d_t does the same for t itself), so membership
// costs about log2(d_v) dependent loads whatever d_v is. The pick is found
// without reading N(v) again: with C(j) = common candidates below position j
// (a wave sum over the lanes' runs; a repeated x counts once) and T(j) =
// copies of t below j, the exclusive prefix is
// S(j) = w_out (j - C - T) + w_common C + w_return T, and m is the smallest i
// with S(i + 1) > r, by binary search over i: the same m as the merge.
constexpr int64_t kShortPrevMinD = 2048;  // shorter N(v): the merge is cheaper
__device__ __forceinline__ int64_t walk_step_n2v_short_prev(const WalkParams& p, Key key, uint32_t c0, int32_t s,
                                                            int32_t v, int64_t beg, int64_t d, int32_t t,
                                                            int64_t tb, int64_t te, bool& stop) {
    const int lane = lane_id();
    const int32_t* __restrict__ col = p.g.col;
    const int64_t dt = te - tb;  // < kWave
    const bool act = lane <= dt;
    const int32_t x = lane < dt ? col[tb + lane] : t;
    // [lo1, lo2): the run of x in N(v) (lower and upper bound, side by side)
    int64_t lo1 = 0, hi1 = act ? d : 0, lo2 = 0, hi2 = act ? d : 0;
    while (ballot(lo1 < hi1 || lo2 < hi2)) {
        const bool s1 = lo1 < hi1, s2 = lo2 < hi2;
        const int64_t m1 = (lo1 + hi1) >> 1, m2 = (lo2 + hi2) >> 1;
        const int32_t y1 = col[beg + (s1 ? m1 : 0)];
        const int32_t y2 = col[beg + (s2 ? m2 : 0)];
        if (s1) {
            if (y1 < x) lo1 = m1 + 1;
            else hi1 = m1;
        }
        if (s2) {
            if (y2 <= x) lo2 = m2 + 1;
            else hi2 = m2;
        }
    }
    const int32_t xprev = __shfl_up(x, 1, kWave);
    const bool common = lane < dt && (lane == 0 || xprev != x) && x != t && lo2 > lo1;
    const int64_t cnt = lo2 - lo1;
    const int64_t pos_t = readlane_i64(lo1, (int)dt);
    const int64_t n_t = readlane_i64(lo2, (int)dt) - pos_t;
    const uint64_t c = (uint64_t)wave_sum_i64(common ? cnt : 0);
    const uint64_t wo = p.w_outward, wc = p.w_common, wr = p.w_return;
    const uint64_t W = wo * ((uint64_t)d - c - (uint64_t)n_t) + wc * c + wr * (uint64_t)n_t;
    stop = W == 0;
    if (stop) return 0;
    const uint64_t r = draw(key, c0, (uint32_t)s, (uint32_t)v, 0u, W);
    int64_t a = 0, b = d - 1;  // S(d) = W > r
    while (a < b) {
        const int64_t mid = (a + b) >> 1, j = mid + 1;
        const int64_t below = j - lo1 < 0 ? 0 : (j - lo1 < cnt ? j - lo1 : cnt);
        const uint64_t C = (uint64_t)wave_sum_i64(common ? below : 0);
        const uint64_t T = j <= pos_t ? 0 : (uint64_t)(j - pos_t < n_t ? j - pos_t : n_t);
        const uint64_t S = wo * ((uint64_t)j - C - T) + wc * C + wr * T;
        if (S > r) b = mid;
        else a = mid + 1;
    }
    return a;
}

template <bool kN2v, bool kMoves>
__device__ __forceinline__ void walk_wave_body(const WalkParams& p) {
    __shared__ WalkLds<kN2v> lds_all[kWavesPerBlock];
    const int lane = lane_id();
    const int wid = uniform_i32(threadIdx.x / kWave);
    WalkLds<kN2v>& lds = lds_all[wid];
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t w = blockIdx.x * (int64_t)kWavesPerBlock + wid; w < p.num_walkers; w += waves) {
        const WalkerCtx wc = walker_ctx(p, w);
        const Key key{(uint32_t)uniform_i32((int32_t)wc.key.k0), (uint32_t)uniform_i32((int32_t)wc.key.k1)};
        const int32_t length = uniform_i32(wc.length);
        const int64_t L1 = (int64_t)length + 1;
        int32_t* path = wc.path;
        int32_t v = uniform_i32(p.starts[w]);
        if (v < 0 || (int64_t)v >= p.g.n) {
            if (lane == 0) *p.bad_start = 1;
            for (int64_t q = lane; q < L1; q += kWave) path[q] = -1;
            continue;
        }
        if (lane == 0) path[0] = v;
        const uint32_t c0 = (uint32_t)uniform_i32((int32_t)wc.c0);
        const int32_t start = v;
        int32_t t = -1;
        int64_t tb = 0, te = 0;
        int32_t s = 0;
        for (; s < length; ++s) {
            int32_t to;
            if (kMoves && walk_move(p, key, c0, s, v, start, to)) {  // uniform: the draw depends on wave-uniform values
                if (lane == 0) path[s + 1] = to;
                v = to;
                t = -1;
                tb = te = 0;
                continue;
            }
            int64_t beg, d;
            row_uniform(p.g.rowptr, v, beg, d);
            // first-order steps: the list's total (for the walk guide) with the
            // row offsets, and the draw's Philox word while they load
            uint64_t u = 0, wt = 0;
            if constexpr (!kN2v) {
                const bool dg = p.bias == kNeighborDegree;
                const uint64_t* tots = dg ? p.g.wtot_deg : p.g.wtot_ew;
                if ((dg ? p.g.wgd_deg : p.g.wgd_ew) != nullptr) wt = ld_uniform(tots + v);
                u = philox_vec(key, c0, (uint32_t)s, (uint32_t)v, 0u);
            }
            if (d == 0) break;
            int64_t m = -1;  // position of the pick (paths that return the neighbor itself leave -1)
            int32_t nx = -1;
            bool stop = false;
            if (kN2v && t < 0) {  // first step: no previous vertex, every bias is 1
                m = (int64_t)draw(key, c0, (uint32_t)s, (uint32_t)v, 0u, (uint64_t)d);
            } else {
                if constexpr (kN2v) {
                    if (te - tb < kWave && d >= kShortPrevMinD)
                        m = walk_step_n2v_short_prev(p, key, c0, s, v, beg, d, t, tb, te, stop);
                    else if (d <= kWalkBits) m = walk_step_n2v(p, lds, key, c0, s, v, beg, d, t, tb, te, stop);
                    else m = walk_step_biased<true>(p, lds, key, c0, s, v, beg, d, t, tb, te, stop);
                } else {
                    const bool dg = p.bias == kNeighborDegree;
                    const uint32_t* wts = dg ? p.g.degw : p.g.ew;
                    const uint64_t* gt = dg ? p.g.gtab_deg : p.g.gtab_ew;
                    const uint64_t* ct = dg ? p.g.ctab_deg : p.g.ctab_ew;
                    const WalkEdge* er = dg ? p.g.wrec_deg : p.g.wrec_ew;
                    const WalkBucket* gd = dg ? p.g.wgd_deg : p.g.wgd_ew;
                    if (d <= kWaveMaxD || (gt && ct)) {
                        if (d <= kWaveMaxD) {
                            nx = walk_step_short(wts, p.g.col, reinterpret_cast<uint32_t*>(lds.tab), u, beg, (int32_t)d,
                                                 stop);
                        } else {
                            if (gd) {
                                stop = wt == 0;
                                if (!stop)
                                    nx = walk_step_guide(er, gd, dg ? p.g.gper_deg : p.g.gper_ew, range_reduce(u, wt), wt, beg,
                                                         d, v);
                            } else {
                                nx = walk_step_long(wts, p.g.col, gt, ct, u, beg, d, stop);
                            }
                        }
                    } else {
                        m = walk_step_biased<false>(p, lds, key, c0, s, v, beg, d, t, tb, te, stop);
                    }
                }
                if (stop) break;
            }
            if (m >= 0) nx = ld_uniform(p.g.col + beg + m);
            nx = uniform_i32(nx);
            if (lane == 0) path[s + 1] = nx;
            t = v;
            tb = beg;
            te = beg + d;
            v = nx;
        }
        for (int64_t q = s + 1 + lane; q < L1; q += kWave) path[q] = -1;
        if (lane == 0 && s) atomicAdd(wc.steps, (unsigned long long)s);
    }
}

// First-order walks are bound by the latency of their dependent loads, so
// they are held to 8 waves per SIMD (the scalar registers this needs spill
// to vector lanes, not to memory); walks with restart / jump moves and
// node2vec keep their larger register sets.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) k_walk_wave_first(WalkParams p) {
    walk_wave_body<false, false>(p);
}

__global__ void __launch_bounds__(kBlock) k_walk_wave_moves(WalkParams p) {
    walk_wave_body<false, true>(p);
}

template <bool kMoves>
__global__ void __launch_bounds__(kBlock) k_walk_wave_n2v(WalkParams p) {
    walk_wave_body<true, kMoves>(p);
}

// Weighted first-order walks through the walk guide, one lane per walker
// (64 walkers per wavefront, each with its own chain of loads). A step:
// the vertex's record, its list and total W (one 16-byte load; the Philox
// word is formed meanwhile), r = floor(u W / 2^64), and r's bucket (one 16-byte
// load), which names the pick nine times in ten; else the edge records of
// kLaneProbe positions at a time from the bucket's first one on, exact prefixes
// beside neighbor ids: m = lo + #{j : S_(lo+j+1) <= r}. The walk is bound by
// the 128-byte lines these scattered reads pull from HBM and by the number of
// scattered reads, so a step makes two where it can: 262,144 walkers x 80 on
// 500M edges took 1.05 ms with pairs of buckets of one position each, two
// per edge; 0.83 ms with this (0.91 with two buckets per edge, 0.76 with eight). (One 128-byte block per two to four positions, with each
// neighbor's own list in it, is one line a step but three or more reads of it, and took
// 1.36 ms; 2.5 ms reading the block whole.) Positions
// past the list's end are read at its end instead, whose prefix exceeds r,
// so every load stays inside the list and needs no mask. The pick is the same m
// as a scan of the whole list.
constexpr int kLaneProbe = 4;
// A lane's round waits for the slowest of its wavefront's 64 scattered loads, so
// an unloaded lane step takes longer than a wavefront's (3.1 against 1.4 us at
// 2,048 walkers); the lane kernel wins once a launch has enough walkers to keep
// many lanes' chains in flight (length 80 on 500M edges: 255 against 205 us at 8,192
// walkers, 261 against 263 at 12,288, 276 against 338 at 16,384).
constexpr int64_t kLaneWalkMin = 12288;

template <bool kMoves, int kRun>
__global__ void __launch_bounds__(kBlock) k_walk_lane(WalkParams p) {
    const bool dg = p.bias == kNeighborDegree;
    const WalkVertex* __restrict__ vt = dg ? p.g.wvtx_deg : p.g.wvtx_ew;
    const WalkEdge* __restrict__ er = dg ? p.g.wrec_deg : p.g.wrec_ew;
    const WalkBucket* __restrict__ gd = dg ? p.g.wgd_deg : p.g.wgd_ew;
    const int per = dg ? p.g.gper_deg : p.g.gper_ew;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t w0 = blockIdx.x * (int64_t)blockDim.x; w0 < p.num_walkers; w0 += stride) {
        const int64_t w = w0 + threadIdx.x;
        int64_t my_steps = 0;
        unsigned long long* my_counter = p.steps;
        if (w < p.num_walkers) {
            const WalkerCtx wc = walker_ctx(p, w);
            const Key key = wc.key;
            const int64_t L1 = (int64_t)wc.length + 1;
            int32_t* path = wc.path;
            my_counter = wc.steps;
            int32_t v = p.starts[w];
            int32_t s = 0;
            if (v < 0 || (int64_t)v >= p.g.n) {
                *p.bad_start = 1;
                for (int64_t q = 0; q < L1; ++q) path[q] = -1;
            } else {
                path[0] = v;
                const int32_t start = v;
                const uint32_t c0 = wc.c0;
                PathRun<kRun> run;
                for (; s < wc.length; ++s) {
                    int32_t to;
                    if (kMoves && walk_move(p, key, c0, s, v, start, to)) {
                        v = to;
                    } else {
                        const WalkVertex x = vt[v];
                        const int64_t beg = x.beg, d = x.d;
                        const uint64_t W = x.W;
                        uint64_t u = philox_u64(key.k0, key.k1, c0, (uint32_t)s, (uint32_t)v, 0u);
                        // formed while the offsets load, not sunk past the test below
                        asm volatile("" : "+v"(u));
                        if (d == 0 || W == 0) break;
                        const uint64_t r = range_reduce(u, W);
                        const int sh = guide_shift(W, d, per);
                        const uint64_t k = r >> sh;
                        const WalkBucket bk = (gd + guide_base(beg, v, per))[k];
                        int32_t nx = (uint32_t)(r - (k << sh)) >= (uint32_t)bk.S ? (int32_t)(bk.S >> 32) : bk.col;
                        if ((uint32_t)(bk.S >> 32) == ~0u) {
                            for (int64_t lo = bk.pos;; lo += kLaneProbe) {
                                uint64_t S[kLaneProbe];
                                int32_t y[kLaneProbe];
#pragma unroll
                                for (int j = 0; j < kLaneProbe; ++j) {
                                    const uint4 e = *(const uint4*)(er + beg + (lo + j < d ? lo + j : d - 1));
                                    S[j] = (uint64_t)e.x | ((uint64_t)e.y << 32);
                                    y[j] = (int32_t)e.z;
                                }
                                int c = 0;
#pragma unroll
                                for (int j = 0; j < kLaneProbe; ++j) c += S[j] <= r ? 1 : 0;
                                nx = y[0];
#pragma unroll
                                for (int j = 1; j < kLaneProbe; ++j) nx = c == j ? y[j] : nx;
                                if (c < kLaneProbe) break;
                            }
                        }
                        v = nx;
                    }
                    run.push(path, v);
                }
                run.flush(path);
                for (int64_t q = s + 1; q < L1; ++q) path[q] = -1;
            }
            my_steps = s;
        }
        if (p.batch.req) {
            count_steps(my_steps, my_counter);
        } else {
            const int64_t ws = wave_sum_i64(my_steps);
            if (lane_id() == 0 && ws) atomicAdd(p.steps, (unsigned long long)ws);
        }
    }
}

// The same, one wavefront per walker, for launches of too few walkers for the
// lanes: what counts is one walker's chain of loads, the vertex's record and the
// bucket (and one time in ten the edge records, 64 at a time), both read
// through the scalar cache while the vector unit forms the draw. Path entries
// are kept one per lane and written 64 at a time. 4,000 walkers x 2,000 on 500M
// edges: 3.63 ms with row offsets and total read apart, pairs of buckets
// and lists of at most 512 scanned whole, 3.55 with these buckets, 2.62 here.
template <bool kMoves>
__global__ void __launch_bounds__(kBlock) k_walk_wave_guide(WalkParams p) {
    const int lane = lane_id();
    const int wid = uniform_i32(threadIdx.x / kWave);
    const bool dg = p.bias == kNeighborDegree;
    const WalkVertex* __restrict__ vt = dg ? p.g.wvtx_deg : p.g.wvtx_ew;
    const WalkEdge* __restrict__ er = dg ? p.g.wrec_deg : p.g.wrec_ew;
    const WalkBucket* __restrict__ gd = dg ? p.g.wgd_deg : p.g.wgd_ew;
    const int per = dg ? p.g.gper_deg : p.g.gper_ew;
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t w = blockIdx.x * (int64_t)kWavesPerBlock + wid; w < p.num_walkers; w += waves) {
        const WalkerCtx wc = walker_ctx(p, w);
        const Key key{(uint32_t)uniform_i32((int32_t)wc.key.k0), (uint32_t)uniform_i32((int32_t)wc.key.k1)};
        const int32_t length = uniform_i32(wc.length);
        const int64_t L1 = (int64_t)length + 1;
        int32_t* path = wc.path;
        int32_t v = uniform_i32(p.starts[w]);
        if (v < 0 || (int64_t)v >= p.g.n) {
            if (lane == 0) *p.bad_start = 1;
            for (int64_t q = lane; q < L1; q += kWave) path[q] = -1;
            continue;
        }
        const uint32_t c0 = (uint32_t)uniform_i32((int32_t)wc.c0);
        const int32_t start = v;
        int32_t mine = v;  // path entry i is kept by lane i % 64
        int32_t s = 0;
        for (; s < length; ++s) {
            int32_t to;
            if (kMoves && walk_move(p, key, c0, s, v, start, to)) {  // uniform: the draw depends on wave-uniform values
                v = uniform_i32(to);
            } else {
                const uint64_t W = ld_uniform(&vt[v].W);
                const int64_t beg = ld_uniform(&vt[v].beg), d = ld_uniform(&vt[v].d);
                const uint64_t u = philox_vec(key, c0, (uint32_t)s, (uint32_t)v, 0u);
                if (d == 0 || W == 0) break;
                v = walk_step_guide(er, gd, per, range_reduce(u, W), W, beg, d, v);
            }
            const int32_t i = s + 1;
            if (lane == (i & (kWave - 1))) mine = v;
            if ((i & (kWave - 1)) == kWave - 1) path[i - (kWave - 1) + lane] = mine;
        }
        const int32_t i0 = s & ~(kWave - 1);  // entries [i0, s] are still in the lanes, unless they fill them
        if ((s & (kWave - 1)) != kWave - 1 && lane <= s - i0) path[i0 + lane] = mine;
        for (int64_t q = (int64_t)s + 1 + lane; q < L1; q += kWave) path[q] = -1;
        if (lane == 0 && s) atomicAdd(wc.steps, (unsigned long long)s);
    }
}

// node2vec through the rank index. A step needs, of the common neighbors of v
// and the previous vertex t, how many there are and where those up to the
// pick stand in N(v). The entries of the shorter list are looked up in the longer
// one (on R-MAT 24 a step's lists have 900 and 8,500 entries on average), where
// a merge reads both. With C(j) = common candidates below position j of
// N(v) and T(j) = copies of t below j, the exclusive prefix is
// S(j) = w_out (j - C - T) + w_common C + w_return T, and S fixes the pick without
// another pass: the last common candidate that begins at or below the draw gives C, the
// rest is a division.
// 65,536 walkers of length 80 on 500M edges: 95.4 ms merging, 34 with every
// entry looked up in memory where the longer list has 3 times the entries and a merge elsewhere,
// 31 with every entry looked up, 28 with the dense stretches staged in LDS,
// 25.0 with the next chunks' loads issued a block ahead, 24.3 at six waves per
// SIMD (five or seven: 25.1, 25.3). The vector unit is then busy 45% of the
// time, the address units 54%, and 179 GB come from beyond the L2s (7.3 TB/s).
constexpr int kRankQ = 4;                        // chunks of 64 entries looked up together
constexpr uint32_t kRankWin = 256 * kRankQ;      // entries of the longer list staged for them
struct RankStep {
    const int32_t* sh;     // the shorter list
    uint32_t ns;
    const int32_t* lg;     // the longer one
    uint32_t nl, lg_at;    // its entries; its first edge (low bits)
    const uint32_t* rank;  // its rank index (nl >= kRankMinD)
    int bits;              // the index's shift
    bool of_t;             // the shorter list is N(t)
    int32_t t;
    int32_t* win;          // LDS, kRankWin entries
};
struct alignas(4) RankPair {
    uint32_t lo, hi;
};
struct alignas(16) RankQuad {
    int32_t e[4];
};

// Entry i of a list: 32-bit byte offsets (lists are shorter than 2^30).
__device__ __forceinline__ int32_t list_at(const int32_t* list, uint32_t i) {
    return *(const int32_t*)((const char*)list + (i << 2));
}

// The stretch of the longer list that ids x0 to x1 span, from the index.
__device__ __forceinline__ void rank_span(const RankStep& st, int32_t x0, int32_t x1, uint32_t& lo, uint32_t& len) {
    lo = 0;
    len = st.nl;
    if (st.nl >= kRankMinD) {
        lo = ld_uniform(st.rank + ((uint32_t)x0 >> st.bits));
        len = ld_uniform(st.rank + (((uint32_t)x1 >> st.bits) + 1)) - lo;
    }
}

// Where n entries x of the shorter list (an entry a lane, Q chunks) stand in the
// longer one, and whether they are in it (a copy, if it is repeated); they span its
// entries [lo, lo + len). Where that is up to four times as many as they are, the
// stretch is staged in LDS and searched there: each line is read once (up to
// twice as many: 28.1 against 25.0 ms, eight times: the 8 KB a wave that needs cost more
// than it gave). Otherwise every entry has its own range from the index, which
// in lists of 10,000 leaves four to five of 13 halvings, Q loads in flight.
// ahead() issues the loads of the chunks that follow.
template <int Q, typename Ahead>
__device__ __forceinline__ void rank_find(const RankStep& st, uint32_t n, const int32_t (&x)[Q], uint32_t lo, uint32_t len,
                                          uint32_t (&pos)[Q], bool (&hit)[Q], const Ahead& ahead) {
    const uint32_t lane = lane_id();
    if (len <= 256 * Q - 4) {
        // whole 16-byte quads of the column ids (whose array is padded to one); what lies
        // outside the stretch becomes -1 and the largest int
        const uint32_t skew = (st.lg_at + lo) & 3u, top = skew + len;
        const int32_t* from = st.lg + (int64_t)lo - skew;
        const int log = top < 256 ? 8 : 32 - __builtin_clz(top);  // 2^log > top
        RankQuad y[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const uint32_t i = (k * kWave + lane) * 4;
            if (k * 256u < top) y[k] = *(const RankQuad*)((const char*)from + ((i < top ? i : 0u) << 2));
        }
        ahead();
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            if (k * 256u < (1u << log)) {
                const uint32_t i = (k * kWave + lane) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) y[k].e[j] = i + j >= top ? INT32_MAX : (i + j < skew ? -1 : y[k].e[j]);
                *(RankQuad*)(st.win + i) = y[k];
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < Q; ++q) pos[q] = 0;
        for (uint32_t step = 1u << (log - 1); step; step >>= 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q) pos[q] += st.win[pos[q] + step - 1] < x[q] ? step : 0u;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            hit[q] = q * kWave + lane < n && st.win[pos[q]] == x[q];
            pos[q] += lo - skew;
        }
        wave_lds_sync();
        return;
    }
    ahead();
    uint32_t hi[Q];
    RankPair r[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) r[q] = *(const RankPair*)((const char*)st.rank + (((uint32_t)x[q] >> st.bits) << 2));
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        pos[q] = r[q].lo;
        hi[q] = q * kWave + lane < n ? r[q].hi : r[q].lo;
        hit[q] = false;
    }
    while (true) {
        bool more = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) more |= pos[q] < hi[q];
        if (ballot(more) == 0) break;
        uint32_t mid[Q];
        int32_t y[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            mid[q] = pos[q] < hi[q] ? (pos[q] + hi[q]) >> 1 : 0u;
            y[q] = list_at(st.lg, mid[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool open = pos[q] < hi[q], eq = open && y[q] == x[q], lt = y[q] < x[q];
            hit[q] |= eq;
            hi[q] = open && !lt ? mid[q] : hi[q];
            pos[q] = eq ? mid[q] : (open && lt ? mid[q] + 1 : pos[q]);
        }
    }
}

// The copies of x around position pos of the longer list (one of them): pos
// becomes the first.
__device__ __forceinline__ uint32_t rank_run(const RankStep& st, int32_t x, uint32_t& pos) {
    uint32_t lo = 0, hi = pos, lo2 = pos + 1, hi2 = st.nl;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (list_at(st.lg, mid) < x) lo = mid + 1;
        else hi = mid;
    }
    while (lo2 < hi2) {
        const uint32_t mid = (lo2 + hi2) >> 1;
        if (list_at(st.lg, mid) <= x) lo2 = mid + 1;
        else hi2 = mid;
    }
    pos = lo;
    return lo2 - lo;
}

// The copies of t in the longer list, N(v), by the whole wavefront: one load
// where its range has at most 64 entries, else one more for each 64-fold.
template <bool kRepeats>
__device__ __forceinline__ void rank_find_t(const RankStep& st, uint32_t& pos_t, uint32_t& n_t) {
    const uint32_t lane = lane_id();
    uint32_t lo = 0, hi = st.nl;
    if (st.nl >= kRankMinD) {
        const uint32_t k = (uint32_t)st.t >> st.bits;
        lo = ld_uniform(st.rank + k);
        hi = ld_uniform(st.rank + (k + 1));
    }
    while (hi - lo > (uint32_t)kWave) {  // the first entry >= t lies in [lo, hi]
        const uint32_t seg = (hi - lo + kWave - 1) / kWave, i = lo + lane * seg;
        const uint32_t below = (uint32_t)__popcll(ballot(i < hi && list_at(st.lg, i < hi ? i : lo) < st.t));
        if (below == 0) {
            hi = lo + 1;
        } else {
            hi = lo + below * seg + 1 < hi ? lo + below * seg + 1 : hi;
            lo += (below - 1) * seg + 1;
        }
    }
    const uint32_t i = lo + lane;
    const int32_t y = i < hi ? list_at(st.lg, i) : INT32_MAX;
    pos_t = lo + (uint32_t)__popcll(ballot(y < st.t));
    n_t = (uint32_t)__popcll(ballot(y == st.t));
    if (kRepeats && n_t) {
        n_t = rank_run(st, st.t, pos_t);
        pos_t = (uint32_t)uniform_i32((int32_t)pos_t);
        n_t = (uint32_t)uniform_i32((int32_t)n_t);
    }
}

// Q chunks of the shorter list from entry base on, an entry a lane.
template <int Q>
__device__ __forceinline__ uint32_t rank_load(const RankStep& st, uint32_t base, int32_t (&x)[Q]) {
    const uint32_t lane = lane_id();
    const uint32_t n = st.ns - base < (uint32_t)(Q * kWave) ? st.ns - base : (uint32_t)(Q * kWave);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t i = q * kWave + lane;
        x[q] = list_at(st.sh, base + (i < n ? i : 0u));
    }
    return n;
}

// Their positions in N(v), and cnt[q] = common candidates there (t itself is
// none), from their places in the longer list. Where the shorter list is N(v), adds to the copies
// of t and sets the first one's position.
template <bool kRepeats, int Q>
__device__ __forceinline__ void rank_count(const RankStep& st, uint32_t base, const int32_t (&x)[Q], const bool (&hit)[Q],
                                           uint32_t (&pos)[Q], uint32_t (&cnt)[Q], uint32_t& pos_t, uint32_t& n_t) {
    const uint32_t lane = lane_id();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t i = base + q * kWave + lane;
        cnt[q] = hit[q] && x[q] != st.t ? 1u : 0u;
        if (!st.of_t) {
            pos[q] = i;
            const uint64_t at_t = ballot(i < st.ns && x[q] == st.t);
            if (at_t) {
                if (n_t == 0) pos_t = base + q * kWave + __ffsll((unsigned long long)at_t) - 1;
                n_t += (uint32_t)__popcll(at_t);
            }
        } else if (kRepeats) {
            uint32_t run = 0;
            if (hit[q]) run = rank_run(st, x[q], pos[q]);
            const bool again = i > 0 && i < st.ns && list_at(st.sh, i - 1) == x[q];  // counted at its first copy
            cnt[q] = again || x[q] == st.t ? 0u : run;
            if (again) pos[q] += run;
        }
    }
}

// One chunk, its loads one after the other.
template <bool kRepeats>
__device__ __forceinline__ void rank_chunk(const RankStep& st, uint32_t base, uint32_t& pos, uint32_t& cnt, uint32_t& pos_t,
                                           uint32_t& n_t) {
    int32_t x[1];
    uint32_t at[1], c[1], lo, len;
    bool hit[1];
    const uint32_t n = rank_load(st, base, x);
    rank_span(st, ld_uniform(st.sh + base), ld_uniform(st.sh + (base + n - 1)), lo, len);
    rank_find(st, n, x, lo, len, at, hit, [] {});
    rank_count<kRepeats>(st, base, x, hit, at, c, pos_t, n_t);
    pos = at[0];
    cnt = c[0];
}

// floor(a / w) where it is below 2^30: inv = 1 / w in double gives it to within one.
__device__ __forceinline__ uint32_t small_quotient(uint64_t a, uint32_t w, double inv) {
    uint32_t q = (uint32_t)((double)a * inv);
    if ((uint64_t)q * w > a) --q;
    else if ((uint64_t)(q + 1) * w <= a) ++q;
    return q;
}

// Lane k keeps the first position of chunk k << g and the common candidates
// before it (g > 0 above 4,096 entries), so one chunk in 64 is looked
// up again to find the pick, or none if it is among the last ones looked up.
template <bool kRepeats>
__device__ __forceinline__ uint32_t walk_step_rank(const WalkParams& p, const RankStep& st, uint64_t u, uint32_t d,
                                                   const double (&inv)[3], bool& stop) {
    const int lane = lane_id();
    const uint32_t chunks = (st.ns + kWave - 1) / kWave;
    int g = 0;
    while (chunks > (uint32_t)kWave << g) ++g;
    const uint32_t low = (1u << g) - 1;
    uint32_t pos_t = 0, n_t = 0, c = 0;
    uint32_t at_pos = 0, at_c = 0;
    if (st.of_t) rank_find_t<kRepeats>(st, pos_t, n_t);
    // chunk k is done: its table entry, its common candidates
    const auto take = [&](uint32_t k, uint32_t pos, uint32_t cnt) {
        if ((k & low) == 0) {
            const uint32_t first = readlane_u32(pos, 0);
            if (lane == (int)(k >> g)) {
                at_pos = first;
                at_c = c;
            }
        }
        c += kRepeats ? (uint32_t)readlane_u32(wave_incl_scan_u32(cnt), kWave - 1)
                        : (uint32_t)__popcll(ballot(cnt != 0));
    };
    uint32_t pos[kRankQ], cnt[kRankQ];  // of the last chunks looked up, from chunk kept on
    uint32_t kept = 0, k = 0;
    if (chunks > 1) {
        int32_t xn[kRankQ];
        uint32_t lo, len, n = rank_load(st, 0, xn);
        rank_span(st, ld_uniform(st.sh), ld_uniform(st.sh + (n - 1)), lo, len);
        const auto first = [&](uint32_t at) { return ld_uniform(st.sh + (at < st.ns ? at : st.ns - 1)); };
        int32_t x0 = first(kRankQ * kWave), x1 = first(2 * kRankQ * kWave - 1);
        for (; k + 1 < chunks; k += kRankQ) {
            int32_t x[kRankQ];
            bool hit[kRankQ];
#pragma unroll
            for (int q = 0; q < kRankQ; ++q) x[q] = xn[q];
            const uint32_t base = k * kWave, m = n, lo1 = lo, len1 = len;
            rank_find(st, m, x, lo1, len1, pos, hit, [&] {
                if (k + kRankQ + 1 < chunks) {
                    n = rank_load(st, base + kRankQ * kWave, xn);
                    rank_span(st, x0, x1, lo, len);
                    x0 = first(base + 2 * kRankQ * kWave);
                    x1 = first(base + 3 * kRankQ * kWave - 1);
                }
            });
            rank_count<kRepeats>(st, base, x, hit, pos, cnt, pos_t, n_t);
#pragma unroll
            for (int q = 0; q < kRankQ; ++q)
                if (k + q < chunks) take(k + q, pos[q], cnt[q]);
            kept = k;
        }
    }
    if (k < chunks) {
        rank_chunk<kRepeats>(st, k * kWave, pos[0], cnt[0], pos_t, n_t);
        take(k, pos[0], cnt[0]);
        kept = k;
    }
    const uint32_t wo = p.w_outward, wc = p.w_common, wr = p.w_return;
    const uint64_t W = (uint64_t)wo * (d - c - n_t) + (uint64_t)wc * c + (uint64_t)wr * n_t;
    stop = W == 0;
    if (stop) return 0;
    const uint64_t r = range_reduce(u, W);
    const auto prefix = [&](uint32_t j, uint32_t C) {
        const uint32_t T = j <= pos_t ? 0u : (j - pos_t < n_t ? j - pos_t : n_t);
        return (uint64_t)wo * (j - C - T) + (uint64_t)wc * C + (uint64_t)wr * T;
    };
    const int sel = __popcll(ballot((uint32_t)lane << g < chunks && prefix(at_pos, at_c) <= r)) - 1;
    uint32_t j0 = 0, C0 = 0;  // C0 common candidates below j0, none from there to the pick
    if (sel >= 0) {
        j0 = readlane_u32(at_pos, sel);
        uint32_t C = C0 = readlane_u32(at_c, sel);
        const uint32_t end = ((uint32_t)sel + 1) << g;
        for (uint32_t k1 = (uint32_t)sel << g; k1 < end && k1 < chunks; ++k1) {
            uint32_t pos1 = pos[0], cnt1 = cnt[0];
            if (k1 < kept) {
                uint32_t unused_p = 0, unused_n = 1;
                rank_chunk<kRepeats>(st, k1 * kWave, pos1, cnt1, unused_p, unused_n);
            } else {
#pragma unroll
                for (int q = 1; q < kRankQ; ++q)
                    if (k1 == kept + q) {
                        pos1 = pos[q];
                        cnt1 = cnt[q];
                    }
            }
            const uint64_t one = ballot(cnt1 != 0);
            if (one == 0) continue;
            uint32_t before, all;  // common candidates before this lane's; all of them
            if (kRepeats) {
                const uint32_t incl = wave_incl_scan_u32(cnt1);
                before = C + incl - cnt1;
                all = readlane_u32(incl, kWave - 1);
            } else {
                before = C + (uint32_t)__popcll(one & ((1ull << lane) - 1));
                all = (uint32_t)__popcll(one);
            }
            const uint64_t below = ballot(cnt1 != 0 && prefix(pos1, before) <= r);
            if (below) {
                const int i = 63 - __builtin_clzll(below);
                const uint32_t ji = readlane_u32(pos1, i), ni = readlane_u32(cnt1, i), Ci = readlane_u32(before, i);
                const uint64_t Si = prefix(ji, Ci);
                if (r < Si + (uint64_t)wc * ni) return ji + small_quotient(r - Si, wc, inv[1]);
                j0 = ji + ni;
                C0 = Ci + ni;
            }
            if (below != one) break;
            C += all;
        }
    }
    uint64_t rem = r - prefix(j0, C0);
    if (pos_t + n_t > j0) {  // copies of t from j0 on (a chunk may begin among them)
        const uint32_t from = pos_t > j0 ? pos_t : j0, left = pos_t + n_t - from;
        const uint64_t gap = (uint64_t)wo * (from - j0), run = (uint64_t)wr * left;
        if (rem >= gap) {
            rem -= gap;
            if (rem < run) return from + small_quotient(rem, wr, inv[2]);
            rem -= run;
            j0 = from + left;
        }
    }
    return j0 + small_quotient(rem, wo, inv[0]);
}

template <bool kMoves, bool kRepeats>
__global__ void __launch_bounds__(kBlock, 6) k_walk_n2v_rank(WalkParams p) {
    __shared__ __align__(16) int32_t win[kWavesPerBlock][kRankWin];
    const int lane = lane_id();
    const double inv[3] = {1.0 / p.w_outward, 1.0 / p.w_common, 1.0 / p.w_return};
    const int wid = uniform_i32(threadIdx.x / kWave);
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t w = blockIdx.x * (int64_t)kWavesPerBlock + wid; w < p.num_walkers; w += waves) {
        const WalkerCtx wc = walker_ctx(p, w);
        const Key key{(uint32_t)uniform_i32((int32_t)wc.key.k0), (uint32_t)uniform_i32((int32_t)wc.key.k1)};
        const int32_t length = uniform_i32(wc.length);
        const int64_t L1 = (int64_t)length + 1;
        int32_t* path = wc.path;
        int32_t v = uniform_i32(p.starts[w]);
        if (v < 0 || (int64_t)v >= p.g.n) {
            if (lane == 0) *p.bad_start = 1;
            for (int64_t q = lane; q < L1; q += kWave) path[q] = -1;
            continue;
        }
        const uint32_t c0 = (uint32_t)uniform_i32((int32_t)wc.c0);
        const int32_t start = v;
        int32_t mine = v;  // path entry i is kept by lane i % 64
        int32_t t = -1;
        int64_t tb = 0;
        uint32_t dt = 0;
        int32_t s = 0;
        for (; s < length; ++s) {
            int32_t to;
            if (kMoves && walk_move(p, key, c0, s, v, start, to)) {  // uniform: the draw depends on wave-uniform values
                v = uniform_i32(to);
                t = -1;
            } else {
                int64_t beg, d64;
                row_uniform(p.g.rowptr, v, beg, d64);
                const uint64_t u = philox_vec(key, c0, (uint32_t)s, (uint32_t)v, 0u);
                const uint32_t d = (uint32_t)d64;
                if (d == 0) break;
                uint32_t m;
                if (t < 0) {  // no previous vertex: every bias is 1
                    m = (uint32_t)range_reduce(u, (uint64_t)d);
                } else {
                    RankStep st;
                    st.of_t = d > dt;
                    st.sh = p.g.col + (st.of_t ? tb : beg);
                    st.ns = st.of_t ? dt : d;
                    const int64_t lb = st.of_t ? beg : tb;
                    st.lg = p.g.col + lb;
                    st.lg_at = (uint32_t)lb;
                    st.nl = st.of_t ? d : dt;
                    st.rank = p.g.rank + rank_base(lb, st.of_t ? v : t);
                    st.bits = rank_shift(p.g.n, st.nl);
                    st.t = t;
                    st.win = win[wid];
                    bool stop;
                    m = walk_step_rank<kRepeats>(p, st, u, d, inv, stop);
                    if (stop) break;
                }
                t = v;
                tb = beg;
                dt = d;
                v = ld_uniform(p.g.col + beg + uniform_i32((int32_t)m));
            }
            const int32_t i = s + 1;
            if (lane == (i & (kWave - 1))) mine = v;
            if ((i & (kWave - 1)) == kWave - 1) path[i - (kWave - 1) + lane] = mine;
        }
        const int32_t i0 = s & ~(kWave - 1);  // entries [i0, s] are still in the lanes, unless they fill them
        if ((s & (kWave - 1)) != kWave - 1 && lane <= s - i0) path[i0 + lane] = mine;
        for (int64_t q = (int64_t)s + 1 + lane; q < L1; q += kWave) path[q] = -1;
        if (lane == 0 && s) atomicAdd(wc.steps, (unsigned long long)s);
    }
}

// One wavefront per vertex u, a lane per edge (u, x): is u in the sorted N(x)?
__global__ void __launch_bounds__(kBlock) k_symmetric_check(RowPtr rowptr, const int32_t* __restrict__ col,
                                                            int64_t n, int32_t* __restrict__ flag) {
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t u = blockIdx.x * (int64_t)kWavesPerBlock + threadIdx.x / kWave; u < n; u += waves) {
        const int64_t b = rowptr[u], e = rowptr[u + 1];
        bool missing = false;
        for (int64_t i = b + lane; i < e; i += kWave) {
            const int32_t x = col[i];
            missing |= !in_sorted(col, rowptr[x], rowptr[x + 1], (int32_t)u);
        }
        if (ballot(missing) && lane == 0) atomicOr(flag, 1);
    }
}

// Rank index, one wavefront per list of at least kRankMinD entries: entry i
// writes its position at the ranges that begin above entry i - 1 and not above
// entry i, the last one also the length at those behind it. Entries are taken
// kRankPer a lane, so that long lists have several loads in flight; wide gaps
// are written by the whole wavefront. Every list is looked over for repeated entries.
constexpr int kRankPer = 4;
constexpr uint32_t kRankLaneFill = 16;
__global__ void __launch_bounds__(kBlock) k_walk_ranks(RowPtr rowptr, const int32_t* __restrict__ col, int64_t n,
                                                       uint32_t* __restrict__ rank, int32_t* __restrict__ repeats) {
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    bool twice = false;
    for (int64_t v = blockIdx.x * (int64_t)kWavesPerBlock + uniform_i32(threadIdx.x / kWave); v < n; v += waves) {
        const int64_t b = uniform_i64(rowptr[v]), d = uniform_i64(rowptr[v + 1]) - b;
        if (d < 2) continue;
        const bool own = d >= kRankMinD;
        const int sh = rank_shift(n, d);
        const uint32_t K = 1u << rank_log(d);
        uint32_t* R = rank + rank_base(b, v);
        for (int64_t base = 0; base <= d; base += kRankPer * kWave) {
            int32_t x[kRankPer], y[kRankPer];
#pragma unroll
            for (int q = 0; q < kRankPer; ++q) {
                const int64_t i = base + q * kWave + lane;
                x[q] = i < d ? col[b + i] : 0;
                y[q] = i > 0 && i <= d ? col[b + i - 1] : 0;
            }
#pragma unroll
            for (int q = 0; q < kRankPer; ++q) {
                const int64_t i = base + q * kWave + lane;
                twice |= i > 0 && i < d && x[q] == y[q];
                const uint32_t k0 = i == 0 ? 0u : ((uint32_t)y[q] >> sh) + 1u;
                const uint32_t k1 = i < d ? ((uint32_t)x[q] >> sh) + 1u : K + 1u;
                const uint32_t nk = own && i <= d && k1 > k0 ? k1 - k0 : 0u;
                if (nk <= kRankLaneFill)
                    for (uint32_t k = k0; k < k0 + nk; ++k) R[k] = (uint32_t)i;
                for (uint64_t wide = ballot(nk > kRankLaneFill); wide; wide &= wide - 1) {
                    const int src = __ffsll((unsigned long long)wide) - 1;
                    const uint32_t a0 = readlane_u32(k0, src), a1 = readlane_u32(k1, src);
                    const uint32_t at = (uint32_t)(base + q * kWave + src);
                    for (uint32_t k = a0 + lane; k < a1; k += kWave) R[k] = at;
                }
            }
        }
    }
    if (ballot(twice) && lane == 0) atomicOr(repeats, 1);
}

// Walk guide tables, one wavefront per list with a positive total: the inclusive prefix of every edge (64 at a time, one
// scan each, carried), and the buckets of the list's guide. The edge whose
// interval holds a bucket's start writes it: edge i those from
// ceil(S_i / 2^s) to ceil(S_(i+1) / 2^s) - 1 (none for a zero
// weight), so every bucket is written once; the second position of a bucket is
// the next edge, if its interval reaches the bucket's end. A lane writes up to
// kGuideLaneFill buckets itself; an edge heavier than that many buckets is
// written by the whole wavefront, 64 buckets at a time.
constexpr uint64_t kGuideLaneFill = 8;

// Bucket k of a list of total W: position i holds its start and ends at S1, the
// next position at S2.
__device__ __forceinline__ WalkBucket guide_bucket(uint64_t k, int sh, uint64_t W, uint64_t S1, uint64_t S2, uint32_t i,
                                                   int32_t y, int32_t y1) {
    const uint64_t start = k << sh, full = start + (uint64_t(1) << sh), end = full < W ? full : W;
    uint32_t bound = ~0u, second = ~0u;  // (searched in the edge records)
    if (S1 >= end) {
        second = 0u;  // one position: the bound is never reached
    } else if (S2 >= end) {
        bound = (uint32_t)(S1 - start);
        second = (uint32_t)y1;
    }
    return WalkBucket{(uint64_t)bound | ((uint64_t)second << 32), i, y};
}

// Edge i of a list and the next one (zeros past the end). A hub's list is one wavefront's
// serial work and sets the time of the build, so edges are loaded 256 at a time, one
// such step ahead: R-MAT 22 (longest list 163,000) 5.6 ms, 6.9 with 64 at a time.
constexpr int kGuidePer = 4;
struct GuideEdges {
    uint32_t x, x1;
    int32_t y, y1;
};
__device__ __forceinline__ void load_edges(const uint32_t* __restrict__ w, const int32_t* __restrict__ col, int64_t d,
                                           int64_t base, GuideEdges (&e)[kGuidePer]) {
#pragma unroll
    for (int q = 0; q < kGuidePer; ++q) {
        const int64_t i = base + q * kWave + lane_id();
        e[q].x = i < d ? w[i] : 0u;
        e[q].y = i < d ? col[i] : 0;
        e[q].x1 = i + 1 < d ? w[i + 1] : 0u;
        e[q].y1 = i + 1 < d ? col[i + 1] : 0;
    }
}

__global__ void __launch_bounds__(kBlock) k_walk_guides(RowPtr rowptr, const int32_t* __restrict__ col,
                                                        const uint32_t* __restrict__ w,
                                                        const uint64_t* __restrict__ wtot, int64_t n,
                                                        WalkEdge* __restrict__ rec, WalkVertex* __restrict__ vtx,
                                                        WalkBucket* __restrict__ gd, int per) {
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t v = blockIdx.x * (int64_t)kWavesPerBlock + threadIdx.x / kWave; v < n; v += waves) {
        int64_t b, d;
        row_uniform(rowptr, v, b, d);
        const uint64_t W = ld_uniform(wtot + v);
        if (vtx && lane == 0) vtx[v] = WalkVertex{W, (uint32_t)b, (uint32_t)d};
        if (W == 0) continue;
        const int sh = guide_shift(W, d, per);
        const uint64_t K = ((W - 1) >> sh) + 1;
        const uint64_t low = (uint64_t(1) << sh) - 1;
        WalkBucket* G = gd + guide_base(b, v, per);
        uint64_t run = 0;
        GuideEdges ahead[kGuidePer];
        load_edges(w + b, col + b, d, 0, ahead);
        for (int64_t base = 0; base < d; base += kGuidePer * kWave) {
            GuideEdges at[kGuidePer];
#pragma unroll
            for (int q = 0; q < kGuidePer; ++q) at[q] = ahead[q];
            load_edges(w + b, col + b, d, base + kGuidePer * kWave, ahead);
#pragma unroll
            for (int q = 0; q < kGuidePer; ++q) {
                if (base + q * kWave >= d) break;
                const int64_t i = base + q * kWave + lane;
                const uint64_t x = at[q].x, x1 = at[q].x1;
                const int32_t y = at[q].y, y1 = at[q].y1;
                const uint64_t incl = run + wave_incl_scan_u64(x);
                const uint64_t excl = incl - x;
                const uint64_t k0 = (excl >> sh) + ((excl & low) != 0);
                uint64_t k1 = (incl >> sh) + ((incl & low) != 0);
                k1 = k1 < K ? k1 : K;
                const uint64_t nk = i < d && k1 > k0 ? k1 - k0 : 0;
                if (i < d) {
                    rec[b + i] = WalkEdge{incl, y, (uint32_t)x};
                    if (nk <= kGuideLaneFill)
                        for (uint64_t k = k0; k < k1; ++k) G[k] = guide_bucket(k, sh, W, incl, incl + x1, (uint32_t)i, y, y1);
                }
                for (uint64_t wide = ballot(nk > kGuideLaneFill); wide; wide &= wide - 1) {
                    const int src = __ffsll((unsigned long long)wide) - 1;
                    const uint64_t a0 = readlane_u64(k0, src), a1 = readlane_u64(k1, src);
                    const uint64_t si = readlane_u64(incl, src), sx = readlane_u64(x1, src);
                    const int32_t sy = readlane_i32(y, src), sy1 = readlane_i32(y1, src);
                    for (uint64_t k = a0 + lane; k < a1; k += kWave)
                        G[k] = guide_bucket(k, sh, W, si, si + sx, (uint32_t)(base + q * kWave + src), sy, sy1);
                }
                run = readlane_u64(incl, kWave - 1);
            }
        }
    }
}

}  // namespace

void launch_walk_hops(RowPtr rowptr, const int32_t* col, int64_t m, WalkHop* hops, hipStream_t s) {
    if (m <= 0) return;
    int64_t g = (m + kBlock - 1) / kBlock;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_walk_hops, dim3((unsigned)g), dim3(kBlock), 0, s, rowptr, col, m, hops);
}

void launch_walk_ranks(RowPtr rowptr, const int32_t* col, int64_t n, uint32_t* rank, int32_t* repeats, hipStream_t s) {
    if (n <= 0) return;
    int64_t g = (n + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_walk_ranks, dim3((unsigned)g), dim3(kBlock), 0, s, rowptr, col, n, rank, repeats);
}

void launch_walk_guides(RowPtr rowptr, const int32_t* col, const uint32_t* w, const uint64_t* wtot, int64_t n,
                        WalkEdge* rec, WalkVertex* vtx, WalkBucket* gd, hipStream_t s) {
    launch_walk_guides(rowptr, col, w, wtot, n, rec, vtx, gd, kGuideBucketsPerEdge, s);
}

void launch_walk_guides(RowPtr rowptr, const int32_t* col, const uint32_t* w, const uint64_t* wtot, int64_t n,
                        WalkEdge* rec, WalkVertex* vtx, WalkBucket* gd, int per, hipStream_t s) {
    if (n <= 0) return;
    int64_t g = (n + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_walk_guides, dim3((unsigned)g), dim3(kBlock), 0, s, rowptr, col, w, wtot, n, rec, vtx, gd, per);
}

void launch_symmetric_check(RowPtr rowptr, const int32_t* col, int64_t n, int32_t* flag, hipStream_t s) {
    if (n <= 0) return;
    int64_t g = (n + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_symmetric_check, dim3((unsigned)g), dim3(kBlock), 0, s, rowptr, col, n, flag);
}

namespace {
template <bool kMH, bool kMoves>
void (*uniform_kernel(const WalkParams& p))(WalkParams) {
    if (p.num_walkers < kUniformRunMin)
        return p.g.hops ? k_walk_uniform<kMH, true, kMoves, 1> : k_walk_uniform<kMH, false, kMoves, 1>;
    return p.g.hops ? k_walk_uniform<kMH, true, kMoves, 64> : k_walk_uniform<kMH, false, kMoves, 64>;
}
}  // namespace

void launch_walk(const WalkParams& p, int grid, hipStream_t s, LaunchEvents ev) {
    if (p.num_walkers <= 0) return;
    const bool flat_n2v = p.bias == kNode2vec && p.w_return == p.w_common && p.w_common == p.w_outward &&
                          p.w_return > 0;
    if (p.bias == kUniform || flat_n2v || p.bias == kMetropolis) {
        int64_t g = (p.num_walkers + kBlock - 1) / kBlock;
        if (g > grid) g = grid;
        const bool mh = p.bias == kMetropolis;
        const bool moves = (p.restart | p.jump) != 0;
        launch_kernel(mh ? (moves ? uniform_kernel<true, true>(p) : uniform_kernel<true, false>(p))
                         : (moves ? uniform_kernel<false, true>(p) : uniform_kernel<false, false>(p)),
                      dim3((unsigned)g), dim3(kBlock), s, ev, p);
    } else {
        int64_t g = (p.num_walkers + kWavesPerBlock - 1) / kWavesPerBlock;
        if (g > grid) g = grid;
        const bool moves = (p.restart | p.jump) != 0;
        if (p.bias == kNode2vec && p.g.rank) {
            launch_kernel(p.g.repeats ? (moves ? k_walk_n2v_rank<true, true> : k_walk_n2v_rank<false, true>)
                                      : (moves ? k_walk_n2v_rank<true, false> : k_walk_n2v_rank<false, false>),
                          dim3((unsigned)g), dim3(kBlock), s, ev, p);
        } else if (p.bias == kNode2vec) {
            if (moves) launch_kernel(k_walk_wave_n2v<true>, dim3((unsigned)g), dim3(kBlock), s, ev, p);
            else launch_kernel(k_walk_wave_n2v<false>, dim3((unsigned)g), dim3(kBlock), s, ev, p);
        } else {
            const bool dg = p.bias == kNeighborDegree;
            const bool guide = (dg ? p.g.wgd_deg : p.g.wgd_ew) && (dg ? p.g.wrec_deg : p.g.wrec_ew) &&
                               (dg ? p.g.wvtx_deg : p.g.wvtx_ew);
            if (guide && p.num_walkers < kLaneWalkMin) {
                launch_kernel(moves ? k_walk_wave_guide<true> : k_walk_wave_guide<false>, dim3((unsigned)g), dim3(kBlock), s,
                              ev, p);
            } else if (guide) {
                int64_t gl = (p.num_walkers + kBlock - 1) / kBlock;
                if (gl > grid) gl = grid;
                launch_kernel(p.num_walkers < kLaneRunMin ? (moves ? k_walk_lane<true, 1> : k_walk_lane<false, 1>)
                                                          : (moves ? k_walk_lane<true, 32> : k_walk_lane<false, 32>),
                              dim3((unsigned)gl), dim3(kBlock), s, ev, p);
            } else if (moves) {
                launch_kernel(k_walk_wave_moves, dim3((unsigned)g), dim3(kBlock), s, ev, p);
            } else {
                launch_kernel(k_walk_wave_first, dim3((unsigned)g), dim3(kBlock), s, ev, p);
            }
        }
    }
}

}  // namespace csaw
