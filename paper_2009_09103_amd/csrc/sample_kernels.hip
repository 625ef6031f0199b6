// sample_kernels.hip -- gfx950 kernels of neighbor sampling.
//
// One layer of the generic sampling loop (fig:api(b)) is
//   frontier build : next bitmap -> sorted frontier entries, each with its
//                    edge count min(k, P), edge offset, list fields and
//                    route (one pass with a decoupled look-back);
//                    visited |= next
//   select         : EdgeBias, exact prefix, Philox draws, inverse transform
//                    search, collision rounds, direct draw from the updated
//                    prefix; writes the edges and marks new neighbors in the
//                    instance's next bitmap. A lane per slot, several
//                    entries to a wavefront (k_select_slots); weighted lists
//                    without a walk guide that are too long for a lane to scan
//                    take a wavefront each, in registers (k_select_wave) or
//                    through the graph's chunk prefix tables (k_select_big).
// Frontier entries are (vertex, instance) pairs sorted by (instance, vertex),
// so edges come out in (layer, instance, source, slot) order without a sort.
#include "device_common.h"
#include "kernels.h"

namespace csaw {

namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

inline int grid_for(int64_t items, int per_block, int cap = 1 << 20) {
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// ------------------------------------------------------------------ misc
__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Edges of a batch to their requests' result arrays: segment j (edges
// [off[j], off[j+1]) of the batch's layer-major arrays, off non-decreasing)
// goes to to_src[j] and to_dst[j] (null: nowhere). A thread per edge finds
// its segment by binary search over off (a few hundred entries, cached), so
// a long segment is spread over the whole grid.
__global__ void k_scatter_segments(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                   const int64_t* __restrict__ off, int64_t nseg, int32_t* const* __restrict__ to_src,
                                   int32_t* const* __restrict__ to_dst) {
    const int64_t total = off[nseg];
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = nseg;  // the last j with off[j] <= k
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (off[mid] <= k) lo = mid;
            else hi = mid;
        }
        int32_t* ts = to_src[lo];
        int32_t* td = to_dst[lo];
        if (!ts || !td) continue;
        ts[k - off[lo]] = src[k];
        td[k - off[lo]] = dst[k];
    }
}

__global__ void k_degree_weights(RowPtr rowptr, const int32_t* __restrict__ col,
                                 int64_t m, uint32_t* __restrict__ degw) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = col[e];
        degw[e] = (uint32_t)(rowptr[x + 1] - rowptr[x]);
    }
}

// one wavefront per vertex: number of positive weights in its list, with
// kWideList set when the list's total weight needs more than 32 bits, and
// the total itself
__global__ void k_positive_counts(RowPtr rowptr, const uint32_t* __restrict__ w,
                                  int64_t n, int32_t* __restrict__ ppos, uint64_t* __restrict__ wtot) {
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t v = blockIdx.x * (int64_t)kWavesPerBlock + threadIdx.x / kWave; v < n; v += waves) {
        const int64_t b = rowptr[v], e = rowptr[v + 1];
        int64_t c = 0;
        uint64_t tot = 0;
        for (int64_t i = b + lane; i < e; i += kWave) {
            c += (w[i] > 0);
            tot += w[i];
        }
        c = wave_sum_i64(c);
        tot = wave_sum_u64(tot);
        if (lane == 0) {
            ppos[v] = (int32_t)c | ((tot >> 32) ? kWideList : 0);
            wtot[v] = tot;
        }
    }
}

// ------------------------------------------------------------- frontier
// Seeds -> next bitmap of their instance (instance of seed s: the largest i
// with seed_offsets[i] <= s).
__global__ void k_mark_seeds(const int32_t* __restrict__ seeds, int64_t num_seeds,
                             const int64_t* __restrict__ seed_off, int32_t ni, int64_t n,
                             uint32_t* __restrict__ next, int64_t nwp, uint32_t* __restrict__ summ, int64_t nsw,
                             SampleCtl* ctl) {
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < num_seeds;
         s += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = seeds[s];
        if (v < 0 || (int64_t)v >= n) {
            ctl->bad_seed = 1;
            continue;
        }
        int32_t lo = 0, hi = ni;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (seed_off[mid] <= s) lo = mid;
            else hi = mid;
        }
        const uint32_t old = atomicOr(&next[(int64_t)lo * nwp + (v >> 5)], 1u << (v & 31));
        if (summ && old == 0u) atomicOr(&summ[(int64_t)lo * nsw + (v >> 10)], 1u << ((v >> 5) & 31));
    }
}

// ------------------------------------------------------------------ count
// Weighted lists that need draws are routed by length: up to kWaveMaxD
// candidates with a total weight below 2^32 to the wavefront kernel (list and
// 32-bit prefix resident in registers); the others to the long-list path,
// which draws with one wavefront per list from a coarse table built out of
// the graph's chunk prefix table (lists longer than kWaveMaxD; the table is
// computed once per graph and weight array, since it depends on the list
// alone, not on the instance) or, for shorter lists with a wide total, out of
// the list's one chunk reduced on the spot.

enum { kRouteWave = 0, kRouteBig = 1 };

__device__ __forceinline__ int route_of(int32_t kind, int32_t k, int32_t P, int64_t d, bool wide) {
    if (kind == kUniform || k <= 0 || k >= P || (d <= kWaveMaxD && !wide)) return kRouteWave;
    return kRouteBig;
}

// Forest fire NeighborSize (Section II-A): vertex v burns G neighbors, G
// geometric with P(G >= j) = (burn / 2^32)^j, capped at cap. Trial j
// succeeds iff word j mod 4 of the Philox block with counter
// (c0, c1, c2, kBurnRound << 16 | j / 4) is below burn.
__device__ __forceinline__ int32_t burn_count(Key key, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t burn,
                                              int32_t cap) {
    int32_t g = 0;
    for (uint32_t blk = 0; g < cap; ++blk) {
        const uint4 x = philox4(key.k0, key.k1, c0, c1, c2, (kBurnRound << 16) | blk);
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (g >= cap || w[q] >= burn) return g;
            ++g;
        }
    }
    return g;
}

// NeighborSize of frontier vertex v of an instance with layer fanout k. The
// kernels that call it are instantiated with and without forest fire, so
// the burning code costs the fixed-fanout kernels no registers.
template <bool kBurn>
__device__ __forceinline__ int32_t neighbor_size(int32_t k, uint32_t burn, uint64_t key, uint32_t c0,
                                                 int32_t layer, int32_t v) {
    if (!kBurn || !burn || k == 0) return k;
    return burn_count(Key{(uint32_t)key, (uint32_t)(key >> 32)}, c0, (uint32_t)layer, (uint32_t)v, burn,
                      k < 0 ? kBurnCapAll : k);
}

// Positive biases of v's list with the kWideList flag (the list length if
// unbiased).
__device__ __forceinline__ int32_t positive_info(const GraphDev& g, int32_t kind, int32_t v, int64_t d) {
    if (kind == kUniform) return (int32_t)d;
    return kind == kEdgeWeight ? g.ppos_ew[v] : g.ppos_deg[v];
}

__device__ __forceinline__ int32_t entry_count(const GraphDev& g, int32_t k, int32_t kind, int32_t v,
                                               int32_t& route, int64_t& beg, int64_t& d, int32_t& pinfo,
                                               SampleCtl* ctl) {
    beg = g.rowptr[v];
    d = g.rowptr[v + 1] - beg;
    pinfo = positive_info(g, kind, v, d);
    const int32_t P = pinfo & ~kWideList;
    const bool wide = (pinfo & kWideList) != 0;
    route = kRouteWave;
    if (k == 0 || P == 0) return 0;
    if (k < 0 || k >= P) return P;
    if (k > kMaxDrawFanout) {
        ctl->unsupported = 1;
        return 0;
    }
    route = route_of(kind, k, P, d, wide);
    return k;
}

__device__ __forceinline__ int64_t chunks_of(int64_t d) { return (d + kChunk - 1) / kChunk; }

// Look-back status words: a 48-bit value, a valid bit and the build's epoch
// in one 64-bit word, so a reader never sees a value without its flag.
constexpr uint64_t kStatusValid = 1ull << 48;
constexpr uint64_t kStatusMask = kStatusValid - 1;

__device__ __forceinline__ uint64_t status_pack(int64_t v, uint32_t epoch) {
    return ((uint64_t)v & kStatusMask) | kStatusValid | ((uint64_t)(epoch & 0x7FFF) << 49);
}
__device__ __forceinline__ bool status_ok(uint64_t w, uint32_t epoch) {
    return (w & kStatusValid) && (w >> 49) == (epoch & 0x7FFF);
}
__device__ __forceinline__ void status_store(unsigned long long* p, uint64_t v) {
    __hip_atomic_store(p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t status_load(unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Entries of a layer's frontier; none where a build gave up, whose entries are not whole.
__device__ __forceinline__ int64_t frontier_size(const SampleCtl* ctl, int32_t layer) {
    return ctl->gave_up() ? 0 : ctl->fcount[layer];
}

// Next set bit of a word (cleared from it), or -1.
__device__ __forceinline__ int32_t pop_bit(uint32_t& bits) {
    if (!bits) return -1;
    const int32_t b = __ffs(bits) - 1;
    bits &= bits - 1;
    return b;
}

// Place of this block in the chain of a frontier build's blocks, whose later ones
// wait for the earlier ones. The block index is such a place as long as the chip
// takes blocks in its order; beside other kernels each XCD does so by
// itself, and the waiting blocks of two chains can fill one XCD each while
// either waits for a block that the other one keeps out (two builds of 2,048
// and 4,096 blocks, once in about 2,000 bursts of a server's requests). So the wait
// of such a chain is short; a call whose chain gave up runs again in order: blocks
// take tickets as they start and wait for blocks that run. Tickets in every call
// would cost it a queue at one address, 8 us for 512 blocks.
__device__ __forceinline__ int64_t chain_place(uint32_t* tickets, bool ordered) {
    if (!ordered) return blockIdx.x;
    __shared__ uint32_t ticket;
    if (threadIdx.x == 0) ticket = atomicAdd(tickets, 1u);
    __syncthreads();
    return ticket;
}

// Decoupled look-back of block b for two running totals (a, c), called by
// the 64 lanes of one wavefront: publishes b's aggregates, then sums its
// predecessors' published values 64 blocks at a time, nearest first; a
// predecessor's inclusive prefix ends the walk (predecessors run or are done:
// chain_place). The spin is bounded and
// reports through *stuck instead of hanging; the prefixes are then those of the
// nearer predecessors, so positions formed from them are too small and stay inside
// their arrays. Publishes b's inclusive prefix and returns the exclusive ones (every lane).
__device__ __forceinline__ void lookback2(unsigned long long* status, int64_t b, int64_t tot_a, int64_t tot_c,
                                          uint32_t epoch, uint32_t limit, int32_t* stuck, int64_t& pa, int64_t& pc) {
    const int lane = lane_id();
    unsigned long long* st = status + 4 * b;
    if (b > 0 && lane == 0) {
        status_store(st + 0, status_pack(tot_a, epoch));
        status_store(st + 1, status_pack(tot_c, epoch));
    }
    pa = 0;
    pc = 0;
    int64_t end = b - 1;  // window covers predecessors end, end-1, ..., end-63
    uint32_t spins = 0;
    while (end >= 0) {
        const int64_t q = end - lane;
        int flag = 2;  // before block 0: an inclusive prefix of zero
        int64_t va = 0, vc = 0;
        if (q >= 0) {
            unsigned long long* sq = status + 4 * q;
            const uint64_t ia = status_load(sq + 2), ic = status_load(sq + 3);
            if (status_ok(ia, epoch) && status_ok(ic, epoch)) {
                va = (int64_t)(ia & kStatusMask);
                vc = (int64_t)(ic & kStatusMask);
            } else {
                const uint64_t aa = status_load(sq + 0), ac = status_load(sq + 1);
                if (status_ok(aa, epoch) && status_ok(ac, epoch)) {
                    flag = 1;
                    va = (int64_t)(aa & kStatusMask);
                    vc = (int64_t)(ac & kStatusMask);
                } else {
                    flag = 0;
                }
            }
        }
        const uint64_t incl = ballot(flag == 2);
        const uint64_t notready = ballot(flag == 0 || limit == 0);
        const int first = incl ? __ffsll((unsigned long long)incl) - 1 : kWave;  // nearest inclusive
        const uint64_t upto = first >= kWave - 1 ? ~0ull : ((2ull << first) - 1);
        if (notready & upto) {  // a nearer predecessor has published nothing yet
            if (++spins > limit) {  // the call runs again in order, or (then never expected) reports it
                if (lane == 0) *stuck = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        const bool take = ((upto >> lane) & 1ull) != 0;
        pa += (int64_t)wave_sum_u64(take ? (uint64_t)va : 0ull);
        pc += (int64_t)wave_sum_u64(take ? (uint64_t)vc : 0ull);
        if (first < kWave) break;
        end -= kWave;
        spins = 0;
    }
    if (lane == 0) {
        status_store(st + 2, status_pack(pa + tot_a, epoch));
        status_store(st + 3, status_pack(pc + tot_c, epoch));
    }
}

// Exclusive scans of four int64 per thread over the block in one pass (one
// pair of barriers); totals in tot[0..3]. Every thread must call it.
__device__ __forceinline__ void block_excl_scan4(int64_t (&x)[4], int64_t (&tot)[4]) {
    constexpr int kW = kBlock / kWave;
    __shared__ int64_t wsum[4][kW];
    const int lane = lane_id();
    const int wid = threadIdx.x / kWave;
    uint64_t incl[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        incl[j] = wave_incl_scan_u64((uint64_t)x[j]);
        if (lane == kWave - 1) wsum[j][wid] = (int64_t)incl[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int64_t base = 0, t = 0;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
            const int64_t v = wsum[j][w];
            if (w < wid) base += v;
            t += v;
        }
        tot[j] = t;
        x[j] = base + (int64_t)incl[j] - x[j];
    }
    __syncthreads();
}

// Frontier build of one layer, one pass: each thread takes kPer consecutive
// bitmap words, of all of them (dense) or of those in the dirty list (sparse, one
// word). Dense builds take one up to kSparseWords, and kWidePer above, where a
// call is short of memory: a sixteenth of the look-back words. The thread counts
// the new bits (entries), their edge counts min(k, P)
// (edges) and their long-list route (the words and the list fields are
// loaded again in the write pass rather than held in registers across the
// scan, which keeps occupancy up); a block scan plus a decoupled look-back
// over the blocks before it give global positions. The thread then writes its entries in
// (instance, vertex) order with count, edge offset, list fields and route,
// sets visited |= next, clears next, and the first word of an instance writes
// that instance's segment offset. The last block writes the layer's totals
// and the output base of the next layer.
constexpr int kWidePer = 16;
template <bool kBurn, bool kSparse, int kPer>
__global__ void __launch_bounds__(kBlock) k_frontier_build(FrontierBuild fb) {
    static_assert(!kSparse || kPer == 1, "the dirty list gives one word per thread");
    __shared__ int64_t s_base_e, s_base_g;
    const int tid = threadIdx.x;
    // dense: every word of the bitmaps; sparse: the words of the dirty list
    // (grid sized by capacity, blocks past the list end at once)
    int64_t nwords = fb.nwords, nb = fb.nb;
    if (kSparse) {
        if (fb.ctl->list_stuck) return;  // the list is not whole (uniform: no block of this launch writes it)
        nwords = fb.ctl->ndirty[fb.layer];
        nb = nwords > 0 ? (nwords + kBlock - 1) / kBlock : 1;
        if (blockIdx.x >= nb) return;
    }
    const int64_t b = chain_place(&fb.ctl->tickets[fb.layer][0], fb.ordered);
    const int64_t w0 = (b * kBlock + tid) * kPer;  // the thread's first word, or its dirty word
    int64_t iw = kSparse ? (w0 < nwords ? fb.dirty[w0] : 0) : w0;
    const int64_t out_base = fb.ctl->out_base[fb.layer];
    uint32_t raw = 0, vis = 0, w = 0;  // word iw, its visited bits, the new ones
    int64_t inst = 0;
    int32_t vbase = 0, k = 0, kind = 0;
    uint64_t key = 0;
    uint32_t iid = 0;
    const auto load = [&](int t) {
        if (!kSparse) iw = w0 + t;
        raw = w0 + t < nwords ? fb.next[iw] : 0u;
        vis = w0 + t < nwords && (kPer == 1 || raw) ? fb.visited[iw] : 0u;
        w = raw & ~vis;  // picks of visited vertices are not new
        inst = iw / fb.nwp;
        vbase = (int32_t)((iw - inst * fb.nwp) * 32);
        if (w) {
            k = fb.fanout[inst];
            kind = fb.bias[inst];
            if (kBurn) {
                key = fb.inst_key[inst];
                iid = fb.inst_id[inst];
            }
        }
    };
    int64_t cnt4[4] = {0, 0, 0, 0};  // entries, edges, long lists, (unused)
    for (int at = 0; at < kPer; ++at) {
        load(at);
        cnt4[0] += __popc(w);
        for (uint32_t bits = w; bits;) {  // four bits at a time so that their loads overlap
            int32_t bv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) bv[t] = pop_bit(bits);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                int32_t route = kRouteWave, pinfo = 0;
                int64_t beg = 0, d = 0;
                if (bv[t] >= 0) {
                    const int32_t kv = neighbor_size<kBurn>(k, fb.burn, key, iid, fb.layer, vbase + bv[t]);
                    cnt4[1] += entry_count(fb.g, kv, kind, vbase + bv[t], route, beg, d, pinfo, fb.ctl);
                    if (route == kRouteBig) ++cnt4[2];
                }
            }
        }
    }
    int64_t tot4[4];
    int64_t ex4[4] = {cnt4[0], cnt4[1], cnt4[2], cnt4[3]};
    block_excl_scan4(ex4, tot4);
    const int64_t ex_e = ex4[0], ex_g = ex4[1];
    int64_t ex_big = ex4[2];
    const int64_t tot_e = tot4[0], tot_g = tot4[1], tot_big = tot4[2];
    __shared__ int64_t s_big_base;
    if (tid == kWave) {  // wave 1: one reservation per block for its long lists
        s_big_base = tot_big ? (int64_t)atomicAdd(&fb.ctl->nbig[fb.layer], (unsigned long long)tot_big) : 0;
    }
    if (tid < kWave) {  // wave 0: publish, then look back 64 predecessors per step
        int64_t pe = 0, pg = 0;
        lookback2(fb.status, b, tot_e, tot_g, kSparse ? 2u * fb.layer + 2u : (uint32_t)fb.layer + 1u,
                  fb.spins, &fb.ctl->lookback_stuck, pe, pg);
        if (tid == 0) {
            s_base_e = pe;
            s_base_g = pg;
        }
    }
    __syncthreads();
    int64_t pos = s_base_e + ex_e;
    int64_t eoff = s_base_g + ex_g;
    for (int at = 0; at < kPer && w0 + at < nwords; ++at) {
        if (kPer > 1) load(at);
        if (fb.offsets && fb.layer < fb.num_layers) {
            if (!kSparse) {
                if (vbase == 0) fb.offsets[(int64_t)fb.layer * fb.num_instances + inst] = out_base + eoff;
            } else {
                // the first dirty word of an instance starts its segment, and
                // those of the instances since the previous dirty word's (empty)
                const int64_t prev = w0 > 0 ? fb.dirty[w0 - 1] / fb.nwp : -1;
                for (int64_t i = prev + 1; i <= inst; ++i)
                    fb.offsets[(int64_t)fb.layer * fb.num_instances + i] = out_base + eoff;
            }
        }
        for (uint32_t bits = w; bits;) {
            int32_t bv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) bv[t] = pop_bit(bits);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (bv[t] < 0) continue;
                const int32_t v = vbase + bv[t];
                int32_t route, c, pinfo;
                int64_t beg, d;
                c = entry_count(fb.g, neighbor_size<kBurn>(k, fb.burn, key, iid, fb.layer, v), kind, v, route, beg, d, pinfo,
                                fb.ctl);
                fb.fv[pos] = v;
                fb.fi[pos] = (int32_t)inst;
                fb.cnt[pos] = c;
                fb.off[pos] = eoff;
                fb.fbeg[pos] = beg;
                fb.fdeg[pos] = (int32_t)d;
                fb.fpos[pos] = pinfo;
                if (route == kRouteBig) fb.bigs[s_big_base + ex_big++] = (int32_t)pos;
                ++pos;
                eoff += c;
            }
        }
        if (w) fb.visited[iw] = vis | w;
        if (raw) fb.next[iw] = 0u;  // also words that held only visited picks
    }
    if (b == nb - 1) {  // last block: totals, and the bases of the layers after this one
        const int64_t te = s_base_e + tot_e, tg = s_base_g + tot_g;
        const int64_t ob = out_base + tg;
        if (tid == 0) {
            fb.ctl->fcount[fb.layer] = te;
            fb.ctl->total[fb.layer] = tg;
            for (int j = fb.layer + 1; j <= fb.num_layers; ++j) fb.ctl->out_base[j] = ob;
        }
        if (fb.offsets) {
            const int64_t ni = fb.num_instances;
            const int64_t first_l = fb.nwp > 0 ? fb.layer + 1 : fb.layer;
            for (int64_t j = first_l; j < fb.num_layers; ++j)
                for (int64_t i = tid; i < ni; i += kBlock) fb.offsets[j * ni + i] = (j == fb.layer ? out_base : ob);
            if (tid == 0) fb.offsets[(int64_t)fb.num_layers * ni] = ob;
            if (kSparse && fb.layer < fb.num_layers) {  // instances after the last dirty word's: empty at the end
                const int64_t last = nwords > 0 ? fb.dirty[nwords - 1] / fb.nwp : -1;
                for (int64_t i = last + 1 + tid; i < ni; i += kBlock) fb.offsets[(int64_t)fb.layer * ni + i] = ob;
            }
        }
    }
}

// Sparse frontier build, first pass: the summary bitmap (one bit per word of
// the instances' next bitmaps, set by the claim that made the word non-zero)
// is compacted into the list of dirty words, in increasing order, with a
// decoupled look-back over the blocks; the summary is cleared as it is read.
// Each thread takes four summary words (the summary of an instance is a
// multiple of four words).
__global__ void __launch_bounds__(kBlock) k_dirty_compact(FrontierBuild fb) {
    __shared__ int64_t s_base;
    const int tid = threadIdx.x;
    const int64_t b = chain_place(&fb.ctl->tickets[fb.layer][1], fb.ordered);
    const int64_t nsumm = (int64_t)fb.num_instances * fb.nsw;
    const int64_t i0 = (b * kBlock + tid) * 4;
    const uint4 s4 = i0 < nsumm ? *(const uint4*)(fb.summ + i0) : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t sw[4] = {s4.x, s4.y, s4.z, s4.w};
    int64_t cnt4[4] = {(int64_t)(__popc(sw[0]) + __popc(sw[1]) + __popc(sw[2]) + __popc(sw[3])), 0, 0, 0};
    int64_t tot4[4];
    block_excl_scan4(cnt4, tot4);
    if (tid < kWave) {
        int64_t pa = 0, pc = 0;
        lookback2(fb.status, b, tot4[0], 0, 2u * fb.layer + 1u, fb.spins, &fb.ctl->list_stuck, pa, pc);
        if (tid == 0) s_base = pa;
    }
    __syncthreads();
    int64_t pos = s_base + cnt4[0];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t i = i0 + q;
        const int64_t inst = i / fb.nsw;
        const int64_t wbase = inst * fb.nwp + (i - inst * fb.nsw) * 32;
        for (uint32_t bits = sw[q]; bits; bits &= bits - 1) fb.dirty[pos++] = wbase + (__ffs(bits) - 1);
    }
    if ((s4.x | s4.y | s4.z | s4.w) != 0u) *(uint4*)(fb.summ + i0) = make_uint4(0u, 0u, 0u, 0u);
    if (b == fb.nb_dirty - 1 && tid == 0) fb.ctl->ndirty[fb.layer] = s_base + tot4[0];
}

// ----------------------------------------------------------------- select
// Lists of k_select_wave (weighted, d <= kWaveMaxD) are searched in registers
// (draw_resident). Long lists without a walk guide use a coarse table: groups of
// g = 16 consecutive candidates, C[t] = S[t*g] (exclusive prefix at the group
// starts) and C[nc] = W in LDS; a search finds the group by binary search in
// C and the candidate by scanning the group's weights from global memory / L2.
//
// Chunk reduction stages weights through LDS in tiles of 1024: 16 coalesced
// loads per lane are issued together, stored transposed (element i at
// i + i/16, so that lane L's 16 consecutive elements sit in 16 distinct
// banks) and summed per lane.
constexpr int kTile = 1024;
constexpr int kTilePad = kTile + kTile / 16;

__device__ __forceinline__ int tpad(int i) { return i + (i >> 4); }

struct CoarsePool {
    const uint64_t* C;      // LDS, nc + 1 entries
    int64_t nc;             // groups
    int64_t g;              // group length
    int64_t d;              // list length
    const uint32_t* w;      // weights of the list in global memory
};

// Scan weights w[i..end) from global memory, 16 loads in flight, for the
// first candidate whose running total (from acc) exceeds r: running totals
// are monotone, so its index in a batch is the number of totals <= r.
__device__ __forceinline__ void fine_scan_global(const uint32_t* __restrict__ w, int64_t i, int64_t end,
                                                 uint64_t acc, uint64_t r, int64_t& m, uint64_t& Sm,
                                                 uint32_t& bm) {
    m = i;
    Sm = acc;
    bm = 0;
    for (; i < end; i += 16) {
        const uint32_t* wp = w + i;
        const int n = end - i < 16 ? (int)(end - i) : 16;
        uint32_t x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = q < n ? wp[q] : 0u;
        int cnt = 0;
        uint64_t run = acc, before = acc;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            run += x[q];
            const bool le = run <= r;
            cnt += le;
            before = le ? run : before;
        }
        if (cnt < n) {
            m = i + cnt;
            Sm = before;
            bm = wp[cnt];
            return;
        }
        acc = run;
    }
}

// m = max{i in [0,d) : S_i <= r} with S_m and b_m; per lane: binary search
// for the group in the LDS table C, then the group's weights from global
// memory / L2.
__device__ __forceinline__ void coarse_search(const CoarsePool& pl, uint64_t r, int64_t& m, uint64_t& Sm,
                                              uint32_t& bm) {
    int64_t lo = 0, hi = pl.nc;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (pl.C[mid] <= r) lo = mid;
        else hi = mid;
    }
    const int64_t i = lo * pl.g;
    const int64_t end = (i + pl.g < pl.d) ? i + pl.g : pl.d;
    fine_scan_global(pl.w, i, end, pl.C[lo], r, m, Sm, bm);
}

// Draw k distinct candidates with one lane per slot (lane j = slot j < k) and
// a per-lane inverse transform search(r, m, Sm, bm) (k <= 64; lanes from k on stay out).
// Each round every open slot draws; taken in slot order, a slot keeps its candidate unless it is
// already held -- which also covers a lower slot that took the same candidate
// in this round, so the lowest slot wins. Slots still open after `rounds` take
// direct draws from the prefix without the held candidates, in slot order:
// r0 in [0, W - held mass), mapped by the skip map (every held candidate whose
// start in the updated prefix is at or below r0 adds its bias) and searched
// with search_all (same r on every lane).
template <class Search, class SearchAll>
__device__ __forceinline__ int64_t draw_slots(Key key, uint32_t c0, uint32_t c1, uint32_t c2, int32_t k, int32_t rounds,
                                              uint64_t W, const Search& search, const SearchAll& search_all) {
    const int lane = lane_id();
    bool held = false;
    int64_t pos = 0;
    uint64_t Spos = 0;
    uint32_t bpos = 0;
    uint64_t open = k >= kWave ? ~0ull : ((1ull << k) - 1);
    for (int a = 0; a < rounds && open; ++a) {
        int64_t m = -1;
        uint64_t Sm = 0;
        uint32_t bm = 0;
        if ((open >> lane) & 1ull) search(draw(key, c0, c1, c2, (uint32_t)lane | ((uint32_t)a << 16), W), m, Sm, bm);
        if (a == 0) {  // nothing is held: a slot yields to a lower one with the same candidate
            bool dup = false;
            for (int j = 0; j + 1 < k; ++j) {
                const int64_t mj = readlane_i64(m, j);
                dup |= lane > j && m == mj;
            }
            dup = dup && lane < k;
            held = lane < k && !dup;
            pos = m;
            Spos = Sm;
            bpos = bm;
            open &= ballot(dup);
            continue;
        }
        for (uint64_t todo = open; todo; todo &= todo - 1) {
            const int j = __ffsll((unsigned long long)todo) - 1;
            const int64_t mj = readlane_i64(m, j);
            if (ballot(held && pos == mj) == 0) {
                if (lane == j) {
                    held = true;
                    pos = m;
                    Spos = Sm;
                    bpos = bm;
                }
                open &= ~(1ull << j);
            }
        }
    }
    if (open) {
        const uint64_t heldmask = ballot(held);
        // before = total bias of held candidates at smaller positions
        uint64_t before = 0;
        for (uint64_t hm = heldmask; hm; hm &= hm - 1) {
            const int q = __ffsll((unsigned long long)hm) - 1;
            const int64_t pq = readlane_i64(pos, q);
            const uint32_t bq = readlane_u32(bpos, q);
            if (held && pq < pos) before += bq;
        }
        uint64_t removed = wave_sum_u64(held ? (uint64_t)bpos : 0ull);
        for (; open; open &= open - 1) {
            const int j = __ffsll((unsigned long long)open) - 1;
            const uint64_t r0 = draw(key, c0, c1, c2, (uint32_t)j | (kFallbackRound << 16), W - removed);
            const uint64_t r = r0 + wave_sum_u64((held && Spos - before <= r0) ? (uint64_t)bpos : 0ull);
            int64_t m = 0;
            uint64_t Sm = 0;
            uint32_t bm = 0;
            search_all(r, m, Sm, bm);  // same r on every lane
            m = readlane_i64(m, j);
            Sm = readlane_u64(Sm, j);
            bm = readlane_u32(bm, j);
            const uint64_t bef_new = wave_sum_u64((held && pos < m) ? (uint64_t)bpos : 0ull);
            if (held && pos > m) before += bm;
            if (lane == j) {
                held = true;
                pos = m;
                Spos = Sm;
                bpos = bm;
                before = bef_new;
            }
            removed += bm;
        }
    }
    return pos;
}

// Weighted lists of at most 64*E candidates, resident in registers: lane L
// holds candidates [L*E, L*E+E) and their inclusive prefix S (width T; the
// wavefront route sends only lists with W < 2^32, so T = 32 bits there). A draw r is resolved by the whole wavefront: the
// owning lane is the number of lanes whose last prefix is <= r, the position
// inside it the number of its prefixes <= r. Held candidates are one bit per
// element in the owning lane. Slots are taken in slot order within a round,
// as in draw_slots; direct draws rescan the prefix with held weights removed,
// which is the updated prefix whose inverse the skip map computes.
template <int E, typename T>
__device__ __forceinline__ int32_t find_resident(const T (&S)[E], T r) {
    const int L = __popcll(ballot(S[E - 1] <= r));
    if (E == 1) return L;
    int32_t cl = 0;
#pragma unroll
    for (int e = 0; e < E - 1; ++e) cl += S[e] <= r ? 1 : 0;
    return L * E + readlane_i32(cl, L);
}

template <int E, typename T>
__device__ __forceinline__ int32_t draw_resident_t(const uint32_t (&x)[E], T excl, T W, Key key, uint32_t c0,
                                                   uint32_t c1, uint32_t c2, int32_t k, int32_t rounds) {
    const int lane = lane_id();
    T S[E];
    {
        T acc = excl;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            acc += (T)x[e];
            S[e] = acc;
        }
    }
    uint32_t hb = 0;  // held bits of this lane's candidates
    int32_t pos = 0;
    uint64_t open = k >= kWave ? ~0ull : ((1ull << k) - 1);
    for (int a = 0; a < rounds && open; ++a) {
        T rl = 0;
        if ((open >> lane) & 1ull) rl = (T)draw(key, c0, c1, c2, (uint32_t)lane | ((uint32_t)a << 16), (uint64_t)W);
        for (uint64_t todo = open; todo; todo &= todo - 1) {
            const int j = __ffsll((unsigned long long)todo) - 1;
            const int32_t m = find_resident<E, T>(S, readlane_t(rl, j));
            const int owner = m / E, bit = m % E;
            if (((readlane_u32(hb, owner) >> bit) & 1u) == 0) {
                if (lane == owner) hb |= 1u << bit;
                if (lane == j) pos = m;
                open &= ~(1ull << j);
            }
        }
    }
    if (open) {
        uint64_t u = 0;
        if ((open >> lane) & 1ull) u = philox_u64(key.k0, key.k1, c0, c1, c2, (uint32_t)lane | (kFallbackRound << 16));
        for (; open; open &= open - 1) {
            const int j = __ffsll((unsigned long long)open) - 1;
            T Sp[E];
            T ls = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                ls += ((hb >> e) & 1u) ? (T)0 : (T)x[e];
                Sp[e] = ls;
            }
            const T incl = wave_incl_scan_t(ls);
            const T ex = incl - ls;
#pragma unroll
            for (int e = 0; e < E; ++e) Sp[e] += ex;
            const T Wp = readlane_t(incl, kWave - 1);
            const T r0 = (T)range_reduce(readlane_u64(u, j), (uint64_t)Wp);
            const int32_t m = find_resident<E, T>(Sp, r0);
            if (lane == m / E) hb |= 1u << (m % E);
            if (lane == j) pos = m;
        }
    }
    return pos;
}

template <int E>
__device__ __forceinline__ int32_t draw_resident(const uint32_t* __restrict__ w, int64_t d, Key key, uint32_t c0,
                                                 uint32_t c1, uint32_t c2, int32_t k, int32_t rounds) {
    const int lane = lane_id();
    // d <= kWaveMaxD: 32-bit indices; every load is issued (clamped into the
    // list) and the tail zeroed after, so no lane branches
    const int32_t last = (int32_t)d - 1;
    uint32_t x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = w[min(lane * E + e, last)];
    uint32_t ls = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        x[e] = lane * E + e <= last ? x[e] : 0u;
        ls += x[e];
    }
    // routing guarantees W < 2^32, so every prefix fits 32 bits
    const uint32_t incl = wave_incl_scan_u32((uint32_t)ls);
    const uint32_t W = readlane_u32(incl, kWave - 1);
    return draw_resident_t<E, uint32_t>(x, incl - (uint32_t)ls, W, key, c0, c1, c2, k, rounds);
}

// A picked neighbor joins the instance's next bitmap unless it is already
// there: picks concentrate on hubs, and skipping those atomics keeps them from
// queueing on a few hot words. Visited vertices join too and are masked by the
// frontier build: testing the visited bit here reads a second random line per
// pick (batched R-MAT 22: 2 x 50M lines of a 4 GB pair of bitmaps) to save few
// atomics.
__device__ __forceinline__ void claim(bool do_claim, uint32_t* nextb, uint32_t* summb, int32_t x) {
    if (!do_claim) return;
    const uint32_t bit = 1u << (x & 31);
    const int64_t wd = x >> 5;
    if (!(nextb[wd] & bit)) {
        // the claim that makes a word non-zero records it in the summary (sparse builds)
        const uint32_t old = atomicOr(&nextb[wd], bit);
        if (summb && old == 0u) atomicOr(&summb[wd >> 5], 1u << (wd & 31));
    }
}

// The instance's summary bitmap (sparse builds) or null.
__device__ __forceinline__ uint32_t* summary_of(const SampleLayer& p, int64_t inst) {
    return p.summ ? p.summ + inst * p.nsw : nullptr;
}

// Load one tile of up to 1024 weights (from list offset base) into an LDS
// tile and return this lane's sum of its 16 consecutive elements.
__device__ __forceinline__ uint64_t tile_group_sums(const uint32_t* __restrict__ w, int64_t base, int64_t d,
                                                    uint32_t* tile) {
    const int lane = lane_id();
    uint32_t x[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const int64_t idx = base + c * kWave + lane;
        x[c] = idx < d ? w[idx] : 0u;
    }
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 16; ++c) tile[tpad(c * kWave + lane)] = x[c];
    wave_lds_sync();
    uint64_t s = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += tile[tpad(lane * 16 + q)];
    return s;
}

struct EntryInfo {
    int32_t c, v, inst, k, kind, P;
    int64_t o, beg, d;
    bool do_claim, wide;
    uint64_t key;
    uint32_t c0;
};

// A run of up to 64 consecutive frontier entries, one per lane: the entry's
// fields are read coalesced, then its instance's tables, so a wavefront pays
// two memory round trips for the whole run instead of several per entry.
struct EntryRun {
    int32_t c, v, inst, pinfo, k, kind, do_claim, c0;
    int32_t d;
    int64_t o, beg;
    uint64_t key;
};

// An entry's edge count c is k when it draws and P when it takes every positive
// candidate, so c < P tells the two apart.
__device__ __forceinline__ void load_run(const SampleLayer& p, int64_t e, bool valid, int64_t out_base,
                                         EntryRun& R) {
    R.c = valid ? p.cnt[e] : 0;
    R.v = valid ? p.fv[e] : 0;
    R.inst = valid ? p.fi[e] : 0;
    R.o = valid ? out_base + p.off[e] : 0;
    R.beg = valid ? p.fbeg[e] : 0;
    R.d = valid ? p.fdeg[e] : 0;
    R.pinfo = valid ? p.fpos[e] : 0;
    if (R.v < p.vlo || R.v >= p.vhi) R.c = 0;  // another partition's entry (out-of-memory schedule)
    R.k = R.kind = R.do_claim = 0;
    R.c0 = 0;
    R.key = 0;
    if (R.c) {
        R.k = R.c < (R.pinfo & ~kWideList) ? R.c : -1;
        R.kind = p.bias[R.inst];
        R.do_claim = p.fanout_next[R.inst] != 0;
        R.key = p.inst_key[R.inst];
        R.c0 = p.inst_id[R.inst];
    }
}

// The fields of run entry j, wave-uniform.
__device__ __forceinline__ EntryInfo run_entry(const EntryRun& R, int j) {
    EntryInfo E;
    E.c = readlane_i32(R.c, j);
    E.v = readlane_i32(R.v, j);
    E.inst = readlane_i32(R.inst, j);
    E.o = readlane_i64(R.o, j);
    E.beg = readlane_i64(R.beg, j);
    E.d = readlane_i32(R.d, j);
    const int32_t pinfo = readlane_i32(R.pinfo, j);
    E.P = pinfo & ~kWideList;
    E.wide = (pinfo & kWideList) != 0;
    E.k = readlane_i32(R.k, j);
    E.kind = readlane_i32(R.kind, j);
    E.do_claim = readlane_i32(R.do_claim, j) != 0;
    E.key = readlane_u64(R.key, j);
    E.c0 = readlane_u32(R.c0, j);
    return E;
}

__device__ __forceinline__ void emit_slots(const SampleLayer& p, const EntryInfo& E, int64_t pos) {
    const int lane = lane_id();
    if (lane < E.k) {
        const int32_t x = p.g.col[E.beg + pos];
        p.src[E.o + lane] = E.v;
        p.dst[E.o + lane] = x;
        claim(E.do_claim, p.next + (int64_t)E.inst * p.nwp, summary_of(p, E.inst), x);
    }
}

// ---------------------------------------------------------- slot per lane
// Main selection kernel: a lane is one slot of one entry. A wavefront loads a
// run of entries and packs whole entries into its 64 lanes (a draw takes its
// k slots, a take-all list of up to 64 candidates its d candidates), so one
// Philox block, one search and one column load serve the slots of several
// entries at once, and small fanouts leave few lanes idle. A slot finds its
// candidate by itself: an unbiased draw is its position; a weighted draw goes
// through the list's walk guide (one bucket, which decides nine draws in ten,
// whatever the list's length); without a guide a list of at most
// `bound` weights is scanned by each lane (the lanes of an entry read the
// same few words). Longer lists without a guide are left to k_select_wave and
// k_select_big.
// Collisions: in the first round a slot is accepted iff no lower slot of its
// entry drew the same candidate (a lower slot that was itself rejected was
// rejected for a still lower one), found by shifting the picks one lane at a
// time, for all entries side by side; the few open slots of the later rounds
// are taken one at a time in slot order, and those left after the last round
// by direct draws, one per entry at a time. The same picks, in the same
// order, as a wavefront per entry makes.
constexpr int kDppWaveShr1 = 0x138;
constexpr int32_t kScanMax = 32;  // longest list a lane scans

template <bool kWeighted>
struct SlotRun {
    int32_t v[kWave], inst[kWave], d[kWave], c0[kWave], info[kWave], own[kWave], stage[kWave];
    int64_t o[kWave], beg[kWave];
    uint64_t key[kWave];
    uint64_t W[kWeighted ? kWave : 1];
};
constexpr int kInfoKind = 3, kInfoTake = 4, kInfoClaim = 8, kInfoZeros = 16;

// Short lists (unbiased, or weighted with a walk guide; d at most kStagePer times
// the slots, a total below 2^32) are drawn from in LDS: their inclusive prefixes,
// copied from the edge records by the entry's own lanes (a list of 8 k edges
// takes as many lines as a bucket per slot), and a claim word per candidate.
// What these lists wait for is the chain of their rounds, and the
// direct draws, one after the other, of lists hardly longer than k or with a
// few heavy weights: a search per round and a slot at a time for its
// acceptance, through the buckets or through LDS, took 52 us for the 8,192 lists of a
// degree-biased layer.
// Here a round is one search and one atomic minimum for all open
// slots: the claim word keeps the smallest round * 64 + slot, so a held
// candidate stays held and the lowest slot of a round wins. A direct draw
// counts the updated prefixes at or below it with all lanes of the entry.
// (5 wavefronts per SIMD: more spilled registers to scratch memory)
template <bool kWeighted>
constexpr int kStageWords = kWeighted ? 368 : 220;
constexpr int kStagePer = 8;
constexpr int64_t kSlotResident = 5120;  // wavefronts of the weighted kernel on the chip at once
constexpr int64_t kSlotBatch = 6;        // entries of about ten slots that fill a wavefront

// Long take-all entry: every positive-bias neighbor in list order, one
// wavefront, 64 candidates (weighted with zero weights: 512) at a time.
__device__ __forceinline__ void take_all_entry(const SampleLayer& p, int32_t v, int32_t inst, int32_t info, int64_t o,
                                               int64_t beg, int32_t d) {
    const int lane = lane_id();
    const bool do_claim = (info & kInfoClaim) != 0;
    uint32_t* nextb = p.next + (int64_t)inst * p.nwp;
    uint32_t* summb = summary_of(p, inst);
    const int32_t* col = p.g.col + beg;
    int32_t* src = p.src + o;
    int32_t* dst = p.dst + o;
    if (!(info & kInfoZeros)) {
        for (int64_t j = lane; j < d; j += kWave) {
            const int32_t x = col[j];
            src[j] = v;
            dst[j] = x;
            claim(do_claim, nextb, summb, x);
        }
        return;
    }
    const uint32_t* w = ((info & kInfoKind) == kEdgeWeight ? p.g.ew : p.g.degw) + beg;
    int64_t run = 0;
    for (int64_t base = 0; base < d; base += 8 * kWave) {
        uint32_t x[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int64_t idx = base + c * kWave + lane;
            x[c] = idx < d ? w[idx] : 0u;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int64_t idx = base + c * kWave + lane;
            const bool pos = x[c] > 0;
            const uint64_t mask = ballot(pos);
            if (pos) {
                const int64_t slot = run + __popcll(mask & lanemask_lt());
                const int32_t nb = col[idx];
                src[slot] = v;
                dst[slot] = nb;
                claim(do_claim, nextb, summb, nb);
            }
            run += __popcll(mask);
        }
    }
}

__device__ __forceinline__ bool has_guide(const GraphDev& g, int32_t kind) {
    return kind == kEdgeWeight ? g.wgd_ew != nullptr : g.wgd_deg != nullptr;
}

// Does the slot kernel serve run entry R? (The others: k_select_wave, k_select_big.)
__device__ __forceinline__ bool slot_served(const SampleLayer& p, const EntryRun& R) {
    if (R.k < 0 || R.kind == kUniform || has_guide(p.g, R.kind)) return true;
    const int32_t bound = p.group32 > p.group16 ? p.group32 : p.group16;
    return !(R.pinfo & kWideList) && R.d <= (bound < kScanMax ? bound : kScanMax);
}

// m = max{i : S_i <= r}, r in [0, W), of the weighted list of vertex v (first
// edge beg, length d): nb receives the neighbor where the guide's records
// hold it, else -1.
__device__ __forceinline__ int32_t slot_search(const GraphDev& g, int32_t kind, int32_t v, int64_t beg, int32_t d,
                                               uint64_t W, uint64_t r, int32_t& nb) {
    const bool ew = kind == kEdgeWeight;
    nb = -1;
    if (!has_guide(g, kind)) {  // at most kScanMax weights, 8 loads in flight
        const uint32_t* w = (ew ? g.ew : g.degw) + beg;
        uint64_t run = 0;
        int32_t m = 0;
        for (int32_t i = 0; i < d; i += 8) {
            uint32_t x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = w[i + q < d ? i + q : d - 1];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                run += x[q];
                m += i + q < d && run <= r ? 1 : 0;
            }
        }
        return m;
    }
    const int per = ew ? g.gper_ew : g.gper_deg;
    const int sh = guide_shift(W, d, per);
    const uint64_t k = r >> sh;
    const WalkBucket b = ((ew ? g.wgd_ew : g.wgd_deg) + guide_base(beg, v, per))[k];
    if ((uint32_t)(b.S >> 32) != ~0u) {
        const bool second = (uint32_t)(r - (k << sh)) >= (uint32_t)b.S;
        nb = second ? (int32_t)(b.S >> 32) : b.col;
        return (int32_t)b.pos + (second ? 1 : 0);
    }
    int32_t lo = (int32_t)b.pos;
    const int32_t hi = d - 1;
    const WalkEdge* er = (ew ? g.wrec_ew : g.wrec_deg) + beg;
    constexpr int kProbe = 4;
    for (;;) {  // edge records from lo on (positions past hi read hi, whose prefix exceeds r)
        uint64_t S[kProbe];
        int32_t y[kProbe];
#pragma unroll
        for (int j = 0; j < kProbe; ++j) {
            const WalkEdge* e = er + (lo + j < hi ? lo + j : hi);
            S[j] = e->S;
            y[j] = e->col;
        }
        int c = 0;
#pragma unroll
        for (int j = 0; j < kProbe; ++j) c += S[j] <= r ? 1 : 0;
        if (c < kProbe) {
            nb = y[0];
#pragma unroll
            for (int j = 1; j < kProbe; ++j) nb = c == j ? y[j] : nb;
            return lo + c;
        }
        lo += kProbe;
    }
}

// S_m and b_m of a position of such a list.
__device__ __forceinline__ void slot_bias(const GraphDev& g, int32_t kind, int64_t beg, int32_t m, uint64_t& Sm,
                                          uint32_t& bm) {
    const bool ew = kind == kEdgeWeight;
    if (has_guide(g, kind)) {
        const WalkEdge e = (ew ? g.wrec_ew : g.wrec_deg)[beg + m];
        Sm = e.S - e.w;
        bm = e.w;
        return;
    }
    const uint32_t* w = (ew ? g.ew : g.degw) + beg;
    Sm = 0;
    for (int32_t i = 0; i < m; ++i) Sm += w[i];
    bm = w[m];
}

__device__ __forceinline__ uint64_t bperm_u64(uint64_t x, int from) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from * 4, (int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from * 4, (int)(uint32_t)(x >> 32));
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Sum of x over the lanes [sl, se) of the calling lane's entry (every lane active).
__device__ __forceinline__ uint64_t segment_sum(uint64_t x, int sl, int se) {
    const uint64_t run = wave_incl_scan_u64(x);
    const uint64_t upto = bperm_u64(run, se > 0 ? se - 1 : 0), from = bperm_u64(run, sl > 0 ? sl - 1 : 0);
    return upto - (sl > 0 ? from : 0ull);
}

// The draws of the staged entries of a wavefront's batch (every lane calls it;
// lanes [sl, se) are an entry, lane sl + j its slot j): returns this lane's
// position, or m for a lane of no staged entry. The staged words of the batch
// are pre[0, words) and claim[0, words); an entry's begin at `at`: pre[at] = 0,
// pre[at + 1 + i] the inclusive prefix of candidate i, claim[at + i].
template <bool kWeighted>
__device__ __forceinline__ int32_t draw_staged(const SampleLayer& p, const SlotRun<kWeighted>& L, uint32_t* pre, uint32_t* claim,
                                               int q, bool staged, int at, int sl, int se, uint64_t segmask, int words,
                                               int32_t m) {
    const int lane = lane_id();
    const int slot = lane - sl, k = se - sl;
    const int32_t d = L.d[q];
    const int32_t kind = kWeighted ? L.info[q] & kInfoKind : kUniform;
    const uint32_t c0 = (uint32_t)L.c0[q], v = (uint32_t)L.v[q];
    const Key key{(uint32_t)L.key[q], (uint32_t)(L.key[q] >> 32)};
    if (staged) {
        if (slot == 0) {
            pre[at] = 0u;
            claim[at + d] = ~0u;  // the last prefix's word has no candidate
        }
        if (kWeighted && kind != kUniform) {
            const WalkEdge* er = (kind == kEdgeWeight ? p.g.wrec_ew : p.g.wrec_deg) + L.beg[q];
            for (int32_t i = slot; i < d; i += 4 * k) {
                uint32_t x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = (uint32_t)er[i + t * k < d ? i + t * k : d - 1].S;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (i + t * k < d) {
                        pre[at + 1 + i + t * k] = x[t];
                        claim[at + i + t * k] = ~0u;
                    }
                }
            }
        } else {
            for (int32_t i = slot; i < d; i += k) {
                pre[at + 1 + i] = (uint32_t)i + 1;
                claim[at + i] = ~0u;
            }
        }
    }
    wave_lds_sync();
    uint32_t W = staged ? pre[at + d] : 0u;
    uint64_t open = ballot(staged);
    for (int a = 0; a < p.rounds && open; ++a) {
        const bool mine = ((open >> lane) & 1ull) != 0;
        uint32_t tag = 0;
        if (mine) {
            const uint64_t u = philox_u64(key.k0, key.k1, c0, (uint32_t)p.layer, v, (uint32_t)slot | ((uint32_t)a << 16));
            const uint32_t r = (uint32_t)range_reduce(u, W);
            int32_t i = (int32_t)r;
            if (kWeighted && kind != kUniform) {
                int32_t hi = d - 1;  // the first candidate whose prefix exceeds r
                for (i = 0; i < hi;) {
                    const int32_t mid = (i + hi) >> 1;
                    if (pre[at + 1 + mid] > r) hi = mid;
                    else i = mid + 1;
                }
            }
            m = i;
            tag = (uint32_t)(a * kWave + slot);
            atomicMin(&claim[at + m], tag);
        }
        wave_lds_sync();
        open &= ~ballot(mine && claim[at + m] == tag);
        wave_lds_sync();
    }
    if (!open) return m;
    // the prefixes without the held candidates: one running sum of the held
    // biases over all staged words (an entry's leading zero takes the sum before
    // it, so that differences from it are the entry's own; 32 bits wrap alike)
    uint64_t u = 0;
    if ((open >> lane) & 1ull)
        u = philox_u64(key.k0, key.k1, c0, (uint32_t)p.layer, v, (uint32_t)slot | (kFallbackRound << 16));
    uint32_t carry = 0;
    for (int w0 = 0; w0 < words; w0 += kWave) {
        const int w = w0 + lane;
        const uint32_t lo = w < words ? pre[w] : 0u;
        const uint32_t hi = w + 1 < words ? pre[w + 1] : 0u;
        const bool held = w + 1 < words && claim[w] != ~0u;
        const uint32_t b = held ? hi - lo : 0u;
        const uint32_t incl = wave_incl_scan_u32(b);
        wave_lds_sync();
        if (w < words) pre[w] = lo - (carry + incl - b);
        carry += readlane_u32(incl, kWave - 1);
        wave_lds_sync();
    }
    for (; open;) {
        const uint64_t o = open & segmask;
        const int j = o ? __ffsll((unsigned long long)o) - 1 : lane;  // the entry's lowest open slot
        const uint32_t zero = staged ? pre[at] : 0u;
        const uint32_t Wp = staged ? pre[at + d] - zero : 0u;
        const uint32_t r = (uint32_t)__builtin_amdgcn_ds_bpermute(j * 4, (int)(uint32_t)range_reduce(u, Wp));
        int32_t c = 0;  // candidates whose updated prefix is at or below r
        for (int32_t i = slot; ballot(o && i < d); i += k) {
            const bool le = o && i < d && pre[at + 1 + (i < d ? i : 0)] - zero <= r;
            c += __popcll(ballot(le) & segmask);
        }
        const uint32_t b = o ? pre[at + 1 + c] - pre[at + c] : 0u;
        wave_lds_sync();
        if (o) {
            for (int32_t i = slot; i < d; i += k)
                if (i >= c) pre[at + 1 + i] -= b;
        }
        wave_lds_sync();
        if (o && j == lane) m = c;
        open &= ~ballot(o && j == lane);
    }
    return m;
}

// kWeighted: some instance of the call draws by weight.
template <bool kWeighted>
__global__ void __launch_bounds__(kBlock, 5) k_select_slots(SampleLayer p) {
    __shared__ SlotRun<kWeighted> runs[kWavesPerBlock];
    __shared__ uint32_t stage_prefix[kWavesPerBlock][kStageWords<kWeighted>], stage_claim[kWavesPerBlock][kStageWords<kWeighted>];
    const int wid = uniform_i32(threadIdx.x / kWave);
    SlotRun<kWeighted>& L = runs[wid];
    const int lane = lane_id();
    const int64_t fcount = frontier_size(p.ctl, p.layer);
    const int64_t out_base = p.ctl->out_base[p.layer];
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave = blockIdx.x * (int64_t)kWavesPerBlock + wid;
    // one entry a wavefront while the resident wavefronts last (the chain of one
    // entry is then all there is to wait for), then up to a batch's worth, so
    // that a second round of wavefronts starts only with full lanes: 206 -> 172 us
    // for a degree-biased call of 1M edges against an even share of the grid
    const int64_t share = (fcount + kSlotResident - 1) / kSlotResident, even = (fcount + waves - 1) / waves;
    const int64_t least = share < kSlotBatch ? share : kSlotBatch;
    const int64_t per = even > least ? even : least;
    const int64_t lo = wave * per < fcount ? wave * per : fcount;
    const int64_t hi = lo + per < fcount ? lo + per : fcount;
    for (int64_t e0 = lo; e0 < hi; e0 += kWave) {
        const int n = (int)(hi - e0 < kWave ? hi - e0 : kWave);
        uint32_t ln;           // lanes the entry takes
        uint32_t sincl, sd = 0;  // words staged in LDS, summed over the run, and the entry's own
        uint64_t long_take;
        {
            EntryRun R;
            load_run(p, e0 + lane, lane < n, out_base, R);
            bool ok = R.c != 0;
            if (ok && R.o + R.c > p.capacity) {
                p.ctl->overflow = 1;
                ok = false;
            }
            ok = ok && (!kWeighted || slot_served(p, R));
            const bool take = R.k < 0;
            ln = !ok ? 0u : (uint32_t)(take ? R.d : R.k);
            long_take = ballot(ln > (uint32_t)kWave);
            if (ln > (uint32_t)kWave) ln = 0;
            uint64_t W = (uint64_t)(uint32_t)R.d;
            if (kWeighted && ln && !take && R.kind != kUniform)
                W = (R.kind == kEdgeWeight ? p.g.wtot_ew : p.g.wtot_deg)[R.v];
            if (ln && !take && R.d <= kStagePer * R.k && R.d < kStageWords<kWeighted> &&
                (R.kind == kUniform || (has_guide(p.g, R.kind) && !(W >> 32))))
                sd = (uint32_t)R.d + 1;  // a zero, then the prefixes
            sincl = wave_incl_scan_u32(sd);
            wave_lds_sync();
            L.v[lane] = R.v;
            L.inst[lane] = R.inst;
            L.d[lane] = R.d;
            L.c0[lane] = R.c0;
            L.info[lane] = R.kind | (take ? kInfoTake : 0) | (R.do_claim ? kInfoClaim : 0) |
                           (take && R.kind != kUniform && (R.pinfo & ~kWideList) != R.d ? kInfoZeros : 0);
            L.o[lane] = R.o;
            L.beg[lane] = R.beg;
            L.key[lane] = R.key;
            if (kWeighted) L.W[lane] = W;
        }
        const uint32_t incl = wave_incl_scan_u32(ln);
        const uint32_t excl = incl - ln;
        for (int s0 = 0; s0 < n;) {
            // entries [s0, s1): as many as fit the 64 lanes and the staging words
            const uint32_t base = s0 ? readlane_u32(incl, s0 - 1) : 0u;
            const uint32_t sbase = s0 ? readlane_u32(sincl, s0 - 1) : 0u;
            const uint64_t fit = ballot(incl - base <= (uint32_t)kWave && sincl - sbase <= (uint32_t)kStageWords<kWeighted>) >> s0;
            const int s1 = s0 + (~fit ? __ffsll((unsigned long long)~fit) - 1 : kWave);
            const int total = (int)(readlane_u32(incl, s1 - 1) - base);
            const int total_words = (int)(readlane_u32(sincl, s1 - 1) - sbase);
            const bool mine = lane >= s0 && lane < s1 && ln > 0;
            s0 = s1;
            if (total == 0) continue;
            wave_lds_sync();
            L.own[lane] = -1;
            wave_lds_sync();
            if (mine) {
                L.own[excl - base] = lane;
                L.stage[lane] = sd ? (int32_t)(sincl - sd - sbase) : -1;
            }
            wave_lds_sync();
            // lanes [sl, se) are the entry of run position q
            const uint64_t starts = ballot(L.own[lane] >= 0);
            const bool valid = lane < total;
            const uint64_t upto = starts & (~0ull >> (63 - lane)), after = starts & ~(~0ull >> (63 - lane));
            const int sl = 63 - __clzll((long long)(upto | 1ull));
            const int se = after ? __ffsll((unsigned long long)after) - 1 : total;
            const uint64_t segmask = valid ? (~0ull >> (64 - (se - sl))) << sl : 0ull;
            const int q = valid ? L.own[sl] : 0;
            const int slot = lane - sl;
            const int32_t info = L.info[q];
            bool draws = valid && !(info & kInfoTake);
            int32_t m = slot, nb = -1;  // this slot's position, and its neighbor once known
            int at = slot;              // edge slot of this lane
            bool emit = valid;
            if (kWeighted && ballot(valid && (info & kInfoZeros))) {  // take-all lists with zero weights: positives only
                const bool z = valid && (info & kInfoZeros);
                const bool pos = z && ((info & kInfoKind) == kEdgeWeight ? p.g.ew : p.g.degw)[L.beg[q] + slot] > 0;
                const uint64_t pm = ballot(pos);
                if (z) {
                    emit = pos;
                    at = __popcll(pm & segmask & lanemask_lt());
                }
            }
            const int stage_at = draws ? L.stage[q] : -1;
            const bool staged = stage_at >= 0;
            if (ballot(staged))
                m = draw_staged<kWeighted>(p, L, stage_prefix[wid], stage_claim[wid], q, staged, stage_at, sl, se,
                                           segmask, total_words, m);
            draws = draws && !staged;
            uint64_t open = ballot(draws);
            // direct draws: start in the updated prefix and bias of this held
            // slot, and the held bias of its entry
            uint64_t start = 0, removed = 0;
            uint32_t bias = 0;
            for (int a = 0; open; ++a) {
                // the entry's fields again from LDS: held in registers across
                // the rounds they cost occupancy
                wave_lds_sync();
                const int32_t kind = kWeighted ? L.info[q] & kInfoKind : kUniform;
                const int32_t v = L.v[q], d = L.d[q];
                const int64_t beg = L.beg[q];
                const uint64_t W = kWeighted ? L.W[q] : (uint64_t)(uint32_t)d;
                const uint64_t key = L.key[q];
                const bool direct = a >= p.rounds;
                const uint64_t eopen = open & segmask;  // the entry's open slots
                const bool myopen = ((open >> lane) & 1ull) != 0;
                const bool held = draws && eopen && !myopen;  // (direct draws)
                const int j = eopen ? __ffsll((unsigned long long)eopen) - 1 : lane;
                const bool turn = direct ? draws && eopen && j == lane : myopen;
                uint64_t r = 0;
                if (turn)
                    r = philox_u64((uint32_t)key, (uint32_t)(key >> 32), (uint32_t)L.c0[q], (uint32_t)p.layer, (uint32_t)v,
                                   (uint32_t)slot | ((direct ? kFallbackRound : (uint32_t)a) << 16));
                if (direct) {
                    if (a == p.rounds) {
                        if (held) {
                            start = (uint64_t)(uint32_t)m;
                            bias = 1;
                            if (kWeighted && kind != kUniform) slot_bias(p.g, kind, beg, m, start, bias);
                        }
                        const uint64_t S0 = start;
                        for (uint64_t hm = ballot(held); hm; hm &= hm - 1) {
                            const int h = __ffsll((unsigned long long)hm) - 1;
                            const uint64_t Sh = readlane_u64(S0, h);
                            const uint32_t bh = readlane_u32(bias, h);
                            if (eopen && h >= sl && h < se) {
                                removed += bh;
                                if (held && Sh < S0) start -= bh;
                            }
                        }
                    }
                    // r0 in [0, W - held bias), plus every held candidate whose
                    // start in the updated prefix is at or below it
                    r = range_reduce(r, W - removed);
                    const uint64_t rj = bperm_u64(r, j);
                    r += segment_sum(held && start <= rj ? bias : 0u, sl, se);
                } else if (turn) {
                    r = range_reduce(r, W);
                }
                if (turn) {
                    m = (int32_t)r;
                    if (kWeighted && kind != kUniform) m = slot_search(p.g, kind, v, beg, d, W, r, nb);
                }
                if (direct) {
                    uint64_t Sj = (uint64_t)(uint32_t)m;
                    uint32_t bj = 1;
                    if (kWeighted && turn && kind != kUniform) slot_bias(p.g, kind, beg, m, Sj, bj);
                    const int32_t mt = __builtin_amdgcn_ds_bpermute(j * 4, m);
                    const uint32_t bt = (uint32_t)__builtin_amdgcn_ds_bpermute(j * 4, (int)bj);
                    const uint64_t below = segment_sum(held && m < mt ? bias : 0u, sl, se);
                    if (eopen) {
                        removed += bt;
                        if (held && m > mt) start -= bt;
                    }
                    if (turn) {
                        start = Sj - below;
                        bias = bj;
                    }
                    open &= ~ballot(turn);
                } else if (a == 0) {
                    // a slot yields to a lower one of its entry with the same pick
                    bool dup = false;
                    int32_t y = m;
                    for (int t = 1; ballot(draws && slot >= t); ++t) {
                        y = __builtin_amdgcn_update_dpp(0, y, kDppWaveShr1, 0xf, 0xf, false);
                        dup |= slot >= t && y == m;
                    }
                    open = ballot(draws && dup);
                } else {
                    for (uint64_t todo = open; todo; todo &= todo - 1) {  // slot order
                        const int i = __ffsll((unsigned long long)todo) - 1;
                        const int32_t mi = readlane_i32(m, i);
                        const uint64_t si = readlane_u64(segmask, i);
                        if ((ballot(m == mi) & si & ~open) == 0) open &= ~(1ull << i);
                    }
                }
            }
            if (emit) {
                if (nb < 0) nb = p.g.col[L.beg[q] + m];
                const int64_t o = L.o[q] + at;
                const int32_t inst = L.inst[q];
                p.src[o] = L.v[q];
                p.dst[o] = nb;
                claim((info & kInfoClaim) != 0, p.next + (int64_t)inst * p.nwp, summary_of(p, inst), nb);
            }
        }
        for (; long_take; long_take &= long_take - 1) {
            const int q = __ffsll((unsigned long long)long_take) - 1;
            take_all_entry(p, uniform_i32(L.v[q]), uniform_i32(L.inst[q]), uniform_i32(L.info[q]),
                           uniform_i64(L.o[q]), uniform_i64(L.beg[q]), uniform_i32(L.d[q]));
        }
    }
}

// Weighted draws from lists without a walk guide, longer than a lane scans
// and of at most kWaveMaxD candidates: one wavefront per entry, the list and
// its prefix in registers. Each wavefront takes a contiguous share of the
// frontier, loaded 64 entries at a time; a share holds few such entries when
// the call is mixed, and the launch is left out when every weighted kind of
// the call has its guide. kTake: the take-all lists too, where every instance
// draws by such a kind and no list is scanned by a lane: the slot kernel would
// have nothing else to do (8,192 seeds, 456,000 degree-biased edges on R-MAT 22: 0.252
// ms a call with it, 0.233 without).
template <bool kTake>
__global__ void __launch_bounds__(kBlock) k_select_wave(SampleLayer p) {
    const int wid = uniform_i32(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t fcount = frontier_size(p.ctl, p.layer);
    const int64_t out_base = p.ctl->out_base[p.layer];
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave = blockIdx.x * (int64_t)kWavesPerBlock + wid;
    const int64_t per = (fcount + waves - 1) / waves;
    const int64_t lo = wave * per < fcount ? wave * per : fcount;
    const int64_t hi = lo + per < fcount ? lo + per : fcount;
    for (int64_t e0 = lo; e0 < hi; e0 += kWave) {
        const int n = (int)(hi - e0 < kWave ? hi - e0 : kWave);
        EntryRun R;
        load_run(p, e0 + lane, lane < n, out_base, R);
        if (kTake && R.c != 0 && R.o + R.c > p.capacity) p.ctl->overflow = 1;
        uint64_t todo = ballot(R.c != 0 && R.o + R.c <= p.capacity &&
                               (slot_served(p, R) ? kTake && R.k < 0 : R.d <= kWaveMaxD && !(R.pinfo & kWideList)));
        for (; todo; todo &= todo - 1) {
            const int i = __ffsll((unsigned long long)todo) - 1;
            if (kTake && readlane_i32(R.k, i) < 0) {
                const int32_t info = R.kind | kInfoTake | (R.do_claim ? kInfoClaim : 0) |
                                     (R.kind != kUniform && (R.pinfo & ~kWideList) != R.d ? kInfoZeros : 0);
                take_all_entry(p, readlane_i32(R.v, i), readlane_i32(R.inst, i), readlane_i32(info, i),
                               readlane_i64(R.o, i), readlane_i64(R.beg, i), readlane_i32(R.d, i));
                continue;
            }
            const EntryInfo E = run_entry(R, i);
            const Key key{(uint32_t)E.key, (uint32_t)(E.key >> 32)};
            const uint32_t* w = (E.kind == kEdgeWeight ? p.g.ew : p.g.degw) + E.beg;
            const uint32_t c1 = (uint32_t)p.layer, c2 = (uint32_t)E.v;
            int64_t pos;
            if (E.d <= 64) pos = draw_resident<1>(w, E.d, key, E.c0, c1, c2, E.k, p.rounds);
            else if (E.d <= 128) pos = draw_resident<2>(w, E.d, key, E.c0, c1, c2, E.k, p.rounds);
            else if (E.d <= 256) pos = draw_resident<4>(w, E.d, key, E.c0, c1, c2, E.k, p.rounds);
            else pos = draw_resident<8>(w, E.d, key, E.c0, c1, c2, E.k, p.rounds);
            emit_slots(p, E, pos);
        }
    }
}

// ------------------------------------------------------ long-list path
// Chunk prefix table, once per graph and weight array: one wavefront per
// list longer than kWaveMaxD, chunk by chunk (coalesced loads, LDS
// transpose, one 16-weight group per lane, a 64-lane scan): row
// (b >> kTabShift) + j holds the inclusive group prefixes of chunk j of the
// list starting at edge b. A list of d > 512 weights spans at least
// floor(d / 512) >= ceil(d / 1024) rows of 512 edges, so the rows of
// different lists never meet, and every row is below (m >> kTabShift).
// ctab (may be null) gets the list's running total at the end of each chunk:
// ctab[(b >> kTabShift) + j] = total weight of chunks 0..j.
__global__ void __launch_bounds__(kBlock) k_chunk_table(RowPtr rowptr,
                                                        const uint32_t* __restrict__ w, int64_t n,
                                                        uint64_t* __restrict__ tab, uint64_t* __restrict__ ctab) {
    __shared__ uint32_t tiles[kWavesPerBlock][kTilePad];
    const int wid = uniform_i32(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t v = blockIdx.x * (int64_t)kWavesPerBlock + wid; v < n; v += waves) {
        const int64_t b = uniform_i64(rowptr[v]);
        const int64_t d = uniform_i64(rowptr[v + 1]) - b;
        if (d <= kWaveMaxD) continue;
        uint64_t* row = tab + (b >> kTabShift) * kChunkGroups;
        uint64_t run = 0;
        for (int64_t j = 0; j < chunks_of(d); ++j) {
            const int64_t len = d - j * kChunk < kChunk ? d - j * kChunk : kChunk;
            const uint64_t s = tile_group_sums(w + b + j * kChunk, 0, len, tiles[wid]);
            const uint64_t incl = wave_incl_scan_u64(s);
            row[j * kChunkGroups + lane] = incl;
            run += readlane_u64(incl, kWave - 1);
            if (ctab && lane == 0) ctab[(b >> kTabShift) + j] = run;
        }
    }
}

// The group of chunk row `row` (64 inclusive group prefixes) that holds r,
// given the total acc before the chunk: the first i with acc + row[i] > r,
// and the prefix before it. Two rounds of eight independent loads (octant
// ends, then the octant) instead of a six-step binary search.
__device__ __forceinline__ int32_t row_group(const uint64_t* __restrict__ row, uint64_t acc, uint64_t r,
                                             uint64_t& before) {
    uint64_t ends[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) ends[q] = row[8 * q + 7];
    int32_t o = 0;
#pragma unroll
    for (int q = 0; q < 7; ++q) o += acc + ends[q] <= r ? 1 : 0;  // r lies inside the chunk: octant 7 ends past it
    uint64_t g8[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) g8[k] = row[8 * o + k];
    int32_t c = 0;
    before = 0;
    for (int q = 0; q < 8; ++q)
        if (q < o) before = ends[q];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const bool le = acc + g8[k] <= r;
        c += le ? 1 : 0;
        before = le ? g8[k] : before;
    }
    return 8 * o + c;
}

// Per-lane search of a long list through its chunk prefixes (pass 1) and a
// coarse LDS table over units of 2^shift chunks: tab[u] = total weight of
// the chunks before unit u, tab[nu] = W. Finds the unit by binary search in
// LDS, the chunk by a walk over the unit's chunk totals, the group by binary
// search in the chunk's G row and the candidate by scanning the group's
// weights (global memory / L2).
struct UnitPool {
    const uint64_t* tab;    // LDS, nu + 1 entries
    int64_t nu;
    int shift;
    int64_t nch;            // chunks of the list
    const uint64_t* G;      // G rows of the list's chunks
    const uint32_t* w;      // weights of the list
    int64_t d;
};

__device__ __forceinline__ void unit_search(const UnitPool& pl, uint64_t r, int64_t& m, uint64_t& Sm,
                                            uint32_t& bm) {
    int64_t lo = 0, hi = pl.nu;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (pl.tab[mid] <= r) lo = mid;
        else hi = mid;
    }
    uint64_t acc = pl.tab[lo];
    int64_t j = lo << pl.shift;
    const int64_t jend = ((lo + 1) << pl.shift) < pl.nch ? ((lo + 1) << pl.shift) : pl.nch;
    for (; j + 1 < jend; ++j) {  // chunk totals of the unit
        const uint64_t t = pl.G[j * kChunkGroups + kChunkGroups - 1];
        if (acc + t > r) break;
        acc += t;
    }
    uint64_t before;
    const int32_t ghi = row_group(pl.G + j * kChunkGroups, acc, r, before);
    const int64_t i = j * kChunk + (int64_t)ghi * 16;
    const int64_t end = i + 16 < pl.d ? i + 16 : pl.d;
    fine_scan_global(pl.w, i, end, acc + before, r, m, Sm, bm);
}

// One wavefront per long list. Lists of up to kGroupTabD weights get a
// group-level table (C[t] = weight before group t, from the chunk totals and
// the G rows), searched like the wavefront path with the group's weights
// read from global memory; longer lists get a unit-level table (UnitPool).
// The G rows come from the graph's chunk prefix table, or for a list of at
// most kWaveMaxD weights (wide total) from its one chunk reduced here.
constexpr int kBigTab = 512;
constexpr int64_t kGroupTabD = (int64_t)kBigTab * 16;

__device__ void select_big_entry(const SampleLayer& p, const EntryInfo& E, uint64_t* tab) {
    const int lane = lane_id();
    if (E.c == 0) return;
    if (E.o + E.c > p.capacity) {
        if (lane == 0) p.ctl->overflow = 1;
        return;
    }
    const int64_t d = E.d;
    const Key key{(uint32_t)E.key, (uint32_t)(E.key >> 32)};
    const uint32_t c0 = E.c0, c1 = (uint32_t)p.layer, c2 = (uint32_t)E.v;
    const int64_t nch = chunks_of(d);
    const uint32_t* w = (E.kind == kEdgeWeight ? p.g.ew : p.g.degw) + E.beg;
    const uint64_t* G = (E.kind == kEdgeWeight ? p.g.gtab_ew : p.g.gtab_deg) + (E.beg >> kTabShift) * kChunkGroups;
    const bool onchip = d <= kWaveMaxD;  // one chunk, not in the table
    int64_t pos;
    if (d <= kGroupTabD) {
        const int64_t nc = (d + 15) / 16;
        uint64_t rows[kGroupTabD / kChunk];
        uint64_t tj;
        if (onchip) {  // (rare) group sums straight from the list, lane = group
            const int64_t i0 = (int64_t)lane * 16;
            uint64_t s = 0;
#pragma unroll 4
            for (int q = 0; q < 16; ++q) s += i0 + q < d ? w[i0 + q] : 0u;
            rows[0] = wave_incl_scan_u64(s);
#pragma unroll
            for (int j = 1; j < kGroupTabD / kChunk; ++j) rows[j] = 0ull;
            tj = lane == 0 ? readlane_u64(rows[0], kWave - 1) : 0ull;
        } else {
#pragma unroll
            for (int j = 0; j < kGroupTabD / kChunk; ++j) rows[j] = j < nch ? G[j * kChunkGroups + lane] : 0ull;
            tj = lane < nch ? G[lane * kChunkGroups + kChunkGroups - 1] : 0ull;
        }
        const uint64_t cincl = wave_incl_scan_u64(tj);
        const uint64_t cex = cincl - tj;
#pragma unroll
        for (int j = 0; j < kGroupTabD / kChunk; ++j) {
            const uint64_t base = readlane_u64(cex, j);
            const int64_t t = (int64_t)j * kChunkGroups + lane;
            if (j < nch && t < nc) tab[t + 1] = base + rows[j];
        }
        if (lane == 0) tab[0] = 0;
        const uint64_t W = readlane_u64(cincl, (int)nch - 1);
        wave_lds_sync();
        const CoarsePool pl{tab, nc, 16, d, w};
        const auto search = [&pl](uint64_t r, int64_t& m, uint64_t& Sm, uint32_t& bm) {
            coarse_search(pl, r, m, Sm, bm);
        };
        pos = draw_slots(key, c0, c1, c2, E.k, p.rounds, W, search, search);
    } else {
        int shift = 0;
        while (((nch + (1ll << shift) - 1) >> shift) > kBigTab) ++shift;
        const int64_t nu = (nch + (1ll << shift) - 1) >> shift;
        uint64_t carry = 0;
        for (int64_t u0 = 0; u0 < nu; u0 += kWave) {
            const int64_t u = u0 + lane;
            uint64_t s = 0;
            if (u < nu) {
                const int64_t j0 = u << shift;
                const int64_t j1 = j0 + (1ll << shift) < nch ? j0 + (1ll << shift) : nch;
                for (int64_t j = j0; j < j1; ++j) s += G[j * kChunkGroups + kChunkGroups - 1];
            }
            const uint64_t incl = wave_incl_scan_u64(s);
            if (u < nu) tab[u + 1] = carry + incl;
            carry += readlane_u64(incl, kWave - 1);
        }
        if (lane == 0) tab[0] = 0;
        wave_lds_sync();
        const UnitPool pl{tab, nu, shift, nch, G, w, d};
        const auto search = [&pl](uint64_t r, int64_t& m, uint64_t& Sm, uint32_t& bm) {
            unit_search(pl, r, m, Sm, bm);
        };
        pos = draw_slots(key, c0, c1, c2, E.k, p.rounds, carry, search, search);
    }
    emit_slots(p, E, pos);
    wave_lds_sync();  // the table is rewritten by the wave's next list
}

__global__ void __launch_bounds__(kBlock) k_select_big(SampleLayer p) {
    __shared__ uint64_t tabs[kWavesPerBlock][kBigTab + 1];
    const int wid = uniform_i32(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t nb = p.ctl->gave_up() ? 0 : (int64_t)p.ctl->nbig[p.layer];
    const int64_t out_base = p.ctl->out_base[p.layer];
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave = blockIdx.x * (int64_t)kWavesPerBlock + wid;
    const int64_t per = (nb + waves - 1) / waves;
    const int64_t lo = wave * per < nb ? wave * per : nb;
    const int64_t hi = lo + per < nb ? lo + per : nb;
    for (int64_t h0 = lo; h0 < hi; h0 += kWave) {
        const int n = (int)(hi - h0 < kWave ? hi - h0 : kWave);
        const bool valid = lane < n;
        const int64_t pos = valid ? p.bigs[h0 + lane] : 0;
        EntryRun R;
        load_run(p, pos, valid, out_base, R);
        // (a kind with its walk guide is the slot kernel's)
        for (uint64_t todo = ballot(R.c != 0 && !has_guide(p.g, R.kind)); todo; todo &= todo - 1)
            select_big_entry(p, run_entry(R, __ffsll((unsigned long long)todo) - 1), tabs[wid]);
    }
}

// ------------------------------------------------------ layer sampling
// One wavefront per instance, every layer in the kernel (Section II-A:
// layer sampling selects a constant number of neighbors for the whole
// frontier). Per layer: per frontier vertex its list's total bias and
// length, two exclusive prefixes over the frontier in LDS (bias and
// position), then k slots drawn like one list (rounds in slot order, direct
// draws) with counter (instance id, layer, 0xFFFFFFFF, slot | round << 16):
// a draw r finds its frontier vertex by binary search in the bias prefix and
// its neighbor in that list (the walk guide or list_search; the position itself
// if unbiased). Picks not visited, deduplicated and sorted, form the next frontier (at
// most 64 vertices).
__device__ __forceinline__ int32_t lds_upper(const uint64_t* a, int32_t n, uint64_t r) {
    // largest f in [0, n) with a[f] <= r (a[0] = 0 <= r)
    int32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (a[mid] <= r) lo = mid;
        else hi = mid;
    }
    return lo;
}

// m = max{i : S_i <= r} inside one weighted list (weights w, first edge beg,
// length d, prefix acc before it), with S_m and b_m: a scan of the list for
// up to kWaveMaxD weights, kWeightPad of them in flight (past the list's end too, where
// r, below its total, is never looked for; the arrays are padded); else through the graph's
// chunk prefix table (the running chunk totals, the chunk's group prefixes, one group).
struct alignas(4) WeightQuad {
    uint32_t x[4];
};
__device__ __forceinline__ void list_search(const uint32_t* __restrict__ w, const uint64_t* __restrict__ gtab,
                                            const uint64_t* __restrict__ ctab, int64_t beg, int64_t d, uint64_t acc,
                                            uint64_t r, int64_t& m, uint64_t& Sm, uint32_t& bm) {
    constexpr int kQuads = kWeightPad / 4;
    if (d <= kWaveMaxD) {
        for (int32_t i0 = 0; i0 < (int32_t)d; i0 += 4 * kQuads) {
            WeightQuad y[kQuads];
#pragma unroll
            for (int q = 0; q < kQuads; ++q) y[q] = *(const WeightQuad*)(w + i0 + 4 * q);
            uint64_t run = acc;  // the quad that ends above r, then the weight
            int32_t c = 0;
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                run += (uint64_t)y[q].x[0] + y[q].x[1] + ((uint64_t)y[q].x[2] + y[q].x[3]);
                const bool le = run <= r;
                c += le ? 1 : 0;
                acc = le ? run : acc;
            }
            if (c == kQuads) continue;
            uint32_t z0 = y[0].x[0], z1 = y[0].x[1], z2 = y[0].x[2], z3 = y[0].x[3];
#pragma unroll
            for (int q = 1; q < kQuads; ++q) {
                const bool at = q == c;
                z0 = at ? y[q].x[0] : z0;
                z1 = at ? y[q].x[1] : z1;
                z2 = at ? y[q].x[2] : z2;
                z3 = at ? y[q].x[3] : z3;
            }
            const uint64_t s0 = acc + z0, s1 = s0 + z1, s2 = s1 + z2;
            const int32_t k = (s0 <= r ? 1 : 0) + (s1 <= r ? 1 : 0) + (s2 <= r ? 1 : 0);
            Sm = k == 0 ? acc : k == 1 ? s0 : k == 2 ? s1 : s2;
            bm = k == 0 ? z0 : k == 1 ? z1 : k == 2 ? z2 : z3;
            m = i0 + 4 * c + k;
            return;
        }
        return;
    }
    const int64_t row0 = beg >> kTabShift, nch = chunks_of(d);
    const uint64_t* G = gtab + row0 * kChunkGroups;
    int64_t j = 0;
    if (ctab) {
        const uint64_t* C = ctab + row0;
        int64_t hi = nch - 1;  // the first chunk whose running total exceeds r
        while (j < hi) {
            const int64_t mid = (j + hi) >> 1;
            if (acc + C[mid] <= r) j = mid + 1;
            else hi = mid;
        }
        if (j > 0) acc += C[j - 1];
    } else {
        for (; j + 1 < nch; ++j) {
            const uint64_t t = G[j * kChunkGroups + kChunkGroups - 1];
            if (acc + t > r) break;
            acc += t;
        }
    }
    uint64_t before;
    const int32_t ghi = row_group(G + j * kChunkGroups, acc, r, before);
    const int64_t i = j * kChunk + (int64_t)ghi * 16;
    fine_scan_global(w, i, i + 16 < d ? i + 16 : d, acc + before, r, m, Sm, bm);
}

// LDS of one wavefront, sized by the call's largest seed set mf and its
// layers. A frontier holds the seeds, then at most 64 picks: cf = max(mf, 64)
// entries. The two prefixes (uint64, cf + 1 each), then the visited list (mf +
// 64 per layer: each layer's frontier, sorted, behind the one before it) and the
// picks (64).
__host__ __device__ inline int32_t layer_frontier_cap(int32_t mf) { return mf > kWave ? mf : kWave; }
inline size_t layer_lds_bytes(int32_t mf, int32_t L) {
    const size_t cf = (size_t)layer_frontier_cap(mf);
    return 2 * sizeof(uint64_t) * (cf + 1) + sizeof(int32_t) * ((size_t)mf + 64 * (size_t)L + kWave);
}

// An instance is one wavefront's chain of loads, and 2,000 instances leave a SIMD two
// of them: the time is the chain's length. So the seeds, and a frontier's totals,
// are read with eight loads of a kind in flight, each lane summing a run of the
// frontier (one scan per layer); a pick is looked for in the earlier frontiers by
// binary search, and not at all in the last layer.
// 2,000 instances of 512 seeds, two layers of 64 degree-biased picks on R-MAT 22: 90 us
// through a walk guide (110 with the positive positions of every vertex read and its
// record in two tables). Without one (list_search), calls on new seeds: 324 us with 16
// weights in flight and linear chunk walks, 253 with 64 compared one by one, 216 with
// their quads compared first; 500 instances of 16 seeds, one layer of 5: 80, 99 and 68.
constexpr int kLayerPer = 8;
__global__ void __launch_bounds__(kWave) k_layer_sample(LayerParams p) {
    extern __shared__ __align__(16) unsigned char layer_lds[];
    const int32_t cf = layer_frontier_cap(p.max_f);
    uint64_t* Wp = (uint64_t*)layer_lds;
    uint64_t* Dp = Wp + (cf + 1);
    int32_t* vis = (int32_t*)(Dp + (cf + 1));
    int32_t* pk = vis + p.max_f + 64 * p.L;  // this layer's picks by slot
    const int lane = lane_id();
    const Key key{p.k0, p.k1};
    const bool guide = p.bias != kUniform && has_guide(p.g, p.bias);
    const WalkVertex* vt = !guide ? nullptr : p.bias == kEdgeWeight ? p.g.wvtx_ew : p.g.wvtx_deg;
    const uint32_t* wts = p.bias == kEdgeWeight ? p.g.ew : p.g.degw;
    const int32_t* ppos = p.bias == kEdgeWeight ? p.g.ppos_ew : p.g.ppos_deg;
    const uint64_t* wtot = p.bias == kEdgeWeight ? p.g.wtot_ew : p.g.wtot_deg;
    const uint64_t* gtab = p.bias == kEdgeWeight ? p.g.gtab_ew : p.g.gtab_deg;
    const uint64_t* ctab = p.bias == kEdgeWeight ? p.g.ctab_ew : p.g.ctab_deg;
    for (int64_t i = blockIdx.x; i < p.num_instances; i += gridDim.x) {
        const int64_t o0 = uniform_i64(p.seed_off[i]);
        int32_t nf = (int32_t)(uniform_i64(p.seed_off[i + 1]) - o0);  // <= kMaxPool (checked by the host)
        const uint32_t iid = (uint32_t)(p.instance_base + (uint64_t)i);
        bool bad = false;
        for (int32_t f0 = 0; f0 < nf; f0 += kLayerPer * kWave) {
            int32_t v[kLayerPer], prev[kLayerPer];
#pragma unroll
            for (int q = 0; q < kLayerPer; ++q) {
                const int32_t f = f0 + q * kWave + lane;
                v[q] = f < nf ? p.seeds[o0 + f] : 0;
                prev[q] = f > 0 && f < nf ? p.seeds[o0 + f - 1] : -1;
            }
#pragma unroll
            for (int q = 0; q < kLayerPer; ++q) {
                const int32_t f = f0 + q * kWave + lane;
                if (f < nf) {
                    bad |= v[q] < 0 || (int64_t)v[q] >= p.g.n || v[q] <= prev[q];
                    vis[f] = v[q];
                }
            }
        }
        if (ballot(bad)) {  // outputs of the call are unspecified; the host reports the error
            if (lane == 0) *p.bad = 1;
            wave_lds_sync();
            continue;
        }
        int32_t* F = vis;        // this layer's frontier
        int32_t ends = nf;       // lane l: end of layer l's frontier in the visited list (lane 0's so far)
        int32_t nvis = nf;
        wave_lds_sync();
        for (int32_t l = 0; l < p.L; ++l) {
            const int32_t k = p.fan[l];
            int32_t* src = p.src + (i * p.L + l) * p.K;
            int32_t* dst = p.dst + (i * p.L + l) * p.K;
            // totals per frontier vertex and both prefixes: lane L sums vertices [L c, L c + c)
            const int32_t c1 = (nf + kWave - 1) / kWave, first = lane * c1;
            uint64_t sw = 0, sd = 0;
            uint32_t lists = 0;  // with a positive total
            for (int32_t q0 = 0; q0 < c1; q0 += kLayerPer) {
                uint64_t wv[kLayerPer], dv[kLayerPer];
#pragma unroll
                for (int q = 0; q < kLayerPer; ++q) {
                    const int32_t f = first + q0 + q;
                    wv[q] = dv[q] = 0;
                    if (q0 + q < c1 && f < nf) {
                        const int32_t v = F[f];
                        if (vt) {
                            const WalkVertex h = vt[v];
                            dv[q] = h.d;
                            wv[q] = h.W;
                        } else {
                            dv[q] = (uint64_t)(p.g.rowptr[v + 1] - p.g.rowptr[v]);
                            if (p.bias != kUniform) wv[q] = wtot[v];
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < kLayerPer; ++q) {
                    const int32_t f = first + q0 + q;
                    if (p.bias == kUniform) wv[q] = dv[q];
                    sw += wv[q];
                    sd += dv[q];
                    lists += wv[q] != 0 ? 1u : 0u;
                    if (q0 + q < c1 && f < nf) {  // within the lane's run
                        Wp[f + 1] = sw;
                        Dp[f + 1] = sd;
                    }
                }
            }
            const uint64_t iw = wave_incl_scan_u64(sw), id = wave_incl_scan_u64(sd);
            const uint64_t W = readlane_u64(iw, kWave - 1);
            // positive positions: at least one in each list with a positive total, counted where that leaves it open
            uint64_t npos = p.bias == kUniform ? readlane_u64(id, kWave - 1) : wave_sum_u64(lists);
            if (p.bias != kUniform && npos <= (uint64_t)k) {
                uint64_t sp = 0;
                for (int32_t f = lane; f < nf; f += kWave) sp += (uint64_t)(ppos[F[f]] & ~kWideList);
                npos = wave_sum_u64(sp);
            }
            if (lane == 0) Wp[0] = Dp[0] = 0;
            for (int32_t q = 0; q < c1; ++q) {
                const int32_t f = first + q;
                if (f < nf) {
                    Wp[f + 1] += iw - sw;
                    Dp[f + 1] += id - sd;
                }
            }
            wave_lds_sync();
            const int32_t c = W == 0 ? 0 : ((uint64_t)k >= npos ? (int32_t)npos : k);
            int64_t pos = -1;  // this lane's pool position (slot lane < c)
            if (c > 0 && (uint64_t)k >= npos) {
                // every positive position, pool order
                int32_t run = 0;
                for (int32_t f = 0; f < nf; ++f) {
                    const int64_t beg = p.g.rowptr[F[f]];
                    const int64_t d = (int64_t)(Dp[f + 1] - Dp[f]);
                    for (int64_t b0 = 0; b0 < d; b0 += kWave) {
                        const int64_t e = b0 + lane;
                        const bool posv = e < d && (p.bias == kUniform || wts[beg + e] > 0);
                        const uint64_t m = ballot(posv);
                        const int32_t slot = run + __popcll(m & lanemask_lt());
                        if (posv) {
                            const int32_t nb = p.g.col[beg + e];
                            src[slot] = F[f];
                            dst[slot] = nb;
                            pk[slot] = nb;
                        }
                        run += __popcll(m);
                    }
                }
            } else if (c > 0) {
                const auto search = [&](uint64_t r, int64_t& m, uint64_t& Sm, uint32_t& bm) {
                    if (p.bias == kUniform) {
                        m = (int64_t)r;
                        Sm = r;
                        bm = 1;
                        return;
                    }
                    const int32_t f = lds_upper(Wp, nf, r);
                    const int32_t v = F[f];
                    const int64_t beg = vt ? (int64_t)vt[v].beg : p.g.rowptr[v];
                    const uint64_t S0 = Wp[f], d = Dp[f + 1] - Dp[f];
                    if (guide) {
                        int32_t nb;
                        const int32_t ml = slot_search(p.g, p.bias, v, beg, (int32_t)d, Wp[f + 1] - S0, r - S0, nb);
                        slot_bias(p.g, p.bias, beg, ml, Sm, bm);
                        Sm += S0;
                        m = (int64_t)Dp[f] + ml;
                    } else {
                        int64_t ml = 0;
                        list_search(wts + beg, gtab, ctab, beg, (int64_t)d, S0, r, ml, Sm, bm);
                        m = (int64_t)Dp[f] + ml;
                    }
                };
                pos = draw_slots(key, iid, (uint32_t)l, 0xFFFFFFFFu, c, p.rounds, W, search, search);
                if (lane < c) {
                    const int32_t f = lds_upper(Dp, nf, (uint64_t)pos);
                    const int32_t v = F[f];
                    const int32_t nb = p.g.col[p.g.rowptr[v] + (pos - (int64_t)Dp[f])];
                    src[lane] = v;
                    dst[lane] = nb;
                    pk[lane] = nb;
                }
            }
            for (int32_t j = c + lane; j < p.K; j += kWave) src[j] = dst[j] = -1;
            if (lane == 0) p.counts[i * p.L + l] = c;
            wave_lds_sync();
            if (l + 1 == p.L) break;
            // next frontier: the picks, deduplicated, minus visited, sorted
            const int32_t x = lane < c ? pk[lane] : -1;
            bool keep = lane < c;
            for (int32_t q = 0, b0 = 0; q <= l; ++q) {  // the frontiers so far, each sorted
                const int32_t e0 = readlane_i32(ends, q);
                int32_t lo = b0, hi = e0;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (vis[mid] < x) lo = mid + 1;
                    else hi = mid;
                }
                keep = keep && !(lo < e0 && vis[lo] == x);
                b0 = e0;
            }
            for (int j = 0; j < kWave; ++j) {
                const int32_t y = readlane_i32(x, j);
                if (j < lane && y == x) keep = false;
            }
            const uint64_t km = ballot(keep);
            int32_t rank = 0;
            for (int j = 0; j < kWave; ++j) {
                const int32_t y = readlane_i32(x, j);
                if (((km >> j) & 1ull) && y < x) ++rank;
            }
            F = vis + nvis;
            if (keep) F[rank] = x;
            nf = __popcll(km);
            nvis += nf;
            if (lane == l + 1) ends = nvis;
            wave_lds_sync();
        }
        wave_lds_sync();  // the next instance rewrites the lists
    }
}

__global__ void k_call_setup(uint32_t* __restrict__ ctl, int64_t nctl, const uint32_t* __restrict__ host_tab,
                             uint32_t* __restrict__ tab, int64_t ntab) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nctl; i += stride) ctl[i] = 0u;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ntab; i += stride) tab[i] = host_tab[i];
}

// End of a call: clear the visited bits of every frontier entry, and hand
// the control block to the host.
__global__ void k_clear_visited(ClearVisited c) {
    if (blockIdx.x == 0 && c.host_ctl != c.ctl) {
        constexpr int kWords = (int)(sizeof(SampleCtl) / 4);
        const uint32_t* from = (const uint32_t*)c.ctl;
        uint32_t* to = (uint32_t*)c.host_ctl;
        for (int i = threadIdx.x; i < kWords; i += blockDim.x) to[i] = from[i];
        __threadfence_system();
    }
    for (int l = 0; l < c.num_layers; ++l) {
        const int64_t fcount = frontier_size(c.ctl, l);
        const int32_t* __restrict__ fv = c.fv[l];
        const int32_t* __restrict__ fi = c.fi[l];
        for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < fcount;
             e += (int64_t)gridDim.x * blockDim.x)
            c.visited[(int64_t)fi[e] * c.nwp + (fv[e] >> 5)] = 0u;
    }
}

// Frontier entries and their edges per vertex-range partition of a layer
// (out-of-memory schedule): partition p holds vertices [bounds[p],
// bounds[p+1]); block-local sums in LDS, one atomic per partition and block.
constexpr int kMaxPartitions = 64;

__global__ void __launch_bounds__(kBlock) k_partition_work(const int32_t* __restrict__ fv,
                                                           const int32_t* __restrict__ cnt, const SampleCtl* ctl,
                                                           int32_t layer, const int64_t* __restrict__ bounds,
                                                           int32_t np, unsigned long long* __restrict__ work) {
    __shared__ unsigned long long s_work[2 * kMaxPartitions];
    for (int i = threadIdx.x; i < 2 * kMaxPartitions; i += blockDim.x) s_work[i] = 0ull;
    __syncthreads();
    const int64_t fcount = frontier_size(ctl, layer);
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < fcount;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = fv[e];
        int32_t lo = 0, hi = np;  // the partition: largest p with bounds[p] <= v
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (bounds[mid] <= v) lo = mid;
            else hi = mid;
        }
        atomicAdd(&s_work[2 * lo], 1ull);
        atomicAdd(&s_work[2 * lo + 1], (unsigned long long)cnt[e]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * np; i += blockDim.x)
        if (s_work[i]) atomicAdd(&work[i], s_work[i]);
}

}  // namespace

// ---------------------------------------------------------------- launchers}  // namespace

// ---------------------------------------------------------------- launchers
size_t free_device_bytes() {
    size_t free_b = 0, total = 0;
    return hipMemGetInfo(&free_b, &total) == hipSuccess ? free_b : 0;
}

void launch_partition_work(const int32_t* fv, const int32_t* cnt, const SampleCtl* ctl, int32_t layer,
                           int64_t capacity, const int64_t* bounds, int32_t np, unsigned long long* work,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_partition_work, dim3(grid_for(capacity, kBlock, 1024)), dim3(kBlock), 0, s, fv, cnt, ctl,
                       layer, bounds, np, work);
}

void launch_scatter_segments(const int32_t* src, const int32_t* dst, const int64_t* off, int64_t nseg,
                             int64_t total, int32_t* const* to_src, int32_t* const* to_dst, hipStream_t s) {
    if (nseg <= 0 || total <= 0) return;
    hipLaunchKernelGGL(k_scatter_segments, dim3(grid_for(total, kBlock, 8192)), dim3(kBlock), 0, s, src, dst, off,
                       nseg, to_src, to_dst);
}

void launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t s) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(count, kBlock, 65536)), dim3(kBlock), 0, s, p, value, count);
}

void launch_degree_weights(RowPtr rowptr, const int32_t* col, int64_t m, uint32_t* degw,
                           hipStream_t s) {
    if (m <= 0) return;
    hipLaunchKernelGGL(k_degree_weights, dim3(grid_for(m, kBlock, 65536)), dim3(kBlock), 0, s, rowptr, col,
                       m, degw);
}

void launch_positive_counts(RowPtr rowptr, const uint32_t* w, int64_t n, int32_t* ppos, uint64_t* wtot,
                            hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_positive_counts, dim3(grid_for(n, kWavesPerBlock, 65536)), dim3(kBlock), 0, s,
                       rowptr, w, n, ppos, wtot);
}

void launch_mark_seeds(const int32_t* seeds, int64_t num_seeds, const int64_t* seed_offsets, int32_t ni,
                       int64_t n, uint32_t* next, int64_t nwp, uint32_t* summ, int64_t nsw, SampleCtl* ctl,
                       hipStream_t s) {
    if (num_seeds <= 0) return;
    hipLaunchKernelGGL(k_mark_seeds, dim3(grid_for(num_seeds, kBlock, 65536)), dim3(kBlock), 0, s, seeds,
                       num_seeds, seed_offsets, ni, n, next, nwp, summ, nsw, ctl);
}

// Bitmap words per thread of a dense build.
static int dense_words(int64_t words) { return words > kSparseWords ? kWidePer : 1; }

int64_t frontier_build_blocks(int64_t words) {
    const int64_t per = (int64_t)kBlock * dense_words(words);
    const int64_t nb = (words + per - 1) / per;
    return nb > 0 ? nb : 1;
}

void launch_frontier_build(const FrontierBuild& fb, hipStream_t s, LaunchEvents ev) {
    const dim3 grid((unsigned)fb.nb), block(kBlock);
    if (fb.summ) {  // sparse: compact the summary, then one thread per dirty word
        hipLaunchKernelGGL(k_dirty_compact, dim3((unsigned)fb.nb_dirty), block, 0, s, fb);
        launch_kernel(fb.burn ? k_frontier_build<true, true, 1> : k_frontier_build<false, true, 1>, grid, block, s, ev, fb);
    } else if (dense_words(fb.nwords) == 1) {
        launch_kernel(fb.burn ? k_frontier_build<true, false, 1> : k_frontier_build<false, false, 1>, grid, block, s, ev, fb);
    } else {
        launch_kernel(fb.burn ? k_frontier_build<true, false, kWidePer> : k_frontier_build<false, false, kWidePer>, grid,
                      block, s, ev, fb);
    }
}

int64_t sparse_build_blocks(int64_t capacity) {
    const int64_t nb = (capacity + kBlock - 1) / kBlock;
    return nb > 0 ? nb : 1;
}

int64_t dirty_compact_blocks(int64_t summary_words) {
    const int64_t per = (int64_t)kBlock * 4;
    const int64_t nb = (summary_words + per - 1) / per;
    return nb > 0 ? nb : 1;
}

void launch_select(const SampleLayer& p, int grid, hipStream_t s, LaunchEvents ev) {
    launch_kernel(p.wave_only ? k_select_wave<true> : p.weighted ? k_select_slots<true> : k_select_slots<false>, dim3(grid),
                  dim3(kBlock), s, ev, p);
}

void launch_layer_sample(const LayerParams& p, hipStream_t s, LaunchEvents ev) {
    if (p.num_instances <= 0) return;
    const int grid = (int)(p.num_instances < 8192 ? p.num_instances : 8192);
    const size_t lds = layer_lds_bytes(p.max_f, p.L);
    if (ev.start || ev.stop)
        hipExtLaunchKernelGGL(k_layer_sample, dim3(grid), dim3(kWave), lds, s, ev.start, ev.stop, 0, p);
    else
        hipLaunchKernelGGL(k_layer_sample, dim3(grid), dim3(kWave), lds, s, p);
}

int64_t chunk_table_rows(int64_t m) { return (m >> kTabShift) + 1; }

void launch_chunk_table(RowPtr rowptr, const uint32_t* w, int64_t n, uint64_t* tab, uint64_t* ctab,
                        hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_chunk_table, dim3(grid_for(n, kWavesPerBlock, 65536)), dim3(kBlock), 0, s, rowptr, w, n,
                       tab, ctab);
}

void launch_select_big(const SampleLayer& p, int grid, hipStream_t s, LaunchEvents ev) {
    if (!p.wave_only) hipLaunchKernelGGL(k_select_wave<false>, dim3(grid), dim3(kBlock), 0, s, p);
    launch_kernel(k_select_big, dim3(grid), dim3(kBlock), s, ev, p);
}

void launch_clear_visited(const ClearVisited& c, hipStream_t s, LaunchEvents ev) {
    launch_kernel(k_clear_visited, dim3(grid_for(c.cap_entries, kBlock, 16384)), dim3(kBlock), s, ev, c);
}

void launch_call_setup(uint32_t* ctl, int64_t nctl, const uint32_t* host_tab, uint32_t* tab, int64_t ntab,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_call_setup, dim3(grid_for(nctl > ntab ? nctl : ntab, kBlock, 1024)), dim3(kBlock), 0, s,
                       ctl, nctl, host_tab, tab, ntab);
}

}  // namespace csaw
