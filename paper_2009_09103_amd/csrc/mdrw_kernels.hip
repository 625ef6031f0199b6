// mdrw_kernels.hip -- gfx950 kernel of the multi-dimensional random walk
// (frontier sampling, Section II-A; the VertexBias select site of
// fig:api(b)).
//
// One wavefront per instance; its frontier pool lives in LDS (vertex, first
// edge and degree per slot). Lane L owns the slots [L*c, L*c + c),
// c = ceil(P / 64): the owning lane of a draw is the number of lanes whose
// inclusive degree total is <= r, the slot inside it the
// number of its slots whose running total is <= the remainder. A step changes
// one slot, so the lanes' inclusive totals are kept and those from the owning
// lane on shifted. Edges are kept one per lane and written 64 steps at a time.
// The steps of an instance are a chain, so the time is the chain's latency
// times the rounds of instances that fit the chip:
//   - one load a step where the graph has its hop table (the picked edge's
//     neighbor and its list in one record; else the id, then its row offsets);
//   - the owning lane's slots are read, and a neighbor draw formed for each
//     of them, beside the scan that decides which is picked; the next
//     step's pool draw is formed while the edge loads;
//   - 10 bytes of LDS a slot where list offsets fit 32 bits (degrees of
//     65,535 and more, a handful of hubs, are looked up again), sized by the
//     call's largest pool: 8 instances of 2,000 vertices per CU, so that 2,000
//     instances are one round, where 16 bytes and room for 2,048 made two.
// 2,000 pools of 2,000 on R-MAT 22, 1,703 steps each: 4.67 ms before, 1.99 now
// (1.17 us a step; 2.28 with a scan of the lanes' totals in every step, 2.11
// with the neighbor draw formed after the pick).
#include "device_common.h"
#include "kernels.h"

namespace csaw {

namespace {

constexpr uint32_t kBigDeg = 0xFFFFu;  // a degree that does not fit 16 bits

// kWide: 64-bit list offsets (m >= 2^32) and 32-bit degrees in the pool.
template <bool kWide>
struct PoolTypes {
    typedef uint32_t Beg;
    typedef uint16_t Deg;
};
template <>
struct PoolTypes<true> {
    typedef int64_t Beg;
    typedef uint32_t Deg;
};

template <bool kWide>
inline size_t mdrw_lds_bytes(int32_t pool) {
    typedef PoolTypes<kWide> T;
    return ((size_t)pool * (sizeof(typename T::Beg) + sizeof(int32_t) + sizeof(typename T::Deg)) + 15) / 16 * 16;
}

// floor(u * W / 2^64) of a 32-bit W
__device__ __forceinline__ uint32_t range_reduce(uint64_t u, uint32_t W) {
    const uint64_t lo = (uint64_t)(uint32_t)u * W, hi = (u >> 32) * (uint64_t)W;
    return (uint32_t)((hi + (lo >> 32)) >> 32);
}
using csaw::range_reduce;

// Sum: type of the pool's degree totals, 32 bits where the largest pool times
// the largest degree fit.
template <bool kWide, bool kHops, typename Sum>
__global__ void __launch_bounds__(kWave) k_mdrw(MdrwParams p) {
    typedef typename PoolTypes<kWide>::Beg Beg;
    typedef typename PoolTypes<kWide>::Deg Deg;
    extern __shared__ __align__(16) unsigned char mdrw_lds[];
    Beg* pb = (Beg*)mdrw_lds;
    int32_t* pv = (int32_t*)(pb + p.max_pool);
    Deg* pd = (Deg*)(pv + p.max_pool);
    const int lane = lane_id();
    const Key key{p.k0, p.k1};
    const auto short_deg = [](uint32_t d) { return kWide || d < kBigDeg ? (Deg)d : (Deg)kBigDeg; };
    // a slot's degree, looked up again where its 16 bits do not hold it
    const auto degree = [&p](Deg x, int32_t v) -> uint32_t {
        if (kWide || (uint32_t)x != kBigDeg) return x;
        return (uint32_t)(p.g.rowptr[v + 1] - p.g.rowptr[v]);
    };
    for (int64_t i = blockIdx.x; i < p.num_instances; i += gridDim.x) {
        const int64_t o0 = uniform_i64(p.pool_off[i]);
        const int64_t P = uniform_i64(p.pool_off[i + 1]) - o0;  // <= max_pool (the host's maximum)
        const uint32_t iid = (uint32_t)(p.instance_base + (uint64_t)i);
        int32_t* src = p.src + i * p.budget;
        int32_t* dst = p.dst + i * p.budget;
        bool bad = false;
        for (int64_t j = lane; j < P; j += kWave) {
            int32_t v = p.pool[o0 + j];
            if (v < 0 || (int64_t)v >= p.g.n) {
                bad = true;
                v = 0;
            }
            const int64_t b = p.g.rowptr[v];
            pv[j] = v;
            pd[j] = short_deg((uint32_t)(p.g.rowptr[v + 1] - b));
            pb[j] = (Beg)b;
        }
        if (ballot(bad)) {  // outputs of the call are unspecified; the host reports the error
            if (lane == 0) *p.bad = 1;
            wave_lds_sync();
            continue;
        }
        wave_lds_sync();
        const int c = (int)((P + kWave - 1) / kWave);
        Sum incl = 0;  // degree total of the lanes up to this one
        for (int q = 0; q < c; ++q) {
            const int64_t j = (int64_t)lane * c + q;
            if (j < P) incl += degree(pd[j], pv[j]);
        }
        incl = wave_incl_scan_t(incl);
        int64_t s = 0;
        int32_t bv = -1, bu = -1;  // edge of step s is kept by lane s % 64
        uint64_t pool_draw = philox_u64(key.k0, key.k1, iid, 0u, 0xFFFFFFFFu, 0u);
        for (; s < p.budget; ++s) {
            const Sum W = readlane_t(incl, kWave - 1);
            if (W == 0) break;
            const Sum r = range_reduce(pool_draw, W);
            const int L = __popcll(ballot(incl <= r));  // owning lane of r
            const Sum rr = r - (L ? readlane_t(incl, L - 1) : (Sum)0);
            const int64_t jq = (int64_t)L * c + lane;
            const bool in = lane < c && jq < P;
            const int32_t vq = in ? pv[jq] : 0;
            const Deg xq = in ? pd[jq] : (Deg)0;
            const Beg bq = in ? pb[jq] : (Beg)0;
            const uint32_t dq = degree(xq, vq);
            const uint32_t nq = range_reduce(philox_u64(key.k0, key.k1, iid, (uint32_t)s, (uint32_t)vq, 1u), dq);
            const Sum iq = wave_incl_scan_t((Sum)dq);
            const int t = __popcll(ballot(lane < c && iq <= rr));  // its slot in that lane
            const int64_t j = (int64_t)L * c + t;
            const int32_t v = readlane_i32(vq, t);
            const uint32_t d = readlane_u32(dq, t);
            const int64_t e = (kWide ? readlane_i64((int64_t)bq, t) : (int64_t)readlane_u32((uint32_t)bq, t)) +
                              (int64_t)readlane_u32(nq, t);
            int32_t u;
            int64_t ub;
            uint32_t ud;
            if (kHops) {
                const uint4 h = *(const uint4*)(p.g.hops + e);
                pool_draw = philox_u64(key.k0, key.k1, iid, (uint32_t)s + 1u, 0xFFFFFFFFu, 0u);
                __builtin_amdgcn_sched_barrier(0);  // formed while the record loads
                u = uniform_i32((int32_t)h.x);
                ub = (int64_t)(uint32_t)uniform_i32((int32_t)h.y);
                ud = (uint32_t)uniform_i32((int32_t)h.z);
            } else {
                u = ld_uniform(p.g.col + e);
                int64_t udl;
                row_uniform(p.g.rowptr, u, ub, udl);
                ud = (uint32_t)udl;
                pool_draw = philox_u64(key.k0, key.k1, iid, (uint32_t)s + 1u, 0xFFFFFFFFu, 0u);
            }
            wave_lds_sync();
            if (lane == 0) {
                pv[j] = u;
                pd[j] = short_deg(ud);
                pb[j] = (Beg)ub;
            }
            if (lane >= L) incl += (Sum)ud - (Sum)d;
            wave_lds_sync();
            if (lane == (int)(s & (kWave - 1))) {
                bv = v;
                bu = u;
            }
            if ((s & (kWave - 1)) == kWave - 1) {
                src[s - (kWave - 1) + lane] = bv;
                dst[s - (kWave - 1) + lane] = bu;
            }
        }
        const int64_t s0 = s & ~(int64_t)(kWave - 1);
        if (lane < s - s0) {
            src[s0 + lane] = bv;
            dst[s0 + lane] = bu;
        }
        for (int64_t q = s + lane; q < p.budget; q += kWave) {
            src[q] = -1;
            dst[q] = -1;
        }
        if (lane == 0) {
            if (p.steps) p.steps[i] = s;
            if (s) atomicAdd(p.total, (unsigned long long)s);
        }
        wave_lds_sync();  // the next instance rewrites the pool
    }
}

}  // namespace

void launch_mdrw(const MdrwParams& p, hipStream_t s, LaunchEvents ev) {
    if (p.num_instances <= 0) return;
    const dim3 grid(p.num_instances < 8192 ? p.num_instances : 8192), block(kWave);
    const bool wide = p.g.rowptr.p64 != nullptr;
    const size_t lds = wide ? mdrw_lds_bytes<true>(p.max_pool) : mdrw_lds_bytes<false>(p.max_pool);
    const bool narrow = (uint64_t)p.max_pool * p.max_degree < (uint64_t(1) << 32);
    void (*const kernel)(MdrwParams) =
        wide ? k_mdrw<true, false, uint64_t>
             : (narrow ? (p.g.hops ? k_mdrw<false, true, uint32_t> : k_mdrw<false, false, uint32_t>)
                       : (p.g.hops ? k_mdrw<false, true, uint64_t> : k_mdrw<false, false, uint64_t>));
    if (ev.start || ev.stop) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, ev.start, ev.stop, 0, p);
    else hipLaunchKernelGGL(kernel, grid, block, lds, s, p);
}

}  // namespace csaw
