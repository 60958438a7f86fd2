// Plan execution and baseline placements on the device (App. C.2 metrics,
// App. B comparison schedulers), in fp64 like the host executor.
//
// One 64-lane wave per instance; lane d stands for device d and keeps that
// device's state in registers (free time, resident models, the model it ran
// last) and its prefix slots in LDS, so a stage's shards on the devices of
// S(v) are computed side by side, and the HEFT-style scheduler tries every
// feasible device at once.  A stage's parents are loaded one per lane and
// handed to the device lanes with readlane.  Stages run in (order key, id)
// order; the order is found by counting, for each stage, the stages that
// precede it (the keys staged through LDS).
//
// Execution rule (the same as the host executor): a shard of v on d (k =
// |S(v)|) starts when d is free and every parent's output has arrived (1/k of
// a remote parent's output from its cheapest holder); it pays the switch
// time if m(v) is absent (then Load with eviction), and runs c(v, d) / k, less
// kappa_prefix * L(v) / k (not below 0) when grp(v) is in d's prefix slots;
// grp(v) then joins the slots.  v finishes with its last shard and is then
// held by S(v).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fate_device.h"
#include "fate_internal.h"

// The host executor rounds every product and quotient before it adds; so does this code.
#pragma clang fp contract(off)

namespace fate {
namespace {

constexpr int kRing = FATE_MAX_DEVICES * FATE_MAX_PREFIX_SLOTS;  // prefix slots of one instance
constexpr int kChunk = 512;  // keys per LDS chunk of the ordering count
constexpr int kPer = 4;      // stages ranked per lane and pass

__device__ __forceinline__ uint64_t rl64(uint64_t x, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double rld(double x, int l) { return __longlong_as_double((long long)rl64((uint64_t)__double_as_longlong(x), l)); }

// Order-preserving image of a double (no NaN): a larger value, a larger key.
__device__ __forceinline__ uint64_t dkey(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x + 0.0);
    return (u >> 63) ? ~u : (u | (1ull << 63));
}
__device__ __forceinline__ double dkey_inv(uint64_t k) {
    const uint64_t u = (k >> 63) ? (k & ~(1ull << 63)) : ~k;
    return __longlong_as_double((long long)u);
}

// Maximum / minimum of a 64-bit key over the wave (every lane active).
__device__ __forceinline__ uint64_t wave_max64(uint64_t x) {
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t y = ((uint64_t)(uint32_t)__shfl_xor((int)(x >> 32), off) << 32) | (uint32_t)__shfl_xor((int)(uint32_t)x, off);
        x = y > x ? y : x;
    }
    return x;
}
__device__ __forceinline__ uint64_t wave_min64(uint64_t x) { return ~wave_max64(~x); }

// Make this wave's global and LDS writes visible to its own later reads.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Per-instance context of the walk.
struct Inst {
    int64_t base, n;
    double t0;
    int lane, D, K;
    bool live;
    // lane d: device d
    double fr;       // free time
    uint64_t res;    // resident models
    int lastm;       // model of the stage it ran last, -1 before the first
};

// Position of each of the cnt stages ids[0..cnt) in (key ascending, index
// ascending) order: out[position] = ids[i].
__device__ void order_by_count(const uint64_t *keys, const uint32_t *ids, int64_t cnt, uint32_t *out,
                               uint64_t *chunk, int lane) {
    for (int64_t i0 = 0; i0 < cnt; i0 += 64 * kPer) {  // uniform
        uint64_t ki[kPer];
        int64_t ii[kPer];
        uint32_t r[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            ii[p] = i0 + p * 64 + lane;
            ki[p] = ii[p] < cnt ? keys[ii[p]] : ~0ull;
            r[p] = 0u;
        }
        for (int64_t j0 = 0; j0 < cnt; j0 += kChunk) {  // uniform
            const int jn = (int)min((int64_t)kChunk, cnt - j0);
            wave_fence();
            for (int t = lane; t < jn; t += 64) chunk[t] = keys[j0 + t];
            wave_fence();
            for (int t = 0; t < jn; ++t) {
                const uint64_t kj = chunk[t];
                const int64_t j = j0 + t;
#pragma unroll
                for (int p = 0; p < kPer; ++p) r[p] += (kj < ki[p] || (kj == ki[p] && j < ii[p])) ? 1u : 0u;
            }
        }
#pragma unroll
        for (int p = 0; p < kPer; ++p)
            if (ii[p] < cnt) out[r[p]] = ids[ii[p]];
    }
    wave_fence();
}

// Finish time of v's shard on this lane's device (k shards) with the parent
// data one per lane in (ph, pf, ps) for parents q0 .. q0+nq-1, folded into
// `ready`; the caller loops over chunks of 64 parents.
__device__ __forceinline__ double arrivals(const SimLaunch &a, const Inst &x, int d, int k, uint64_t ph, double pf,
                                           float ps, int nq, double ready) {
    for (int q = 0; q < nq; ++q) {  // uniform
        const uint64_t h = rl64(ph, q);
        const double f = rld(pf, q);
        const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ps), q));
        double arr;
        if ((h >> d) & 1ull) {
            arr = f;
        } else {
            double bmin = __builtin_huge_val();
            for (uint64_t t = h; t; t &= t - 1) bmin = fmin(bmin, (double)a.beta[__builtin_ctzll(t) * x.D + d]);
            arr = f + ((double)s * bmin) / (double)k;
        }
        ready = fmax(ready, arr);
    }
    return ready;
}

// Shard of stage g (flat) on this lane's device d after the parents' latest
// arrival `ready`: finish time, and whether grp(g) is cached on d.
__device__ __forceinline__ double shard_finish(const SimLaunch &a, const Inst &x, const uint64_t *ring, const StageRec &r,
                                               int d, int k, double ready, bool &hit) {
    const double start = fmax(x.fr, ready);
    const int m = r.model;
    const double sw = ((x.res >> m) & 1ull) ? 0.0 : (double)a.ksw[m * x.D + d];
    hit = false;
    if (r.hash != 0)
        for (int e = 0; e < x.K; ++e) hit = hit || ring[d * x.K + e] == r.hash;
    double run = (double)a.exec[m * x.D + d] / (double)k;
    if (hit) run = fmax(0.0, run - ((a.kpf * (double)r.tokens) / (double)k));
    return (start + sw) + run;
}

// The parents' latest arrival on this lane's device for stage g with k
// shards; also whether every parent has finished (held somewhere) and how
// many parent edges reach no device of S (S = 0: not counted).
__device__ __forceinline__ double parent_ready(const SimLaunch &a, const Inst &x, const StageRec &r, int d, int k,
                                               uint64_t S, bool &all_done, int64_t &xdev) {
    double ready = x.t0;
    all_done = true;
    for (int q0 = 0; q0 < (int)r.npar; q0 += 64) {  // uniform
        const int nq = min(64, (int)r.npar - q0);
        uint64_t ph = 1ull;
        double pf = 0.0;
        float ps = 0.0f;
        if (x.lane < nq) {
            const uint32_t u = a.par_idx[r.par_begin + q0 + x.lane];
            ph = a.hold[u];
            pf = a.fin[u];
            ps = a.rec[u].sigma;
        }
        all_done = all_done && __ballot(ph == 0ull) == 0ull;
        xdev += __popcll(__ballot(x.lane < nq && (ph & S) == 0ull));
        ready = arrivals(a, x, d, k, ph, pf, ps, nq, ready);
    }
    return ready;
}

// Run stage g on the devices of S (lanes of S apply the shard's effects);
// returns its finish, and whether the first device of S hit the prefix
// cache and continued the same model.
__device__ __forceinline__ double run_stage(const SimLaunch &a, Inst &x, uint64_t *ring, const StageRec &r, int64_t g,
                                            uint64_t S, double ready, bool &hit0, bool &cont0) {
    const int k = __popcll(S);
    const int d = x.lane;
    const bool mine = x.live && ((S >> d) & 1ull);
    bool hit = false;
    double fd = x.t0;
    if (mine) fd = shard_finish(a, x, ring, r, d, k, ready, hit);
    const int d0 = __builtin_ctzll(S);
    hit0 = __builtin_amdgcn_readlane(hit ? 1 : 0, d0) != 0;
    cont0 = __builtin_amdgcn_readlane(x.lastm, d0) == (int)r.model;
    if (mine) {
        x.fr = fd;
        x.res = load_model(x.res, r.model, a.cap[d], a.weight);
        // grp(v) joins the slots: the first empty one, else drop the oldest and append
        if (r.hash != 0 && x.K > 0) {
            uint64_t *row = ring + d * x.K;
            bool have = false;
            int empty = -1;
            for (int e = 0; e < x.K; ++e) {
                have = have || row[e] == r.hash;
                if (empty < 0 && row[e] == 0ull) empty = e;
            }
            if (!have) {
                if (empty >= 0) {
                    row[empty] = r.hash;
                } else {
                    for (int e = 0; e + 1 < x.K; ++e) row[e] = row[e + 1];
                    row[x.K - 1] = r.hash;
                }
            }
        }
        x.lastm = r.model;
    }
    const double f = dkey_inv(wave_max64(mine ? dkey(fd) : dkey(x.t0)));  // max(t0, shard finishes)
    if (d == 0) {
        a.fin[g] = f;
        a.hold[g] = S;
    }
    wave_fence();
    return f;
}

template <int MODE>  // 0: execute a plan; 1: round-robin placement; 2: HEFT-style placement
__global__ __launch_bounds__(64) void k_sim(SimLaunch a) {
    __shared__ uint64_t ring[kRing];
    __shared__ uint64_t chunk[kChunk];
    const int b = blockIdx.x;
    Inst x;
    x.lane = threadIdx.x;
    x.D = a.D;
    x.K = a.K;
    x.base = a.stage_off[b];
    x.n = a.stage_off[b + 1] - x.base;
    x.t0 = (double)a.tnow[b];
    x.live = x.lane < x.D;
    const int D = x.D, K = x.K, lane = x.lane;
    const uint64_t dm = D >= 64 ? ~0ull : ((1ull << D) - 1ull);
    x.fr = x.live ? fmax((double)a.tau[(int64_t)b * D + lane], x.t0) : 0.0;
    x.res = x.live ? a.resident[(int64_t)b * D + lane] : 0ull;
    x.lastm = -1;
    for (int e = lane; e < D * K; e += 64) ring[e] = a.pcache[(int64_t)b * D * K + e];
    const int64_t base = x.base, n = x.n;

    // working copies of finish times and holders; children marks
    bool bad = false;
    for (int64_t v = lane; v < n; v += 64) {
        const int64_t g = base + v;
        const uint64_t h = a.holders[g];
        a.hold[g] = h;
        a.fin[g] = h != 0 ? x.t0 : 0.0;
        a.flags[g] = 0;
        if (MODE == 0 && (a.devices[g] & ~dm) != 0) bad = true;
        if (MODE != 0 && h != 0) {  // completed stages are not placed
            a.dev_out[g] = 0ull;
            a.ord_out[g] = 0;
        }
    }
    if (__ballot(bad) != 0ull) {
        if (lane == 0) {
            a.status[b] = FATE_EINVAL;
            a.out[b] = fate_sim_metrics_t{};
        }
        return;
    }
    wave_fence();
    for (int64_t v = lane; v < n; v += 64) {  // a stage with a child is no sink
        const StageRec r = a.rec[base + v];
        for (uint32_t q = 0; q < r.npar; ++q) a.flags[a.par_idx[r.par_begin + q]] = 1;
    }
    wave_fence();

    if (MODE == 1) {  // round robin: each pending stage, in id order, on the next feasible device
        int nxt = 0;
        for (int64_t v = 0; v < n; ++v) {  // uniform
            const int64_t g = base + v;
            uint64_t dev = 0;
            if (a.hold[g] == 0ull) {
                const StageRec r = a.rec[g];
                const uint64_t fm = r.elig & a.fits[r.model] & dm;
                const uint64_t hi = nxt < 64 ? fm & (~0ull << nxt) : 0ull;
                const int d = hi ? __builtin_ctzll(hi) : __builtin_ctzll(fm);
                dev = 1ull << d;
                nxt = d + 1;
            }
            if (lane == 0) {
                a.dev_out[g] = dev;
                a.ord_out[g] = dev ? v : 0;
            }
        }
        if (lane == 0) a.status[b] = FATE_OK;
        return;
    }

    // the stages to run and their order keys
    int64_t cnt = 0;
    if (MODE == 2) {  // HEFT-style: upward ranks, children first (a child has a larger id)
        double bmean = 0.0;  // mean off-diagonal transfer coefficient, summed in row order
        for (int i = 0; i < D; ++i)
            for (int j = 0; j < D; ++j)
                if (i != j) bmean += (double)a.beta[i * D + j];
        bmean = D > 1 ? bmean / (double)(D * (D - 1)) : 0.0;
        double rank_v = 0.0;
        for (int64_t v = n - 1; v >= 0; --v) {  // uniform
            const int64_t g = base + v;
            const StageRec r = a.rec[g];
            double wsum = 0.0;
            int nf = 0;
            const uint64_t fm = r.elig & a.fits[r.model] & dm;
            for (int d = 0; d < D; ++d)
                if ((fm >> d) & 1ull) {
                    wsum += (double)a.exec[r.model * D + d];
                    ++nf;
                }
            const double tail = (a.flags[g] & 2) ? a.tail[g] : 0.0;
            rank_v = wsum / (double)nf + tail;
            // each parent's tail: the largest sigma(u) * mean beta + rank over its children
            for (uint32_t q0 = 0; q0 < r.npar; q0 += 64) {
                const uint32_t q = q0 + lane;
                if (q < r.npar) {
                    const uint32_t u = a.par_idx[r.par_begin + q];
                    const double t = ((double)a.rec[u].sigma * bmean) + rank_v;
                    const uint8_t fl = a.flags[u];
                    a.tail[u] = (fl & 2) ? fmax(a.tail[u], t) : t;
                    a.flags[u] = fl | 2;
                }
            }
            if (lane == 0) a.aux[g] = rank_v;
            wave_fence();
        }
        // pending stages by rank descending, then id
        for (int64_t v0 = 0; v0 < n; v0 += 64) {
            const int64_t v = v0 + lane;
            const bool take = v < n && a.hold[base + v] == 0ull;
            const uint64_t bal = __ballot(take);
            if (take) {
                const int64_t o = cnt + __popcll(bal & ((1ull << lane) - 1ull));
                a.keys[base + o] = ~dkey(a.aux[base + v]);
                a.ids[base + o] = (uint32_t)v;
            }
            cnt += __popcll(bal);
        }
    } else {  // placed pending stages by (order key, id)
        for (int64_t v0 = 0; v0 < n; v0 += 64) {
            const int64_t v = v0 + lane;
            const bool take = v < n && a.hold[base + v] == 0ull && a.devices[base + v] != 0ull;
            const uint64_t bal = __ballot(take);
            if (take) {
                const int64_t o = cnt + __popcll(bal & ((1ull << lane) - 1ull));
                a.keys[base + o] = (uint64_t)a.order[base + v] ^ (1ull << 63);
                a.ids[base + o] = (uint32_t)v;
            }
            cnt += __popcll(bal);
        }
    }
    wave_fence();
    order_by_count(a.keys + base, a.ids + base, cnt, a.todo + base, chunk, lane);

    // the walk
    fate_sim_metrics_t m{};
    int32_t st = FATE_OK;
    for (int64_t p = 0; p < cnt; ++p) {  // uniform
        const int64_t g = base + a.todo[base + p];
        const StageRec r = a.rec[g];
        uint64_t S;
        bool all_done;
        int64_t xdev = 0;
        double ready;
        if (MODE == 2) {  // every feasible device at once; the earliest finish, ties to the lower device
            const int d = lane;
            const bool feas = x.live && ((r.elig & a.fits[r.model]) >> d) & 1ull;
            ready = parent_ready(a, x, r, x.live ? d : 0, 1, ~0ull, all_done, xdev);
            bool hit;
            const double fd = feas ? shard_finish(a, x, ring, r, d, 1, ready, hit) : 0.0;
            const uint64_t best = wave_min64(feas ? dkey(fd) : ~0ull);
            const int bd = (int)wave_min64(feas && dkey(fd) == best ? (uint64_t)d : ~0ull);
            S = 1ull << bd;
            if (lane == 0) {
                a.dev_out[g] = S;
                a.ord_out[g] = p;
            }
        } else {
            S = a.devices[g];
            ready = parent_ready(a, x, r, x.live ? lane : 0, __popcll(S), S, all_done, xdev);
        }
        if (!all_done) {  // the order runs a stage before one of its parents
            st = FATE_ESTATE;
            break;
        }
        bool hit0, cont0;
        run_stage(a, x, ring, r, g, S, ready, hit0, cont0);
        m.tasks += 1;
        m.xdev_edges += xdev;
        m.cache_hits += hit0 ? 1 : 0;
        m.model_cont += cont0 ? 1 : 0;
    }
    if (st != FATE_OK) {
        if (lane == 0) {
            a.status[b] = st;
            a.out[b] = fate_sim_metrics_t{};
        }
        return;
    }
    if (MODE == 2) {
        if (lane == 0) a.status[b] = FATE_OK;
        return;
    }

    // makespan and the p95 of the sinks' completion times
    uint64_t lastk = dkey(x.t0);
    int64_t ns = 0;
    for (int64_t p0 = 0; p0 < cnt; p0 += 64) {
        const int64_t p = p0 + lane;
        bool sink = false;
        double f = x.t0;
        if (p < cnt) {
            const int64_t g = base + a.todo[base + p];
            f = a.fin[g];
            sink = (a.flags[g] & 1) == 0;
        }
        const uint64_t fk = dkey(f);
        lastk = fk > lastk ? fk : lastk;
        const uint64_t bal = __ballot(sink);
        if (sink) a.aux[base + ns + __popcll(bal & ((1ull << lane) - 1ull))] = f - x.t0;
        ns += __popcll(bal);
    }
    m.makespan = dkey_inv(wave_max64(lastk)) - x.t0;
    wave_fence();
    if (ns > 0) {  // nearest rank: the element at 0-based position ceil(0.95 ns) - 1 in ascending order
        const int64_t rk = max((int64_t)0, (int64_t)ceil(0.95 * (double)ns) - 1);
        uint64_t pick = 0ull;
        for (int64_t i0 = 0; i0 < ns; i0 += 64) {
            const int64_t i = i0 + lane;
            const double xi = i < ns ? a.aux[base + i] : 0.0;
            int64_t lt = 0, le = 0;
            for (int64_t j = 0; j < ns; ++j) {
                const double xj = a.aux[base + j];
                lt += xj < xi ? 1 : 0;
                le += xj <= xi ? 1 : 0;
            }
            if (i < ns && lt <= rk && rk < le) pick = dkey(xi);
        }
        m.p95 = dkey_inv(wave_max64(pick));
    }
    if (lane == 0) {
        a.out[b] = m;
        a.status[b] = FATE_OK;
    }
}

// ---- k_sim_lds: execution and HEFT-style placement with the instance in LDS
//
// The walk is one serial chain per instance (a stage needs its parents'
// finish times and the free time its device's last stage left), so its time
// is the latency of one link times the stages.  k_sim's link goes through
// global memory some six times; here the stages' finish times and holders,
// the order, the cluster tables and the prefix slots stay in LDS, everything
// that does not depend on the walk (records, parent lists, run times, the
// devices caching a stage's group) is prepared for 64 stages at a time, one
// per lane, and reductions over the lanes are DPP moves.
//
//   ranks   64 stages at a time, last ids first: every lane computes its
//           stage's rank from the largest rank its children have pushed, and
//           pushes its own to its parents (LDS maximum); lanes whose value
//           grew go round again until none does, as often as the 64 stages
//           are deep.  sigma * mean beta is the same for all children and
//           adding it is monotone, so the maximum commutes with the addition
//           and the rank is the sequential one to the bit.
//   order   bitonic sort of (key, id) in LDS.
//   walk    HEFT: lane d tries device d, each parent's finish and holders
//           read by all lanes at once; execution: lane q holds parent q.
//           Lane i keeps the mask of devices caching the group of the batch's
//           stage i; a placement that changes a device's slots updates all
//           64 masks with two comparisons.
struct SimPlan {
    uint32_t rank, key, idx, ring, par, tab, fits, wts, beta, total;
};
constexpr int kParBuf = 256;  // prefetched parents of 64 stages

struct alignas(16) FinHold {
    double fin;     // finish time (t for a stage completed at the start)
    uint64_t hold;  // devices holding the output, 0 = not finished
};
struct alignas(16) ParL {  // a prefetched parent
    uint32_t u;    // stage
    float sigma;   // its output size
    double tr;     // sigma * beta0 (uniform beta)
};

__host__ __device__ inline SimPlan sim_plan(int64_t max_stages, int D, int K, int M, bool uni) {
    SimPlan q;
    uint32_t n = (uint32_t)max_stages, np2 = 64;
    while (np2 < n) np2 <<= 1;
    uint32_t o = 0;
    q.rank = o; o += 8 * n;   // ranks; the walk's FinHold[n] takes the place
    q.key = o; o += 8 * np2;  // of ranks and keys
    o = (o + 15u) & ~15u;
    q.idx = o; o += 4 * np2;  // stages in order
    q.ring = o; o += 8 * (uint32_t)(D * K);
    o = (o + 15u) & ~15u;
    q.par = o; o += (uint32_t)sizeof(ParL) * (uint32_t)kParBuf;
    q.tab = o; o += 8 * (uint32_t)(M * D);
    q.fits = o; o += 8 * (uint32_t)M;
    q.wts = o; o += 8 * (uint32_t)M;
    q.beta = o; o += uni ? 0u : 4 * (uint32_t)(D * D);
    q.total = (o + 15u) & ~15u;
    return q;
}

// Order this wave's LDS accesses (one wave per workgroup; LDS serves a wave
// in program order, so only the compiler has to be held back).
__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL>
__device__ __forceinline__ double dpp64(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// Minimum / maximum over the first `used` lanes (uniform; the lanes up to the
// next multiple of 4 or 16 hold the neutral value): exchanges within quads,
// then rotations within the rows of 16, then the rows' first lanes.
template <bool MAX>
__device__ __forceinline__ double lanes_reduce(double x, int used) {
    auto op = [](double a, double b) { return MAX ? fmax(a, b) : fmin(a, b); };
    x = op(x, dpp64<0xB1>(x));  // quad_perm [1,0,3,2]
    x = op(x, dpp64<0x4E>(x));  // quad_perm [2,3,0,1]
    if (used <= 4) return rld(x, 0);
    x = op(x, dpp64<0x124>(x));  // row_ror:4
    x = op(x, dpp64<0x128>(x));  // row_ror:8
    double r = rld(x, 0);
    if (used > 16) r = op(r, rld(x, 16));
    if (used > 32) r = op(r, rld(x, 32));
    if (used > 48) r = op(r, rld(x, 48));
    return r;
}

// Sort (key, idx) ascending, cnt entries, the arrays holding the next power
// of two (at least 64) of them: bitonic, four pairs' loads in flight per lane.
__device__ void sort_lds(uint64_t *key, uint32_t *idx, int cnt, int lane) {
    int np = 64;
    while (np < cnt) np <<= 1;
    for (int t = cnt + lane; t < np; t += 64) {
        key[t] = ~0ull;
        idx[t] = 0xffffffffu;
    }
    lds_order();
    const int pairs = np >> 1;
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t0 = lane; t0 < pairs; t0 += 256) {
                constexpr int P = 4;
                uint64_t ki[P], kl[P];
                uint32_t xi[P], xl[P];
                int at[P];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int t = min(t0 + 64 * p, pairs - 1);
                    at[p] = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                    ki[p] = key[at[p]];
                    kl[p] = key[at[p] | j];
                    xi[p] = idx[at[p]];
                    xl[p] = idx[at[p] | j];
                }
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const bool gt = ki[p] > kl[p] || (ki[p] == kl[p] && xi[p] > xl[p]);
                    if (t0 + 64 * p < pairs && gt == ((at[p] & k) == 0)) {
                        key[at[p]] = kl[p];
                        key[at[p] | j] = ki[p];
                        idx[at[p]] = xl[p];
                        idx[at[p] | j] = xi[p];
                    }
                }
            }
            lds_order();
        }
}

template <int MODE, bool UNI>  // MODE 0: execute a plan; 2: HEFT-style placement
__global__ __launch_bounds__(64) void k_sim_lds(SimLaunch a) {
    extern __shared__ uint64_t smem[];
    uint8_t *sb = reinterpret_cast<uint8_t *>(smem);
    const int b = blockIdx.x, lane = threadIdx.x;
    const int D = a.D, K = a.K, M = a.M;
    const SimPlan pl = sim_plan(a.max_stages, D, K, M, UNI);
    int64_t *top = reinterpret_cast<int64_t *>(sb + pl.rank);
    uint64_t *key = reinterpret_cast<uint64_t *>(sb + pl.key);
    FinHold *fh = reinterpret_cast<FinHold *>(sb + pl.rank);
    uint32_t *todo = reinterpret_cast<uint32_t *>(sb + pl.idx);
    uint64_t *ring = reinterpret_cast<uint64_t *>(sb + pl.ring);
    ParL *pbuf = reinterpret_cast<ParL *>(sb + pl.par);
    float2 *tab = reinterpret_cast<float2 *>(sb + pl.tab);  // (run time, switch time) of model m on device d
    uint64_t *fits = reinterpret_cast<uint64_t *>(sb + pl.fits), *wts = reinterpret_cast<uint64_t *>(sb + pl.wts);
    float *bt = reinterpret_cast<float *>(sb + pl.beta);

    const int64_t base = a.stage_off[b];
    const int n = (int)(a.stage_off[b + 1] - base);
    const double t0 = (double)a.tnow[b];
    const bool live = lane < D;
    const int dl = live ? lane : D - 1;
    const uint64_t dm = D >= 64 ? ~0ull : ((1ull << D) - 1ull);
    for (int i = lane; i < M * D; i += 64) tab[i] = make_float2(a.exec[i], a.ksw[i]);
    if (lane < M) {
        fits[lane] = a.fits[lane];
        wts[lane] = a.weight[lane];
    }
    if (!UNI)
        for (int i = lane; i < D * D; i += 64) bt[i] = a.beta[i];
    for (int i = lane; i < D * K; i += 64) ring[i] = a.pcache[(int64_t)b * D * K + i];
    double fr = live ? fmax((double)a.tau[(int64_t)b * D + lane], t0) : 0.0;  // lane d: free time of device d
    uint64_t res = live ? a.resident[(int64_t)b * D + lane] : 0ull;           // its resident models
    const uint64_t cap = live ? a.cap[lane] : 0ull;
    int lastm = -1;  // lane d: model of the stage device d ran last
    const double b0 = (double)a.beta0;
    lds_order();
    uint64_t tot = 0;  // lane d: weight of the resident models
    for (int m = 0; m < M; ++m) tot += ((res >> m) & 1ull) ? wts[m] : 0ull;
    // lane d: the empty slots of device d, the slot the next group takes (the
    // first empty one, or the oldest) and what it holds
    uint32_t emask = 0, pos = 0;
    uint64_t victim = 0;
    if (live && K > 0) {
        for (int e = 0; e < K; ++e) emask |= (ring[lane * K + e] == 0 ? 1u : 0u) << e;
        pos = emask ? (uint32_t)__builtin_ctz(emask) : 0u;
        victim = ring[lane * K + (int)pos];
    }

    // ---- the stages to run and their order
    int cnt = 0;
    if (MODE == 0) {
        bool bad = false;
        for (int v0 = 0; v0 < n; v0 += 64) {
            const int v = v0 + lane;
            const uint64_t S = v < n ? a.devices[base + v] : 0ull;
            bad = bad || (S & ~dm) != 0;
            const bool take = S != 0 && a.holders[base + v] == 0ull;
            const uint64_t bal = __ballot(take);
            if (take) {
                const int o = cnt + __popcll(bal & ((1ull << lane) - 1ull));
                key[o] = (uint64_t)a.order[base + v] ^ (1ull << 63);
                todo[o] = (uint32_t)v;
            }
            cnt += __popcll(bal);
        }
        if (__ballot(bad) != 0ull) {
            if (lane == 0) {
                a.status[b] = FATE_EINVAL;
                a.out[b] = fate_sim_metrics_t{};
            }
            return;
        }
    } else {
        double bmean = a.bmean;  // mean off-diagonal transfer coefficient, summed in row order
        if (!UNI) {
            bmean = 0.0;
            for (int i = 0; i < D; ++i)
                for (int j = 0; j < D; ++j)
                    if (i != j) bmean += (double)bt[i * D + j];
            bmean = D > 1 ? bmean / (double)(D * (D - 1)) : 0.0;
        }
        // top[v]: largest rank pushed by a child of v (bits of a double >= 0),
        // -1 = none; then v's rank
        for (int v = lane; v < n; v += 64) top[v] = -1;
        lds_order();
        constexpr int kP = 4;
        auto fetch = [&](int hi) { return a.rec[base + max(0, hi - 64 + lane)]; };
        StageRec nx{};
        if (n > 0) nx = fetch(n);
        for (int hi = n; hi > 0; hi -= 64) {  // uniform
            const int v = hi - 64 + lane;
            const bool in = v >= 0;
            const StageRec r = nx;
            uint32_t pid[kP];
#pragma unroll
            for (int q = 0; q < kP; ++q) pid[q] = in && q < (int)r.npar ? a.par_idx[r.par_begin + q] - (uint32_t)base : 0u;
            if (hi > 64) nx = fetch(hi - 64);
            double wsum = 0.0;
            int nf = 0;
            const uint64_t fm = r.elig & fits[r.model] & dm;
            for (int d = 0; d < D; ++d)
                if ((fm >> d) & 1ull) {
                    wsum += (double)tab[r.model * D + d].x;
                    ++nf;
                }
            const double wbar = wsum / (double)nf, sg = (double)r.sigma * bmean;
            double rank = -1.0;  // a rank is never negative
            for (int it = 0; it <= 64; ++it) {  // 64 stages are at most 64 deep
                const int64_t t = in ? top[v] : -1;
                const double x = wbar + (t < 0 ? 0.0 : sg + __longlong_as_double((long long)t));
                const bool grew = in && x != rank;
                if (__ballot(grew) == 0ull) break;
                if (grew) {
                    rank = x;
                    const int64_t bits = (int64_t)__double_as_longlong(x + 0.0);
#pragma unroll
                    for (int q = 0; q < kP; ++q)
                        if (q < (int)r.npar)
                            __hip_atomic_fetch_max(&top[pid[q]], bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    for (int q = kP; q < (int)r.npar; ++q)
                        __hip_atomic_fetch_max(&top[a.par_idx[r.par_begin + q] - (uint32_t)base], bits, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                lds_order();
            }
            // every child has a larger id, so v's maximum is not read again
            if (in) top[v] = (int64_t)__double_as_longlong(rank);
            lds_order();
        }
        for (int v0 = 0; v0 < n; v0 += 64) {
            const int v = v0 + lane;
            const bool done = v < n && a.holders[base + v] != 0ull;
            const bool take = v < n && !done;
            if (done) {  // completed stages are not placed
                a.dev_out[base + v] = 0ull;
                a.ord_out[base + v] = 0;
            }
            const uint64_t bal = __ballot(take);
            if (take) {  // by rank descending, then id
                const int o = cnt + __popcll(bal & ((1ull << lane) - 1ull));
                key[o] = ~dkey(__longlong_as_double((long long)top[v]));
                todo[o] = (uint32_t)v;
            }
            cnt += __popcll(bal);
        }
    }
    lds_order();
    sort_lds(key, todo, cnt, lane);
    for (int v = lane; v < n; v += 64) {
        const uint64_t h = a.holders[base + v];
        fh[v] = FinHold{h != 0 ? t0 : 0.0, h};
    }
    lds_order();

    // ---- the walk
    fate_sim_metrics_t mt{};
    int32_t st = FATE_OK;
    double last = t0;
    uint32_t xdev = 0, hits = 0, conts = 0;
    StageRec nx{};
    uint32_t nv = 0;
    uint64_t nS = 0;
    auto fetch = [&](int p) {  // the record of the stage at position p (and its devices)
        nv = p < cnt ? todo[p] : 0u;
        nx = a.rec[base + nv];
        if (MODE == 0) nS = p < cnt ? a.devices[base + nv] : 0ull;
    };
    if (cnt > 0) fetch(lane);
    for (int p0 = 0; p0 < cnt && st == FATE_OK; p0 += 64) {  // uniform: 64 stages, stage i of them on lane i
        const int nb = min(64, cnt - p0);
        const bool in = lane < nb;
        const uint32_t bv = nv;
        const StageRec r = nx;
        const uint64_t bS = MODE == 0 ? nS : (r.elig & fits[r.model] & dm);
        const double bpf = a.kpf * (double)r.tokens;
        const uint32_t nbuf = in && r.npar <= 64 ? r.npar : 0u;
        uint32_t all = 0;
        const uint32_t off = wave_exscan_u32(nbuf, all);
        const bool buffered = nbuf == r.npar && off + nbuf <= (uint32_t)kParBuf;
        uint32_t u0 = 0;   // the first parent
        double tr0 = 0.0;
        if (in && buffered)
            for (uint32_t q0 = 0; q0 < nbuf; q0 += 4) {
                uint32_t u[4];
                float sg[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) u[j] = a.par_idx[r.par_begin + min(q0 + j, nbuf - 1u)];
#pragma unroll
                for (int j = 0; j < 4; ++j) sg[j] = a.rec[u[j]].sigma;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (q0 + j < nbuf) {
                        const ParL e{u[j] - (uint32_t)base, sg[j], (double)sg[j] * b0};
                        pbuf[off + q0 + j] = e;
                        if (q0 + j == 0) {
                            u0 = e.u;
                            tr0 = e.tr;
                        }
                    }
            }
        const uint32_t bnp = buffered ? off : 0xffffu;  // 0xffff: no prefetched list
        uint64_t cached = 0;  // devices caching the stage's group
        if (r.hash != 0)
            for (int d = 0; d < D; ++d) {
                bool c = false;
#pragma unroll 8
                for (int e = 0; e < K; ++e) c = c | (ring[d * K + e] == r.hash);
                cached |= (uint64_t)c << d;
            }
        double run0 = 0.0, run1 = 0.0, swt = 0.0;  // execution: on the stage's first device
        if (MODE == 0 && in) {
            const int d0 = __builtin_ctzll(bS);
            const double k = (double)__popcll(bS);
            const float2 c = tab[r.model * D + d0];
            run0 = (double)c.x / k;
            run1 = fmax(0.0, run0 - bpf / k);
            swt = (double)c.y;
        }
        const uint32_t pbeg = r.par_begin, bm = r.model | (uint32_t)r.npar << 8;
        // the common stages, whose link is straight-line code: a prefetched list of
        // at most 16 parents and one device (execution), of at most 4 parents (HEFT)
        const bool common = UNI && buffered && (MODE == 2 ? r.npar <= 4 : r.npar <= 16 && (bS & (bS - 1)) == 0);
        const uint64_t bcom = __ballot(common);
        const uint64_t bhash = r.hash;
        lds_order();
        if (p0 + 64 < cnt) fetch(p0 + 64 + lane);
        uint64_t placed = 0;  // HEFT: lane i, the device of stage i

        // up to 64 parents of stage i, one per lane
        FinHold pe;
        ParL px;
        auto parents = [&](int i, uint32_t po, bool buf, int q0, int nq) {
            pe = FinHold{t0, 1ull};
            px = ParL{0u, 0.0f, 0.0};
            if (lane < nq) {
                if (buf) {
                    px = pbuf[po + (uint32_t)lane];
                } else {
                    const uint32_t gu = a.par_idx[(uint32_t)__builtin_amdgcn_readlane((int)pbeg, i) + (uint32_t)(q0 + lane)];
                    px.sigma = a.rec[gu].sigma;
                    px.tr = (double)px.sigma * b0;
                    px.u = gu - (uint32_t)base;
                }
                pe = fh[px.u];
            }
        };
        // the cheapest of the holders h into device d
        auto cheapest = [&](uint64_t h, int d) {
            double x = __builtin_huge_val();
            for (uint64_t t = h; t; t &= t - 1) x = fmin(x, (double)bt[__builtin_ctzll(t) * D + d]);
            return x;
        };
        // stage i's group joins the slots of device d (uniform), which lacks it
        auto join_slots = [&](int i, int d) {
            const uint64_t hash = rl64(bhash, i), old = rl64(victim, d);
            if (hash == 0 || K == 0) return;
            // the group dropped leaves the device unless another slot has it too
            // (an initial state may repeat one); seldom does a stage of the
            // batch ask for it
            if (old != 0 && __ballot(bhash == old) != 0) {
                const uint64_t row = lane < K ? ring[d * K + lane] : 0ull;
                if (__popcll(__ballot(row == old)) == 1) cached &= bhash == old ? ~(1ull << d) : ~0ull;
            }
            cached |= bhash == hash ? 1ull << d : 0ull;
            if (lane == d) {
                ring[d * K + (int)pos] = hash;
                const uint32_t left = emask & (emask - 1u);  // pos was the lowest of them
                const uint32_t next = pos + 1u == (uint32_t)K ? 0u : pos + 1u;
                pos = emask == 0 ? next : left ? (uint32_t)__builtin_ctz(left) : 0u;
                emask = emask ? left : 0u;
                victim = ring[d * K + (int)pos];
            }
        };
        // device d (uniform) loads model m, which it lacks
        auto load = [&](int d, int m) {
            if (lane == d) {
                res |= 1ull << m;
                tot += wts[m];
                for (uint64_t t = res & ~(1ull << m); t && tot > cap; t &= t - 1) {
                    const int x = __builtin_ctzll(t);
                    res &= ~(1ull << x);
                    tot -= wts[x];
                }
            }
        };

        for (int i = 0; i < nb; ++i) {  // uniform
            const int v = __builtin_amdgcn_readlane((int)bv, i);
            const uint32_t mn = (uint32_t)__builtin_amdgcn_readlane((int)bm, i);
            const uint32_t po = (uint32_t)__builtin_amdgcn_readlane((int)bnp, i);
            const int m = (int)(mn & 0xffu), np = (int)(mn >> 8);
            const bool buf = po != 0xffffu, com = (bcom >> i) & 1ull;
            const uint64_t S0 = rl64(bS, i), cm = rl64(cached, i);
            double f;
            uint64_t S;
            if (MODE == 2) {  // every feasible device at once; the earliest finish, ties to the lower device
                const float2 c = tab[m * D + dl];
                double ready = t0;
                auto arrive = [&](const FinHold &x, double tr, float sg) {
                    if (!UNI) tr = (double)sg * cheapest(x.hold, dl);
                    const double far = x.fin + tr;
                    ready = fmax(ready, (x.hold >> lane) & 1ull ? x.fin : far);
                };
                auto four = [&](int q0) {  // a repeated parent changes nothing
                    ParL e[4];
                    FinHold x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) e[j] = pbuf[po + (uint32_t)min(q0 + j, np - 1)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = fh[e[j].u];
#pragma unroll
                    for (int j = 0; j < 4; ++j) arrive(x[j], e[j].tr, e[j].sigma);
                };
                if (com) {
                    if (np > 1) four(0);
                    else if (np == 1) arrive(fh[__builtin_amdgcn_readlane((int)u0, i)], rld(tr0, i), 0.0f);
                } else if (buf) {
                    for (int q0 = 0; q0 < np; q0 += 4) four(q0);
                } else {
                    for (int q = 0; q < np; ++q) {
                        const uint32_t gu = a.par_idx[(uint32_t)__builtin_amdgcn_readlane((int)pbeg, i) + (uint32_t)q];
                        const float sg = a.rec[gu].sigma;
                        arrive(fh[gu - (uint32_t)base], (double)sg * b0, sg);
                    }
                }
                const bool hit = __builtin_amdgcn_inverse_ballot_w64(cm), feas = __builtin_amdgcn_inverse_ballot_w64(S0);
                const bool has = (res >> m) & 1ull;
                const double r0 = (double)c.x, r1 = fmax(0.0, r0 - rld(bpf, i));
                const double fd = (fmax(fr, ready) + (has ? 0.0 : (double)c.y)) + (hit ? r1 : r0);
                f = lanes_reduce<false>(feas ? fd : __builtin_huge_val(), D);
                const uint64_t who = __ballot(feas && fd == f);
                if (who == 0) {  // no device: packing excludes it
                    st = FATE_ESTATE;
                    break;
                }
                const int d = __builtin_ctzll(who);
                S = 1ull << d;
                if (!((__ballot(has) >> d) & 1ull)) load(d, m);
                if (!((cm >> d) & 1ull)) join_slots(i, d);
                fr = lane == d ? f : fr;
                f = fmax(t0, f);
                placed = lane == i ? S : placed;
            } else if (com) {
                S = S0;
                const int d = __builtin_ctzll(S);
                pe = FinHold{t0, ~0ull};
                px.tr = 0.0;
                if (lane < np) {
                    px = pbuf[po + (uint32_t)lane];
                    pe = fh[px.u];
                }
                const double far = pe.fin + px.tr;
                const bool here = (pe.hold >> d) & 1ull;
                if (__ballot(pe.hold == 0ull) != 0ull) {  // the order runs a stage before one of its parents
                    st = FATE_ESTATE;
                    break;
                }
                xdev += (uint32_t)__popcll(__ballot(!here));
                double x = here ? pe.fin : far;
                x = fmax(x, dpp64<0xB1>(x));
                x = fmax(x, dpp64<0x4E>(x));
                x = fmax(x, dpp64<0x124>(x));
                x = fmax(x, dpp64<0x128>(x));  // lane 0: the latest arrival (at least t)
                const bool hit = (cm >> d) & 1ull, has = (rl64(res, d) >> m) & 1ull;
                const double run = hit ? rld(run1, i) : rld(run0, i), sw = rld(swt, i);
                f = rld((fmax(rld(fr, d), x) + (has ? 0.0 : sw)) + run, 0);
                hits += hit ? 1u : 0u;
                conts += __builtin_amdgcn_readlane(lastm, d) == m ? 1u : 0u;
                if (!has) load(d, m);
                if (!hit) join_slots(i, d);
                fr = lane == d ? f : fr;
                lastm = lane == d ? m : lastm;
                f = fmax(t0, f);
                last = fmax(last, f);
            } else {
                S = S0;
                const int d0 = __builtin_ctzll(S), k = __popcll(S);
                const double kd = (double)k;
                f = t0;
                uint64_t dead = 0;
                for (uint64_t t = S; t; t &= t - 1) {  // uniform
                    const int d = __builtin_ctzll(t);
                    double ready = t0;
                    for (int q0 = 0; q0 < np; q0 += 64) {
                        const int nq = min(64, np - q0);
                        if (np > 64 || d == d0) parents(i, po, buf, q0, nq);
                        if (d == d0) {
                            dead |= __ballot(pe.hold == 0ull);
                            xdev += (uint32_t)__popcll(__ballot(lane < nq && (pe.hold & S) == 0ull));
                        }
                        double tr = px.tr;
                        if (!UNI) tr = (double)px.sigma * cheapest(lane < nq ? pe.hold : 0ull, d);
                        tr = tr / kd;
                        const double arr = lane >= nq || ((pe.hold >> d) & 1ull) ? pe.fin : pe.fin + tr;
                        ready = fmax(ready, lanes_reduce<true>(arr, nq));
                    }
                    if (dead != 0) break;
                    const bool hit = (cm >> d) & 1ull, has = (rl64(res, d) >> m) & 1ull;
                    const float2 c = tab[m * D + d];
                    double run = (double)c.x / kd;
                    if (hit) run = fmax(0.0, run - rld(bpf, i) / kd);
                    if (d == d0) {
                        hits += hit ? 1u : 0u;
                        conts += __builtin_amdgcn_readlane(lastm, d) == m ? 1u : 0u;
                    }
                    const double fd = (fmax(rld(fr, d), ready) + (has ? 0.0 : (double)c.y)) + run;
                    if (!has) load(d, m);
                    if (!hit) join_slots(i, d);
                    fr = lane == d ? fd : fr;
                    lastm = lane == d ? m : lastm;
                    f = fmax(f, fd);
                }
                if (dead != 0) {  // the order runs a stage before one of its parents
                    st = FATE_ESTATE;
                    break;
                }
                last = fmax(last, f);
            }
            if (lane == 0) fh[v] = FinHold{f, S};
            lds_order();
        }
        if (MODE == 2 && in) {
            a.dev_out[base + bv] = placed;
            a.ord_out[base + bv] = p0 + lane;
        }
    }
    if (MODE == 2) {
        if (lane == 0) a.status[b] = st;
        return;
    }
    if (st != FATE_OK) {
        if (lane == 0) {
            a.status[b] = st;
            a.out[b] = fate_sim_metrics_t{};
        }
        return;
    }

    // makespan, and the p95 of the sinks' completion times: the element at
    // 0-based position ceil(0.95 ns) - 1 in ascending order (the times pass
    // through the workspace: the keys' place is still in use)
    int ns = 0;
    for (int p0 = 0; p0 < cnt; p0 += 64) {
        const int p = p0 + lane;
        const uint32_t v = p < cnt ? todo[p] : 0u;
        const bool sink = p < cnt && a.ch_off[base + v] == a.ch_off[base + v + 1];
        const uint64_t bal = __ballot(sink);
        if (sink) a.aux[base + ns + __popcll(bal & ((1ull << lane) - 1ull))] = fh[v].fin - t0;
        ns += __popcll(bal);
    }
    mt.tasks = cnt;
    mt.xdev_edges = xdev;
    mt.cache_hits = hits;
    mt.model_cont = conts;
    mt.makespan = last - t0;
    wave_fence();
    if (ns > 0) {
        for (int i = lane; i < ns; i += 64) {
            key[i] = dkey(a.aux[base + i]);
            todo[i] = (uint32_t)i;
        }
        lds_order();
        sort_lds(key, todo, ns, lane);
        const int rk = max(0, (int)ceil(0.95 * (double)ns) - 1);
        mt.p95 = dkey_inv(key[rk]);
    }
    if (lane == 0) {
        a.out[b] = mt;
        a.status[b] = FATE_OK;
    }
}

}  // namespace

// Whether a batch takes k_sim_lds.  The choice is the batch's: its largest
// instance has to fit the LDS (20 to 32 bytes per stage and the tables: 29 KB
// for 1,000 stages on 16 devices), or all of its instances walk through the
// workspace in k_sim, the only place that holds the large one: 1,023 instances
// of 200 stages beside one of 9,000 are placed in 73.5 ms, as long as the large
// one takes.  Fork-join, 1,024 instances of 1,000 stages (700 to run) on 16
// devices, one wave per SIMD: HEFT placement 6.44 ms in k_sim, 0.65 ms here;
// execution 3.60 ms, 0.66 ms.  Of the 0.65 ms the walk takes 0.53 (1,700 cycles
// a stage: arrivals 500, finish and choice 300, Load and slots 450), the
// ranks 0.04 and the sort 0.05; the chain of single instructions binds, not
// memory.
//
// k_sim keeps eight walks per compute unit whatever their size.  While the LDS
// leaves room for two, k_sim_lds is ahead also of that (4,096 layered instances
// of 1,500 stages on 48 devices with links of two speeds, execution 11.6 ms
// against 12.3).  With room for one, placement stays ahead (2,048 power-law
// instances of 4,000 stages on 64 devices 28.8 ms against 57.4), and execution,
// whose link in k_sim is shorter, while few instances are many rounds of one
// per compute unit, or where the devices are few.  Execution in ms, k_sim_lds
// and k_sim, 4,000 stages, uniform links:
//   64 devices, power-law  1,024 instances 12.1, 18.4; 1,536 18.2, 20.0; 2,048 24.3, 20.9
//   32 devices, 2,048      power-law 21.1, 21.0; layered 20.7, 19.4
//   24 devices             layered 2,048 19.5, 19.1; power-law 4,096 40.7, 41.9
//   16 devices, fork-join  4,096 39.9, 53.7
// and with links of several speeds, where the walk reads the link of every
// holder:
//   64 devices, power-law, 2,500 stages  1,024 9.5, 10.5; 1,280 11.9, 11.1; 2,048 19.3, 12.2
//   2,048 of 4,000 stages  16 devices, layered 25.2, 19.1; 8 devices 17.5, 18.9
static bool sim_in_lds(const SimLaunch &a, int mode) {
    constexpr int kCus = 256, kLds = 160 * 1024;
    const bool uni = a.beta_uniform != 0;
    if (!a.ch_off || a.max_stages > 16384) return false;
    const uint32_t lds = sim_plan(a.max_stages, a.D, a.K, a.M, uni).total;
    if (lds > (uint32_t)kLds) return false;
    const bool few = a.D <= (uni ? 24 : 8);
    return mode == 2 || lds <= (uint32_t)kLds / 2 || few || a.N <= (uni ? 6 : 4) * kCus * a.max_stages;
}

int launch_sim(const SimLaunch &a, int mode, void *stream) {
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a.B <= 0) return 0;
    const dim3 grid((unsigned)a.B), block(64);
    if (mode != 1 && sim_in_lds(a, mode)) {
        const bool uni = a.beta_uniform != 0;
        const size_t lds = sim_plan(a.max_stages, a.D, a.K, a.M, uni).total;
        if (mode == 0) {
            if (uni) hipLaunchKernelGGL((k_sim_lds<0, true>), grid, block, lds, s, a);
            else hipLaunchKernelGGL((k_sim_lds<0, false>), grid, block, lds, s, a);
        } else {
            if (uni) hipLaunchKernelGGL((k_sim_lds<2, true>), grid, block, lds, s, a);
            else hipLaunchKernelGGL((k_sim_lds<2, false>), grid, block, lds, s, a);
        }
        return (int)hipGetLastError();
    }
    if (mode == 0) hipLaunchKernelGGL(k_sim<0>, grid, block, 0, s, a);
    else if (mode == 1) hipLaunchKernelGGL(k_sim<1>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(k_sim<2>, grid, block, 0, s, a);
    return (int)hipGetLastError();
}

}  // namespace fate
