// Frontier planning wave on the device (Alg. 1 planner step, under the wave
// constraints of App. A.2: each device takes at most one shard-slot
// assignment per wave, each stage at most one choice; a window candidate is
// the stage's slots 0..k-1 on k devices, so slot order holds by itself).
// The choices of a frontier stage are its top-k (fate_topk's output); the
// wave is built greedily: the best remaining choice whose stage is still
// unassigned and whose devices are all free is taken, ties going to the
// lower frontier slot, then the lower rank, until no choice is left.
//
//   k_plan_wave  one 64-lane wave per instance.  The instance's choices are
//                kept as (order-preserving score key, device mask, stage and
//                candidate), up to sixteen in each lane's registers; each
//                round every lane takes the best of its keys, a wave-wide
//                maximum picks the round's winner, and the keys of the
//                winner's stage and of choices on its devices are cleared
//                (neither comes back, so a key that is set is a valid choice).
//                At most D rounds take a choice.  Instances of more choices
//                stage keys and candidates in LDS, and read those past its
//                capacity from HBM each round.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fate_device.h"
#include "fate_internal.h"

namespace fate {
namespace {

// Choices held in registers: 64 lanes of kPlanRegs (fork-join instances hold
// about 460 at k = 4; instances of at most half run the half-sized loop).  A
// round is one pass over the lane's keys and one wave maximum: with the choices
// in LDS (sixteen bytes each), two barriers and a global load of the winner's
// candidate per round, a wave of 4,096 fork-join instances took 28.4 us; 15.6
// from registers.  The rounds are sequential: their latency binds.
constexpr int kPlanRegs = 16;
// Choices staged in LDS for larger instances: 8 KB, so that the instances that
// need none of it still share a compute unit sixteen at a time.
constexpr int kPlanCap = 1024;

// Order-preserving map of a finite or +infinite score to a nonzero 32-bit key
// (a larger score gives a larger key, -0 and +0 the same one); 0 marks "no
// valid choice".
__device__ __forceinline__ uint32_t score_key(float v) {
    const uint32_t u = __float_as_uint(v + 0.0f);  // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Devices of candidate j (the numbering of candidate_window, without its loop).
__device__ __forceinline__ uint64_t window_mask(int32_t j, int D) {
    static_assert(FATE_MAX_SHARD == 4, "window sizes 2 to 4");
    const int32_t j2 = j - D, j3 = j2 - (D - 1), j4 = j3 - (D - 2);
    const uint64_t m = j2 < 0 ? 1ull : j3 < 0 ? 3ull : j4 < 0 ? 7ull : 15ull;
    return m << ((j2 < 0 ? j : j3 < 0 ? j2 : j4 < 0 ? j3 : j4) & 63);
}

// Devices of candidate j of a stage with nc candidates, or 0 when j is not
// one of them; -infinity and padding are no choice.
__device__ __forceinline__ uint64_t choice_mask(int32_t j, float v, int D, uint32_t nc) {
    if (j < 0 || (uint32_t)j >= nc || !(v > -inf_f())) return 0ull;
    return window_mask(j, D);
}

struct ChoiceL {
    uint32_t key;
    int32_t j;  // candidate
};

// Maximum over the wave (all 64 lanes active), returned to every lane: DPP
// steps within each 16-lane row (pairs, quads, half-rows, rows), then the four
// row maxima through scalar registers.  No LDS round trips.
template <int CTRL>
__device__ __forceinline__ uint32_t umax_dpp(uint32_t x) {
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    x = umax_dpp<0xB1>(x);   // quad_perm [1, 0, 3, 2]
    x = umax_dpp<0x4E>(x);   // quad_perm [2, 3, 0, 1]
    x = umax_dpp<0x141>(x);  // row_half_mirror
    x = umax_dpp<0x140>(x);  // row_mirror
    const uint32_t r0 = __builtin_amdgcn_readlane(x, 0), r1 = __builtin_amdgcn_readlane(x, 16);
    const uint32_t r2 = __builtin_amdgcn_readlane(x, 32), r3 = __builtin_amdgcn_readlane(x, 48);
    return max(max(r0, r1), max(r2, r3));
}
// 64-bit maximum: the high words first, then the low words of the lanes
// holding the highest high word.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t x) {
    const uint32_t hi = wave_max_u32((uint32_t)(x >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(x >> 32) == hi ? (uint32_t)x : 0u);
    return ((uint64_t)hi << 32) | lo;
}

// The wave of one instance (frontier slots lo .. hi) from registers: n <= 64 R
// choices, choice c on lane c mod 64.  Mask holds the devices of D <= 32, or 64.
template <int R, class Mask>
__device__ __forceinline__ void plan_in_registers(const PlanLaunch &a, int64_t lo, int64_t base, uint32_t n) {
    const int lane = threadIdx.x, D = a.D;
    const uint32_t k = (uint32_t)a.k;
    uint32_t key[R], sj[R];  // sj: stage slot << 8 | candidate (below 256)
    Mask mask[R];
    int32_t jj[R];
    float vv[R];
    uint32_t nc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {  // the loads first
        const uint32_t c = (uint32_t)(r * 64 + lane);
        jj[r] = -1;
        vv[r] = 0.0f;
        nc[r] = 0u;
        if (c < n) {
            const int64_t f = lo + c / k;
            jj[r] = a.idx[base + c];
            vv[r] = a.val[base + c];
            nc[r] = a.cand_off[f + 1] - a.cand_off[f];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t m = choice_mask(jj[r], vv[r], D, nc[r]);
        mask[r] = (Mask)m;
        key[r] = m ? score_key(vv[r]) : 0u;
        sj[r] = ((uint32_t)(r * 64 + lane) / k) << 8 | ((uint32_t)jj[r] & 0xffu);
    }
    Mask dev = 0;                // the last winner's devices
    uint32_t wst = 0xffffffffu;  // and stage slot
    for (;;) {                   // uniform: one assignment per round
        uint32_t bk = 0u, br = 0u, bsj = 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            key[r] = (mask[r] & dev) != 0 || (sj[r] >> 8) == wst ? 0u : key[r];
            const bool gt = key[r] > bk;  // among equal keys the lowest choice index
            bk = gt ? key[r] : bk;
            br = gt ? (uint32_t)r : br;
            bsj = gt ? sj[r] : bsj;
        }
        const uint32_t m = wave_max_u32(bk);
        if (m == 0u) break;
        const uint64_t who = __ballot(bk == m);
        int L = __builtin_ctzll(who);
        if (who & (who - 1)) {  // several lanes: the lowest row of choices, then the lowest lane
            const uint32_t w = wave_max_u32(bk == m ? (uint32_t)(R - br) << 6 | (uint32_t)(63 - lane) : 0u);
            L = 63 - (int)(w & 63u);
        }
        const uint32_t wsj = __builtin_amdgcn_readlane(bsj, L);
        const int32_t j = (int32_t)(wsj & 0xffu);
        dev = (Mask)window_mask(j, D);
        wst = wsj >> 8;
        if (lane == 0) a.sel[lo + wst] = j;
    }
}

__global__ __launch_bounds__(64) void k_plan_wave(PlanLaunch a) {
    __shared__ ChoiceL ch[kPlanCap];
    __shared__ uint32_t taken[64];  // local stages assigned so far (one device each at least)
    const int b = (int)a.order[blockIdx.x], lane = threadIdx.x, k = a.k;  // largest frontiers first
    const int64_t lo = a.fr_off[b], hi = a.fr_off[b + 1];
    const int64_t base = lo * k;
    const uint32_t n = (uint32_t)((hi - lo) * k);
    const uint32_t nl = n < (uint32_t)kPlanCap ? n : (uint32_t)kPlanCap;
    for (int64_t f = lo + lane; f < hi; f += 64) a.sel[f] = -1;
    __syncthreads();  // the winners' candidates go over them
    if (n <= 64u * (kPlanRegs / 2)) {  // uniform
        if (a.D <= 32) plan_in_registers<kPlanRegs / 2, uint32_t>(a, lo, base, n);
        else plan_in_registers<kPlanRegs / 2, uint64_t>(a, lo, base, n);
        return;
    }
    if (n <= 64u * kPlanRegs) {
        if (a.D <= 32) plan_in_registers<kPlanRegs, uint32_t>(a, lo, base, n);
        else plan_in_registers<kPlanRegs, uint64_t>(a, lo, base, n);
        return;
    }
    for (uint32_t c = lane; c < nl; c += 64) {
        const int64_t f = lo + c / (uint32_t)k;
        ChoiceL x;
        x.j = a.idx[base + c];
        x.key = choice_mask(x.j, a.val[base + c], a.D, a.cand_off[f + 1] - a.cand_off[f]) ? score_key(a.val[base + c]) : 0u;
        ch[c] = x;
    }
    __syncthreads();
    uint64_t used = 0;
    int ntaken = 0;
    for (;;) {  // uniform: one assignment per round
        uint64_t best = 0;
        for (uint32_t c = lane; c < n; c += 64) {
            uint64_t m;
            uint32_t key;
            if (c < nl) {
                const ChoiceL x = ch[c];
                m = x.key ? window_mask(x.j, a.D) : 0ull;
                key = x.key;
            } else {  // past the LDS capacity: read again, and skip assigned stages
                const float v = a.val[base + c];
                const uint32_t s = c / (uint32_t)k;
                m = choice_mask(a.idx[base + c], v, a.D, a.cand_off[lo + s + 1] - a.cand_off[lo + s]);
                key = m ? score_key(v) : 0u;
                for (int t = 0; t < ntaken; ++t) key = taken[t] == s ? 0u : key;
            }
            // highest key first; among equal keys the lowest choice index
            const uint64_t cand = ((uint64_t)key << 32) | (uint64_t)(0xffffffffu - c);
            if (key != 0u && (m & used) == 0ull && cand > best) best = cand;
        }
        best = wave_max_u64(best);
        if (best == 0ull) break;
        const uint32_t c = 0xffffffffu - (uint32_t)best;
        const uint32_t s = c / (uint32_t)k;
        const int32_t j = c < nl ? ch[c].j : a.idx[base + c];
        used |= window_mask(j, a.D);
        __syncthreads();  // every lane has read the winner
        if (lane == 0) {
            a.sel[lo + s] = j;
            taken[ntaken] = s;
        }
        if (lane < k && s * (uint32_t)k + (uint32_t)lane < nl) ch[s * k + lane].key = 0u;
        ++ntaken;
        __syncthreads();
    }
}

}  // namespace

int launch_plan(const PlanLaunch &a, void *stream) {
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a.B > 0) hipLaunchKernelGGL(k_plan_wave, dim3((unsigned)a.B), dim3(64), 0, s, a);
    return (int)hipGetLastError();
}

}  // namespace fate
