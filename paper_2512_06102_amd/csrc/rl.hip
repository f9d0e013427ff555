// rl.hip -- the reinforcement-learning layer over the batched step.
//
// Section 4 of the paper trains an air-tanker agent: it sees an egocentric
// window of the fire, moves, and opens a valve to drop a limited amount of
// water, which turns burning cells burnt; each step costs a penalty
// proportional to the number of burning cells, and putting the fire out
// earns a terminal bonus; episodes start from a random fire and agent
// position.  One RL step of every env is:
//   rl_act_kernel   move each agent, turn an open valve into a water drop
//                   (drop row of the step kernel), spend one unit of water;
//   the step kernel one stochastic step with those drops (water mode) and
//                   the BURNING count of every env;
//   rl_obs_kernel   reward and done from the count, then the (2R+1)^2
//                   window of the new state around each agent.
// rl_reset_kernel redraws the fire and the agent of selected envs.
#include <algorithm>

#include "bitplane.hpp"
#include "devmath.hpp"
#include "framed.hpp"
#include "internal.hpp"
#include "rl.hpp"
#include "stepcell.hpp"

namespace firesim {
namespace {

constexpr int kRlWaves = 4;       // waves per workgroup
// An env of more cells (on average) is reset by 4 waves, not 1.  Measured, us per
// reset with 1 and 4: 4096 envs of 64 x 64 12.9 13.9; 1024 of 76 x 76 11.7 11.0;
// 64 of 128 x 128 17.5 11.3; 1 of 1000 x 1000 626 186.
constexpr int64_t kRlLargeCells = 4096;
// A window of more cells is written by 4 waves in batches of no more envs.
// Measured, us per step in separate launches: 64 envs of 92 x 92, windows of 121
// cells 20.1 19.8, 289 20.8 20.4, 3969 36.3 21.1; 65536 envs of 20 x 20, 289 86 103,
// 3969 190 204; 4096 of 64 x 64, 289 35.0 34.1, 3969 57.8 45.0.
constexpr int kRlLargeWindow = 256, kRlLargeWindowEnvs = 8192;
constexpr int kRlWaveList = 128;  // front cells listed per wave
constexpr uint8_t kOutside = 4;  // observation code of cells beyond the grid

__device__ __forceinline__ int32_t scale_draw(uint32_t w, int32_t n)
{
    return (int32_t)(((uint64_t)w * (uint64_t)n) >> 32);  // uniform in 0..n-1
}

// kWaves waves per env, kRlWaves waves per workgroup: lanes 0 to 7 of each draw
// the eight ignition attempts at once, then the env's waves write the cells, the
// ignited one among them.
template <int kWaves>
__global__ __launch_bounds__(64 * kRlWaves) void rl_reset_kernel(const EnvDev* __restrict__ envs, int32_t n_env,
                                                       const uint8_t* __restrict__ cls,
                                                       uint32_t unburnable_mask,
                                                       uint8_t* __restrict__ states, RlAgent* __restrict__ agents,
                                                       const int32_t* __restrict__ reset_mask, uint2 key,
                                                       uint64_t episode, int32_t water)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = blockIdx.x * (kRlWaves / kWaves) + wv / kWaves;
    const int me = 64 * (wv % kWaves) + lane;  // of the env's 64 kWaves lanes
    if (e >= n_env || (reset_mask && reset_mask[e] == 0)) return;
    const EnvDev ed = envs[e];
    const int64_t n = (int64_t)ed.H * ed.W;
    static_assert(kRlIgnitionAttempts <= 64, "one lane per attempt");
    const uint4 w = philox4x32_10(make_uint4(ed.env_id, (uint32_t)episode, (uint32_t)(episode >> 32),
                                             0x80000000u | (uint32_t)lane),
                                  key);
    const int32_t row = scale_draw(w.x, ed.H), col = scale_draw(w.y, ed.W);
    int64_t cell = (int64_t)row * ed.W + col;
    const bool burns = lane < (int)kRlIgnitionAttempts && !((unburnable_mask >> cls[ed.offset + cell]) & 1u);
    const uint64_t hits = __ballot(burns);
    const int first = hits ? __ffsll((unsigned long long)hits) - 1 : 0;
    // the first attempt on a burnable cell (at most 2^30 cells per env)
    const int32_t ignited = hits ? __builtin_amdgcn_readlane((int)cell, first) : -1;
    auto fresh = [&](uint32_t c, int64_t i) -> uint32_t {
        if (i == ignited) return kBurning;
        return ((unburnable_mask >> c) & 1u) ? kUnburnable : kFlammable;
    };
    // (the handle's classes start on a 4-byte boundary, the caller's states need not)
    if (((ed.offset | n | (int64_t)(uintptr_t)states) & 3) == 0) {
        const uint32_t* c4 = reinterpret_cast<const uint32_t*>(cls + ed.offset);
        uint32_t* s4 = reinterpret_cast<uint32_t*>(states + ed.offset);
        for (int64_t i = me; i < (n >> 2); i += 64 * kWaves) {
            const uint32_t c = c4[i];
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) v |= fresh((c >> (8 * b)) & 0xFFu, 4 * i + b) << (8 * b);
            s4[i] = v;
        }
    } else {
        for (int64_t i = me; i < n; i += 64 * kWaves) states[ed.offset + i] = (uint8_t)fresh(cls[ed.offset + i], i);
    }
    if (me != 0) return;
    RlAgent a{};
    a.row = scale_draw(w.z, ed.H);
    a.col = scale_draw(w.w, ed.W);
    a.water = water;
    agents[e] = a;
}

__global__ __launch_bounds__(256) void rl_act_kernel(const EnvDev* __restrict__ envs, RlAgent* __restrict__ agents,
                                                     const int32_t* __restrict__ actions,
                                                     int32_t* __restrict__ drop_row, int32_t n_env)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_env) return;
    RlAgent a = agents[e];
    int32_t drop = -1;
    if (!a.done) {
        const int32_t act = actions[e];
        const int32_t move = (act >= 0 && act < 32) ? (act & 15) : 0;
        const bool valve = act >= 0 && act < 32 && ((act >> 4) & 1);
        if (move >= 1 && move <= 8) {
            const EnvDev ed = envs[e];
            a.row = min(max(a.row + kDRow[move - 1], 0), ed.H - 1);
            a.col = min(max(a.col + kDCol[move - 1], 0), ed.W - 1);
        }
        if (valve && a.water > 0) {
            drop = (a.row << 16) | a.col;
            a.water -= 1;
        }
        agents[e] = a;
    }
    drop_row[e] = drop;
}

// counts == nullptr: observation only (after a reset), reward 0.
// kWaves waves per env, kRlWaves waves per workgroup.
template <int kWaves>
__global__ __launch_bounds__(64 * kRlWaves) void rl_obs_kernel(const EnvDev* __restrict__ envs, int32_t n_env,
                                                     const uint8_t* __restrict__ states,
                                                     RlAgent* __restrict__ agents,
                                                     const int32_t* __restrict__ counts, RlConfigDev cfg,
                                                     uint8_t* __restrict__ obs, float* __restrict__ reward,
                                                     int32_t* __restrict__ done)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = blockIdx.x * (kRlWaves / kWaves) + wv / kWaves;
    const int me = 64 * (wv % kWaves) + lane;  // of the env's 64 kWaves lanes
    static_assert(kWaves == 1 || kWaves == kRlWaves, "a barrier of the env's waves is one of the workgroup");
    if (e >= n_env) return;
    const EnvDev ed = envs[e];
    RlAgent a = agents[e];
    if (kWaves > 1) __syncthreads();  // every wave has the agent as it was
    float r = 0.0f;
    if (counts && !a.done) {
        const int32_t c = counts[e];
        r = -cfg.burn_penalty * (float)c;
        if (c == 0) r = r + cfg.extinguish_bonus;
        a.steps += 1;
        a.last_count = c;
        a.done = (c == 0 || a.steps >= cfg.max_steps) ? 1 : 0;
        if (me == 0) agents[e] = a;
    }
    if (me == 0) {
        if (reward) reward[e] = r;
        if (done) done[e] = a.done;
    }
    const int R = cfg.obs_radius, side = 2 * R + 1, n = side * side;
    const float inv_side = 1.0f / (float)side;
    uint8_t* o = obs + (int64_t)e * n;
    for (int i = me; i < n; i += 64 * kWaves) {
        const int di = small_div(i, side, inv_side);
        const int gi = a.row - R + di, gj = a.col - R + (i - di * side);
        o[i] = (gi >= 0 && gi < ed.H && gj >= 0 && gj < ed.W) ? states[ed.offset + (int64_t)gi * ed.W + gj]
                                                              : kOutside;
    }
}

// One whole RL step, one env per wave (up to kRlWaves envs per workgroup):
// the agent's move and water drop, the fire step (same per-cell pieces,
// counters and operation order as the step kernels, hence the same bits), the
// BURNING count, reward and done, and the observation window.  The waves of a
// workgroup never wait for each other.
//
// An env with no BURNING cell cannot change (fire only spreads from burning
// cells, and water only removes it): its wave reads the state, the agent and
// the window, and touches no LDS.  A burning env goes to LDS as bit planes F
// and B (wave_words words per wave, the new state beside them); each lane
// works out 4-cell groups, with a front cell's rates from the table.
//
// What bounds it: the chain of dependent loads of each wave and, with most
// fires out, the launch of the waves.  65536 envs of 20 x 20, rollout of 50
// steps: one env per 64-lane workgroup, byte states and exponentials worked out
// per step 65 us per step, now 41 us (a call of the reset included).
template <int RATES>
__global__ __launch_bounds__(64 * kRlWaves) void rl_step_kernel(
    const EnvDev* __restrict__ envs, int32_t n_env, StaticFields F0, StepArgs A, const float4* __restrict__ phi,
    uint8_t* __restrict__ states, RlAgent* __restrict__ agents, const int32_t* __restrict__ actions, RlConfigDev cfg,
    uint32_t t, uint32_t keep_below, int32_t wave_words, uint8_t* __restrict__ obs, float* __restrict__ reward,
    int32_t* __restrict__ done)
{
    extern __shared__ uint4 lds_dyn[];
    __shared__ float s_ew[kRlWaves][8];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = blockIdx.x * (blockDim.x >> 6) + wv;
    if (e >= n_env) return;  // (no workgroup barrier below)
    const EnvDev ed = envs[e];
    RlAgent a = agents[e];
    const int32_t act = actions[e];
    const int H = ed.H, W = ed.W, WD = W >> 2, n_dw = H * WD;
    const float inv_wd = 1.0f / (float)WD;
    const int64_t base = ed.offset;

    // -- 1. the state; the agent's action (every lane alike)
    uint32_t* const st = reinterpret_cast<uint32_t*>(states + base);
    constexpr int kKeep = 2;  // dwords kept in registers; further ones are read again
    uint32_t kept[kKeep];
    uint32_t any_burn = 0;
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
        const int i = 64 * k + lane;
        kept[k] = i < n_dw ? st[i] : 0u;
        any_burn |= burning_flags(kept[k]);
    }
    for (int i = 64 * kKeep + lane; i < n_dw; i += 64) any_burn |= burning_flags(st[i]);
    bool drop = false;
    int drop_r = 0, drop_c = 0;  // centre of the drop, a cell of the env
    if (!a.done) {
        const int32_t move = (act >= 0 && act < 32) ? (act & 15) : 0;
        const bool valve = act >= 0 && act < 32 && ((act >> 4) & 1);
        if (move >= 1 && move <= 8) {
            a.row = min(max(a.row + kDRow[move - 1], 0), H - 1);
            a.col = min(max(a.col + kDCol[move - 1], 0), W - 1);
        }
        if (valve && a.water > 0) {
            // as in a row of drops: one that lies outside the grid (the agents
            // are the caller's to set) spends its water and wets nothing
            const int32_t code = (int32_t)(((uint32_t)a.row << 16) | (uint32_t)a.col);
            drop_r = (code >> 16) & 0x7FFF;
            drop_c = code & 0xFFFF;
            drop = code >= 0 && drop_r < H && drop_c < W;
            a.water -= 1;
        }
    }
    const bool quiet = !__any(any_burn != 0u);
    int32_t count = 0;  // BURNING cells after the step
    const int WW = (W + 31) >> 5, S = WW + 1, fw = (H + 2) * S + 1;
    uint32_t* const pF = reinterpret_cast<uint32_t*>(lds_dyn) + wv * wave_words;
    uint32_t* const pB = pF + fw;
    uint32_t* const sN = pB + fw;  // the new state, dense
    if (!quiet) {
        // -- 2. the planes
        for (int i = lane; i < 2 * fw; i += 64) pF[i] = 0u;
        if (RATES == kRatesEnvWind && lane < 8) {
            float V = ed.V, Vx = ed.Vx, Vy = ed.Vy;
            if (F0.env_wind) {
                const float* w = F0.env_wind + ((int64_t)t * F0.n_env + e) * 3;
                V = w[0];
                Vx = w[1];
                Vy = w[2];
            }
            s_ew[wv][lane] = wind_exponent(lane, A.alpha_w1, A.alpha_w2, V, Vx, Vy);
        }
        wave_sync();
        auto own = [&](int k, int i) { return k == 0 ? kept[0] : (k == 1 ? kept[1] : (i < n_dw ? st[i] : 0u)); };
        for (int k = 0; 64 * k < n_dw; ++k) {
            const int i = 64 * k + lane;
            const uint32_t w = own(k, i);
            const uint32_t f = pack4(flammable_flags(w)), b = pack4(burning_flags(w));
            const int r = small_div(i, WD, inv_wd), g = i - r * WD;
            const int at = (r + 1) * S + 1 + (g >> 3), sh = 4 * (g & 7);
            if (f) atomicOr(&pF[at], f << sh);
            if (b) atomicOr(&pB[at], b << sh);
        }
        wave_sync();
        if (drop) {  // water on F_t: BURNING cells of the square go out
            const int R = A.drop_radius;
            const int r0 = max(drop_r - R, 0), r1 = min(drop_r + R, H - 1);
            const int c0 = max(drop_c - R, 0), c1 = min(drop_c + R, W - 1);
            const int wa = c0 >> 5, nw = (c1 >> 5) - wa + 1;
            for (int q = lane; q < (r1 - r0 + 1) * nw; q += 64) {
                const int w = wa + q % nw;
                pB[(r0 + q / nw + 1) * S + 1 + w] &= ~column_mask(w, c0, c1 + 1);
            }
            wave_sync();
        }

        // -- 3. draws, survivals and ignitions, one 4-cell group per lane
        const uint2 key = make_uint2(A.key0, A.key1);
        StaticFields F = F0;
        if (RATES == kRatesCellWind && F0.wind_stride != 0) F.wind = F0.wind + (int64_t)t * F0.wind_stride;
        uint2* const wl = reinterpret_cast<uint2*>(pF + wave_words - 2 * kRlWaveList);  // (without the table)
        int wn = 0;
        auto eval = [&](int n) {  // the last n (<= 64) front cells of the list
            wave_sync();
            bool ign = false;
            if (lane < n) {
                const uint2 c = wl[wn - n + lane];
                const float p = ignite_prob<RATES == kRatesCellWind>(c.x >> 16, base + (c.x & 0xFFFFu), W, F, A, s_ew[wv]);
                ign = word_to_uniform(c.y) < p;
                if (ign) reinterpret_cast<uint8_t*>(sN)[c.x & 0xFFFFu] = kBurning;
            }
            count += __popcll(__ballot(ign));
            wn -= n;
            wave_sync();
        };
        for (int k = 0; 64 * k < n_dw; ++k) {
            const int i = 64 * k + lane;
            const bool on = i < n_dw;
            const uint32_t w = own(k, i);
            const int r = on ? small_div(i, WD, inv_wd) : 0, g = on ? i - r * WD : 0;
            const int at = (r + 1) * S + 1 + (g >> 3), sh = 4 * (g & 7);
            // the 6 columns from one left of the group lie in its word and the
            // next one on that side
            const uint32_t* p = pB + at - (sh == 0 ? 1 : 0);
            auto window = [&](const uint32_t* q) {
                return __builtin_amdgcn_alignbit(q[1], q[0], (sh - 1) & 31) & 0x3Fu;
            };
            const uint32_t up6 = window(p - S), md6 = window(p), dn6 = window(p + S);
            const uint32_t ud = up6 | dn6;
            const uint32_t burn = (md6 >> 1) & 0xFu;
            const uint32_t front =
                pack4(flammable_flags(w)) & (ud | (ud >> 1) | (ud >> 2) | md6 | (md6 >> 2)) & 0xFu;
            uint32_t next = 0;  // its cells that burn after the step
            uint4 rnd = make_uint4(0u, 0u, 0u, 0u);
            if (on && (burn | front)) {
                float4 ra[4], rb[4];
                float gv[4];
                if constexpr (RATES == kRatesTable) {
                    const float4* ph = phi + 2 * (base + 4 * i);
                    const float* pg = F.g + base + 4 * i;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        ra[c] = rb[c] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        gv[c] = 0.0f;
                        if ((front >> c) & 1u) {
                            ra[c] = ph[2 * c];
                            rb[c] = ph[2 * c + 1];
                            gv[c] = pg[c];
                        }
                    }
                }
                rnd = group_words<true>(4 * i, t, ed.env_id, key);  // 4 i = r W + 4 g
                next = burn & ((rnd.x >> 8 < keep_below ? 1u : 0u) | (rnd.y >> 8 < keep_below ? 2u : 0u) |
                               (rnd.z >> 8 < keep_below ? 4u : 0u) | (rnd.w >> 8 < keep_below ? 8u : 0u));
                if constexpr (RATES == kRatesTable) {
                    uint32_t ign = 0;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t win = ((up6 >> c) & 7u) | (((md6 >> c) & 7u) << 3) | (((dn6 >> c) & 7u) << 6);
                        const float lambda = rate_sum(ra[c], rb[c], win);
                        const float q = 1.0f - exp_c(-((A.alpha_gamma * gv[c]) * lambda));
                        ign |= word_to_uniform(compu(rnd, c)) < (lambda > 0.0f ? q : 0.0f) ? 1u << c : 0u;
                    }
                    next |= ign & front;
                }
            }
            // BURNING (10): stays, or BURNT (11), as where the drop put it out;
            // FLAMMABLE (01) that ignites: BURNING
            const uint32_t was = burning_flags(w), will = spread4(next);
            const uint32_t fresh = will & ~was;
            const uint32_t out = (w | (was & ~will)) ^ (fresh * 3u);
            if (on) sN[i] = out;
            if (RATES == kRatesTable && on && out != w) st[i] = out;
#pragma unroll
            for (int c = 0; c < 4; ++c) count += __popcll(__ballot((next >> c) & 1u));
            if constexpr (RATES != kRatesTable) {
                const bool last = 64 * (k + 1) >= n_dw;
#pragma unroll 1
                for (int c = 0; c < 4; ++c) {
                    const bool is_front = on && ((front >> c) & 1u);
                    const uint64_t m = __ballot(is_front);
                    if (is_front)
                        wl[wn + lanes_below(m)] = make_uint2((uint32_t)(4 * i + c) | (direction_mask(up6, md6, dn6, c) << 16),
                                                             compu(rnd, c));
                    wn += __popcll(m);
                    const int full = last && c == 3 ? 1 : 64;
                    while (wn >= full) eval(min(wn, 64));
                }
            }
        }
        wave_sync();
        if constexpr (RATES != kRatesTable)
            for (int i = lane; i < n_dw; i += 64) st[i] = sN[i];
    }

    // -- 4. reward and done from the count
    float rw = 0.0f;
    if (!a.done) {
        rw = -cfg.burn_penalty * (float)count;
        if (count == 0) rw = rw + cfg.extinguish_bonus;
        a.steps += 1;
        a.last_count = count;
        a.done = (count == 0 || a.steps >= cfg.max_steps) ? 1 : 0;
    }
    if (lane == 0) {
        agents[e] = a;
        reward[e] = rw;
        done[e] = a.done;
    }

    // -- 5. the observation window
    const int R = cfg.obs_radius, side = 2 * R + 1, n_obs = side * side;
    const float inv_side = 1.0f / (float)side;
    uint8_t* o = obs + (int64_t)e * n_obs;
    const uint8_t* seen = quiet ? states + base : reinterpret_cast<const uint8_t*>(sN);
    for (int i = lane; i < n_obs; i += 64) {
        const int di = small_div(i, side, inv_side);
        const int gi = a.row - R + di, gj = a.col - R + (i - di * side);
        o[i] = (gi >= 0 && gi < H && gj >= 0 && gj < W) ? seen[gi * W + gj] : kOutside;
    }
}

}  // namespace

hipError_t launch_rl_step_fused(hipStream_t s, const EnvDev* envs, int32_t n_env, const StaticFields& F,
                                const StepArgs& A, const RlFusedShape& shape, const float* phi, uint8_t* states,
                                RlAgent* agents, const int32_t* actions, const RlConfigDev& cfg, uint32_t t,
                                uint8_t* obs, float* reward, int32_t* done)
{
    if (n_env <= 0) return hipSuccess;
    if (!shape.fits) return hipErrorInvalidValue;
    // two planes and the new state per wave, and the list where rates are worked out
    const int32_t words = 2 * shape.plane_words + shape.cell_cap / 4;
    const int32_t wave_words = ((phi ? words : words + 2 * kRlWaveList) + 3) & ~3;
    const int waves = std::max(1, std::min<int>(kRlWaves, (int)(kRlFusedMaxLds / (4 * (size_t)wave_words))));
    const size_t lds = 4 * (size_t)wave_words * (size_t)waves;
    if (lds > kRlFusedMaxLds) return hipErrorInvalidValue;
    const dim3 grid((n_env + waves - 1) / waves), block(64 * waves);
    const float4* table = reinterpret_cast<const float4*>(phi);
    const uint32_t keep = keep_threshold(A.p_continue);
#define RL_LAUNCH(RT)                                                                                                \
    hipLaunchKernelGGL((rl_step_kernel<RT>), grid, block, lds, s, envs, n_env, F, A, table, states, agents, actions, \
                       cfg, t, keep, wave_words, obs, reward, done)
    if (phi) RL_LAUNCH(kRatesTable);
    else if (F.wind) RL_LAUNCH(kRatesCellWind);
    else RL_LAUNCH(kRatesEnvWind);
#undef RL_LAUNCH
    return hipGetLastError();
}

hipError_t launch_rl_reset(hipStream_t s, const EnvDev* envs, int32_t n_env, const uint8_t* cls,
                           uint32_t unburnable_mask, uint8_t* states, RlAgent* agents,
                           const int32_t* reset_mask, uint32_t key0, uint32_t key1, uint64_t episode,
                           int32_t water, int64_t n_cells)
{
    if (n_env <= 0) return hipSuccess;
    const bool large = n_cells > kRlLargeCells * n_env;
    auto kernel = large ? rl_reset_kernel<kRlWaves> : rl_reset_kernel<1>;
    const int grid = large ? n_env : (n_env + kRlWaves - 1) / kRlWaves;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * kRlWaves), 0, s, envs, n_env, cls, unburnable_mask, states,
                       agents, reset_mask, make_uint2(key0, key1), episode, water);
    return hipGetLastError();
}

hipError_t launch_rl_act(hipStream_t s, const EnvDev* envs, int32_t n_env, RlAgent* agents,
                         const int32_t* actions, int32_t* drop_row)
{
    if (n_env <= 0) return hipSuccess;
    hipLaunchKernelGGL(rl_act_kernel, dim3((n_env + 255) / 256), dim3(256), 0, s, envs, agents, actions,
                       drop_row, n_env);
    return hipGetLastError();
}

hipError_t launch_rl_obs(hipStream_t s, const EnvDev* envs, int32_t n_env, const uint8_t* states,
                         RlAgent* agents, const int32_t* counts, const RlConfigDev& cfg, uint8_t* obs,
                         float* reward, int32_t* done)
{
    if (n_env <= 0) return hipSuccess;
    const int side = 2 * cfg.obs_radius + 1;
    const bool large = side * side > kRlLargeWindow && n_env <= kRlLargeWindowEnvs;
    auto kernel = large ? rl_obs_kernel<kRlWaves> : rl_obs_kernel<1>;
    const int grid = large ? n_env : (n_env + kRlWaves - 1) / kRlWaves;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * kRlWaves), 0, s, envs, n_env, states, agents, counts, cfg, obs,
                       reward, done);
    return hipGetLastError();
}

}  // namespace firesim
