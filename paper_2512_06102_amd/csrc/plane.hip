// plane.hip -- many stochastic steps per launch on bit planes held in LDS.
//
// One workgroup takes a tile (a whole env where it fits, else a part of one
// with a halo) through all steps of the launch.  The state lives in LDS as
// bit planes, one bit per cell: F (FLAMMABLE), B (BURNING, before and after
// the step) and, where a retardant drop or a history needs it, U
// (UNBURNABLE); a cell in none of them is BURNT, or what the source buffer
// says.  A 256 x 256 env takes 9.3 KB per plane.
//
// Every step is the one of the step kernels (the paper's section 3, Eqs. 1-4
// and the "Stochastic update"), with their counters and fp32 operation order,
// so the results are bit-identical:
//  1. The words of the region are scanned 32 cells at a time: front = F and
//     (B of the 3 x 3 neighbourhood), need = front or B.  The 4-cell groups
//     with a needed cell are listed in LDS by the whole workgroup; B of the
//     next step is cleared.
//  2. The lanes share the list, one group each: a Philox block, the burning
//     cells' survival and the front cells' ignitions, and the group's bits of
//     the next B.  A front cell's rates come from the table phi[cell][8] (32
//     bytes, the same for every step under static wind), so its probability
//     costs two 16-byte loads (on their way during the Philox block), eight
//     masked adds and one exponential.  Under a wind series, or without the
//     table, the front cells go to the wave's own short list, 64 of which are
//     evaluated at a time.
// Two barriers per step (three with a drop; one less where a region is small
// enough for one group per lane, and is not scanned).  No state goes to memory
// between the steps of a launch.
//
// What bounds it: the chain of a step (LDS round trips, one Philox block, one
// table load, one exponential, the barriers; 4000 to 10000 cycles at one
// workgroup per compute unit), the instructions of the lanes that have little
// to do while the fires burn, and the longest fire of a launch (at 1024 envs of
// 256 x 256 the compute units are busy 57% of it; one env alone takes half its
// time), not memory.  Measured against one launch per step over 64-lane tiles
// (the other step kernel): 1024 envs of 256 x 256, 200 steps, 11.4 -> 2.4 ms;
// 1024 envs of 64 to 512 squared with a drop per step, 300 steps, 18.6 -> 6.1
// ms (its two launches beside each other; 7.6 in order); 8 envs of 2048 x 2048
// with per-cell wind, 1000 steps, 27.9 -> 6.0 ms (parts of 64 x 128 with 24
// steps of halo; 0.6 ms more with 12 steps, 1.7 ms more with 128 x 128).
// Against one workgroup per env with byte states and the exponentials worked
// out per step: 64 envs of 64 x 64, 200 steps, 463 -> 268 us.
//
// With a halo the region is the tile and `steps` rows and 32 columns around
// it; a step works out the cells that the tile's last step still depends on.
#include <type_traits>

#include "bitplane.hpp"
#include "devmath.hpp"
#include "framed.hpp"
#include "internal.hpp"
#include "plane.hpp"
#include "stepcell.hpp"

namespace firesim {
namespace {

constexpr int kScanRows = 4;     // rows scanned between two listings
constexpr int kSmallRounds = 1;  // a region of up to so many groups per lane is not scanned
constexpr int kDeal = 16;        // listed groups a wave takes at a time, without the table

constexpr int32_t kPartRun = 1, kPartRan = 2;  // marks of a part for the next launch

// Workgroup barrier that orders LDS only: stores to memory stay in flight
// (__syncthreads waits for them, about 1000 cycles with a count stored in the
// step before).  The wait for the wave's own LDS operations is explicit: a
// fence on local memory alone emits none, and an add without a result was
// still on its way when another wave read the sum behind the barrier.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Adds x to a word of LDS that every lane names alike, and returns what was
// there.  The address is hidden from the compiler, which would otherwise
// gather the lanes' values in a scalar loop (2500 cycles for 64 lanes, about
// 200 for the conflict in LDS).
__device__ __forceinline__ uint32_t lds_add(uint32_t* p, uint32_t x)
{
    uint32_t i = 0;
    asm volatile("" : "+v"(i));
    return atomicAdd(p + i, x);
}

struct PlaneArgs {
    const PlaneTile* tiles;
    int32_t n_tiles, frame_words, list_cap, has_u;
    const EnvDev* envs;
    int32_t n_env;
    StaticFields F;
    StepArgs A;
    const float4* phi;
    const uint8_t* src;
    uint8_t* dst;
    const uint32_t* t_base;
    uint32_t step0;
    int32_t steps;
    const int32_t* actions;
    int32_t* counts;
    uint8_t* history;
    PlaneParts parts;
    uint32_t keep_below;  // a BURNING cell stays when its 24-bit draw is below this
};

// Waves per SIMD the kernel is compiled for: with the table 80 VGPRs fit
// without a spill (64 spill, and 1024 envs of 256 x 256 run 4% slower).
constexpr int plane_waves_per_eu(int rates) { return rates == kRatesTable ? 6 : 4; }

template <int NT, bool ALIGNED, int RATES, bool HALO>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(plane_waves_per_eu(RATES)))) void stoch_plane_kernel(
    PlaneArgs K)
{
    constexpr int NW = NT / 64;
    // A call of few steps on a small env is little more than its start.  The
    // aligned whole envs therefore start briskly: the env's entry comes with the
    // tile, the first cells are on their way while the planes are cleared, and the
    // lanes' shares take no run-time divisions (64 envs of 64 x 64, 1 step: 10.2 ->
    // 9.5 us).  The variants that have no registers to spare lose more by it (8
    // envs of 2048 x 2048 in parts 1 to 5%).
    constexpr bool kBrisk = ALIGNED && !HALO;
    extern __shared__ uint4 lds_dyn[];
    __shared__ float s_ew[RATES == kRatesEnvWind ? kPlaneChunk : 1][8];
    __shared__ int32_t s_act[kPlaneChunk];
    __shared__ uint32_t s_n[2];               // groups listed in step s, slot s % 2
    // BURNING cells worked out in step s, slot s % 3: step s reads the slot of
    // step s - 1, adds to its own and clears that of step s + 1, which no wave
    // reads or adds to between two openings of a step.  (A small region has no
    // other barrier in a step: of two slots, the clear could meet the adds.)
    __shared__ uint32_t s_all[3];
    __shared__ uint32_t s_tile[kPlaneChunk];  // those of the tile itself, slot s % kPlaneChunk
    __shared__ int32_t s_run;

    // whole envs, and parts on a call's first launch, in the order of the tile
    // list: neighbouring tiles (and the larger envs at the head of the list)
    // spread over the XCDs, as a step's work follows the fire.  Later launches
    // take the parts that the one before put on the next list, so that the
    // parts with fire spread evenly over the compute units.
    int tix = blockIdx.x;
    if (HALO) {
        if (K.parts.n_clear && blockIdx.x == 0 && threadIdx.x == 0) *K.parts.n_clear = 0;
        if (K.parts.list) {
            if (tix >= *K.parts.n_list) return;
            tix = K.parts.list[tix];
        }
    }
    const PlaneTile td = K.tiles[tix];
    const EnvDev ed = kBrisk ? td.dev : K.envs[td.env];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = ed.H, W = ed.W;
    const int64_t base = ed.offset;
    // region: rows [q0, q0 + RH), columns [p0, p0 + RC) of the env; the tile
    // is rows [tr0, tr1), columns [tc0, tc1) of the region
    const int hk = HALO ? K.steps : 0, hc = HALO ? kPlaneHaloCols : 0;
    const int q0 = max(td.r0 - hk, 0), RH = min(td.r0 + td.rows + hk, H) - q0;
    const int p0 = max(td.c0 - hc, 0), RC = min(td.c0 + td.cols + hc, W) - p0;
    const int tr0 = td.r0 - q0, tr1 = tr0 + td.rows, tc0 = td.c0 - p0, tc1 = tc0 + td.cols;
    const int WW = (RC + 31) >> 5, S = WW + 1;       // words per row, row stride
    const int G = (RC + 3) >> 2;                     // 4-cell groups per row
    const int gshift = 32 - __clz(8 * WW - 1);       // group id: row << gshift | group column

    // -- sparse scheduling of parts: a part runs when it or a neighbouring one
    //    still burnt after the previous launch, when a drop may touch its
    //    region, or on the first launch of a call; one that ran in the
    //    previous launch and does not in this one copies its cells over
    if (HALO) {
        if (tid == 0) {
            s_run = K.parts.first ? kPartRun : K.parts.mark[tix];
            K.parts.mark[tix] = 0;
        }
        __syncthreads();
        if (K.actions)
            for (int j = tid; j < K.steps; j += NT) {
                const int32_t a = K.actions[(int64_t)j * K.n_env + td.env];
                const int ar = (a >> 16) & 0x7FFF, ac = a & 0xFFFF, R = K.A.drop_radius;
                if (a >= 0 && ar < H && ac < W && ar + R >= q0 && ar - R < q0 + RH && ac + R >= p0 &&
                    ac - R < p0 + RC)
                    atomicOr(&s_run, kPartRun);
            }
        __syncthreads();
        const int32_t run = s_run;
        if (!(run & kPartRun)) {
            if (run & kPartRan)
                for (int r = wv; r < td.rows; r += NW)
                    for (int c = lane; c < td.cols; c += 64) {
                        const int64_t i = base + (int64_t)(td.r0 + r) * W + td.c0 + c;
                        K.dst[i] = K.src[i];
                    }
            return;
        }
    }

    // the wave's front cells (without the table), then the planes
    uint2* const wl = reinterpret_cast<uint2*>(lds_dyn) + wv * kPlaneWaveList;
    uint32_t* const pF = reinterpret_cast<uint32_t*>(reinterpret_cast<uint2*>(lds_dyn) +
                                                     (RATES == kRatesTable ? 0 : NW * kPlaneWaveList));
    uint32_t* cur = pF + K.frame_words;
    uint32_t* nxt = cur + K.frame_words;
    uint32_t* const pU = nxt + K.frame_words;
    uint16_t* const list = reinterpret_cast<uint16_t*>(pF + (3 + (HALO ? K.has_u : 0)) * K.frame_words);

    // how the lanes share the cells (the store at the end keeps its divisions, and
    // the first drops and wind wait for the planes: 200 steps of 64 envs of 64 x
    // 64 took 274 and 278 us otherwise, now 270)
    auto share = [&](int q, int d, float inv_d) { return kBrisk ? small_div(q, d, inv_d) : q / d; };
    const float inv_g = 1.0f / (float)G;
    const int g_step = G <= NT ? G : NT, g_rows = G <= NT ? share(NT, G, inv_g) : 1;
    const int my_gr = G <= NT ? share(tid, G, inv_g) : 0, my_g = tid - my_gr * G;
    auto load4 = [&](const uint8_t* p, int col) -> uint32_t {
        if constexpr (ALIGNED) {
            return *reinterpret_cast<const uint32_t*>(p);
        } else {
            uint32_t v = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < W) v |= (uint32_t)p[c] << (8 * c);
            return v;
        }
    };
    // this lane's first group
    uint32_t w_first = 0;
    if (kBrisk && my_gr < g_rows && my_g < G && my_gr < RH)
        w_first = load4(K.src + base + (uint32_t)((q0 + my_gr) * W + p0 + 4 * my_g), p0 + 4 * my_g);

    const uint32_t t0 = *K.t_base + K.step0;
    const bool ew_series = RATES == kRatesEnvWind && K.F.env_wind != nullptr;
    if (RATES == kRatesEnvWind && !ew_series && tid < 8)
        s_ew[0][tid] = wind_exponent(tid, K.A.alpha_w1, K.A.alpha_w2, ed.V, ed.Vx, ed.Vy);

    // -- planes cleared (frames included), then filled from the source bytes
    for (int i = tid; i < (3 + (HALO ? K.has_u : 0)) * K.frame_words; i += NT) pF[i] = 0u;
    if (tid < 2) s_n[tid] = 0u;
    if (tid < 3) s_all[tid] = 0u;
    if (tid < kPlaneChunk) s_tile[tid] = 0u;
    __syncthreads();
    {
        uint32_t any = 0;
        if (my_gr < g_rows)
            for (int g = my_g; g < G; g += g_step)
                for (int r = my_gr; r < RH; r += g_rows) {
                    const int col = p0 + 4 * g;
                    const uint32_t w = kBrisk && g == my_g && r == my_gr
                                           ? w_first
                                           : load4(K.src + base + (uint32_t)((q0 + r) * W + col), col);
                    const uint32_t f = pack4(flammable_flags(w)), bu = pack4(burning_flags(w));
                    const int at = (r + 1) * S + 1 + (g >> 3), sh = 4 * (g & 7);
                    if (f) atomicOr(&pF[at], f << sh);
                    if (bu) atomicOr(&cur[at], bu << sh);
                    if (HALO && K.has_u) {
                        uint32_t u = ~pack4((w | (w >> 1)) & 0x01010101u) & 0xFu;
                        if (!ALIGNED && col + 3 >= W) u &= (1u << (W - col)) - 1u;
                        if (u) atomicOr(&pU[at], u << sh);
                    }
                    any |= bu;
                }
        if (any) s_all[2] = 1u;  // read by step 0: does anything burn?
    }

    // bytes of the 4 cells of group g in row r
    auto state4 = [&](int r, int g) -> uint32_t {
        const int at = (r + 1) * S + 1 + (g >> 3), sh = 4 * (g & 7);
        const uint32_t f = pF[at] >> sh, bu = cur[at] >> sh;
        uint32_t z = spread4(~(f | bu));
        if (HALO && K.has_u) {
            z &= ~spread4(pU[at] >> sh);
        } else if (z) {
            const int col = p0 + 4 * g;
            const uint32_t w = load4(K.src + base + (uint32_t)((q0 + r) * W + col), col);
            z &= w | (w >> 1);
        }
        return spread4(f) | (spread4(bu) << 1) | (z * 3u);
    };
    // the tile's cells to an array of whole envs
    auto store_tile = [&](uint8_t* out) {
        const int ga = tc0 >> 2, gn = (tc1 - tc0 + 3) >> 2;
        const int st = gn <= NT ? gn : NT, rows = gn <= NT ? NT / gn : 1;
        const int r0 = gn <= NT ? tid / gn : 0, g0 = tid - r0 * gn;
        if (r0 >= rows) return;
        for (int g = g0; g < gn; g += st)
            for (int r = tr0 + r0; r < tr1; r += rows) {
                const int col = p0 + 4 * (ga + g);
                const uint32_t v = state4(r, ga + g);
                uint8_t* o = out + base + (uint32_t)((q0 + r) * W + col);
                if constexpr (ALIGNED) {
                    *reinterpret_cast<uint32_t*>(o) = v;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (col + c < W) o[c] = (uint8_t)(v >> (8 * c));
                }
            }
    };

    const uint2 key = make_uint2(K.A.key0, K.A.key1);
    // scan: lane (word column, strip of rows)
    const float inv_ww = 1.0f / (float)WW;
    const int w_step = WW <= NT ? WW : NT, n_strips = WW <= NT ? share(NT, WW, inv_ww) : 1;
    const int my_strip = WW <= NT ? share(tid, WW, inv_ww) : 0, my_w = tid - my_strip * WW;

    // the counts of `n` steps from step `first` on, and their slots cleared
    auto flush_counts = [&](int32_t first, int32_t n) {
        if (tid >= kPlaneChunk) return;
        const uint32_t c = s_tile[tid];
        s_tile[tid] = 0u;
        if (!K.counts || tid >= n) return;
        int32_t* row = K.counts + (int64_t)(first + tid) * K.n_env + td.env;
        if (!HALO)
            *row = (int32_t)c;
        else if (c)
            atomicAdd(row, (int32_t)c);
    };

    const int per = share(RH + n_strips - 1, n_strips, 1.0f / (float)n_strips);  // rows of a strip
    // groups per row padded to whole words; this lane's first in a dense pass
    const int GW = 8 * WW, dense_r = share(tid, GW, 0.125f * inv_ww), dense_g = tid - dense_r * GW;
    const bool small = !HALO && RH * GW <= kSmallRounds * NT;
    bool quiet = false, stopped = false;
    int32_t s = 0;
    uint32_t s3 = 0;  // s % 3
    for (; s < K.steps; ++s, s3 = s3 == 2 ? 0 : s3 + 1) {
        const uint32_t t = t0 + (uint32_t)s;
        const int kc = s % kPlaneChunk;
        if (kc == 0) {
            if (s > 0) {
                lds_barrier();  // the last chunk's drops and wind are read, its counts summed
                flush_counts(s - kPlaneChunk, kPlaneChunk);
            }
            const int nk = min(kPlaneChunk, K.steps - s);
            if (K.actions)
                for (int j = tid; j < nk; j += NT) s_act[j] = K.actions[(int64_t)(s + j) * K.n_env + td.env];
            if (ew_series)
                for (int q = tid; q < nk * 8; q += NT) {
                    const int j = q >> 3, d = q & 7;
                    const float* w = K.F.env_wind + ((int64_t)(t + j) * K.F.n_env + td.env) * 3;
                    s_ew[j][d] = wind_exponent(d, K.A.alpha_w1, K.A.alpha_w2, w[0], w[1], w[2]);
                }
        }
        lds_barrier();  // F_t complete, the chunk staged, the last step's cells counted
        const uint32_t prev = s_all[s3 == 0 ? 2 : s3 - 1];
        if (tid == 0) {
            s_all[s3 == 2 ? 0 : s3 + 1] = 0u;
            s_n[(s + 1) & 1] = 0u;
        }
        // nothing burns: no cell can ignite or burn out any more, only the
        // drops can still change the state (the remaining counts stay 0)
        quiet = prev == 0u;
        if (K.history && s > 0) {
            store_tile(K.history + (int64_t)(s - 1) * K.F.n_cells);
            // where no scan follows and rows end within a word (they are padded
            // to whole words for the draws, not for the store), another wave may
            // step the groups that this one stores, and would take ignited cells
            // out of F
            if (small && G != GW) lds_barrier();
        }
        if (quiet && !K.actions && !K.history) {
            stopped = true;
            break;
        }
        const int32_t act = K.actions ? s_act[kc] : -1;
        if (act >= 0) {
            const int ar = (act >> 16) & 0x7FFF, ac = act & 0xFFFF;
            if (ar < H && ac < W) {
                if (K.history && s > 0) lds_barrier();  // the last state is read
                const int R = K.A.drop_radius;
                const int ra = max(ar - R - q0, 0), rb = min(ar + R - q0, RH - 1);
                const int ca = max(ac - R - p0, 0), cb = min(ac + R - p0, RC - 1);
                if (ra <= rb && ca <= cb) {
                    const int wa = ca >> 5, nw = (cb >> 5) - wa + 1;
                    for (int q = tid; q < (rb - ra + 1) * nw; q += NT) {
                        const int w = wa + q % nw, at = (ra + q / nw + 1) * S + 1 + w;
                        const uint32_t m = column_mask(w, ca, cb + 1);
                        if (K.A.drop_mode == 0) {
                            uint32_t gone = (pF[at] | cur[at]) & m;
                            if (HALO) {
                                pU[at] |= gone;
                            } else {
                                // a whole env is stepped in place: its bytes say
                                // which cells are UNBURNABLE
                                uint8_t* o = K.dst + base + (uint32_t)((q0 + ra + q / nw) * W + p0 + 32 * w);
                                for (; gone; gone &= gone - 1) o[__ffs(gone) - 1] = kUnburnable;
                            }
                            pF[at] &= ~m;
                        }
                        cur[at] &= ~m;
                    }
                }
                if (K.history)
                    __syncthreads();  // the next history row reads the dropped bytes
                else
                    lds_barrier();
            }
        }
        if (quiet) continue;

        // -- 1. scan: the cells that this step has to work out
        const int left = K.steps - 1 - s;
        const int lo = HALO ? max(tr0 - left, 0) : 0, hi = HALO ? min(tr1 + left, RH) : RH;
        // strips of one row have a scan of their own: it reads 3 rows, not 6
        auto scan = [&](auto rows_at_once) {
            constexpr int ROWS = decltype(rows_at_once)::value;
            const int rs = n_strips * S;
            for (int w0 = 0; w0 < WW; w0 += w_step)
                for (int j = 0; j < per; j += ROWS) {
                    // a lane's word column and rows ra, ra + n_strips, ...: a
                    // fire's rows fall to different lanes and waves (with
                    // neighbouring rows to a lane, one wave lists most of the
                    // groups while the others wait, 2900 of 11500 cycles)
                    const int cw = w0 + my_w, ra = lo + my_strip + j * n_strips;
                    if (my_strip >= n_strips || cw >= WW || ra >= hi) continue;
                    const int at0 = (ra + 1) * S + 1 + cw;
                    uint32_t m[ROWS], h[ROWS], f[ROWS];
                    int at[ROWS];
                    auto reach = [&](const uint32_t* p, uint32_t& mid) {
                        const uint32_t l = p[-1], r = p[1];
                        mid = p[0];
                        // the row's burning cells and their left and right neighbours
                        return mid | __builtin_amdgcn_alignbit(mid, l, 31) | __builtin_amdgcn_alignbit(r, mid, 1);
                    };
#pragma unroll
                    for (int q = 0; q < ROWS; ++q) {
                        at[q] = ra + q * n_strips < hi ? at0 + q * rs : at0;
                        const uint32_t* p = cur + at[q];
                        uint32_t above, below;
                        h[q] = reach(p - S, above) | reach(p, m[q]) | reach(p + S, below);
                        f[q] = pF[at[q]];
                    }
                    const uint32_t mask = HALO ? column_mask(cw, tc0 - left, tc1 + left) : ~0u;
                    uint32_t todo = 0;  // bit 4 b + q: group b of row q has a needed cell
#pragma unroll
                    for (int q = 0; q < ROWS; ++q) {
                        const bool in = ra + q * n_strips < hi;
                        uint32_t need = (f[q] & h[q]) | m[q];
                        if (HALO) need &= mask;
                        if (in) nxt[at[q]] = 0u;
                        uint32_t nz = need | (need >> 1);
                        nz = (nz | (nz >> 2)) & 0x11111111u;
                        todo |= (in ? nz : 0u) << q;
                    }
                    if (todo == 0u) continue;
                    const uint32_t n = (uint32_t)__popc(todo);
                    const uint32_t slot = lds_add(&s_n[s & 1], n);
                    if (slot + n > (uint32_t)K.list_cap) continue;  // (a list that overflows is not read)
                    const uint32_t id0 = ((uint32_t)ra << gshift) | (uint32_t)(8 * cw);
                    const uint32_t id_row = (uint32_t)n_strips << gshift;
                    uint16_t* put = list + slot;
                    for (; todo; todo &= todo - 1) {
                        const uint32_t bit = (uint32_t)__ffs(todo) - 1u;
                        *put++ = (uint16_t)(id0 + (bit & 3u) * id_row + (bit >> 2));
                    }
                }
        };
        if (!small) {
            if (per == 1)
                scan(std::integral_constant<int, 1>{});
            else
                scan(std::integral_constant<int, kScanRows>{});
            lds_barrier();
        }

        // -- 2. draws, survivals and ignitions
        const uint32_t found = small ? 0u : s_n[s & 1];
        // where more groups were found than the list holds, and in small
        // regions, every group of the rows is looked at (row by row, padded to
        // whole words, so that a wave owns the words it writes)
        const bool dense = small || found > (uint32_t)K.list_cap;
        const int n_work = dense ? (hi - lo) * GW : (int)found;
        const float* ew = s_ew[ew_series ? kc : 0];
        StaticFields F = K.F;
        if (RATES == kRatesCellWind && F.wind_stride != 0) F.wind = K.F.wind + (int64_t)t * K.F.wind_stride;
        uint32_t n_all = 0, n_tile = 0;  // this lane's BURNING cells
        int wn = 0;                      // cells in the wave's list (wave-uniform)
        auto inside = [&](int r, int c) { return r >= tr0 && r < tr1 && c >= tc0 && c < tc1; };
        // without the table: evaluate the last n (<= 64) cells of the wave's list
        auto eval = [&](int n) {
            wave_sync();
            if (lane < n) {
                const uint2 e = wl[wn - n + lane];
                const int r = e.x & 0x7FFF, c = (e.x >> 15) & 0x7FFF;
                const uint32_t win = (e.x >> 30) | ((e.y >> 24) << 2);
                const int64_t v = base + (uint32_t)((q0 + r) * W + p0 + c);
                const uint32_t nbk = direction_mask(win & 7u, (win >> 3) & 7u, (win >> 6) & 7u, 0);
                const float p = ignite_prob<RATES == kRatesCellWind>(nbk, v, W, F, K.A, ew);
                if (word_to_uniform(e.y << 8) < p) {
                    const int at = (r + 1) * S + 1 + (c >> 5);
                    atomicOr(&nxt[at], 1u << (c & 31));
                    atomicAnd(&pF[at], ~(1u << (c & 31)));
                    n_all += 1u;
                    if (HALO && inside(r, c)) n_tile += 1u;
                }
            }
            wn -= n;
            wave_sync();
        };
        int rd = lo + dense_r, gd = dense_g;
        // a list is dealt out entry by entry: a short one keeps every wave busy.
        // Without the table a wave evaluates its front cells 64 at a time, at one
        // price for few and many: kDeal entries at a time fill fewer waves (226
        // envs of 136 x 36, 60 steps of a wind series: 315 us one by one, 270 by
        // 8, 252 by 16, 235 by 32; 8 of 100 x 200 328, 325, 332 and 354 us)
        const int n_rounds = (n_work + NT - 1) / NT;
        for (int k = 0; k < n_rounds; ++k) {
            bool on;
            int r, g;
            if (dense) {
                on = rd < hi;
                r = on ? rd : lo;
                g = gd;
                rd += NT / GW;
                gd += NT % GW;
                if (gd >= GW) {
                    gd -= GW;
                    ++rd;
                }
            } else {
                const int i = RATES == kRatesTable ? NW * (64 * k + lane) + wv
                                                   : kDeal * (NW * (64 / kDeal * k + lane / kDeal) + wv) + lane % kDeal;
                on = i < n_work;
                const uint32_t id = on ? list[i] : 0u;
                r = (int)(id >> gshift);
                g = (int)(id & ((1u << gshift) - 1u));
            }
            const int sh = 4 * (g & 7), col = 4 * g;
            const int at = (r + 1) * S + 1 + (g >> 3);
            // the 6 columns from one left of the group lie in its word and the
            // next one on that side
            const uint32_t* p = cur + at - (sh == 0 ? 1 : 0);
            auto window = [&](const uint32_t* q) {
                return __builtin_amdgcn_alignbit(q[1], q[0], (sh - 1) & 31) & 0x3Fu;
            };
            const uint32_t up6 = window(p - S), md6 = window(p), dn6 = window(p + S);
            const uint32_t flam = pF[at] >> sh;
            if (small && on && sh == 0) nxt[at] = 0u;  // (the scan clears it otherwise)
            const uint32_t ud = up6 | dn6;
            const uint32_t front = on ? flam & (ud | (ud >> 1) | (ud >> 2) | md6 | (md6 >> 2)) & 0xFu : 0u;
            const uint32_t burn = on ? (md6 >> 1) & 0xFu : 0u;
            const bool last = k == n_rounds - 1;
            uint4 w = make_uint4(0u, 0u, 0u, 0u);
            if (burn | front) {
                const int n0 = (q0 + r) * W + p0 + col;  // the group's first cell
                uint32_t next = 0;                       // its cells that burn after the step
                float4 ra[4], rb[4];
                float gv[4];
                if constexpr (RATES == kRatesTable) {
                    // the front cells' rates are on their way while the draws are
                    // worked out (those of the other cells are left: at 1024 envs
                    // of 256 x 256 whole 128-byte groups take 3.3 ms for 2.5)
                    const float4* ph = K.phi + 2 * (base + n0);
                    const float* pg = K.F.g + base + n0;
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
                w = group_words<ALIGNED>((int64_t)n0, t, ed.env_id, key);
                next = burn & ((w.x >> 8 < K.keep_below ? 1u : 0u) | (w.y >> 8 < K.keep_below ? 2u : 0u) |
                               (w.z >> 8 < K.keep_below ? 4u : 0u) | (w.w >> 8 < K.keep_below ? 8u : 0u));
                if constexpr (RATES == kRatesTable) {
                    uint32_t ign = 0;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t win = ((up6 >> c) & 7u) | (((md6 >> c) & 7u) << 3) | (((dn6 >> c) & 7u) << 6);
                        const float lambda = rate_sum(ra[c], rb[c], win);
                        const float q = 1.0f - exp_c(-((K.A.alpha_gamma * gv[c]) * lambda));
                        const float pr = lambda > 0.0f ? q : 0.0f;
                        ign |= word_to_uniform(compu(w, c)) < pr ? 1u << c : 0u;
                    }
                    ign &= front;
                    next |= ign;
                    if (ign) atomicAnd(&pF[at], ~(ign << sh));
                }
                if (next) atomicOr(&nxt[at], next << sh);
                n_all += (uint32_t)__popc(next);
                if (HALO && inside(r, col)) n_tile += (uint32_t)__popc(next);  // tile edges are on group edges
            }
            if constexpr (RATES != kRatesTable) {
                // the front cells into the wave's list, two of the group at a time
                if (!__any(front != 0u) && !(last && wn > 0)) continue;
                const uint32_t rc = (uint32_t)r | ((uint32_t)col << 15);
#pragma unroll 1
                for (int h = 0; h < 2; ++h) {
                    const uint32_t fr = front >> (2 * h);
                    const uint64_t m0 = __ballot((fr & 1u) != 0u), m1 = __ballot((fr & 2u) != 0u);
                    const int n0 = __popcll(m0);
                    const uint32_t w9 = ((up6 >> (2 * h)) & 15u) | (((md6 >> (2 * h)) & 15u) << 8) |
                                        (((dn6 >> (2 * h)) & 15u) << 16);
                    auto entry = [&](int c, uint32_t word) {
                        const uint32_t x = w9 >> c;
                        const uint32_t win = (x & 7u) | ((x >> 5) & 0x38u) | ((x >> 10) & 0x1C0u);
                        return make_uint2((rc + ((uint32_t)(2 * h + c) << 15)) | (win << 30),
                                          (word >> 8) | ((win >> 2) << 24));
                    };
                    if (fr & 1u) wl[wn + lanes_below(m0)] = entry(0, h ? w.z : w.x);
                    if (fr & 2u) wl[wn + n0 + lanes_below(m1)] = entry(1, h ? w.w : w.y);
                    wn += n0 + __popcll(m1);
                    const int full = last && h ? 1 : 64;
                    while (wn >= full) eval(min(wn, 64));
                }
            }
        }
        if (n_all) {
            lds_add(&s_all[s3], n_all);
            if (!HALO || n_tile) lds_add(&s_tile[kc], HALO ? n_tile : n_all);
        }
        uint32_t* tmp = cur;
        cur = nxt;
        nxt = tmp;
    }

    if (!HALO && K.actions)
        __syncthreads();  // the dropped bytes are in memory
    else
        lds_barrier();
    if (!stopped && K.history) store_tile(K.history + (int64_t)(K.steps - 1) * K.F.n_cells);
    if (HALO && tid < 9) {
        // the next launch runs this part and its neighbours if it still burns,
        // and else only copies its cells
        const bool burns = !stopped && s_tile[(K.steps - 1) % kPlaneChunk] != 0u;
        const int nb = tid == 0 ? tix : K.parts.nbr[8 * tix + tid - 1];
        const int32_t mark = tid == 0 ? (burns ? kPartRan | kPartRun : kPartRan) : (burns ? kPartRun : 0);
        if (nb >= 0 && mark && atomicOr(&K.parts.mark_next[nb], mark) == 0 && K.parts.list_next)
            K.parts.list_next[atomicAdd(K.parts.n_next, 1)] = nb;
    }
    // the counts not yet written: of the chunk that the loop was left in
    const int32_t taken = stopped ? s : K.steps;
    const int32_t c0 = ((stopped ? s : K.steps - 1) / kPlaneChunk) * kPlaneChunk;
    flush_counts(c0, taken - c0);
    if (stopped && s == 0 && K.src == K.dst) return;  // nothing burnt: the state is as it was
    store_tile(K.dst);
}

// One lane per cell, a workgroup per run of kLossChunk cells of one env.
template <bool WIND_CELL>
__global__ __launch_bounds__(256) void phi_table_kernel(const EnvDev* __restrict__ envs,
                                                        const int32_t* __restrict__ chunk_env, StaticFields F,
                                                        StepArgs A, float4* __restrict__ phi)
{
    __shared__ float ew[8];
    const int ch = blockIdx.x;
    const EnvDev ed = envs[chunk_env[ch]];
    const int H = ed.H, W = ed.W;
    if (!WIND_CELL && threadIdx.x < 8)
        ew[threadIdx.x] = wind_exponent(threadIdx.x, A.alpha_w1, A.alpha_w2, ed.V, ed.Vx, ed.Vy);
    __syncthreads();
    const int64_t n = (int64_t)H * W, first = (int64_t)(ch - ed.chunk0) * kLossChunk;
    const int64_t last = min(first + (int64_t)kLossChunk, n);
    for (int64_t i = first + threadIdx.x; i < last; i += 256) {
        const int r = (int)i / W, c = (int)i - r * W;
        const int64_t v = ed.offset + i;
        const float E_v = F.E[v];
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int ur = r - kDRow[k], uc = c - kDCol[k];
            x[k] = 0.0f;
            if (ur < 0 || ur >= H || uc < 0 || uc >= W) continue;
            const int64_t u = v - (int64_t)kDRow[k] * W - kDCol[k];
            float wexp;
            if constexpr (WIND_CELL)
                wexp = wind_exponent(k, A.alpha_w1, A.alpha_w2, F.wind[u], F.wind[F.n_cells + u],
                                     F.wind[2 * F.n_cells + u]);
            else
                wexp = ew[k];
            x[k] = edge_rate(k, wexp, F.g[u], E_v, F.E[u], A);
        }
        phi[2 * v] = make_float4(x[0], x[1], x[2], x[3]);
        phi[2 * v + 1] = make_float4(x[4], x[5], x[6], x[7]);
    }
}

template <int NT, bool HALO, class Fn>
hipError_t for_kernel(bool aligned, int rates, Fn fn)
{
    if (aligned) {
        if (rates == kRatesTable) return fn(&stoch_plane_kernel<NT, true, kRatesTable, HALO>);
        if (rates == kRatesEnvWind) return fn(&stoch_plane_kernel<NT, true, kRatesEnvWind, HALO>);
        return fn(&stoch_plane_kernel<NT, true, kRatesCellWind, HALO>);
    }
    if (rates == kRatesTable) return fn(&stoch_plane_kernel<NT, false, kRatesTable, HALO>);
    if (rates == kRatesEnvWind) return fn(&stoch_plane_kernel<NT, false, kRatesEnvWind, HALO>);
    return fn(&stoch_plane_kernel<NT, false, kRatesCellWind, HALO>);
}

// fn(kernel) for the instance that a launch takes; hipErrorInvalidValue where there is none.
template <class Fn>
hipError_t with_kernel(int threads, bool halo, bool aligned, int rates, Fn fn)
{
    if (halo) return threads == kPlaneHaloThreads ? for_kernel<kPlaneHaloThreads, true>(aligned, rates, fn) : hipErrorInvalidValue;
    switch (threads) {
    case 64: return for_kernel<64, false>(aligned, rates, fn);
    case 256: return for_kernel<256, false>(aligned, rates, fn);
    case 512: return for_kernel<512, false>(aligned, rates, fn);
    case 1024: return for_kernel<1024, false>(aligned, rates, fn);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_phi_table(hipStream_t s, const EnvDev* envs, const int32_t* chunk_env, int32_t n_chunks,
                            const StaticFields& F, const StepArgs& A, float* phi)
{
    float4* out = reinterpret_cast<float4*>(phi);
    if (F.wind)
        hipLaunchKernelGGL((phi_table_kernel<true>), dim3(n_chunks), dim3(256), 0, s, envs, chunk_env, F, A, out);
    else
        hipLaunchKernelGGL((phi_table_kernel<false>), dim3(n_chunks), dim3(256), 0, s, envs, chunk_env, F, A, out);
    return hipGetLastError();
}

hipError_t plane_set_lds_limit(int bytes)
{
    for (int threads : {64, 256, 512, 1024})
        for (bool halo : {false, true})
            for (bool aligned : {false, true})
                for (int rates : {kRatesTable, kRatesEnvWind, kRatesCellWind}) {
                    if (halo && threads != kPlaneHaloThreads) continue;
                    const hipError_t e = with_kernel(threads, halo, aligned, rates, [&](auto* kernel) {
                        return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
                    });
                    if (e != hipSuccess) return e;
                }
    return hipSuccess;
}

hipError_t launch_stoch_plane(hipStream_t s, const PlaneLaunch& L, const uint8_t* src, uint8_t* dst,
                              const uint32_t* t_base, uint32_t step0, int32_t steps, const int32_t* actions,
                              int32_t* counts, uint8_t* history, const PlaneParts& parts)
{
    if (L.n_tiles < 1 || steps < 1) return hipErrorInvalidValue;
    if (L.halo && (steps > L.halo || L.halo > kPlaneHaloCols || history || src == dst || !parts.mark_next))
        return hipErrorInvalidValue;
    PlaneArgs K;
    K.tiles = L.tiles;
    K.n_tiles = L.n_tiles;
    K.frame_words = L.frame_words;
    K.list_cap = L.list_cap;
    K.has_u = L.halo && actions && L.args.drop_mode == 0 ? 1 : 0;
    K.envs = L.envs;
    K.n_env = L.n_env;
    K.F = L.fields;
    K.A = L.args;
    K.phi = reinterpret_cast<const float4*>(L.phi);
    K.src = src;
    K.dst = dst;
    K.t_base = t_base;
    K.step0 = step0;
    K.steps = steps;
    K.actions = actions;
    K.counts = counts;
    K.history = history;
    K.parts = parts;
    K.keep_below = keep_threshold(L.args.p_continue);
    const size_t lds = plane_lds_bytes(L.frame_words, 3 + K.has_u, K.phi ? 0 : L.threads, L.list_cap);
    const int rates = K.phi ? kRatesTable : (K.F.wind ? kRatesCellWind : kRatesEnvWind);
    return with_kernel(L.threads, L.halo != 0, L.aligned, rates, [&](auto* kernel) {
        hipLaunchKernelGGL(kernel, dim3(K.n_tiles), dim3(L.threads), lds, s, K);
        return hipGetLastError();
    });
}

}  // namespace firesim
