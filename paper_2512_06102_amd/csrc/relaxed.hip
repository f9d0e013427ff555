// relaxed.hip -- the relaxed (mean-field) fire-spread step, its soft-IoU
// loss and its adjoint, for gradient-based calibration of the model's
// parameters (JaxWildfire, arXiv 2512.06102, section 3, "Deterministic
// (raw-probabilities) update", Eqs. 5-10; Eq. 4 for the ignition term).
//
// State per cell: U = p_un, B = p_burn.  One step:
//   q_k(v) = 1 - exp(-gamma(v) phi(u_k, k)),  u_k = v - D_k   (Eqs. 1-4)
//   P(v)   = 1 - prod_k (1 - q_k(v) B(u_k))
//   N = U P,  U' = U - N,  B' = N + p_continue B             (Eqs. 5-10)
//
// Adjoint of one step (bars are adjoints, primes are step t+1):
//   Nbar = B'bar - U'bar,   Ubar = U'bar + Nbar P,   Pbar = Nbar U,
//   Bbar(u) = p_c B'bar(u) + sum_k c_k(u + D_k),  c_k(v) = Pbar(v) q_k(v) E_k(v),
//   qbar_k(v) = Pbar(v) B(u_k) E_k(v),  E_k = prod_{j != k} (1 - q_j B(u_j))
// (exclusive products from prefix and suffix products, no division since
// q B can be 1), then through q = 1 - exp(-y), y = gamma phi (dq/dy =
// exp(-y)), phi = p_base g(u) exp(x), x = wind exponent + alpha_s S,
// gamma(v) = alpha_gamma g(v), g = (1 + veg[class]) (1 + den), to the 17
// parameters.
//
// Both directions work on 64 x 32 tiles (kAdjW x kAdjR) whose lanes own
// columns and walk the rows, passing neighbouring values and terms by DPP
// lane shifts, so each cell is loaded once per step.  The forward cuts a tile
// into row bands of one wave each.  The adjoint's transpose stencil
// (Bbar(u) gathers the terms of the targets around u, and those need B two
// cells away) runs one wave per tile or band, one launch per step; terms that
// cross into another tile go through an exchange record that the owning tile
// adds in the next step.  Every sum runs in a fixed order (no atomics), so the
// gradient is the same bits on every run.  Parameter gradients are summed per
// lane, reduced per wave and added to the tile's own row of partial sums; a
// last kernel sums the rows.
//
// Precision: the recurrence amplifies small burning mass exponentially (in
// the mean-field model every region reachable from a burning cell
// eventually ignites), so an fp32 state underflows and rounds its way onto a
// different trajectory within ~100 steps on a 128 x 128 grid.  U, B, the
// adjoint and the gradient sums are therefore fp64; the per-edge factors
// exp(x), phi, q = 1 - exp(-y) and exp(-y) are fp32 from the hardware base-2
// exponential (relative error ~1e-6 for |x| < 20), with q from its Taylor
// series below y = 1/16 so that small rates keep their relative accuracy.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "devmath.hpp"
#include "relaxed.hpp"

// Unlike the stochastic step, whose fp32 operation sequence is fixed so that
// it reproduces the oracle bit for bit, the relaxed path is held to a
// tolerance against an fp64 recurrence: from here on multiplies and adds may
// fuse into FMAs.
#pragma clang fp contract(fast)

namespace firesim {
namespace {

struct RelaxedArgs {
    float p_base, alpha_gamma, alpha_w1, alpha_w2, alpha_s, p_continue;
    float inv_orth, inv_diag;
    int32_t slope_mode;  // 0: S = rise / run; 1: S = atan(rise / run)
};

// The per-env wind of the current step: row env of a series row [n_env][3],
// or the env's static wind.
__device__ __forceinline__ float3 env_wind_of(const EnvDev& ed, const float* env_wind, int env)
{
    if (env_wind) return make_float3(env_wind[3 * env], env_wind[3 * env + 1], env_wind[3 * env + 2]);
    return make_float3(ed.V, ed.Vx, ed.Vy);
}

RelaxedArgs relaxed_args(const sim_params& p)
{
    RelaxedArgs a;
    a.p_base = p.p_base;
    a.alpha_gamma = p.alpha_gamma;
    a.alpha_w1 = p.alpha_w1;
    a.alpha_w2 = p.alpha_w2;
    a.alpha_s = p.alpha_s;
    a.p_continue = p.p_continue;
    a.inv_orth = (float)(1.0 / (double)p.cell_size);
    a.inv_diag = (float)(1.0 / ((double)p.cell_size * 1.41421356237309504880));
    a.slope_mode = (int32_t)p.slope_mode;
    return a;
}

bool finite_params(const sim_params& p)
{
    bool ok = true;
    for (float v : {p.p_base, p.alpha_gamma, p.alpha_w1, p.alpha_w2, p.alpha_s, p.p_continue}) ok = ok && std::isfinite(v);
    for (float v : p.veg) ok = ok && std::isfinite(v);
    return ok;
}

struct Veg11 {
    float v[11];
};

// e^x by the hardware base-2 exponential.
__device__ __forceinline__ float hexp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

// 1 - e^{-y} for y >= 0: Taylor series through y^5 below 1/16 (relative
// error < 2e-9 there), 1 - e^{-y} above (where it is at least 0.06).  Both are
// computed: a select, not a divergent branch.
__device__ __forceinline__ float one_minus_exp_neg(float y)
{
    const float qs = y * (1.0f - y * (0.5f - y * ((float)(1.0 / 6.0) - y * ((float)(1.0 / 24.0) - y * (float)(1.0 / 120.0)))));
    float ql = 1.0f - hexp(-y);
    float qt = qs;
    asm volatile("" : "+v"(ql), "+v"(qt));
    return y < 0.0625f ? qt : ql;
}

// q = 1 - e^{-y} as above and the survival e^{-y}: 1 - q below y = 1/16
// (where e^{-y} > 0.94, so the subtraction loses nothing), else from the
// one exponential.
__device__ __forceinline__ float2 q_and_survival(float y)
{
    const float qs = y * (1.0f - y * (0.5f - y * ((float)(1.0 / 6.0) - y * ((float)(1.0 / 24.0) - y * (float)(1.0 / 120.0)))));
    float el = hexp(-y);
    float qt = qs;
    // both are computed: a select, not a divergent branch
    asm volatile("" : "+v"(el), "+v"(qt));
    return y < 0.0625f ? make_float2(qt, 1.0f - qt) : make_float2(1.0f - el, el);
}

// e^{-z} and 1 - e^{-z} in fp64 from one series: z = n ln 2 + r, |r| <= ln 2 / 2
// (ln 2 split into its leading 40 bits, whose product with n is exact, and the
// rest), p = e^{-r} - 1 by its Taylor series through r^14 (truncation below 1e-18), then
// e^{-z} = 2^{-n} (1 + p) and 1 - e^{-z} = (1 - 2^{-n}) - 2^{-n} p, which keeps
// its relative accuracy for small z (n = 0).
struct SurvivalPair {
    double surv, p;
};
__device__ __forceinline__ SurvivalPair survival_pair(double z)
{
    constexpr double kLn2Head = 762123384785.0 / 1099511627776.0, kLn2Tail = 7.37100256516779889989e-13;
    z = z > 800.0 ? 800.0 : z;  // 2^-1154 is 0; a NaN stays
    const double n = __builtin_rint(z * 1.44269504088896340736);
    const double x = fma(n, kLn2Tail, fma(n, kLn2Head, -z));  // -r
    double c = 1.0 / 87178291200.0;
    c = fma(c, x, 1.0 / 6227020800.0);
    c = fma(c, x, 1.0 / 479001600.0);
    c = fma(c, x, 1.0 / 39916800.0);
    c = fma(c, x, 1.0 / 3628800.0);
    c = fma(c, x, 1.0 / 362880.0);
    c = fma(c, x, 1.0 / 40320.0);
    c = fma(c, x, 1.0 / 5040.0);
    c = fma(c, x, 1.0 / 720.0);
    c = fma(c, x, 1.0 / 120.0);
    c = fma(c, x, 1.0 / 24.0);
    c = fma(c, x, 1.0 / 6.0);
    c = fma(c, x, 0.5);
    c = fma(c, x, 1.0);
    const double p = c * x;
    const double two = __builtin_ldexp(1.0, -(int)n);
    return SurvivalPair{fma(two, p, two), fma(-two, p, 1.0 - two)};
}

__global__ __launch_bounds__(256) void relaxed_init_kernel(const uint8_t* __restrict__ st, int64_t n,
                                                           double* __restrict__ U, double* __restrict__ B)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint8_t s = st[i];
        U[i] = s == kFlammable ? 1.0 : 0.0;
        B[i] = s == kBurning ? 1.0 : 0.0;
    }
}

__global__ __launch_bounds__(256) void fuel_kernel(const uint8_t* __restrict__ cls,
                                                   const float* __restrict__ den, int64_t n,
                                                   Veg11 veg, float* __restrict__ g)
{
    __shared__ float sveg[11];
    if (threadIdx.x < 11) sveg[threadIdx.x] = veg.v[threadIdx.x];
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        g[i] = (1.0f + sveg[cls[i]]) * (1.0f + den[i]);
}

// (clear: a word set to 0 on the way, or nullptr)
__global__ __launch_bounds__(256) void copy_f64_kernel(double* __restrict__ dst,
                                                       const double* __restrict__ src, int64_t n,
                                                       int32_t* __restrict__ clear)
{
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;
    const int64_t n2 = n >> 1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2;
         i += (int64_t)gridDim.x * blockDim.x)
        reinterpret_cast<double2*>(dst)[i] = reinterpret_cast<const double2*>(src)[i];
    for (int64_t i = (n2 << 1) + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// (only_if: nullptr, or nothing is filled where it points to 0)
__global__ void fill_f64_kernel(double* p, int64_t n, double v, const int32_t* only_if)
{
    if (only_if && *only_if == 0) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Wind exponent of direction k at source cell u (per env from LDS, or per cell).
template <bool WC>
__device__ __forceinline__ float source_wind(int k, const float* ew, const float* wind, int64_t n_cells,
                                             int64_t u, const RelaxedArgs& A)
{
    if constexpr (WC)
        return wind_exponent(k, A.alpha_w1, A.alpha_w2, wind[u], wind[n_cells + u], wind[2 * n_cells + u]);
    else
        return ew[k];
}

// ---------------------------------------------------------------- adjoint
// Adjoint tiles are AW = 64 columns (one wave, one column per lane) by AR
// rows.  A wave walks its tile's rows top to bottom with the target row r in
// the middle of a three-row window of sources (rows r-1, r, r+1).  Each lane
// loads its own column; the left and right columns come from the
// neighbouring lanes by wave-wide DPP shifts, and lanes 0 and 63 load the
// column just outside the tile (the "ghost" column) themselves.
//
// Every target is evaluated once, by the tile that holds it.  Its terms c_k
// (into Bbar of source u_k) and d_k (into the fuel adjoint of u_k) go to
// running sums of the three source rows of the own column and, by the same
// DPP shifts, of the two neighbouring columns, always added in the same
// order.  Row r-1 is complete once target row r is done and is finished
// then.  Sums that belong to cells of another tile (the rows just above and
// below the tile and the ghost columns) are written to the tile's exchange
// record; the tile that owns those cells adds them, in a fixed order, to
// Bbar_{t+1} when it reads it in the next adjoint step.  Their fuel-adjoint
// part is turned into veg gradient by the producing lane, which reads the
// land-cover class and density of the foreign cell.  No atomics: Bbar, Ubar
// and the gradient are the same bits on every run.
constexpr int AW = kAdjW, AR = kAdjR;
// The reach data of a workspace: [0] the states were written sparsely, from
// [kReachHead] on the envs' integral images.
constexpr int kReachHead = 4;
constexpr int kXTop = 0, kXBot = AW, kXLeft = 2 * AW, kXRight = 2 * AW + AR + 2;
static_assert(kXRight + AR + 2 <= kXTile, "exchange record");

// Wave-wide shifts (DPP wave_shr:1 / wave_shl:1): from_left gives lane i the
// value of lane i-1, from_right that of lane i+1.  The lane with no source
// (0, resp. 63) reads 0 in the *0 forms and keeps `edge` in the *_or forms.
template <bool ZERO>
__device__ __forceinline__ int shr1(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, 0x138, 0xf, 0xf, ZERO); }
template <bool ZERO>
__device__ __forceinline__ int shl1(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, 0x130, 0xf, 0xf, ZERO); }
__device__ __forceinline__ float from_left_or(float edge, float v)
{
    return __int_as_float(shr1<false>(__float_as_int(edge), __float_as_int(v)));
}
__device__ __forceinline__ float from_right_or(float edge, float v)
{
    return __int_as_float(shl1<false>(__float_as_int(edge), __float_as_int(v)));
}
__device__ __forceinline__ int lo32(double v) { return (int)(unsigned)(unsigned long long)__double_as_longlong(v); }
__device__ __forceinline__ int hi32(double v) { return (int)(__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double mk64(int lo, int hi)
{
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double from_left_or(double edge, double v)
{
    return mk64(shr1<false>(lo32(edge), lo32(v)), shr1<false>(hi32(edge), hi32(v)));
}
__device__ __forceinline__ double from_right_or(double edge, double v)
{
    return mk64(shl1<false>(lo32(edge), lo32(v)), shl1<false>(hi32(edge), hi32(v)));
}
__device__ __forceinline__ double from_left0(double v) { return mk64(shr1<true>(0, lo32(v)), shr1<true>(0, hi32(v))); }
__device__ __forceinline__ double from_right0(double v) { return mk64(shl1<true>(0, lo32(v)), shl1<true>(0, hi32(v))); }

// Sum over the 64 lanes of a wave, returned to every lane: within rows of 16
// and across them by DPP moves (a butterfly of lane shuffles goes through LDS,
// 12 round trips per value).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    return v + mk64(__builtin_amdgcn_update_dpp(0, lo32(v), CTRL, ROWS, 0xf, false),
                    __builtin_amdgcn_update_dpp(0, hi32(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = dpp_add<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add<0x118, 0xf>(v);  // row_shr:8
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31
    return mk64(__builtin_amdgcn_readlane(lo32(v), 63), __builtin_amdgcn_readlane(hi32(v), 63));
}

// A source cell as the adjoint reads it: B, fuel g, elevation E and (per-cell
// wind only) V, Vx, Vy.  Off-grid cells are all zero.
struct AdjCell {
    double B;
    float g, E, V, Vx, Vy;
};

// An env's arrays from its first cell (wave-uniform pointers).  Cells are
// addressed by a 32-bit byte offset from them, so loads take a scalar base;
// the relaxed path therefore accepts envs of fewer than 2^29 cells.
struct AdjEnv {
    const double *U, *B, *gU1, *gB1;
    double *gU0, *gB0;
    const float *g, *E, *V, *Vx, *Vy, *den;
    const uint8_t* cls;
};

template <class T>
__device__ __forceinline__ T ld_at(const T* base, uint32_t i)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ void st_at(T* base, uint32_t i, T v)
{
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + i * (uint32_t)sizeof(T)) = v;
}

// The source cell at offset o, which lies on the grid whatever `in` says: no
// lane branches, and an off-grid cell gets no fuel and no burning mass (its
// other values are finite, so all its terms vanish).
template <bool WC>
__device__ __forceinline__ AdjCell load_adj_cell(const AdjEnv& P, uint32_t o, bool in)
{
    AdjCell c{ld_at(P.B, o), ld_at(P.g, o), ld_at(P.E, o), 0.0f, 0.0f, 0.0f};
    if constexpr (WC) {
        c.V = ld_at(P.V, o);
        c.Vx = ld_at(P.Vx, o);
        c.Vy = ld_at(P.Vy, o);
    }
    c.B = in ? c.B : 0.0;
    c.g = in ? c.g : 0.0f;
    return c;
}

// The left (right) neighbour of each lane's cell: the neighbouring lane's
// cell, or for lane 0 (63) its ghost cell, the column just outside the tile.
template <bool WC>
__device__ __forceinline__ AdjCell left_of(const AdjCell& x, const AdjCell& ghost)
{
    AdjCell r{from_left_or(ghost.B, x.B), from_left_or(ghost.g, x.g), from_left_or(ghost.E, x.E), 0.0f, 0.0f, 0.0f};
    if constexpr (WC) {
        r.V = from_left_or(ghost.V, x.V);
        r.Vx = from_left_or(ghost.Vx, x.Vx);
        r.Vy = from_left_or(ghost.Vy, x.Vy);
    }
    return r;
}

template <bool WC>
__device__ __forceinline__ AdjCell right_of(const AdjCell& x, const AdjCell& ghost)
{
    AdjCell r{from_right_or(ghost.B, x.B), from_right_or(ghost.g, x.g), from_right_or(ghost.E, x.E), 0.0f, 0.0f, 0.0f};
    if constexpr (WC) {
        r.V = from_right_or(ghost.V, x.V);
        r.Vx = from_right_or(ghost.Vx, x.Vx);
        r.Vy = from_right_or(ghost.Vy, x.Vy);
    }
    return r;
}

// A row of sources as a lane sees it: its own column and its neighbours.  The
// walk shifts each row once, when it enters the window.
struct AdjRow {
    AdjCell X, L, R;
};
template <bool WC>
__device__ __forceinline__ AdjRow make_row(const AdjCell& x, const AdjCell& ghost)
{
    return AdjRow{x, left_of<WC>(x, ghost), right_of<WC>(x, ghost)};
}

// The wind term (cos Vx + sin Vy) - V of direction k at source u, and the
// exponent of its edge under per-cell wind.  The multiply-adds are written out:
// a source's products serve three targets, and which of two products fuses
// would otherwise depend on what else the compiler shares.
__device__ __forceinline__ float wind_term(int k, const AdjCell& u)
{
    const float along = kCos[k] == 1.0f || kCos[k] == -1.0f ? __builtin_fmaf(kSin[k], u.Vy, kCos[k] * u.Vx)
                                                            : __builtin_fmaf(kCos[k], u.Vx, kSin[k] * u.Vy);
    return along - u.V;
}
__device__ __forceinline__ float cell_wind_exponent(int k, const AdjCell& u, float slope, const RelaxedArgs& A)
{
    return __builtin_fmaf(A.alpha_s, slope, __builtin_fmaf(A.alpha_w1, u.V, A.alpha_w2 * wind_term(k, u)));
}

// Running sums of one source cell: c into Bbar, d into the fuel adjoint.
struct CD {
    double c, d;
};

// The sums of one source row: of the lane's own column, and of the columns to
// its left and right.  The terms of three target rows are summed before the
// one shift that hands the sides to the neighbouring lanes; lane 0's left and
// lane 63's right sums are those of the ghost columns.
struct RowSums {
    CD own, left, right;
};

__device__ __forceinline__ CD cd_add(CD a, CD b) { return CD{a.c + b.c, a.d + b.d}; }
__device__ __forceinline__ CD cd_from_left(CD a) { return CD{from_left0(a.c), from_left0(a.d)}; }
__device__ __forceinline__ CD cd_from_right(CD a) { return CD{from_right0(a.c), from_right0(a.d)}; }

// Sparse adjoint.  The parameter gradient of step s sums over edges u -> v
// with B_s(u) != 0, so u lies within s cells (Chebyshev) of S_0, the cells
// with initial burning mass, and v within s + 1; it needs Bbar_{s+1} and
// Ubar_{s+1} there.  Bbar_s(u) in turn needs the terms of the targets next
// to u, whose inputs are one cell further out, and so on up to the seed at
// T: the adjoint step s must be exact within s + 1 cells of S_0, and it
// evaluates targets within s + 2.  A tile with no cell within s + 2 of S_0 is
// skipped: whatever its cells and exchange record hold (finite: the buffers
// start at zero) only ever meets B = 0 in the gradient sums, so only the
// parameter gradient is returned.
//
// first_state_kernel copies the initial state to its checkpoint and flags the
// tiles holding initial burning mass (or a U that is not finite) on the way, one
// workgroup per tile: with the flags in a pass of their own a forward call of one
// step of 256 envs of 128 x 128 took 94 us, now 83, and of one env of 2048 x 2048
// 85, now 67.  Where an env is one strip wide, its tiles are contiguous and are
// copied as such.
// tile_integral_kernel builds each env's integral image of the flags (one
// workgroup per env, in LDS).
__global__ __launch_bounds__(256) void first_state_kernel(const RelaxedTile* __restrict__ tiles,
                                                          const EnvDev* __restrict__ envs,
                                                          const double* __restrict__ U, const double* __restrict__ B,
                                                          double* __restrict__ Uo, double* __restrict__ Bo,
                                                          int32_t* __restrict__ mass)
{
    const RelaxedTile td = tiles[blockIdx.x];
    const EnvDev ed = envs[td.env];
    const int rows = min(AR, ed.H - td.r0), cols = min(AW, ed.W - td.c0);
    const bool strip = ed.W <= AW;
    const int64_t base = ed.offset + (int64_t)td.r0 * ed.W + td.c0;
    constexpr int N = AW * AR / 256;
    double u[N], b[N];
    int64_t at[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int q = 256 * k + (int)threadIdx.x, r = q / AW, c = q % AW;
        const bool in = strip ? q < rows * ed.W : r < rows && c < cols;
        at[k] = in ? base + (strip ? (int64_t)q : (int64_t)r * ed.W + c) : -1;
        u[k] = in ? U[at[k]] : 0.0;
        b[k] = in ? B[at[k]] : 0.0;
    }
    int any = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (at[k] >= 0) {
            Uo[at[k]] = u[k];
            Bo[at[k]] = b[k];
        }
        // (U P is not 0 where U is no number or infinite)
        if (b[k] != 0.0 || !(fabs(u[k]) < __builtin_inf())) any = 1;
    }
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) mass[blockIdx.x] = any ? 1 : 0;
}

__global__ __launch_bounds__(256) void tile_integral_kernel(const TileGrid* __restrict__ grids,
                                                            const int32_t* __restrict__ mass,
                                                            int32_t* __restrict__ reach)
{
    int32_t* const integ = reach + kReachHead;
    if (blockIdx.x == 0 && threadIdx.x == 0) reach[0] = 1;
    extern __shared__ int32_t sI[];
    const TileGrid tg = grids[blockIdx.x];
    const int W1 = tg.cols + 1, n = (tg.rows + 1) * W1;
    for (int i = threadIdx.x; i < n; i += 256) {
        const int r = i / W1, c = i % W1;
        sI[i] = (r && c) ? mass[tg.first + (r - 1) * tg.cols + (c - 1)] : 0;
    }
    __syncthreads();
    for (int r = threadIdx.x + 1; r <= tg.rows; r += 256) {
        int run = 0;
        for (int c = 1; c <= tg.cols; ++c) sI[r * W1 + c] = (run += sI[r * W1 + c]);
    }
    __syncthreads();
    for (int c = threadIdx.x + 1; c <= tg.cols; c += 256) {
        int run = 0;
        for (int r = 1; r <= tg.rows; ++r) sI[r * W1 + c] = (run += sI[r * W1 + c]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) integ[tg.ioff + i] = sI[i];
}

// The block of tiles that workgroup b takes.  per_xcd > 0: a contiguous run
// of that many blocks per XCD (workgroup b runs on XCD b % 8), so that
// neighbouring tiles meet in its L2; 0: in order.
__device__ __forceinline__ int dealt_block(uint32_t b, int32_t per_xcd)
{
    return per_xcd > 0 ? (int)(b & 7) * per_xcd + (int)(b >> 3) : (int)b;
}

// Is a tile with initial mass within a bands and b strips of tile (i, j)?
__device__ __forceinline__ bool adj_tile_in_reach_by(int i, int j, const TileGrid& tg, const int32_t* integ, int a, int b)
{
    const int i0 = max(i - a, 0), i1 = min(i + a, tg.rows - 1);
    const int j0 = max(j - b, 0), j1 = min(j + b, tg.cols - 1);
    const int32_t* I = integ + tg.ioff;
    const int W1 = tg.cols + 1;
    return I[(i1 + 1) * W1 + (j1 + 1)] - I[i0 * W1 + (j1 + 1)] - I[(i1 + 1) * W1 + j0] + I[i0 * W1 + j0] > 0;
}
// Does the adjoint step s need tile (band i, strip j): is a tile with initial
// mass within a = floor((s + 1) / AR) + 1 bands and b = floor((s + 1) / AW) + 1
// strips (the tiles whose nearest cells are at most s + 2 apart)?
__device__ __forceinline__ bool adj_tile_in_reach(int i, int j, const TileGrid& tg, const int32_t* integ, int32_t s)
{
    return adj_tile_in_reach_by(i, j, tg, integ, (s + 1) / AR + 1, (s + 1) / AW + 1);
}

// One adjoint step: (U_t, B_t), (Ubar_{t+1}, Bbar_{t+1}) -> (Ubar_t, Bbar_t)
// and the step's terms of the parameter gradient, added to the tile's row of
// gsum.  Both forms reduce to per-edge phibar_k and per-target gammabar:
//   FORM 0: ybar_k = Pbar B_k E_k exp(-y_k), phibar_k = ybar_k gamma,
//           gammabar = sum_k ybar_k phi_k, c_k = Pbar q_k E_k;
//   FORM 1: lambdabar = Pbar gamma (1 - P), phibar_k = lambdabar B_k,
//           gammabar = Pbar lambda (1 - P), c_k = lambdabar phi_k;
// d_k = phibar_k p_base exp(x_k) (dphi/dg of the source).  Far ahead of the
// fire (B = 0, U = 1) the adjoint state grows by about p_c + sum_k q_k per
// step backward and can pass the fp64 range after a few hundred steps.  It
// only ever meets B = 0 there: every gradient term it enters carries a factor
// B of a source or of the target, so those terms are 0.  The kernel takes a
// non-finite Pbar as 0 and adds the p_continue term only where B != 0, so the
// overflow never turns into inf x 0 = NaN.
// SL: slope S = rise / run (0) or atan(rise / run) (1).
//
// BANDS: waves per tile.  1: a wave walks the whole tile, four tiles per
// workgroup.  More: the waves walk AR / BANDS rows each and meet in LDS: the
// sums that cross a band edge are handed over there, so tiles, exchange records
// and the workspace are the same.
//
// What bounds it: VALU issue when every tile runs (its instructions alone take
// 56 of the 72 us below), else the walk of one wave.  256 envs of 128 x
// 128: 81 us per step with a shift per term and the rows moved through the
// window, 72 now; with 8 bands 118, so a full chip keeps 1.  One env of 128 x
// 128 (8 tiles): 43 us with 1 band, 13 with 8.  2048 x 2048 with per-cell wind,
// 200 steps, tiles in reach of the fire only: 59 us with 1 band, 41 with 8, 29
// with 4.
template <bool WC, int FORM, int SL, int BANDS>
__global__ __launch_bounds__(BANDS == 1 ? 256 : 64 * BANDS) __attribute__((amdgpu_waves_per_eu(2))) void relaxed_adj_kernel(
    const RelaxedTile* __restrict__ tiles, int32_t n_tiles, int32_t per_xcd, const TileGrid* __restrict__ grids,
    const EnvDev* __restrict__ envs, const float* __restrict__ g, const float* __restrict__ E,
    const float* __restrict__ wind, const uint8_t* __restrict__ cls, const float* __restrict__ den, int64_t n_cells,
    RelaxedArgs A, const double* __restrict__ U, const double* __restrict__ B, const double* __restrict__ gU1,
    const double* __restrict__ gB1, double* __restrict__ gU0, double* __restrict__ gB0,
    const double* __restrict__ Xin, double* __restrict__ Xout, double* __restrict__ gsum,
    const float* __restrict__ env_wind, const int32_t* __restrict__ reach, int32_t step)
{
    constexpr int NW = BANDS == 1 ? 4 : BANDS;  // waves per workgroup
    constexpr int BR = AR / BANDS;              // rows per wave
    __shared__ double sveg[NW][11][64];  // per lane: fuel adjoint x (1 + den) by land-cover class
    __shared__ double sxc[NW][BR][2];    // incoming Bbar terms of the first and last column, per row
    // the sums that a band hands to the one above and below it, per lane, and
    // those of the ghost columns (lanes 0 and 63)
    __shared__ double s_up[BANDS == 1 ? 1 : NW][64], s_down[BANDS == 1 ? 1 : NW][64];
    __shared__ double s_up_ghost[BANDS == 1 ? 1 : NW][2], s_down_ghost[BANDS == 1 ? 1 : NW][2];
    __shared__ double s_sum[BANDS == 1 ? 1 : NW][17];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: tile values in SGPRs
    const int block = dealt_block(blockIdx.x, per_xcd);
    const int tix = BANDS == 1 ? block * 4 + wv : block;
    if (tix >= n_tiles) return;
    const RelaxedTile td = tiles[tix];
    const TileGrid tg = grids[td.env];
    const int tb = td.r0 / AR, ts = td.c0 / AW;  // band and strip of the tile
    // sparse: the whole tile
    if (reach && reach[0] && !adj_tile_in_reach(tb, ts, tg, reach + kReachHead, step)) return;
    const EnvDev ed = envs[td.env];
    const int H = ed.H, W = ed.W;
    const int band = BANDS == 1 ? 0 : wv;
    const int tile_rows = min(AR, H - td.r0);
    const int r0 = td.r0 + band * BR;
    const int rows = min(BR, tile_rows - band * BR);  // <= 0: a band beyond the env
    const bool first_band = band == 0, last_band = (band + 1) * BR >= tile_rows;
    const int c = td.c0 + lane;
    const bool act = c < W;
    // ghost column: c0 - 1 for lane 0, c0 + 64 for lane 63 (if on the grid)
    const int cg = lane == 0 ? td.c0 - 1 : td.c0 + AW;
    const bool ghost = (lane == 0 && td.c0 > 0) || (lane == 63 && td.c0 + AW < W);
    const int64_t base = ed.offset;
    AdjEnv P;
    P.U = U + base;
    P.B = B + base;
    P.gU1 = gU1 + base;
    P.gB1 = gB1 + base;
    P.gU0 = gU0 + base;
    P.gB0 = gB0 + base;
    P.g = g + base;
    P.E = E + base;
    P.den = den + base;
    P.cls = cls + base;
    if constexpr (WC) {
        P.V = wind + base;
        P.Vx = wind + n_cells + base;
        P.Vy = wind + 2 * n_cells + base;
    } else {
        P.V = P.Vx = P.Vy = nullptr;
    }
    auto at = [&](int r, int col) { return (uint32_t)(r * W + col); };
    // the lane's own and ghost columns, and rows, kept on the grid for the loads of the window
    const int cc = min(c, W - 1), gc = min(max(cg, 0), W - 1);
    auto own_cell = [&](int r, bool in) { return load_adj_cell<WC>(P, at(min(max(r, 0), H - 1), cc), act && in); };
    auto ghost_cell = [&](int r, bool in) { return load_adj_cell<WC>(P, at(min(max(r, 0), H - 1), gc), ghost && in); };
    auto tile_of = [&](int bi, int sj) { return (int64_t)(tg.first + bi * tg.cols + sj) * kXTile; };
    const int64_t xrec = (int64_t)tix * kXTile;
    const int64_t xside = xrec + (lane == 0 ? kXLeft : kXRight) + band * BR;  // ghost entry of the row above the band

#pragma unroll
    for (int j = 0; j < 11; ++j) sveg[wv][j][lane] = 0.0;
    // each lane touches only its own slots, in program order: no barrier
    auto veg_add = [&](double fbar, uint32_t cl, float dn, bool on) {
        if (on) {
            double& slot = sveg[wv][cl][lane];
            slot += fbar * (1.0 + (double)dn);
        }
    };

    // this step's per-env wind; the exponent of direction k is
    // (alpha_w1 - alpha_w2) V + cos_k alpha_w2 Vx + sin_k alpha_w2 Vy
    const float3 wenv = env_wind_of(ed, env_wind, td.env);
    const float wA0 = (A.alpha_w1 - A.alpha_w2) * wenv.x, wA1 = A.alpha_w2 * wenv.y, wA2 = A.alpha_w2 * wenv.z;
    const float gp = A.alpha_gamma * A.p_base;
    const double p_c = A.p_continue;

    // sums over the lane's targets of w = ybar dphi/dp_base and of w S; per-cell
    // wind: of w V and w ((cos Vx + sin Vy) - V) of the source (acc_w1, acc_w2);
    // per-env wind: of w cos_k and w sin_k; each times gamma(v)
    double acc_pb = 0.0, acc_w1 = 0.0, acc_w2 = 0.0, acc_s = 0.0, acc_gw = 0.0, acc_pc = 0.0;
    // Bbar of the band's first and last row, and the ghost sums there, wait for
    // the neighbouring bands
    double first_B = 0.0, first_ghost = 0.0, last_B = 0.0, last_ghost = 0.0;

    if (rows > 0) {
        // Bbar terms that neighbouring tiles added to this tile's cells in the
        // previous step: for the tile's first and last row one per lane (xt, xb,
        // corners included), for the first and last column one per row (lanes 0
        // and 63, fetched by lanes 0.. and 32.. into LDS)
        double xt = 0.0, xb = 0.0;
        if (Xin) {
            const bool up = tb > 0 && first_band, dn = tb + 1 < tg.rows && last_band;
            if (act && up) xt = Xin[tile_of(tb - 1, ts) + kXBot + lane];
            if (act && dn) xb = Xin[tile_of(tb + 1, ts) + kXTop + lane];
            if (lane == 0 && ts > 0) {
                if (up) xt += Xin[tile_of(tb - 1, ts - 1) + kXRight + AR + 1];
                if (dn) xb += Xin[tile_of(tb + 1, ts - 1) + kXRight];
            }
            if (lane == 63 && ts + 1 < tg.cols) {
                if (up) xt += Xin[tile_of(tb - 1, ts + 1) + kXLeft + AR + 1];
                if (dn) xb += Xin[tile_of(tb + 1, ts + 1) + kXLeft];
            }
            const int side = lane >> 5, ii = lane & 31;
            double x = 0.0;
            if (ii < rows) {
                if (side == 0 && ts > 0) x = Xin[tile_of(tb, ts - 1) + kXRight + band * BR + ii + 1];
                if (side == 1 && ts + 1 < tg.cols) x = Xin[tile_of(tb, ts + 1) + kXLeft + band * BR + ii + 1];
            }
            if (ii < BR) sxc[wv][ii][side] = x;
            // the wave reads what its own lanes wrote: order the LDS accesses
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }

        // the window of source rows r - 1 (a), r (m), r + 1 (b): R0 to R2 in turn
        // (three rows of the walk per loop pass, so that no row is ever moved);
        // the row after it is on its way in nX (own column) and nG (ghost column)
        AdjRow R0 = make_row<WC>(own_cell(r0 - 1, r0 > 0), ghost_cell(r0 - 1, r0 > 0));
        AdjRow R1 = make_row<WC>(own_cell(r0, true), ghost_cell(r0, true));
        AdjRow R2;
        AdjCell nX = own_cell(r0 + 1, r0 + 1 < H), nG = ghost_cell(r0 + 1, r0 + 1 < H);
        RowSums S0{}, S1{}, S2{};
        double gB_prev = 0.0;

        // loaded one row ahead: the target's U, Ubar, Bbar, and the class and
        // density of the source row finished next (own and ghost column)
        double nU = 0.0, ngU = 0.0, ngB = 0.0;
        if (act) {
            nU = ld_at(P.U, at(r0, c));
            ngU = ld_at(P.gU1, at(r0, c));
            ngB = ld_at(P.gB1, at(r0, c));
        }
        uint32_t fcl = 0, gcl = 0;
        float fdn = 0.0f, gdn = 0.0f;
        if (act && r0 > 0) {
            fcl = ld_at(P.cls, at(r0 - 1, c));
            fdn = ld_at(P.den, at(r0 - 1, c));
        }
        if (ghost && r0 > 0) {
            gcl = ld_at(P.cls, at(r0 - 1, cg));
            gdn = ld_at(P.den, at(r0 - 1, cg));
        }

        // the sums of a finished source row: those of the lane's own column from
        // its three columns of targets, and of the ghost column
        auto column = [&](const RowSums& q) { return cd_add(cd_add(q.own, cd_from_right(q.left)), cd_from_left(q.right)); };
        auto ghost_of = [&](const RowSums& q) { return lane == 0 ? q.left : q.right; };

        auto walk = [&](const AdjRow& a, const AdjRow& m, AdjRow& b, RowSums& Sa, RowSums& Sm, RowSums& Sb, int i) {
            const int r = r0 + i;
            const uint32_t v = at(r, c);
            b = make_row<WC>(nX, nG);
            // the target's adjoint inputs, and what other tiles added to Bbar_{t+1}
            // of this cell in the previous step
            const double Uv = nU, gU = ngU;
            double gB = ngB;
            if (act && Xin)
                gB += ((i == 0 ? xt : 0.0) + (i == rows - 1 ? xb : 0.0)) +
                      (lane == 0 ? sxc[wv][i][0] : (lane == 63 ? sxc[wv][i][1] : 0.0));
            const uint32_t cl_a = fcl, gcl_a = gcl;  // row r - 1
            const float dn_a = fdn, gdn_a = gdn;
            if (act && i + 1 < rows) {
                nU = ld_at(P.U, v + W);
                ngU = ld_at(P.gU1, v + W);
                ngB = ld_at(P.gB1, v + W);
            }
            if (act) {
                fcl = ld_at(P.cls, v);
                fdn = ld_at(P.den, v);
            }
            if (ghost) {
                gcl = ld_at(P.cls, at(r, cg));
                gdn = ld_at(P.den, at(r, cg));
            }
            // next window row (r + 2)
            const bool more = i + 1 < rows && r + 2 < H;
            nX = own_cell(r + 2, more);
            nG = ghost_cell(r + 2, more);

            // ---- the target v = (r, c); its source in direction k is u_k = v - D_k
            const AdjCell* const src[8] = {&m.L, &b.L, &b.X, &b.R, &m.R, &a.R, &a.X, &a.L};
            auto sB = [&](int k) { return src[k]->B; };
            auto sg = [&](int k) { return src[k]->g; };
            const double nbar = gB - gU;
            // a non-finite Pbar comes only from an overflowed far-field adjoint
            // (see above), whose terms all carry B = 0: they are 0, not inf x 0
            const double Pbar = __builtin_isfinite(nbar * Uv) ? nbar * Uv : 0.0;
            const float gv = m.X.g, Ev = m.X.E;
            const float gam = A.alpha_gamma * gv, gpe = gp * gv;  // gamma(v), gamma(v) p_base
            const double gam64 = gam;
            // per-cell wind: the wind term (cos Vx + sin Vy) - V of direction k at the source
            auto wterm = [&](int k) { return wind_term(k, *src[k]); };
            auto slope_k = [&](int k) {
                const float rr = (Ev - src[k]->E) * ((k & 1) ? A.inv_diag : A.inv_orth);
                return SL ? atanf(rr) : rr;
            };
            float q[8], em[8], ex[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                // the exponent sums onto the slope term first, so that the
                // per-env wind constants are not kept per direction
                float x;
                if constexpr (WC) {
                    x = cell_wind_exponent(k, *src[k], slope_k(k), A);
                } else {
                    x = A.alpha_s * slope_k(k) + wA0;
                    if (kCos[k] != 0.0f) x = x + kCos[k] * wA1;
                    if (kSin[k] != 0.0f) x = x + kSin[k] * wA2;
                }
                // off-grid sources have zero fuel and zero B, so their terms
                // vanish; the exponent is capped so that 0 x e^x stays 0
                ex[k] = hexp(fminf(x, 88.0f));
                if constexpr (FORM == 0) {
                    const float2 qe = q_and_survival(gam * (A.p_base * (sg(k) * ex[k])));
                    q[k] = qe.x;
                    em[k] = qe.y;
                }
            }
            // the terms of edge k from ybar_k = phibar_k / gamma: w_k = ybar_k
            // dphi/dp_base for the gradient sums, c_k and d_k into the sums of
            // source u_k's row
            double w[8];
            auto emit = [&](int k, double cterm, double ybar) {
                w[k] = ybar * (double)(sg(k) * ex[k]);
                const CD o{cterm, ybar * (double)(gpe * ex[k])};  // d = phibar p_base e^x
                switch (k) {
                case 0: Sm.left = cd_add(Sm.left, o); break;
                case 1: Sb.left = o; break;
                case 2: Sb.own = o; break;
                case 3: Sb.right = o; break;
                case 4: Sm.right = cd_add(Sm.right, o); break;
                case 5: Sa.right = cd_add(Sa.right, o); break;
                case 6: Sa.own = cd_add(Sa.own, o); break;
                default: Sa.left = cd_add(Sa.left, o); break;
                }
            };
            double Pv;
            if constexpr (FORM == 0) {
                // exclusive products prod over j != k of 1 - q_j B_j, no division:
                // pairs, then pairs of pairs, Pbar carried along
                double om[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) om[k] = 1.0 - (double)q[k] * sB(k);
                const double p01 = om[0] * om[1], p23 = om[2] * om[3], p45 = om[4] * om[5], p67 = om[6] * om[7];
                const double lo = p01 * p23, hi = p45 * p67;
                // P's own product runs in the forward's order: where the burning
                // mass is below 1e-16 its rounding is all there is to P
                double run = 1.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) run = run * om[k];
                Pv = 1.0 - run;
                const double plo = Pbar * lo, phi = Pbar * hi;
                const double e[4] = {p23 * phi, p01 * phi, p67 * plo, p45 * plo};
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const double pe = e[k >> 1] * om[k ^ 1];
                    emit(k, pe * (double)q[k], (pe * sB(k)) * (double)em[k]);  // ybar = qbar dq/dy
                }
            } else {
                double lam = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) lam = lam + (double)(A.p_base * (sg(k) * ex[k])) * sB(k);
                const SurvivalPair sv = survival_pair((double)gam * lam);
                Pv = sv.p;
                const double ls = Pbar * sv.surv, lbar = ls * gam64;  // phibar_k = lbar B_k, ybar_k = phibar_k / gamma
#pragma unroll
                for (int k = 0; k < 8; ++k) emit(k, lbar * (double)(A.p_base * (sg(k) * ex[k])), ls * sB(k));
            }
            double gam_w = w[0], ws = w[0] * (double)slope_k(0);  // sum_k w_k (gammabar / p_base), sum_k w_k S_k
#pragma unroll
            for (int k = 1; k < 8; ++k) {
                gam_w += w[k];
                ws += w[k] * (double)slope_k(k);
            }
            acc_pb += gam64 * gam_w;
            acc_s += gam64 * ws;
            if constexpr (WC) {
                double w1 = 0.0, w2 = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    w1 += w[k] * (double)src[k]->V;
                    w2 += w[k] * (double)wterm(k);
                }
                acc_w1 += gam64 * w1;
                acc_w2 += gam64 * w2;
            } else {  // the env's wind is applied at the end
                const double d15 = w[1] - w[5], d37 = w[3] - w[7];
                acc_w1 += gam64 * ((w[0] - w[4]) + (double)kHalfSqrt2 * (d15 - d37));
                acc_w2 += gam64 * ((w[2] - w[6]) + (double)kHalfSqrt2 * (d15 + d37));
            }
            // gammabar = p_base gam_w; gamma(v) = alpha_gamma g(v)
            const double gam_bar = (double)A.p_base * gam_w;
            acc_gw += gam_w * (double)gv;
            if (m.X.B != 0.0) acc_pc += gB * m.X.B;
            Sm.own.d += gam_bar * (double)A.alpha_gamma;
            if (act) st_at(P.gU0, v, gU + nbar * Pv);

            // ---- source row r - 1 is complete
            const CD own = column(Sa), gh = ghost_of(Sa);
            if (i > 0 || r0 > 0) {
                veg_add(own.d, cl_a, dn_a, act);
                veg_add(gh.d, gcl_a, gdn_a, ghost);
            }
            if (i == 0) {  // the row above the band
                if (!first_band) {
                    s_up[wv][lane] = own.c;
                    if (lane == 0 || lane == 63) s_up_ghost[wv][lane == 63] = gh.c;
                } else if (r0 > 0) {
                    if (act) Xout[xrec + kXTop + lane] = own.c;
                    if (ghost) Xout[xside] = gh.c;
                }
            } else if (BANDS > 1 && i == 1) {
                first_B = p_c * gB_prev + own.c;
                first_ghost = gh.c;
            } else {
                if (act) st_at(P.gB0, v - W, p_c * gB_prev + own.c);
                if (ghost) Xout[xside + i] = gh.c;
            }
            gB_prev = gB;
        };
        int i = 0;
        while (true) {
            walk(R0, R1, R2, S0, S1, S2, i);
            if (++i == rows) break;
            walk(R1, R2, R0, S1, S2, S0, i);
            if (++i == rows) break;
            walk(R2, R0, R1, S2, S0, S1, i);
            if (++i == rows) break;
        }
        // the band's last row, and the row below it: the sums of rows - 1 and
        // rows, by where the walk ended
        const int turn = rows % 3;  // 1: after the first call of a pass, 2: the second, 0: the third
        const RowSums sl = turn == 1 ? S1 : (turn == 2 ? S2 : S0), sb = turn == 1 ? S2 : (turn == 2 ? S0 : S1);
        const int rl = r0 + rows - 1;
        const CD own = column(sl), gh = ghost_of(sl);
        veg_add(own.d, fcl, fdn, act);
        veg_add(gh.d, gcl, gdn, ghost);
        if (BANDS == 1) {
            if (act) st_at(P.gB0, at(rl, c), p_c * gB_prev + own.c);
            if (ghost) Xout[xside + rows] = gh.c;
        } else {
            last_B = p_c * gB_prev + own.c;
            last_ghost = gh.c;
        }
        if (rl + 1 < H) {
            const bool on = act, gon = ghost;
            const uint32_t cl = on ? (uint32_t)ld_at(P.cls, at(rl + 1, c)) : 0u;
            const float dn = on ? ld_at(P.den, at(rl + 1, c)) : 0.0f;
            const uint32_t gcl_b = gon ? (uint32_t)ld_at(P.cls, at(rl + 1, cg)) : 0u;
            const float gd = gon ? ld_at(P.den, at(rl + 1, cg)) : 0.0f;
            const CD bo = column(sb), bg = ghost_of(sb);
            veg_add(bo.d, cl, dn, on);
            veg_add(bg.d, gcl_b, gd, gon);
            if (!last_band) {
                s_down[wv][lane] = bo.c;
                if (lane == 0 || lane == 63) s_down_ghost[wv][lane == 63] = bg.c;
            } else {
                if (act) Xout[xrec + kXBot + lane] = bo.c;
                if (ghost) Xout[xside + rows + 1] = bg.c;
            }
        }
    }

    if constexpr (BANDS > 1) {
        __syncthreads();
        if (rows > 0) {
            const int gi = lane == 63;
            const double down = first_band ? 0.0 : s_down[wv - 1][lane], up = last_band ? 0.0 : s_up[wv + 1][lane];
            const double down_g = first_band ? 0.0 : s_down_ghost[wv - 1][gi], up_g = last_band ? 0.0 : s_up_ghost[wv + 1][gi];
            if (rows == 1) {
                if (act) st_at(P.gB0, at(r0, c), (last_B + down) + up);
                if (ghost) Xout[xside + 1] = (last_ghost + down_g) + up_g;
            } else {
                if (act) {
                    st_at(P.gB0, at(r0, c), first_B + down);
                    st_at(P.gB0, at(r0 + rows - 1, c), last_B + up);
                }
                if (ghost) {
                    Xout[xside + 1] = first_ghost + down_g;
                    Xout[xside + rows] = last_ghost + up_g;
                }
            }
        }
    }

    // ---- the tile's 17 gradient terms (fixed order), added to its gsum row.
    // dphi/dx = phi = p_base dphi/dp_base, so the wind and slope terms are
    // p_base times sums of gamma w
    const double p_base = A.p_base;
    double acc[17];
    acc[0] = acc_pb;
    if constexpr (WC) {
        acc[1] = p_base * acc_w1;
        acc[2] = p_base * acc_w2;
    } else {
        acc[1] = p_base * ((double)wenv.x * acc_pb);
        acc[2] = p_base * (((double)wenv.y * acc_w1 + (double)wenv.z * acc_w2) - (double)wenv.x * acc_pb);
    }
    acc[3] = p_base * acc_s;
    acc[4] = p_base * acc_gw;  // sum gammabar g(v)
    acc[5] = acc_pc;
#pragma unroll
    for (int j = 0; j < 11; ++j) acc[6 + j] = sveg[wv][j][lane];
#pragma unroll
    for (int j = 0; j < 17; ++j) acc[j] = wave_sum(acc[j]);
    double* row = gsum + (int64_t)tix * 17;
    if constexpr (BANDS == 1) {
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 17; ++j) row[j] += acc[j];
        }
    } else {
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 17; ++j) s_sum[wv][j] = acc[j];
        }
        __syncthreads();
        if (threadIdx.x < 17) {
            double sum = 0.0;
            for (int w2 = 0; w2 < NW; ++w2) sum += s_sum[w2][threadIdx.x];
            row[threadIdx.x] += sum;
        }
    }
}

// One relaxed forward step on the adjoint's 64 x AR tiles, each cut into
// SPLIT row bands of one wave (four per workgroup, so that enough loads
// are in flight): lanes own columns and walk the rows with the same
// window as the adjoint (left and right sources by DPP from the neighbouring
// lanes, the ghost columns for lanes 0 and 63), so each cell is loaded once.
// FORM 0: p_ignite = 1 - prod_k (1 - q_k B_k); FORM 1: p_ignite = 1 -
// exp(-gamma sum_k B_k phi_k).  Rows where no lane sees burning mass skip the
// edge terms (P = 0 exactly there).
//
// What bounds it: memory, at the rate of a copy, when every tile runs (256 envs
// of 128 x 128: 38 us per step at 40 bytes per cell); 2048 x 2048 with per-cell
// wind took 42 us per step with every tile and takes 13 with those in reach
// over 200 steps; one env of 128 x 128 8 us with 8-row bands, 4.5 with 2 rows.
//
// Sparse (reach given): after t steps burning mass lies within t cells of the
// cells that hold it at the start (S_0).  Step t runs on the tiles within
// reach, fills the tiles one further out with the initial state (U_0, 0), which
// is what they hold, and leaves the rest unwritten: the next step, and the
// adjoint of step t + 1, read only tiles within reach and their neighbours.
template <bool WC, int FORM, int SL, int SPLIT>
__global__ __launch_bounds__(256) void relaxed_fwd_kernel(
    const RelaxedTile* __restrict__ tiles, int32_t n_tiles, int32_t per_xcd, const TileGrid* __restrict__ grids,
    const EnvDev* __restrict__ envs, const float* __restrict__ g, const float* __restrict__ E,
    const float* __restrict__ wind, int64_t n_cells, RelaxedArgs A, const double* __restrict__ U,
    const double* __restrict__ B, double* __restrict__ Uo, double* __restrict__ Bo,
    const float* __restrict__ env_wind, const int32_t* __restrict__ reach, const double* __restrict__ U_0, int32_t step)
{
    constexpr int BR = AR / SPLIT;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wix = dealt_block(blockIdx.x, per_xcd) * 4 + wv;
    if (wix >= n_tiles * SPLIT) return;
    const RelaxedTile td = tiles[wix / SPLIT];
    const EnvDev ed = envs[td.env];
    const int H = ed.H, W = ed.W, r0 = td.r0 + (wix % SPLIT) * BR;
    if (r0 >= H) return;
    const int rows = min(BR, H - r0);
    const int c = td.c0 + lane;
    const bool act = c < W;
    const int64_t base = ed.offset;
    double* const Uoe = Uo + base;
    double* const Boe = Bo + base;
    auto at = [&](int r, int col) { return (uint32_t)(r * W + col); };
    if (reach && reach[0]) {
        const TileGrid tg = grids[td.env];
        const int tb = td.r0 / AR, ts = td.c0 / AW;
        if (!adj_tile_in_reach(tb, ts, tg, reach + kReachHead, step)) {
            if (!adj_tile_in_reach_by(tb, ts, tg, reach + kReachHead, (step + 2) / AR + 2, (step + 2) / AW + 2)) return;
            if (act)
                for (int i = 0; i < rows; ++i) {
                    const uint32_t v = at(r0 + i, c);
                    st_at(Uoe, v, ld_at(U_0 + base, v));
                    st_at(Boe, v, 0.0);
                }
            return;
        }
    }
    const int cg = lane == 0 ? td.c0 - 1 : td.c0 + AW;
    const bool ghost = (lane == 0 && td.c0 > 0) || (lane == 63 && td.c0 + AW < W);
    AdjEnv P{};
    P.U = U + base;
    P.B = B + base;
    P.g = g + base;
    P.E = E + base;
    if constexpr (WC) {
        P.V = wind + base;
        P.Vx = wind + n_cells + base;
        P.Vy = wind + 2 * n_cells + base;
    }
    const float3 wenv = env_wind_of(ed, env_wind, td.env);
    const float wA0 = (A.alpha_w1 - A.alpha_w2) * wenv.x, wA1 = A.alpha_w2 * wenv.y, wA2 = A.alpha_w2 * wenv.z;
    const double p_c = A.p_continue;

    const int cc = min(c, W - 1), gc = min(max(cg, 0), W - 1);
    auto own_cell = [&](int r, bool in) { return load_adj_cell<WC>(P, at(min(max(r, 0), H - 1), cc), act && in); };
    auto ghost_cell = [&](int r, bool in) { return load_adj_cell<WC>(P, at(min(max(r, 0), H - 1), gc), ghost && in); };
    // the window as in the adjoint; n0 to n2: does the row hold burning mass
    auto holds = [&](const AdjCell& x, const AdjCell& gh) { return __any(x.B != 0.0 || gh.B != 0.0) != 0; };
    AdjCell nX = own_cell(r0 - 1, r0 > 0), nG = ghost_cell(r0 - 1, r0 > 0);
    AdjRow R0 = make_row<WC>(nX, nG), R1, R2;
    bool n0 = holds(nX, nG), n1, n2 = false;
    nX = own_cell(r0, true);
    nG = ghost_cell(r0, true);
    R1 = make_row<WC>(nX, nG);
    n1 = holds(nX, nG);
    nX = own_cell(r0 + 1, r0 + 1 < H);
    nG = ghost_cell(r0 + 1, r0 + 1 < H);
    double nU = act ? ld_at(P.U, at(r0, c)) : 0.0;

    auto walk = [&](const AdjRow& a, const AdjRow& m, AdjRow& b, bool na, bool nm, bool& nb, int i) {
        const int r = r0 + i;
        const uint32_t v = at(r, c);
        b = make_row<WC>(nX, nG);
        nb = holds(nX, nG);
        const double Uv = nU;
        if (act && i + 1 < rows) nU = ld_at(P.U, v + W);
        const bool more = i + 1 < rows && r + 2 < H;
        nX = own_cell(r + 2, more);
        nG = ghost_cell(r + 2, more);

        double Pv = 0.0;
        if (na || nm || nb) {  // wave-uniform
            const AdjCell* const src[8] = {&m.L, &b.L, &b.X, &b.R, &m.R, &a.R, &a.X, &a.L};
            const float Ev = m.X.E, gam = A.alpha_gamma * m.X.g;
            // (the product in ascending order, one factor at a time: where the
            // burning mass is below 1e-16 its rounding is all there is to P)
            double prod = 1.0, lam = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const AdjCell& u = *src[k];
                const float rr = (Ev - u.E) * ((k & 1) ? A.inv_diag : A.inv_orth);
                float x;
                if constexpr (WC) {
                    x = cell_wind_exponent(k, u, SL ? atanf(rr) : rr, A);
                } else {
                    x = A.alpha_s * (SL ? atanf(rr) : rr) + wA0;
                    if (kCos[k] != 0.0f) x = x + kCos[k] * wA1;
                    if (kSin[k] != 0.0f) x = x + kSin[k] * wA2;
                }
                // off-grid sources read 0: no fuel, no burning mass
                const float phi = A.p_base * (u.g * hexp(fminf(x, 88.0f)));
                if constexpr (FORM == 0)
                    prod = prod * (1.0 - (double)one_minus_exp_neg(gam * phi) * u.B);
                else
                    lam = lam + (double)phi * u.B;
            }
            if constexpr (FORM == 0)
                Pv = 1.0 - prod;
            else
                Pv = survival_pair((double)gam * lam).p;
        }
        if (act) {
            const double N = Uv * Pv;
            st_at(Uoe, v, Uv - N);
            st_at(Boe, v, N + p_c * m.X.B);
        }
    };
    int i = 0;
    while (true) {
        walk(R0, R1, R2, n0, n1, n2, i);
        if (++i == rows) break;
        walk(R1, R2, R0, n1, n2, n0, i);
        if (++i == rows) break;
        walk(R2, R0, R1, n2, n0, n1, i);
        if (++i == rows) break;
    }
}

// grad[j] = sum over tiles of gsum[tile][j], one workgroup per j, in a fixed order.
__global__ __launch_bounds__(256) void gsum_reduce_kernel(const double* __restrict__ gsum, int32_t n_tiles,
                                                          double* __restrict__ grad)
{
    __shared__ double red[4];
    const int j = blockIdx.x;
    double a = 0.0;
    for (int t = threadIdx.x; t < n_tiles; t += 256) a += gsum[(int64_t)t * 17 + j];
    a = wave_sum(a);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) grad[j] = ((red[0] + red[1]) + red[2]) + red[3];
}
// ---------------------------------------------------------------- losses
// Every reduction below runs in a fixed order (lane-strided partial sums,
// DPP sums within a wave, then the four wave sums in order), so the losses, the
// objective and the seed are the same bits on every call.

// Sum over a 256-lane workgroup, returned to every lane.
__device__ __forceinline__ double block_sum256(double v, double* red)
{
    v = wave_sum(v);
    __syncthreads();  // red may still be read by a previous call
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}

// Soft IoU, stage 1: per loss chunk (kLossChunk cells of one env), the sums
// I = sum S Y, sum S and sum Y, with S = 1 - U_T on burnable cells.
__global__ __launch_bounds__(256) void iou_partials_kernel(const int32_t* __restrict__ chunk_env,
                                                           const EnvDev* __restrict__ envs,
                                                           const uint8_t* __restrict__ init_states,
                                                           const double* __restrict__ U_T,
                                                           const uint8_t* __restrict__ target,
                                                           double* __restrict__ partial)
{
    __shared__ double red[4];
    const int c = blockIdx.x;
    const EnvDev ed = envs[chunk_env[c]];
    const int64_t n = (int64_t)ed.H * ed.W;
    const int64_t first = (int64_t)(c - ed.chunk0) * kLossChunk;
    const int64_t last = min(first + (int64_t)kLossChunk, n);
    double sy = 0.0, ss = 0.0, yy = 0.0;
    for (int64_t i = first + threadIdx.x; i < last; i += 256) {
        const int64_t v = ed.offset + i;
        const double S = init_states[v] != kUnburnable ? 1.0 - U_T[v] : 0.0;
        const double Y = target[v] ? 1.0 : 0.0;
        sy += S * Y;
        ss += S;
        yy += Y;
    }
    sy = block_sum256(sy, red);
    ss = block_sum256(ss, red);
    yy = block_sum256(yy, red);
    if (threadIdx.x == 0) {
        partial[3 * c] = sy;
        partial[3 * c + 1] = ss;
        partial[3 * c + 2] = yy;
    }
}

// Soft IoU, stage 2 (one wave per env): the env's sums over its chunks and
// L_e = 1 - I / D, D = sum S + sum Y - I (0 when D = 0).
__global__ __launch_bounds__(64) void iou_env_kernel(const EnvDev* __restrict__ envs,
                                                     const double* __restrict__ partial,
                                                     double* __restrict__ sums, double* __restrict__ env_loss,
                                                     float* __restrict__ loss)
{
    const int e = blockIdx.x, lane = threadIdx.x;
    const EnvDev ed = envs[e];
    const int nch = (int)(((int64_t)ed.H * ed.W + kLossChunk - 1) / kLossChunk);
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int c = lane; c < nch; c += 64) {
        const double* p = partial + 3 * (int64_t)(ed.chunk0 + c);
        a0 += p[0];
        a1 += p[1];
        a2 += p[2];
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    a2 = wave_sum(a2);
    if (lane == 0) {
        const double D = (a1 + a2) - a0;
        const double L = D > 0.0 ? 1.0 - a0 / D : 0.0;
        sums[3 * e] = a0;
        sums[3 * e + 1] = a1;
        sums[3 * e + 2] = a2;
        env_loss[e] = L;
        loss[e] = (float)L;
    }
}

// The objective scale * sum_e L_e (one workgroup).
__global__ __launch_bounds__(256) void objective_kernel(const double* __restrict__ env_loss, int32_t n_env,
                                                        double scale, double* __restrict__ objective)
{
    __shared__ double red[4];
    double a = 0.0;
    for (int e = threadIdx.x; e < n_env; e += 256) a += env_loss[e];
    a = block_sum256(a, red);
    if (threadIdx.x == 0) objective[0] = scale * a;
}

// Soft IoU, stage 3: the seed scale * dL_e/dU_T = scale (Y D - I (1 - Y)) / D^2
// on burnable cells (dL/dU = -dL/dS), 0 elsewhere.
__global__ __launch_bounds__(256) void iou_seed_kernel(const int32_t* __restrict__ chunk_env,
                                                       const EnvDev* __restrict__ envs,
                                                       const uint8_t* __restrict__ init_states,
                                                       const uint8_t* __restrict__ target,
                                                       const double* __restrict__ sums, double scale,
                                                       double* __restrict__ gU_T)
{
    const int c = blockIdx.x;
    const int e = chunk_env[c];
    const EnvDev ed = envs[e];
    const int64_t n = (int64_t)ed.H * ed.W;
    const int64_t first = (int64_t)(c - ed.chunk0) * kLossChunk;
    const int64_t last = min(first + (int64_t)kLossChunk, n);
    const double I = sums[3 * e], D = (sums[3 * e + 1] + sums[3 * e + 2]) - I;
    for (int64_t i = first + threadIdx.x; i < last; i += 256) {
        const int64_t v = ed.offset + i;
        double gv = 0.0;
        if (D > 0.0 && init_states[v] != kUnburnable) {
            const double Y = target[v] ? 1.0 : 0.0;
            gv = scale * (Y * D - I * (1.0 - Y)) / (D * D);
        }
        gU_T[v] = gv;
    }
}

// The paper's calibration loss: BCE of the clipped soft scar plus the mean
// squared error of pool x pool block averages.  One lane per pooled block:
// the block means of S and Y, the block's BCE sum and squared error.
__global__ __launch_bounds__(256) void bce_pool_sums_kernel(
    const RelaxedTile* __restrict__ blocks, int32_t n_pool, int32_t pool, const EnvDev* __restrict__ envs,
    const uint8_t* __restrict__ init_states, const double* __restrict__ U_T,
    const uint8_t* __restrict__ target, double eps, double* __restrict__ vals)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_pool) return;
    const RelaxedTile pb = blocks[b];
    const EnvDev ed = envs[pb.env];
    const int i1 = min(pb.r0 + pool, ed.H), j1 = min(pb.c0 + pool, ed.W);
    double sS = 0.0, sY = 0.0, bce = 0.0;
    for (int i = pb.r0; i < i1; ++i)
        for (int j = pb.c0; j < j1; ++j) {
            const int64_t v = ed.offset + (int64_t)i * ed.W + j;
            const double S = init_states[v] != kUnburnable ? 1.0 - U_T[v] : 0.0;
            const double Y = target[v] ? 1.0 : 0.0;
            const double Sc = fmin(fmax(S, eps), 1.0 - eps);
            bce -= Y * log(Sc) + (1.0 - Y) * log(1.0 - Sc);
            sS += S;
            sY += Y;
        }
    const double cnt = (double)(i1 - pb.r0) * (double)(j1 - pb.c0);
    const double pS = sS / cnt, pY = sY / cnt;
    vals[b] = pS;
    vals[n_pool + b] = pY;
    vals[2 * (int64_t)n_pool + b] = bce;
    vals[3 * (int64_t)n_pool + b] = (pS - pY) * (pS - pY);
}

// Per env (one wave): BCE over its cells plus mse_weight times the mean
// squared error over its blocks.
__global__ __launch_bounds__(64) void bce_env_kernel(const EnvDev* __restrict__ envs,
                                                     const int32_t* __restrict__ env_blocks, int32_t n_pool,
                                                     const double* __restrict__ vals, double mse_weight,
                                                     double* __restrict__ env_loss, float* __restrict__ loss)
{
    const int e = blockIdx.x, lane = threadIdx.x;
    const int first = env_blocks[2 * e], nb = env_blocks[2 * e + 1];
    double bce = 0.0, sq = 0.0;
    for (int b = lane; b < nb; b += 64) {
        bce += vals[2 * (int64_t)n_pool + first + b];
        sq += vals[3 * (int64_t)n_pool + first + b];
    }
    bce = wave_sum(bce);
    sq = wave_sum(sq);
    if (lane == 0) {
        const double n_e = (double)envs[e].H * (double)envs[e].W;
        const double L = bce / n_e + mse_weight * sq / (double)nb;
        env_loss[e] = L;
        loss[e] = (float)L;
    }
}

__global__ __launch_bounds__(256) void bce_pool_grad_kernel(
    const RelaxedTile* __restrict__ blocks, int32_t n_pool, int32_t pool, const EnvDev* __restrict__ envs,
    const int32_t* __restrict__ env_blocks, const uint8_t* __restrict__ init_states,
    const double* __restrict__ U_T, const uint8_t* __restrict__ target, double eps, double mse_weight,
    const double* __restrict__ vals, double scale, double* __restrict__ gU_T)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_pool) return;
    const RelaxedTile pb = blocks[b];
    const EnvDev ed = envs[pb.env];
    const int i1 = min(pb.r0 + pool, ed.H), j1 = min(pb.c0 + pool, ed.W);
    const double n_e = (double)ed.H * (double)ed.W, m_e = (double)env_blocks[2 * pb.env + 1];
    const double cnt = (double)(i1 - pb.r0) * (double)(j1 - pb.c0);
    const double dmse = 2.0 * (vals[b] - vals[n_pool + b]) / m_e / cnt;  // d mse / d S of each cell
    for (int i = pb.r0; i < i1; ++i)
        for (int j = pb.c0; j < j1; ++j) {
            const int64_t v = ed.offset + (int64_t)i * ed.W + j;
            double gv = 0.0;
            if (init_states[v] != kUnburnable) {
                const double S = 1.0 - U_T[v];
                const double Y = target[v] ? 1.0 : 0.0;
                const double dbce = (S > eps && S < 1.0 - eps) ? (-(Y / S) + (1.0 - Y) / (1.0 - S)) / n_e : 0.0;
                gv = -scale * (dbce + mse_weight * dmse);  // dL/dU = -dL/dS
            }
            gU_T[v] = gv;
        }
}

int blocks_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 65536));
}

hipError_t copy_f64(hipStream_t s, double* dst, const double* src, int64_t n, int32_t* clear = nullptr)
{
    hipLaunchKernelGGL(copy_f64_kernel, dim3(blocks_for((n >> 1) + 1)), dim3(256), 0, s, dst, src, n, clear);
    return hipGetLastError();
}

hipError_t fill_f64(hipStream_t s, double* p, int64_t n, double v, const int32_t* only_if = nullptr)
{
    hipLaunchKernelGGL(fill_f64_kernel, dim3(blocks_for(n)), dim3(256), 0, s, p, n, v, only_if);
    return hipGetLastError();
}

// Workspace layout (all offsets 256-byte aligned).
struct WsLayout {
    size_t g, ckpt, seg, fwd, adj, xchg, gsum, reach, total;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

WsLayout layout(int64_t n, int64_t n_adj_tiles, int32_t T, int32_t k)
{
    const size_t d = 8 * (size_t)n;
    const size_t n_ckpt = T > 0 ? (size_t)((T + k - 1) / k) : 1;
    WsLayout L;
    size_t o = 0;
    L.g = o;
    o = align256(o + 4 * (size_t)n);
    L.ckpt = o;
    o = align256(o + n_ckpt * 2 * d);
    L.seg = o;
    o = align256(o + (size_t)k * 2 * d);
    L.fwd = o;
    o = align256(o + 2 * d);
    L.adj = o;
    o = align256(o + 4 * d);
    L.xchg = o;  // two exchange records per adjoint tile (steps of either parity)
    o = align256(o + sizeof(double) * 2 * (size_t)n_adj_tiles * kXTile);
    L.gsum = o;  // 17 gradient partial sums per adjoint tile
    o = align256(o + sizeof(double) * 17 * (size_t)n_adj_tiles);
    // the head, the envs' integral images ((rows + 1)(cols + 1) <= 4 rows cols
    // entries each) and the tiles' flags
    L.reach = o;
    o = align256(o + sizeof(int32_t) * (kReachHead + 5 * (size_t)n_adj_tiles));
    L.total = o;
    return L;
}

hipError_t fuel(hipStream_t s, const RelaxedInputs& in, const sim_params& p, float* g)
{
    Veg11 veg;
    for (int c = 0; c < 11; ++c) veg.v[c] = p.veg[c];
    hipLaunchKernelGGL(fuel_kernel, dim3(blocks_for(in.n_cells)), dim3(256), 0, s, in.cls, in.den,
                       in.n_cells, veg, g);
    return hipGetLastError();
}

// The inputs of relaxed step t: a wind series (per env or per cell) moves to
// its row t; static wind is returned as it is.
RelaxedInputs at_step(const RelaxedInputs& in, int32_t t)
{
    RelaxedInputs r = in;
    if (in.wind && in.wind_stride) r.wind = in.wind + (int64_t)t * in.wind_stride;
    if (in.env_wind) r.env_wind = in.env_wind + (int64_t)t * in.n_env * 3;
    return r;
}

// Row bands per tile: where the tiles alone (or those in reach of the fire)
// leave the chip idle, a step lasts as long as one wave's walk, so more waves
// walk fewer rows each.  Measured, many / few, ms of 100 steps, product form,
// envs of 128 x 128 (8 tiles each):
//   tiles   256          512          768          896          1024         2048
//   forward 0.94 / 0.77  1.41 / 1.26  1.70 / 1.59  2.00 / 1.78  2.06 / 1.92  3.64 / 3.26
//   adjoint 5.1  / 2.2   5.6  / 4.1   6.0  / 5.8   6.3  / 7.2   6.5  / 7.5   10.0 / 14.6
// where the fire decides which tiles run (envs of 64 tiles and more, 4 bands
// instead of 1): 512 tiles 3.3 / 3.3, 896 4.0 / 4.6; in one env, which has fewer
// of them in reach, 968 tiles 2.7 / 2.3, 2048 3.2 / 3.7
constexpr int kFwdBands = 4, kFwdBandsFew = 16, kAdjBandsFew = 8, kAdjBandsPart = 4;
constexpr int kFewFwdTiles = 1024, kFewAdjTiles = 800, kFewAdjTilesOneEnv = 1024;

// Tiles per env from which the sparse plan skips any.  In smaller envs the fire is
// in reach of every tile soon, and each wave looks it up in every step: dense and
// sparse, 40 steps forward, 4096 envs of 24 x 24 (1 tile) 1.86 and 1.89 ms, 512 of
// 64 x 64 (2) 0.80 and 0.83, 1000 of 50 x 70 (4) 2.09 and 2.15, 300 of 96 x 128 (6)
// 1.28 and 1.29, 256 of 128 x 128 (8) 1.49 and 1.44, 64 of 160 x 320 (25) 1.16 and
// 1.04; one step forward and back is 2 to 17% longer in the first four.
constexpr int64_t kSparseTiles = 8;

// Do only some of the tiles run in most steps: large envs under a sparse plan?
bool partly_active(const RelaxedInputs& in, const RelaxedState& R)
{
    return in.sparse && R.sparse_lds > 0 && in.n_tiles >= 64 * in.n_env;
}
// Blocks per XCD (0: deal them in order).  In runs per XCD a forward step of 256 envs
// of 128 x 128 takes 37.1 us, in order 38.8; where the fire decides which tiles
// run, they would leave most XCDs idle.
int32_t blocks_per_xcd(const RelaxedInputs& in, const RelaxedState& R, int32_t blocks)
{
    return partly_active(in, R) ? 0 : (blocks + 7) / 8;
}

template <bool WC, int FORM, int SL>
void launch_fwd(hipStream_t s, const RelaxedInputs& in, const RelaxedState& R, const RelaxedArgs& A, const float* g,
                const double* U, const double* B, double* Uo, double* Bo, const int32_t* reach, const double* U_0,
                int32_t step)
{
    const bool few = in.n_tiles < kFewFwdTiles;
    auto kernel = few ? relaxed_fwd_kernel<WC, FORM, SL, kFwdBandsFew> : relaxed_fwd_kernel<WC, FORM, SL, kFwdBands>;
    const int32_t groups = (in.n_tiles * (few ? kFwdBandsFew : kFwdBands) + 3) / 4;
    const int32_t per_xcd = blocks_per_xcd(in, R, groups);
    hipLaunchKernelGGL(kernel, dim3(per_xcd ? 8 * per_xcd : groups), dim3(256), 0, s, in.tiles, in.n_tiles, per_xcd, R.d_tgrid, in.envs, g, in.E,
                       in.wind, in.n_cells, A, U, B, Uo, Bo, in.env_wind, reach, U_0, step);
}

// Calls fn with the wind, form and slope of a launch as template arguments.
template <class Fn>
void with_variant(bool wc, int form, int slope, Fn fn)
{
    auto pick = [&](auto w, auto f) {
        slope ? fn(w, f, std::integral_constant<int, 1>{}) : fn(w, f, std::integral_constant<int, 0>{});
    };
    auto pick_form = [&](auto w) {
        form ? pick(w, std::integral_constant<int, 1>{}) : pick(w, std::integral_constant<int, 0>{});
    };
    wc ? pick_form(std::true_type{}) : pick_form(std::false_type{});
}

// Relaxed step `step`, from (U, B) to (Uo, Bo); U_0: the initial U.
hipError_t fwd_step(hipStream_t s, const RelaxedInputs& in, const RelaxedState& R, const RelaxedArgs& A, const float* g,
                    const double* U, const double* B, double* Uo, double* Bo, const int32_t* reach,
                    const double* U_0, int32_t step)
{
    with_variant(in.wind != nullptr, in.form, A.slope_mode, [&](auto w, auto f, auto sl) {
        launch_fwd<decltype(w)::value, decltype(f)::value, decltype(sl)::value>(s, in, R, A, g, U, B, Uo, Bo, reach,
                                                                                U_0, step);
    });
    return hipGetLastError();
}

template <bool WC, int FORM, int SL>
void launch_adj(hipStream_t s, const RelaxedInputs& in, const RelaxedState& R, const RelaxedArgs& A,
                const float* g, const double* U, const double* B, const double* gU1, const double* gB1,
                double* gU0, double* gB0, const double* Xin, double* Xout, double* gsum, const int32_t* reach,
                int32_t step)
{
    const bool part = partly_active(in, R);
    const bool few = R.n_btiles < (part && in.n_env == 1 ? kFewAdjTilesOneEnv : kFewAdjTiles);
    const int bands = few ? kAdjBandsFew : (part ? kAdjBandsPart : 1);
    auto kernel = bands == kAdjBandsFew    ? relaxed_adj_kernel<WC, FORM, SL, kAdjBandsFew>
                  : bands == kAdjBandsPart ? relaxed_adj_kernel<WC, FORM, SL, kAdjBandsPart>
                                           : relaxed_adj_kernel<WC, FORM, SL, 1>;
    const int32_t blocks = bands > 1 ? R.n_btiles : (R.n_btiles + 3) / 4;
    const int32_t per_xcd = blocks_per_xcd(in, R, blocks);
    hipLaunchKernelGGL(kernel, dim3(per_xcd ? 8 * per_xcd : blocks), dim3(bands > 1 ? 64 * bands : 256), 0, s,
                       R.d_btiles, R.n_btiles, per_xcd, R.d_tgrid, in.envs, g, in.E, in.wind, in.cls, in.den, in.n_cells, A, U,
                       B, gU1, gB1, gU0, gB0, Xin, Xout, gsum, in.env_wind, reach, step);
}

}  // namespace

int64_t relaxed_adj_tiles(const std::vector<sim_env>& envs)
{
    int64_t n = 0;
    for (const sim_env& v : envs) n += (int64_t)((v.H + AR - 1) / AR) * ((v.W + AW - 1) / AW);
    return n;
}

int relaxed_prepare(RelaxedState& R, const std::vector<sim_env>& envs)
{
    if (R.d_btiles) return 0;
    std::vector<RelaxedTile> btiles;
    std::vector<TileGrid> grids;
    int64_t ioff = 0, max_img = 0;
    for (int32_t e = 0; e < (int32_t)envs.size(); ++e) {
        TileGrid tg{(int32_t)btiles.size(), (envs[e].H + AR - 1) / AR, (envs[e].W + AW - 1) / AW, (int32_t)ioff};
        for (int r0 = 0; r0 < envs[e].H; r0 += AR)
            for (int c0 = 0; c0 < envs[e].W; c0 += AW) btiles.push_back(RelaxedTile{e, r0, c0, 0});
        const int64_t img = (int64_t)(tg.rows + 1) * (tg.cols + 1);
        ioff += img;
        max_img = std::max(max_img, img);
        grids.push_back(tg);
    }
    if (hipMalloc(&R.d_btiles, btiles.size() * sizeof(RelaxedTile)) != hipSuccess) return -1;
    if (hipMemcpy(R.d_btiles, btiles.data(), btiles.size() * sizeof(RelaxedTile),
                  hipMemcpyHostToDevice) != hipSuccess)
        return -1;
    if (hipMalloc(&R.d_tgrid, grids.size() * sizeof(TileGrid)) != hipSuccess) return -1;
    if (hipMemcpy(R.d_tgrid, grids.data(), grids.size() * sizeof(TileGrid), hipMemcpyHostToDevice) != hipSuccess)
        return -1;
    R.n_btiles = (int32_t)btiles.size();
    R.n_env = (int32_t)envs.size();
    if (ioff < INT32_MAX && 4 * max_img <= 64 * 1024) R.sparse_lds = (int32_t)(4 * max_img);
    return 0;
}

int relaxed_prepare_pool(RelaxedState& R, const std::vector<sim_env>& envs, int pool)
{
    if (R.d_pool && R.pool_k == pool) return 0;
    for (void** p : {(void**)&R.d_pool, (void**)&R.d_env_blocks, (void**)&R.d_pool_vals,
                     (void**)&R.d_bce_loss}) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
    }
    std::vector<RelaxedTile> blocks;
    std::vector<int32_t> per_env;  // first block, number of blocks
    for (int32_t e = 0; e < (int32_t)envs.size(); ++e) {
        const size_t before = blocks.size();
        for (int r0 = 0; r0 < envs[e].H; r0 += pool)
            for (int c0 = 0; c0 < envs[e].W; c0 += pool) blocks.push_back(RelaxedTile{e, r0, c0, 0});
        per_env.push_back((int32_t)before);
        per_env.push_back((int32_t)(blocks.size() - before));
    }
    R.n_pool = (int32_t)blocks.size();
    if (hipMalloc(&R.d_pool, blocks.size() * sizeof(RelaxedTile)) != hipSuccess ||
        hipMalloc(&R.d_env_blocks, per_env.size() * sizeof(int32_t)) != hipSuccess ||
        hipMalloc(&R.d_pool_vals, 4 * blocks.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&R.d_bce_loss, envs.size() * sizeof(double)) != hipSuccess)
        return -1;
    if (hipMemcpy(R.d_pool, blocks.data(), blocks.size() * sizeof(RelaxedTile), hipMemcpyHostToDevice) !=
            hipSuccess ||
        hipMemcpy(R.d_env_blocks, per_env.data(), per_env.size() * sizeof(int32_t),
                  hipMemcpyHostToDevice) != hipSuccess)
        return -1;
    R.pool_k = pool;
    return 0;
}

void relaxed_free(RelaxedState& R)
{
    for (void* p : {(void*)R.d_btiles, (void*)R.d_pool,
                    (void*)R.d_env_blocks, (void*)R.d_pool_vals, (void*)R.d_bce_loss, (void*)R.d_tgrid})
        if (p) (void)hipFree(p);
    R = RelaxedState{};
}

size_t relaxed_workspace_bytes(int64_t n_cells, int64_t n_adj_tiles, int32_t T, int32_t ckpt_every)
{
    return layout(n_cells, n_adj_tiles, T, ckpt_every).total;
}

hipError_t launch_relaxed_init(hipStream_t s, const uint8_t* init_states, int64_t n, double* U, double* B)
{
    hipLaunchKernelGGL(relaxed_init_kernel, dim3(blocks_for(n)), dim3(256), 0, s, init_states, n, U, B);
    return hipGetLastError();
}

// The forward writes each step's output where it is needed next: the
// checkpoint slot of every k-th state, the segment slots 1.. of the last
// segment's states (so the backward need not recompute that segment), the
// caller's U, B for the final state, and otherwise one of two scratch states
// (the forward buffer and segment slot 0, which the backward never uses).
hipError_t relaxed_forward(hipStream_t s, const RelaxedInputs& in, const sim_params& p, double* U,
                           double* B, int32_t T, int32_t k, void* workspace, RelaxedState& R)
{
    R.last_segment_ws = nullptr;
    if (T == 0) return hipSuccess;
    const int64_t n = in.n_cells;
    const WsLayout L = layout(n, R.n_btiles, T, k);
    char* ws = static_cast<char*>(workspace);
    float* g = reinterpret_cast<float*>(ws + L.g);
    double* ckpt = reinterpret_cast<double*>(ws + L.ckpt);
    double* seg = reinterpret_cast<double*>(ws + L.seg);
    double* spare[2] = {reinterpret_cast<double*>(ws + L.fwd), seg};
    const RelaxedArgs A = relaxed_args(p);
    const int32_t t_last = ((T - 1) / k) * k;  // first step of the last segment
    hipError_t e = fuel(s, in, p, g);
    // sparse: tiles with initial burning mass and their integral images, kept in
    // the workspace for the backward; a dense forward notes that it is one
    // (as it is under parameters that are not finite: what is 0 out of reach of the
    // fire, the terms of edges without burning mass and p_continue B, then is not)
    int32_t* const r = R.sparse_lds > 0 ? reinterpret_cast<int32_t*>(ws + L.reach) : nullptr;
    const int32_t* reach = nullptr;
    if (r && in.sparse && in.n_tiles >= kSparseTiles * (int64_t)in.n_env && finite_params(p)) {
        int32_t* mass = r + kReachHead + 4 * (size_t)R.n_btiles;
        if (e == hipSuccess) {
            hipLaunchKernelGGL(first_state_kernel, dim3(R.n_btiles), dim3(256), 0, s, R.d_btiles, in.envs, U, B, ckpt,
                               ckpt + n, mass);
            hipLaunchKernelGGL(tile_integral_kernel, dim3(R.n_env), dim3(256), (size_t)R.sparse_lds, s, R.d_tgrid,
                               mass, r);
            e = hipGetLastError();
        }
        reach = r;
    } else {
        if (e == hipSuccess) e = copy_f64(s, ckpt, U, n, r);
        if (e == hipSuccess) e = copy_f64(s, ckpt + n, B, n);
    }
    const double* cu = ckpt;  // state t
    const double* cb = ckpt + n;
    for (int32_t t = 0; t < T && e == hipSuccess; ++t) {
        const int32_t t1 = t + 1;
        double *nu, *nb;
        if (t1 == T) {
            nu = U;
            nb = B;
        } else if (t1 % k == 0) {
            nu = ckpt + (size_t)(t1 / k) * 2 * n;
            nb = nu + n;
        } else if (t1 > t_last) {
            nu = seg + (size_t)(t1 - t_last) * 2 * n;
            nb = nu + n;
        } else {
            nu = spare[0] == cu ? spare[1] : spare[0];
            nb = nu + n;
        }
        e = fwd_step(s, at_step(in, t), R, A, g, cu, cb, nu, nb, reach, ckpt, t);
        cu = nu;
        cb = nb;
    }
    if (e == hipSuccess) R.last_segment_ws = workspace;
    return e;
}

hipError_t relaxed_loss(hipStream_t s, const LossBatch& lb, const double* U_T, const uint8_t* target,
                        float* loss, double* gU_T, double scale, double* objective, double* scr)
{
    double* partial = scr;
    double* sums = partial + 3 * (size_t)lb.n_chunks;
    double* env_loss = sums + 3 * (size_t)lb.n_env;
    hipLaunchKernelGGL(iou_partials_kernel, dim3(lb.n_chunks), dim3(256), 0, s, lb.chunk_env, lb.envs,
                       lb.init_states, U_T, target, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(iou_env_kernel, dim3(lb.n_env), dim3(64), 0, s, lb.envs, partial, sums, env_loss, loss);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (objective) {
        hipLaunchKernelGGL(objective_kernel, dim3(1), dim3(256), 0, s, env_loss, lb.n_env, scale, objective);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (gU_T) {
        hipLaunchKernelGGL(iou_seed_kernel, dim3(lb.n_chunks), dim3(256), 0, s, lb.chunk_env, lb.envs,
                           lb.init_states, target, sums, scale, gU_T);
        e = hipGetLastError();
    }
    return e;
}

hipError_t relaxed_loss_bce(hipStream_t s, const RelaxedInputs& in, const uint8_t* init_states,
                            const double* U_T, const uint8_t* target, int pool, double mse_weight,
                            double eps, float* loss, double* gU_T, double scale, double* objective,
                            RelaxedState& R)
{
    const int nb = (R.n_pool + 255) / 256;
    hipLaunchKernelGGL(bce_pool_sums_kernel, dim3(nb), dim3(256), 0, s, R.d_pool, R.n_pool, pool, in.envs,
                       init_states, U_T, target, eps, R.d_pool_vals);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bce_env_kernel, dim3(in.n_env), dim3(64), 0, s, in.envs, R.d_env_blocks, R.n_pool,
                       R.d_pool_vals, mse_weight, R.d_bce_loss, loss);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (objective) {
        hipLaunchKernelGGL(objective_kernel, dim3(1), dim3(256), 0, s, R.d_bce_loss, in.n_env, scale, objective);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (gU_T) {
        hipLaunchKernelGGL(bce_pool_grad_kernel, dim3(nb), dim3(256), 0, s, R.d_pool, R.n_pool, pool, in.envs,
                           R.d_env_blocks, init_states, U_T, target, eps, mse_weight, R.d_pool_vals, scale,
                           gU_T);
        e = hipGetLastError();
    }
    return e;
}

hipError_t relaxed_backward(hipStream_t s, const RelaxedInputs& in, const sim_params& p,
                            const double* gU_T, const double* gB_T, int32_t T, int32_t k,
                            void* workspace, double* grad, RelaxedState& R)
{
    const int64_t n = in.n_cells;
    const WsLayout L = layout(n, R.n_btiles, T, k);
    char* ws = static_cast<char*>(workspace);
    float* g = reinterpret_cast<float*>(ws + L.g);
    double* ckpt = reinterpret_cast<double*>(ws + L.ckpt);
    double* seg = reinterpret_cast<double*>(ws + L.seg);
    double* adj = reinterpret_cast<double*>(ws + L.adj);
    double* xchg = reinterpret_cast<double*>(ws + L.xchg);
    double* gsum = reinterpret_cast<double*>(ws + L.gsum);
    const int64_t xrecs = (int64_t)R.n_btiles * kXTile;
    const RelaxedArgs A = relaxed_args(p);
    hipError_t e = fill_f64(s, gsum, (int64_t)R.n_btiles * 17, 0.0);
    // exchange records start at zero: a tile that the sparse adjoint skips
    // leaves finite values for its neighbours to read
    if (e == hipSuccess) e = fill_f64(s, xchg, 2 * xrecs, 0.0);
    if (e == hipSuccess) e = fuel(s, in, p, g);
    double* cu = adj;  // adjoint at t+1: (Ubar, Bbar)
    double* cb = adj + n;
    double* nu = adj + 2 * n;  // adjoint at t
    double* nb = adj + 3 * n;
    if (e == hipSuccess) e = copy_f64(s, cu, gU_T, n);
    if (e == hipSuccess) e = gB_T ? copy_f64(s, cb, gB_T, n) : fill_f64(s, cb, n, 0.0);
    // sparse adjoint, after a forward that wrote its states sparsely: the reach of
    // the initial burning mass, left in the workspace, and zeroed output buffers
    // (skipped tiles keep them)
    const int32_t* reach = nullptr;
    if (R.sparse_lds > 0 && T > 0 && e == hipSuccess) {
        reach = reinterpret_cast<const int32_t*>(ws + L.reach);
        e = fill_f64(s, nu, 2 * n, 0.0, reach);
    }
    const int32_t n_seg = T > 0 ? (T + k - 1) / k : 0;
    for (int32_t sg = n_seg - 1; sg >= 0 && e == hipSuccess; --sg) {
        const int32_t t0 = sg * k, t1 = std::min(T, t0 + k);
        const double* base = ckpt + (size_t)sg * 2 * n;
        // states t0 .. t1-1 of the segment: slot 0 is the checkpoint itself
        auto state_u = [&](int32_t j) -> const double* { return j == 0 ? base : seg + (size_t)j * 2 * n; };
        auto state_b = [&](int32_t j) -> const double* {
            return j == 0 ? base + n : seg + (size_t)j * 2 * n + n;
        };
        // the last segment's states are in place after the forward, until an
        // earlier segment's recompute overwrites them
        const bool stored = sg == n_seg - 1 && R.last_segment_ws == workspace;
        if (sg < n_seg - 1) R.last_segment_ws = nullptr;
        for (int32_t j = 1; j < t1 - t0 && !stored && e == hipSuccess; ++j)
            e = fwd_step(s, at_step(in, t0 + j - 1), R, A, g, state_u(j - 1), state_b(j - 1),
                         seg + (size_t)j * 2 * n, seg + (size_t)j * 2 * n + n, reach, ckpt, t0 + j - 1);
        for (int32_t t = t1 - 1; t >= t0 && e == hipSuccess; --t) {
            const int32_t j = t - t0;
            const double *Ut = state_u(j), *Bt = state_b(j);
            const RelaxedInputs it = at_step(in, t);
            // step t writes the exchange record of parity t; step t - 1 adds it
            const double* Xin = t == T - 1 ? nullptr : xchg + ((t + 1) & 1) * xrecs;
            double* Xout = xchg + (t & 1) * xrecs;
            with_variant(it.wind != nullptr, it.form, A.slope_mode, [&](auto w, auto f, auto sl) {
                launch_adj<decltype(w)::value, decltype(f)::value, decltype(sl)::value>(
                    s, it, R, A, g, Ut, Bt, cu, cb, nu, nb, Xin, Xout, gsum, reach, t);
            });
            e = hipGetLastError();
            std::swap(cu, nu);
            std::swap(cb, nb);
        }
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(gsum_reduce_kernel, dim3(17), dim3(256), 0, s, gsum, R.n_btiles, grad);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace firesim
