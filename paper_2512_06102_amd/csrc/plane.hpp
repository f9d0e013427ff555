// plane.hpp -- host interface of the bit-plane step kernel: many stochastic
// steps per launch on tiles whose state is held in LDS as bit planes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.hpp"

namespace firesim {

// One workgroup's cells: `rows` x `cols` of env `env` from (r0, c0).  A tile
// is a whole env, or (in a launch with a halo) a part of one with c0 a
// multiple of 32.  It holds the env's own entry, so that a workgroup can start
// with one load and not two in turn.
struct PlaneTile {
    int32_t env, r0, c0, rows, cols;
    EnvDev dev;
};

// Columns kept beyond a tile's left and right edge when it has a halo (one
// word of cells), and so the most steps such a launch may take.
constexpr int kPlaneHaloCols = 32;
// Entries of one wave's front list and steps of drops and wind staged at once.
constexpr int kPlaneWaveList = 192;
constexpr int kPlaneChunk = 32;
// Workgroup size of the launches with a halo.
constexpr int kPlaneHaloThreads = 256;
// Static LDS of the kernel, rounded up.
constexpr size_t kPlaneStaticLds = 1536;

// Words of one bit plane of a region: rows of ceil(cols / 32) words and one
// zero word between rows, a zero row above and below and one word more (the
// right neighbour of the last one).
inline int64_t plane_frame_words(int64_t rows, int64_t cols)
{
    return (rows + 2) * ((cols + 31) / 32 + 1) + 1;
}
// A listed group is rows << shift | group column in 16 bits.
inline bool plane_indexable(int64_t rows, int64_t cols)
{
    int shift = 0;
    while ((int64_t{1} << shift) < 8 * ((cols + 31) / 32)) ++shift;
    return (rows << shift) <= 65536;
}
// Listed 4-cell groups of a region (with more found, every group of the rows
// is looked at): an eighth of them, at least 256 and at most 4096.
inline int32_t plane_list_cap(int64_t rows, int64_t cols)
{
    const int64_t groups = rows * ((cols + 3) / 4);
    return (int32_t)std::min<int64_t>(4096, std::max<int64_t>(256, ((groups / 8 + 63) / 64) * 64));
}
// threads: 0 for the launches that read the table (they keep no wave lists)
inline size_t plane_lds_bytes(int64_t frame_words, int planes, int threads, int32_t list_cap)
{
    return 8 * (size_t)kPlaneWaveList * (size_t)(threads / 64) + 4 * (size_t)planes * (size_t)frame_words +
           2 * (size_t)list_cap;
}

struct PlaneLaunch {
    const PlaneTile* tiles;
    int32_t n_tiles;
    int32_t halo;         // 0: every tile is a whole env; else steps of halo (at most kPlaneHaloCols)
    int32_t threads;      // 64, 256, 512 or 1024
    int32_t frame_words;  // largest plane of the launch's regions
    int32_t list_cap;
    const EnvDev* envs;
    int32_t n_env;
    StaticFields fields;
    StepArgs args;
    bool aligned;         // every env has W % 4 == 0 and a 4-aligned offset
    const float* phi;     // [n_cells][8] ignition rates per edge (launch_phi_table) or nullptr
};

// Scheduling of the launches with a halo.  mark: what this launch does with
// each part (read and cleared), mark_next: the same for the next launch.  list
// (n_list entries): the parts that need anything, or nullptr for all of them;
// list_next receives the next launch's (or nullptr, as with drops, which may
// touch any part); n_clear is set to 0.  Marks, and the counts, start at 0.
struct PlaneParts {
    int32_t *mark, *mark_next;
    const int32_t* nbr;  // the 8 neighbouring parts (-1 off the env)
    const int32_t *list, *n_list;
    int32_t *list_next, *n_next, *n_clear;
    int32_t first;       // the first launch of a call: every part runs
};

// Ignition rate of every edge into a cell: phi[v][k] = p_base g(u) exp(wind
// exponent + alpha_s slope) of the source u = v - D_k, 0 off the grid, in the
// step's fp32 operation order.  Holds for static wind.
hipError_t launch_phi_table(hipStream_t s, const EnvDev* envs, const int32_t* chunk_env, int32_t n_chunks,
                            const StaticFields& F, const StepArgs& A, float* phi);

// Which batches take the `resident` plan: every env W % 4 == 0 at a 4-aligned
// offset, at most 65536 cells, and 8 bytes per dword of its framed state plus
// 16 per cell within the device's LDS per workgroup less kResidentStaticLds
// (on gfx950, squares up to 92 x 92).  The bit-plane kernel holds much larger
// envs whole; the plan's rule stays as it was published.
struct ResidentShape {
    bool fits = false;
    int32_t frame_cap = 0;  // (H + 2)(W/4 + 2) dwords of the largest, a multiple of 4
    int32_t cell_cap = 0;   // cells of the largest
};
constexpr size_t kResidentStaticLds = 2560;
inline size_t resident_lds_bytes(const ResidentShape& s)
{
    return 8 * (size_t)s.frame_cap + 16 * (size_t)s.cell_cap;
}

// Allows every instance of the kernel `bytes` of dynamic LDS.
hipError_t plane_set_lds_limit(int bytes);

// `steps` steps of the launch's tiles from src to dst, the first at absolute
// step *t_base + step0.  Without a halo src may equal dst, and `history` (or
// NULL) receives every state, n_cells bytes per step.  With a halo, src and
// dst differ, steps is at most L.halo, and `parts` schedules them.
// actions and counts point at the rows of the first step or are NULL; count
// rows must hold 0 on entry.
hipError_t launch_stoch_plane(hipStream_t s, const PlaneLaunch& L, const uint8_t* src, uint8_t* dst,
                              const uint32_t* t_base, uint32_t step0, int32_t steps, const int32_t* actions,
                              int32_t* counts, uint8_t* history, const PlaneParts& parts);

}  // namespace firesim
