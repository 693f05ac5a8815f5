// Persistent batched solve (kernels_persist.hip) and its tuning
// (tune.hip): shared declarations.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <functional>

#include "msf_internal.hpp"

namespace msf {

// Arguments of one persistent launch.  Graph g has vtx_off[g+1]-vtx_off[g]
// vertices and edge_off[g+1]-edge_off[g] edges (local endpoint ids, weight
// bits); order lists the graphs to solve (largest first; null: every graph
// in index order), queue is the shared cursor into it.  Each workgroup owns
// slot_bytes of scratch (persist_slot_bytes of the launch's largest n and m)
// for its graph's edge list, forest flags and larger maps.
struct PersistArgs {
    int32_t G = 0;
    const uint32_t *order = nullptr;
    uint32_t *queue = nullptr;
    const int64_t *vtx_off = nullptr;
    const int64_t *edge_off = nullptr;
    const int32_t *edges = nullptr;
    const uint32_t *w = nullptr;
    int32_t *out = nullptr;
    int64_t *counts = nullptr;
    uint64_t *tot_u64 = nullptr;
    double *tot_f64 = nullptr;
    uint8_t *scratch = nullptr;
    size_t slot_bytes = 0;
    uint32_t lds_bytes = 0;
    uint32_t *err = nullptr;
    // one graph of one_n vertices and one_m edges and no queue, order,
    // offsets, counts and totals: everything that the host reads goes to
    // *one_out (pinned host memory, written once at the end).  round_hooks
    // (device): kept hooks of rounds 0..63 and, at [64], the rounds run
    SmallOut *one_out = nullptr;
    uint32_t *round_hooks = nullptr;
    int64_t one_n = 0, one_m = 0;
    // graph g's totals go to tot_u64[g * tot_stride], tot_f64[g * tot_stride]
    // (2 when they are the fields of an msf_total array)
    uint32_t tot_stride = 1;
};

// A launch configuration: threads per workgroup, edges each thread loads per
// step of a pass, dynamic LDS per workgroup (rounds whose minima and map fit
// it need one pass over the edges; it also sets how many workgroups share a
// CU).
struct PersistCfg {
    int nt;
    int ept;
    uint32_t lds;
};

// Edges a thread of the persistent kernel can keep in registers (1024 threads
// have 128 each: eight edges spill), and whether a graph's edges fit them and
// its state (10 bytes a vertex, a bit an edge) LDS: such a graph is solved
// without a list in device memory.
__host__ __device__ constexpr int persist_rq(int nt) { return nt == 1024 ? 4 : 8; }
__host__ __device__ inline bool persist_in_registers(uint32_t n, uint32_t m, int nt, size_t lds)
{
    const uint32_t cap = (uint32_t)(persist_rq(nt) * nt);
    return m <= cap && 10 * (size_t)n + 32 + cap / 8 <= lds;
}

// Graphs above these sizes are not solved by the persistent kernel.
constexpr uint32_t PERSIST_MAX_N = 1u << 20;
constexpr uint32_t PERSIST_MAX_M = 1u << 22;
// Dynamic LDS of the one-workgroup solve of a small graph (msf_solve).
constexpr uint32_t SMALL_LDS = 150u << 10;

// The size by which the server, and msf_solve with other than the default
// settings, choose the one-workgroup path (up to SMALL_LDS), and the part of
// a slot beside 32 bytes per edge.
__host__ __device__ inline size_t persist_state_bytes(uint32_t n, uint32_t m)
{
    return 20 * (size_t)n + 4 * (((size_t)m + 31) / 32);
}

__host__ inline size_t persist_slot_bytes(uint32_t n_cap, uint32_t m_cap)
{
    const size_t b = 2 * 16 * (size_t)m_cap + persist_state_bytes(n_cap, m_cap);
    return (b + 255) & ~(size_t)255;
}

// The form of the kernel, part of the tuner's saved choices: to be raised when
// the kernel or the candidates change enough to change which is the fastest (a
// choice made for the sweeps over edge lists that came before the contracted
// lists: 40000 vertices 7.4 ms, 3.3 ms by the present one).
constexpr int PERSIST_FORM = 2;

// The candidate configurations the tuner times (count in *count).
const PersistCfg *persist_candidates(int *count);

// Zero the queue and error word if reset, then launch `grid` workgroups.
hipError_t launch_persist(hipStream_t s, const PersistArgs &A, const PersistCfg &cfg, int wt,
                          unsigned grid, bool reset = true);

// The one-workgroup path's share where the contracted rounds are the other
// choice: edges + 2 * vertices.  One workgroup takes about 1.5-2 us per 1000
// of them, the contracted rounds 100-140 us at these sizes, mostly launches
// and dependent steps.  One workgroup / contracted rounds, us a solve by
// vertices and edges: 8000, 16000: 90 / 126; grid 20^3, 22K: 110 / 120; 24000,
// 20000: 143 / 160; 8000, 48000: 130 / 129; 16000, 32000: 143 / 141; 12000,
// 40000: 142 / 137; 1000, 64000: 101 / 92; R-MAT s12, 58K: 134 / 100.
constexpr int64_t SMALL_WORK = 68000;

// Whether msf_solve takes the one-workgroup path for this graph: at most
// c->small_m edges, and SMALL_WORK or, where the rounds over an adjacency
// matrix are the other choice, state that fits the largest LDS allocation.
bool small_eligible(const Ctx *c, int32_t n, int64_t m);

// msf_solve of a small graph by one workgroup of the persistent kernel
// (every round in LDS, no host round trips); same outputs as solve_device.
msf_status solve_small(Ctx *c, int32_t n, int64_t m, const int32_t *d_edges, const void *d_w,
                       msf_wtype wt, int32_t *d_ids, int64_t *count, msf_total *total);

// Workgroups of this configuration one compute unit holds at once (0 if the
// configuration cannot run).
int persist_blocks_per_cu(const PersistCfg &cfg, int wt);

// Whether the configuration's dynamic LDS fits this device.
bool persist_cfg_fits(int device, const PersistCfg &cfg);

// Shape of a batch, for the tuning cache key.
struct BatchShape {
    double mean_n = 0.0;    // mean vertices per graph
    double mean_deg = 0.0;  // mean stored entries (2 m) per vertex
};

// Runs candidate `cand` once on a sample of the batch; with ms non-null it
// also times the run (device events).
using PersistTuneRun = std::function<msf_status(int cand, float *ms)>;

// The candidate to use for a batch of this shape: MSF_BATCH_CONFIG if set,
// else the cached choice, else the fastest candidate on the sample (then
// cached).
msf_status persist_pick(Ctx *c, const BatchShape &shape, int wt, const PersistTuneRun &run,
                        int *chosen);

}  // namespace msf
