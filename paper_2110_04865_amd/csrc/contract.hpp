// Rounds over a contracted edge list (kernels_contract.hip): declarations.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "msf_internal.hpp"

namespace msf {

// One edge of the list: its ends (vertices of the current round) and key.
struct __align__(16) CtEdge {
    uint32_t a, b;
    uint64_t key;
};

constexpr uint32_t CT_MAX_WAVES = 8192;  // list segments
constexpr uint32_t CT_TILE = 256;        // input edges a wave takes at a time
constexpr uint32_t CT_WSLOTS = 2048;     // partial weight sums
constexpr uint32_t CT_SMALL = 7680;      // vertices whose minima fit LDS (two workgroups a CU)
constexpr uint32_t CT_FINISH = 2048;     // vertices whose round one workgroup finishes best
constexpr uint32_t CT_PAIR = 32;         // vertices finished on their pairs' minima

// Edges per list segment when the input's tiles are dealt to W waves.
inline size_t ct_segcap(int64_t m, uint32_t W)
{
    const int64_t tiles = (m + CT_TILE - 1) / CT_TILE;
    return (size_t)((tiles + W - 1) / W) * CT_TILE;
}

// Arguments of the kernels of one phase (phase 0: the light edges, or all;
// phase 1: the edges left between the trees of phase 0).
struct CtArgs {
    int32_t n = 0;  // vertices of the graph
    int64_t m = 0;
    int ph = 0;
    int wt = 0;
    const int2 *edges = nullptr;
    const uint32_t *w = nullptr;
    const uint32_t *comp = nullptr;  // phase 1: vertex -> tree of phase 0
    CtEdge *list = nullptr;          // W segments of segcap edges
    uint32_t *cw = nullptr;          // edges in each segment
    uint32_t W = 0;           // waves that write the list, one segment each
    uint32_t pass_waves = 0;  // waves of an edge pass in phase 0 (in phase 1, W)
    uint32_t segcap = 0;
    uint64_t *r[2] = {nullptr, nullptr};  // root minima of even and odd rounds
    uint32_t *h = nullptr;
    uint32_t *map0 = nullptr;  // round 0: vertex -> vertex of round 1
    uint32_t *maps = nullptr;  // later rounds, one after the other
    uint32_t *cum = nullptr;   // first small round's vertices -> current ones
    uint32_t *wlist = nullptr; // weight keys of the small rounds' hooks
    uint64_t *mat = nullptr;   // pair minima of a phase's last vertices
    uint8_t *flags = nullptr;
    int64_t *wpart = nullptr;
    uint32_t sweeps = 0;  // visits of a large round's chase to a vertex
    Counters *cnt = nullptr;
};

// Whether the context's settings leave msf_solve to these rounds.
bool contract_settings(const Ctx *c);

// Words of the maps of rounds 1, 2, ... (round k has at most n >> k
// vertices: every vertex with an edge hooks).
size_t ct_maps_words(int32_t n);
size_t ct_wpart_bytes();

// Set-up, and the threshold for about the `light` lightest edges.
void ct_init(hipStream_t s, const CtArgs &A, size_t flag_words, int64_t light);
void ct_select(hipStream_t s, const CtArgs &A);
// One round; big: also the kernels that a round with many vertices needs
// (bound: the most vertices it can have).
void ct_round(hipStream_t s, const CtArgs &A, int k, bool big, uint32_t bound);
// Round k (of L vertices), whose chase gave up, to its end: every chain
// shortened by launches of its own, then the chase.
void ct_far(hipStream_t s, CtArgs A, int k, uint32_t L);
// Trees of phase 0 per vertex, the largest one's membership bits, and the
// list of the edges between different trees.
void ct_between(hipStream_t s, const CtArgs &A, uint32_t *comp, uint32_t *bits);
// Partial weight sums that graphs of n vertices use.
uint32_t ct_wslots_host(int32_t n);

}  // namespace msf
