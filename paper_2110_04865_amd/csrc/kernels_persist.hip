// Persistent batched solve: one workgroup runs every round of one graph.
//
// A batch of many small and medium graphs (the batched pattern) is solved
// by one launch of a persistent grid (a few workgroups per compute unit).
// Each workgroup takes graphs from a queue, largest first, and runs
// Algorithm 2 with complete shortcutting (section 4.2) on its graph alone,
// with a workgroup barrier between the steps of a round and a per-graph
// termination test, so no round boundary involves the host:
//
//   list      the graph's live edges, dense and in edge-id order, with their
//             ends renumbered every round (0 .. L - 1); a pass maps the ends,
//             drops the edges that became internal, in place, and lowers the
//             minima of both ends (the multilinear kernel of section 3.1 with
//             the projection of Algorithm 2, both stored directions at once);
//   hook      every vertex hooks onto the other end of its minimum edge;
//   tie break of two vertices that hooked onto each other the smaller stays
//             root (Algorithm 2, tie-breaking step; section 2.3);
//   shortcut  complete shortcutting (section 4.2), then new numbers for the
//             roots that can still hook;
//   stop      when no live edge is left.
// Once few edges are left (persist_rq a thread) they move to registers and the
// remaining rounds touch LDS alone; with 128 or fewer vertices and more edges,
// one pass first takes the minimum key of every pair of vertices into a matrix
// in LDS.  A graph that has so few edges from the start never leaves the chip
// (solve_registers).  From PERSIST_TWO_PHASE_M edges on the lightest edges go
// first (see kernels_contract.hip): their forest is built, one pass over the
// graph drops every edge inside one of its trees, and a second phase finishes.
//
// A round's minima, hook records and map take 10 bytes of LDS per vertex of
// the round; where that does not fit (the first round of a graph of more
// than 15K vertices in 150 KB) the minima are taken by ranges of vertices,
// one pass over the list each.  The list and the larger maps are in the
// workgroup's slot of a global scratch area (at most 32 m + 20 n bytes).
// Keys use the graph's local edge ids, so each graph's forest is the one
// msf_solve finds on that graph alone.  Outputs: the forest's local edge ids
// in ascending order from out + vtx_off[g], count and exact totals.
//
// Measured on 10^4 Erdos-Renyi graphs (64 to 65536 vertices, 382M edges):
// 42.3 ms by an earlier form, which swept the edge list with a parent vector
// in LDS and the minima in global memory; 7.6 ms by the list; 7.1 ms with the
// loops over vertices batched (PC_B) and the ids written through LDS.  It
// moves 21 GB (13.0 read, 8.4 written).  The passes over the input run at 4.8
// TB/s, memory's rate; between them a graph's one workgroup on its compute
// unit waits for device memory 70% of the time.
// Smaller graphs, registers against the list before: 10^4 of 1000 vertices
// and 4000 edges 658 / 576 us, 10^4 of 50 to 2000 vertices and six edges each
// 698 / 467 us; one graph of 100 vertices and 400 edges 31 / 28 us a solve.
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "exact_sum.hpp"
#include "msf_internal.hpp"
#include "persist.hpp"
#include "wave.hpp"

// Edges from which a graph takes its light edges first.
#ifndef PERSIST_TWO_PHASE_M
#define PERSIST_TWO_PHASE_M 2048
#endif

namespace msf {

namespace {

__device__ __forceinline__ uint64_t ld_min_u64(uint64_t *p, uint64_t v)
{
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// r[i] <- min(r[i], key) where a read of r[i] (cur) shows that the key can
// lower it: r only decreases during a sweep, so a stale read can cost an
// atomic, never a miss, and most atomics are skipped (measured: sending
// every atomic to global memory made the sweep 3x slower).
__device__ __forceinline__ void lower(uint64_t *r, uint32_t i, uint64_t cur, uint64_t key)
{
    if (key < cur) ld_min_u64(r + i, key);
}

__device__ __forceinline__ uint32_t weight_key(uint32_t bits, int wt)
{
    return wt == MSF_W_F32 ? wkey_f32_bits(bits) : bits;
}

// The list keeps the order of the edge ids, so (weight key, position in the
// list) compares like (weight key, edge id): a minimum names its edge's
// place in the list, where the hook finds both ends.

struct PEdge {
    uint32_t a, b, w, e;
};

// The list as arrays of words: with P16 both ends in one word (12 bytes an
// edge), else a word each.  At most 2^22 edges, so byte offsets fit 32 bits
// and the accesses take a scalar base.
template <bool P16>
struct PList {
    uint32_t *ab, *b, *w, *e;
    __device__ __forceinline__ static uint32_t ld(const uint32_t *p, uint32_t j)
    {
        return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(p) + (j << 2));
    }
    __device__ __forceinline__ static void st(uint32_t *p, uint32_t j, uint32_t v)
    {
        *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(p) + (j << 2)) = v;
    }
    __device__ __forceinline__ PList(uint8_t *at, uint32_t m)
    {
        ab = reinterpret_cast<uint32_t *>(at);
        b = ab + m;
        w = b + m;
        e = w + m;
    }
    __device__ __forceinline__ PEdge get(uint32_t j) const
    {
        const uint32_t x = ld(ab, j);
        if (P16) return PEdge{x & 0xFFFFu, x >> 16, ld(w, j), ld(e, j)};
        return PEdge{x, ld(b, j), ld(w, j), ld(e, j)};
    }
    __device__ __forceinline__ void put(uint32_t j, const PEdge &x) const
    {
        if (P16) {
            st(ab, j, x.a | (x.b << 16));
        } else {
            st(ab, j, x.a);
            st(b, j, x.b);
        }
        st(w, j, x.w);
        st(e, j, x.e);
    }
};

constexpr uint32_t PC_MARK = 0xFFFFFFFFu;
constexpr uint32_t PC_TREE = 0x80000000u;  // with a tree's number
constexpr int PC_LEVELS = 40;

// Shared control words of the contracted solve.
constexpr uint32_t PC_MAT = 128;  // most vertices a pair matrix takes
template <int NT>
struct PCtl {
    uint32_t cnt[2][NT / 64];  // kept edges per wave, alternating tiles
    uint32_t hist[256];
    uint32_t bin, rank, same;
    uint32_t live, dead, hooks;
    uint32_t g;     // graph being solved (NONE32: queue empty)
    uint32_t err;   // ERR_* seen by this workgroup
    uint32_t gerr;  // the current graph failed validation
    uint32_t off[PC_LEVELS];
    // rounds in registers: hooks and edges of even and odd rounds, flags of
    // the pointer jumping
    uint32_t rc[4], rj[3];
};

// A value that every lane of every wave reads alike, in a scalar register
// (what comes from LDS is taken for a vector value otherwise, and with it
// every size, pointer and loop bound derived from it).
__device__ __forceinline__ uint32_t uniform(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ int64_t uniform(int64_t v)
{
    return (int64_t)(((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v));
}

// Items of a tile: wave w takes the 64 U consecutive ones from 64 U w on,
// item q of lane l being 64 q + l of them.  From each wave's count of kept
// items, this wave's first place in the tile; *total gets the tile's count.
// One barrier; the counts alternate between two buffers (par).
template <int NT>
__device__ __forceinline__ uint32_t wave_place(uint32_t c, PCtl<NT> &pc, int par, uint32_t *total)
{
    constexpr int NW = NT / 64;
    static_assert(NW <= 16, "one row of lanes");
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (__lane_id() == 0) pc.cnt[par][w] = c;
    __syncthreads();
    uint32_t v = __lane_id() < NW ? pc.cnt[par][__lane_id()] : 0u;
    v += dpp_move<DPP_ROW_SHR1>(v);
    if (NW > 2) v += dpp_move<DPP_ROW_SHR2>(v);
    if (NW > 4) v += dpp_move<DPP_ROW_SHR4>(v);
    if (NW > 8) v += dpp_move<DPP_ROW_SHR8>(v);
    *total = (uint32_t)__builtin_amdgcn_readlane((int)v, NW - 1);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, w) - c;
}

// A thread's first item (item q is 64 q further).  Opaque, so that each pass
// computes its own offsets: shared by all the passes inlined into the kernel
// they cost some 40 registers everywhere.
__device__ __forceinline__ uint32_t opaque_tid()
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

template <int U>
__device__ __forceinline__ uint32_t tile_item0()
{
    const uint32_t t = opaque_tid();
    return (t >> 6) * (64u * U) + (t & 63u);
}

// How a pass lowers minima: not at all; r[end] by an LDS atomic each; the
// same behind a read (few vertices: most edges change nothing, and atomics
// on few addresses serialise); only ends in [lo, lo + len), behind a read;
// the pair's entry of a matrix, behind a read (nothing else is kept).
enum { PM_NONE, PM_MIN, PM_MINF, PM_RANGE, PM_MAT };

struct PMinArgs {
    uint64_t *r = nullptr;  // minima, or the matrix (rows of 1 << lo entries)
    uint32_t lo = 0, len = 0;
};

template <int MODE, int U>
__device__ __forceinline__ void lower_ends(const PMinArgs &M, const PEdge (&x)[U],
                                           const bool (&live)[U], const uint32_t (&pos)[U])
{
    if (MODE == PM_MIN) {
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (!live[q]) continue;
            const uint64_t key = ((uint64_t)x[q].w << 32) | pos[q];
            ld_min_u64(M.r + x[q].a, key);
            ld_min_u64(M.r + x[q].b, key);
        }
    }
    if (MODE == PM_MINF || MODE == PM_RANGE) {
        uint32_t ia[U], ib[U];
        uint64_t ra[U], rb[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            ia[q] = x[q].a - (MODE == PM_RANGE ? M.lo : 0u);
            ib[q] = x[q].b - (MODE == PM_RANGE ? M.lo : 0u);
            const bool in = live[q];
            ra[q] = M.r[in && (MODE != PM_RANGE || ia[q] < M.len) ? ia[q] : 0u];
            rb[q] = M.r[in && (MODE != PM_RANGE || ib[q] < M.len) ? ib[q] : 0u];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (!live[q]) continue;
            const uint64_t key = ((uint64_t)x[q].w << 32) | pos[q];
            if (MODE != PM_RANGE || ia[q] < M.len) lower(M.r, ia[q], ra[q], key);
            if (MODE != PM_RANGE || ib[q] < M.len) lower(M.r, ib[q], rb[q], key);
        }
    }
    if (MODE == PM_MAT) {
        uint32_t at[U];
        uint64_t cur[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            at[q] = live[q] ? (min(x[q].a, x[q].b) << M.lo) + max(x[q].a, x[q].b) : 0u;
            cur[q] = M.r[at[q]];
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (live[q]) lower(M.r, at[q], cur[q], ((uint64_t)x[q].w << 32) | x[q].e);
    }
}

// One pass over the list.  MAP: ends go through the map (MT in LDS, or u32 in
// the slot) and only edges between different vertices stay, in place (not
// with a matrix: the list is not needed after it).  Returns the edges kept.
template <int NT, int U, bool MAP, int MODE, typename MT, bool P16>
__device__ __forceinline__ uint32_t list_pass(const PList<P16> list, uint32_t E, const MT *map,
                                              const PMinArgs M, PCtl<NT> &pc)
{
    constexpr bool KEEP = MAP && MODE != PM_MAT;
    const uint32_t me = tile_item0<U>();
    uint32_t out = 0;
    int par = 0;
    PEdge nx[U];
#pragma unroll
    for (int q = 0; q < U; ++q) nx[q] = list.get(min((me + 64u * q), E - 1));
    for (uint32_t base = 0; base < E; base += NT * U) {
        PEdge x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = nx[q];
        // the next tile's loads are in flight while this one is worked on
        // (in place: a tile's edges are written below its own end only)
        if (base + NT * U < E) {
#pragma unroll
            for (int q = 0; q < U; ++q)
                nx[q] = list.get(min(base + NT * U + (me + 64u * q), E - 1));
        }
        if (MAP) {
#pragma unroll
            for (int q = 0; q < U; ++q) {
                x[q].a = map[x[q].a];
                x[q].b = map[x[q].b];
            }
        }
        bool live[U];
        uint32_t pos[U];
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t j = base + (me + 64u * q);
            live[q] = j < E && x[q].a != x[q].b;
            pos[q] = j;
            if (KEEP) {
                const uint64_t mask = __ballot(live[q]);
                pos[q] = c + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                c += (uint32_t)__popcll(mask);
            }
        }
        if (KEEP) {
            uint32_t tot;
            const uint32_t first = out + wave_place<NT>(c, pc, par, &tot);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                pos[q] += first;
                if (live[q]) list.put(pos[q], x[q]);
            }
            out += tot;
            par ^= 1;
        }
        lower_ends<MODE, U>(M, x, live, pos);
    }
    __syncthreads();
    return KEEP ? out : E;
}

// Hook records of the vertices [lo, lo + len) from their minima r (weight
// key, place in the list), in place: x = target, y = edge, PC_MARK for none.
// With many vertices per edge one more pass over the list lets every edge
// that is a minimum leave its other end there (streamed, 12 bytes an edge);
// otherwise each vertex reads its edge (two cache lines a vertex).
template <int NT, int U, bool P16>
__device__ __forceinline__ void hook_records(const PList<P16> list, uint32_t E, uint64_t *r,
                                             uint32_t lo, uint32_t len, uint32_t L)
{
    const uint32_t tid = threadIdx.x;
    constexpr uint32_t DONE = 0x80000000u;  // places stay below it
    const bool pass = (uint64_t)L * 8 > E;
    if (pass && E) {
        const uint32_t me = tile_item0<U>();
        PEdge nx[U];
#pragma unroll
        for (int q = 0; q < U; ++q) nx[q] = list.get(min((me + 64u * q), E - 1));
        for (uint32_t base = 0; base < E; base += NT * U) {
            PEdge x[U];
#pragma unroll
            for (int q = 0; q < U; ++q) x[q] = nx[q];
            if (base + NT * U < E) {
#pragma unroll
                for (int q = 0; q < U; ++q)
                    nx[q] = list.get(min(base + NT * U + (me + 64u * q), E - 1));
            }
            uint64_t ra[U], rb[U];
            uint32_t ia[U], ib[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const bool in = base + (me + 64u * q) < E;
                ia[q] = in ? x[q].a - lo : len;
                ib[q] = in ? x[q].b - lo : len;
                ra[q] = r[ia[q] < len ? ia[q] : 0u];
                rb[q] = r[ib[q] < len ? ib[q] : 0u];
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const uint64_t key = ((uint64_t)x[q].w << 32) | (base + (me + 64u * q));
                if (ia[q] < len && ra[q] == key) r[ia[q]] = ((uint64_t)x[q].e << 32) | DONE | x[q].b;
                if (ib[q] < len && rb[q] == key) r[ib[q]] = ((uint64_t)x[q].e << 32) | DONE | x[q].a;
            }
        }
        __syncthreads();
    }
    for (uint32_t i = tid; i < len; i += NT) {
        const uint64_t key = r[i];
        uint64_t v = ((uint64_t)PC_MARK << 32) | (lo + i);
        if (key != KEY_INF) {
            if (pass) {
                v = key & ~(uint64_t)DONE;
            } else {
                const PEdge x = list.get((uint32_t)key);
                v = ((uint64_t)x.e << 32) | (x.a == lo + i ? x.b : x.a);
            }
        }
        r[i] = v;
    }
    __syncthreads();
}

// The matrix of the pairs' minimum keys (rows of 1 << sh entries, upper
// triangle) of L vertices as the list: one edge a pair.  Returns the edges.
template <int NT, bool P16>
__device__ __forceinline__ uint32_t matrix_list(const uint64_t *mat, uint32_t L, uint32_t sh,
                                                const PList<P16> list, PCtl<NT> &pc)
{
    if (threadIdx.x == 0) pc.hooks = 0;
    __syncthreads();
    const uint32_t cells = L << sh, colm = (1u << sh) - 1u;
    for (uint32_t x0 = threadIdx.x & ~63u; x0 < cells; x0 += NT) {
        const uint32_t x = x0 + __lane_id();
        const uint64_t key = x < cells ? mat[x] : KEY_INF;  // (only i < j were lowered)
        const uint64_t mk = __ballot(key != KEY_INF);
        if (!mk) continue;
        uint32_t at = 0;
        if (__lane_id() == 0) at = atomicAdd(&pc.hooks, (uint32_t)__popcll(mk));
        at = __shfl(at, 0, 64);
        if (key != KEY_INF)
            list.put(at + __popcll(mk & lanemask_lt()),
                     PEdge{x >> sh, x & colm, (uint32_t)(key >> 32), (uint32_t)key});
    }
    __syncthreads();
    return uniform(pc.hooks);
}

// All remaining rounds of a graph with at most persist_rq(NT) * NT edges: edges in
// registers (key, ends in ab; key KEY_INF: none; qa of them a thread), minima
// and parents of its L vertices in LDS (10 bytes each, from smem on; what is
// left of its S bytes serves to deal edges out).  The edge that is a root's minimum hooks it (of two roots with the
// same one the larger), then pointer jumping; an edge whose ends meet is
// dropped, and the rest are dealt out again when a register fewer a thread
// holds them.  forest(key) is called for every forest edge; with did, did[v]
// = the number of v's tree.  A round takes 1-2 us; through the list it takes
// a pass to lower the minima, one to write the hook records and a dozen
// barriers.
template <int NT, typename F>
__device__ __forceinline__ void register_rounds(uint64_t (&key)[persist_rq(NT)], uint32_t (&ab)[persist_rq(NT)],
                                                int qa, uint32_t L, uint8_t *smem, size_t S,
                                                F forest, uint32_t *did, PCtl<NT> &pc,
                                                uint32_t *round_hooks, uint32_t &nrounds)
{
    constexpr int Q = persist_rq(NT);
    const uint32_t lane = __lane_id();
    uint64_t *r = reinterpret_cast<uint64_t *>(smem);
    uint16_t *par = reinterpret_cast<uint16_t *>(smem + 8 * (size_t)L);
    const size_t used = (10 * (size_t)L + 15) & ~(size_t)15;
    uint64_t *s_key = reinterpret_cast<uint64_t *>(smem + used);
    const uint32_t stage = (uint32_t)((S - used) / 12);  // edges there is room to deal out
    for (uint32_t v = opaque_tid(); v < L; v += NT) {
        par[v] = (uint16_t)v;
        r[v] = KEY_INF;
    }
    if (threadIdx.x < 4) pc.rc[threadIdx.x] = 0;
    if (threadIdx.x < 3) pc.rj[threadIdx.x] = 0;
    __syncthreads();
    uint32_t jump = 0;
    for (uint32_t p = 0;; p ^= 1) {  // rc[p]: this round's hooks, rc[2 + p]: its edges
        uint32_t mine = 0, at = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= qa) continue;
            if (key[q] != KEY_INF) {
                const uint32_t a = par[ab[q] & 0xFFFFu], b = par[ab[q] >> 16];
                if (a == b) key[q] = KEY_INF;
                ab[q] = a | (b << 16);
            }
            mine += (uint32_t)__popcll(__ballot(key[q] != KEY_INF));
        }
        if (lane == 0 && mine) at = atomicAdd(&pc.rc[2 + p], mine);
        __syncthreads();
        const uint32_t live = uniform(pc.rc[2 + p]);
        const int qn = (int)((live + NT - 1) / NT);
        if (qn < qa && live <= stage) {
            uint32_t *s_ab = reinterpret_cast<uint32_t *>(s_key + stage);
            at = __shfl(at, 0, 64);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint64_t mk = __ballot(key[q] != KEY_INF);
                if (key[q] != KEY_INF) {
                    const uint32_t i = at + __popcll(mk & lanemask_lt());
                    s_key[i] = key[q];
                    s_ab[i] = ab[q];
                }
                at += (uint32_t)__popcll(mk);
            }
            __syncthreads();
            qa = qn;
            const uint32_t i0 = opaque_tid();
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint32_t i = q * NT + i0;
                key[q] = KEY_INF;
                if (q < qa && i < live) {
                    key[q] = s_key[i];
                    ab[q] = s_ab[i];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= qa || key[q] == KEY_INF) continue;
            const uint32_t a = ab[q] & 0xFFFFu, b = ab[q] >> 16;
            const uint64_t ra = r[a], rb = r[b];
            lower(r, a, ra, key[q]);
            lower(r, b, rb, key[q]);
        }
        __syncthreads();
        // keys are distinct: one edge has each minimum
        uint32_t hooks = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= qa) continue;
            bool wa = false, wb = false;
            if (key[q] != KEY_INF) {
                const uint32_t a = ab[q] & 0xFFFFu, b = ab[q] >> 16;
                wa = r[a] == key[q];
                wb = r[b] == key[q];
                if (wa && (!wb || a > b)) par[a] = (uint16_t)b;
                else if (wb) par[b] = (uint16_t)a;
                if (wa || wb) forest(key[q]);
            }
            hooks += (uint32_t)__popcll(__ballot(wa || wb));
        }
        if (lane == 0 && hooks) atomicAdd(&pc.rc[p], hooks);
        __syncthreads();
        hooks = uniform(pc.rc[p]);
        if (!hooks) break;
        if (threadIdx.x == 0) {
            pc.rc[1 - p] = pc.rc[3 - p] = 0;
            if (round_hooks && nrounds < 64) round_hooks[nrounds] = hooks;
        }
        ++nrounds;
        // pointer jumping in place (a value read is always an ancestor)
        for (bool first = true;; first = false) {
            bool any = false;
            for (uint32_t v = opaque_tid(); v < L; v += NT) {
                const uint32_t x = par[v], z = par[par[x]];
                if (z != x) {
                    par[v] = (uint16_t)z;
                    any = true;
                }
                if (first) r[v] = KEY_INF;
            }
            if (any) pc.rj[jump] = 1;
            const uint32_t next = jump == 2 ? 0 : jump + 1;
            if (threadIdx.x == 0) pc.rj[next] = 0;
            __syncthreads();
            const uint32_t more = uniform(pc.rj[jump]);
            jump = next;
            if (!more) break;
        }
    }
    if (did) {
        // numbers of the trees, by their roots
        uint32_t *s_id = reinterpret_cast<uint32_t *>(smem);
        for (uint32_t v0 = opaque_tid() & ~63u; v0 < L; v0 += NT) {
            const uint32_t v = v0 + lane;
            const bool root = v < L && par[v] == v;
            const uint64_t mk = __ballot(root);
            uint32_t at = 0;
            if (lane == 0 && mk) at = atomicAdd(&pc.dead, (uint32_t)__popcll(mk));
            at = __shfl(at, 0, 64);
            if (root) s_id[v] = at + __popcll(mk & lanemask_lt());
        }
        __syncthreads();
        for (uint32_t v = opaque_tid(); v < L; v += NT) did[v] = s_id[par[v]];
    }
    __syncthreads();
}

// The same for the edges on the list, with the forest flags in the slot.
template <int NT, bool P16>
__device__ __forceinline__ void list_rounds(const PList<P16> list, uint32_t E, uint32_t L,
                                            uint8_t *smem, size_t S, uint8_t *flags,
                                            uint32_t *did, PCtl<NT> &pc, uint32_t *round_hooks,
                                            uint32_t &nrounds)
{
    const uint32_t tid = opaque_tid();
    uint64_t key[persist_rq(NT)];
    uint32_t ab[persist_rq(NT)];
    const int qa = (int)uniform((E + NT - 1) / NT);
#pragma unroll
    for (int q = 0; q < persist_rq(NT); ++q) {
        key[q] = KEY_INF;
        ab[q] = 0;
        if (q >= qa) continue;
        const uint32_t j = q * NT + tid;
        const PEdge x = list.get(min(j, E - 1));
        ab[q] = x.a | (x.b << 16);
        if (j < E) key[q] = ((uint64_t)x.w << 32) | x.e;
    }
    register_rounds<NT>(key, ab, qa, L, smem, S,
                        [=](uint64_t k) { flags[(uint32_t)k] = 1; }, did, pc, round_hooks,
                        nrounds);
}

// Targets of a round's vertices: 16-bit in LDS, or the x words of the hook
// records in the slot (more than 2^16 vertices, or a launch with little LDS).
struct H16 {
    uint16_t *h;
    __device__ __forceinline__ uint32_t get(uint32_t i) const
    {
        return __hip_atomic_load(h + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void set(uint32_t i, uint32_t v) const
    {
        __hip_atomic_store(h + i, (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};
struct HRec {
    uint2 *h;
    __device__ __forceinline__ uint32_t get(uint32_t i) const
    {
        return __hip_atomic_load(&h[i].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void set(uint32_t i, uint32_t v) const
    {
        __hip_atomic_store(&h[i].x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// Loops over a graph's vertices in device memory: items of a thread whose
// loads are issued together.  One at a time, such a loop takes a load's
// latency, 1-2 us, per NT vertices (40000 vertices, 1024 threads: 60 us).
constexpr int PC_B = 4;

// Steps along a chain of hooks before a thread turns to its next vertex.  To
// the end at once, a chain into vertices that nobody has shortened yet takes a
// step per vertex: a path of 20000 vertices with falling weights 13.0 ms a
// solve, 0.11 ms with this (0.39 ms over an adjacency matrix).  Unrolled, so
// that a step needs no count: 20000 vertices and random edges 129 us before,
// 127 us; as a loop 132 us.
constexpr int PC_WALK = 16;

// Tie break and shortcut over the targets h of a round's L vertices and the
// hooked edges in rec[i].y (PC_MARK: no edge).  Afterwards h[i] is i's root,
// and rec[root].y the root's number in the next round; a vertex without an
// edge gets dead number did[i] (if wanted) and rec[i].y = PC_MARK.
template <int NT, typename H, typename C>
__device__ __forceinline__ void tie_and_chase(const H h, uint2 *rec, uint32_t L, uint8_t *flags,
                                              uint32_t *did, C &pc)
{
    if (threadIdx.x == 0) pc.live = pc.hooks = 0;
    __syncthreads();
    uint32_t kept = 0;
    for (uint32_t i0 = opaque_tid(); i0 < L; i0 += PC_B * NT) {
        uint32_t e[PC_B], t[PC_B];
#pragma unroll
        for (int q = 0; q < PC_B; ++q) e[q] = rec[min(i0 + q * NT, L - 1)].y;
#pragma unroll
        for (int q = 0; q < PC_B; ++q) t[q] = h.get(min(i0 + q * NT, L - 1));
#pragma unroll
        for (int q = 0; q < PC_B; ++q) {
            const uint32_t i = i0 + q * NT;
            if (i >= L || e[q] == PC_MARK) continue;
            // the larger of a mutual pair never reverts, whatever it reads
            if (i < t[q] && h.get(t[q]) == i) {
                h.set(i, i);
            } else {
                flags[e[q]] = 1;
                ++kept;
            }
        }
    }
    kept = wave_sum(kept);
    if (__lane_id() == 0 && kept) atomicAdd(&pc.hooks, kept);
    __syncthreads();
    // each vertex follows its chain to the root, writing improvements back, at
    // most PC_WALK steps at a time: a thread that has not come to every root
    // goes over its vertices once more, so that every chain gets shorter
    // everywhere
    for (bool far = true; far;) {
        far = false;
        for (uint32_t i = threadIdx.x; i < L; i += NT) {
            uint32_t x = h.get(i);
            if (x == i) continue;
            bool there = false;
#pragma unroll
            for (int q = 0; q < PC_WALK; ++q) {
                const uint32_t y = h.get(x);
                there = y == x;
                if (there) break;
                x = y;
                h.set(i, x);
            }
            far = far || !there;
        }
    }
    __syncthreads();
    // numbers: roots with an edge from 0, finished trees from pc.dead
    for (uint32_t base = 0; base < L; base += PC_B * NT) {
        const uint32_t i0 = base + opaque_tid();
        bool root[PC_B];
        uint32_t y[PC_B];
#pragma unroll
        for (int q = 0; q < PC_B; ++q) {
            const uint32_t i = i0 + q * NT;
            root[q] = i < L && h.get(i) == i;
            y[q] = PC_MARK;
            if (root[q]) y[q] = rec[i].y;
        }
        uint64_t ms[PC_B], md[PC_B];
        uint32_t cs = 0, cd = 0, as = 0, ad = 0;
#pragma unroll
        for (int q = 0; q < PC_B; ++q) {
            ms[q] = __ballot(root[q] && y[q] != PC_MARK);
            md[q] = __ballot(root[q] && y[q] == PC_MARK);
            cs += (uint32_t)__popcll(ms[q]);
            cd += (uint32_t)__popcll(md[q]);
        }
        if (__lane_id() == 0) {
            if (cs) as = atomicAdd(&pc.live, cs);
            if (cd && did) ad = atomicAdd(&pc.dead, cd);
        }
        as = __shfl(as, 0, 64);
        ad = __shfl(ad, 0, 64);
#pragma unroll
        for (int q = 0; q < PC_B; ++q) {
            const uint32_t i = i0 + q * NT;
            if (root[q] && y[q] != PC_MARK) rec[i].y = as + __popcll(ms[q] & lanemask_lt());
            if (root[q] && y[q] == PC_MARK && did) did[i] = ad + __popcll(md[q] & lanemask_lt());
            as += (uint32_t)__popcll(ms[q]);
            ad += (uint32_t)__popcll(md[q]);
        }
    }
    __syncthreads();
}

// A graph's count (minus its error flags if it failed validation) and totals.
template <int NT, int WT>
__device__ __forceinline__ void graph_results(const PersistArgs &A, uint32_t g, WSum &ws,
                                              bool failed, uint32_t err, uint32_t pos,
                                              PCtl<NT> &pc, int64_t *s_sum, int64_t *s_tot)
{
    wsum_block<NT, WT>(ws, s_sum, s_tot, 1);
    if (err) atomicOr(&pc.err, err);
    if (threadIdx.x == 0) {
        const int64_t count = failed ? -(int64_t)pc.gerr : (int64_t)pos;
        const uint64_t tu = WT == MSF_W_U32 ? (uint64_t)s_tot[0] : 0;
        const double tf = exact_total_f64((uint64_t)s_tot[0], s_tot + 1,
                                          (uint32_t)s_tot[1 + ACC_DIGITS],
                                          (uint32_t)s_tot[2 + ACC_DIGITS], WT);
        if (A.one_out) {
            A.one_out->count = count;
            A.one_out->tot_u64 = tu;
            A.one_out->tot_f64 = tf;
        } else {
            A.counts[g] = count;
            A.tot_u64[(size_t)g * A.tot_stride] = tu;
            A.tot_f64[(size_t)g * A.tot_stride] = tf;
        }
    }
    __syncthreads();
}

// The edge that thread t samples for the threshold of the light edges.
template <int NT>
__device__ __forceinline__ uint32_t sampled_edge(uint32_t t, uint32_t m)
{
    return min((uint32_t)((uint64_t)m * t / NT) + (t * 0x9E3779B9u >> 8) % max(1u, m / NT), m - 1);
}

// The forest of graph g; flags (one byte per edge, in the slot) are set for
// its edges.  A graph that failed validation writes no ids (pc.gerr).
template <int NT, int U, int WT, bool P16>
__device__ __forceinline__ void solve_contracted(const PersistArgs &A, uint32_t g, uint8_t *smem,
                                                 uint8_t *slot, PCtl<NT> &pc, int64_t *s_sum, int64_t *s_tot, uint32_t *s_scan)
{
    const uint32_t tid = threadIdx.x;
    const bool one = A.one_out != nullptr;
    const int64_t v0 = one ? 0 : uniform(A.vtx_off[g]);
    const uint32_t n = uniform((uint32_t)(one ? A.one_n : A.vtx_off[g + 1] - v0));
    const int64_t e0 = one ? 0 : uniform(A.edge_off[g]);
    const uint32_t m = uniform((uint32_t)(one ? A.one_m : A.edge_off[g + 1] - e0));
    const int2 *E = reinterpret_cast<const int2 *>(A.edges) + e0;
    const uint32_t *W = A.w + e0;
    const size_t S = A.lds_bytes;
    // light edges: n ln(4 m / n) / 2, which balances the edges of the two
    // phases (here an edge costs much the same in both); below a few thousand
    // edges, or with few edges per vertex, every edge at once
    const uint32_t light = (uint32_t)(0.5f * n * __logf(4.0f * (float)m / (float)(n ? n : 1u)));
    const bool two = !A.round_hooks && m >= PERSIST_TWO_PHASE_M && m >= 2 * n && light * 5ull <= m * 3ull;
    // the slot: list 16 m, flags m (16 at a time), hook records 8 n, maps 8 n
    // (all levels), with two phases tree numbers 8 n: at most 32 m + 20 n
    // bytes (two phases only with m >= 2 n)
    const PList<P16> list(slot, m);
    uint8_t *flags = slot + 16 * (size_t)m;
    uint4 *fw = reinterpret_cast<uint4 *>(flags);
    const uint32_t nw = (m + 15) / 16;
    uint2 *rec = reinterpret_cast<uint2 *>(fw + nw);
    uint32_t *mapg = reinterpret_cast<uint32_t *>(rec + n);
    uint32_t *didg = mapg + 2 * (size_t)n;
    for (uint32_t k = tid; k < nw; k += NT) fw[k] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) {
        pc.gerr = 0;
        pc.dead = 0;
    }
    uint32_t T = 0xFFFFFFFFu, Te = 0xFFFFFFFFu;  // weight key, edge
    if (two) {
        // the threshold: the weight at the light edges' share of a sample, and
        // the last edge of that weight (with the weight alone, equal weights
        // would all be light: 3 graphs of 10^6 vertices and 3 * 10^6 edges of
        // one weight 102 ms, 52 ms with the edge)
        const uint32_t wk = weight_key(W[sampled_edge<NT>(tid, m)], WT);
        uint32_t pre = 0, want = (uint32_t)((uint64_t)light * NT / m);
        for (int sh = 24; sh >= 0; sh -= 8) {
            for (uint32_t k = tid; k < 256; k += NT) pc.hist[k] = 0;
            __syncthreads();
            if (sh == 24 || (wk >> (sh + 8)) == pre) atomicAdd(&pc.hist[(wk >> sh) & 255u], 1u);
            __syncthreads();
            if (tid < 64) {
                uint32_t c[4], t = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) t += c[q] = pc.hist[tid * 4 + q];
                uint32_t ex = wave_incl_sum(t) - t;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (want >= ex && want < ex + c[q]) {
                        pc.bin = tid * 4 + q;
                        pc.rank = want - ex;
                        pc.same = c[q];
                    }
                    ex += c[q];
                }
            }
            __syncthreads();
            pre = (pre << 8) | uniform(pc.bin);
            want = uniform(pc.rank);
            __syncthreads();
        }
        T = pre;
        if (uniform(pc.same) > 1) {
            // (the sample lies in the order of the edges; read once more, since
            // held in registers it slows the rest down by 2%)
            const uint32_t t = opaque_tid(), pos = sampled_edge<NT>(t, m);
            const bool same = weight_key(W[pos], WT) == T;
            const uint64_t eq = __ballot(same);
            if (__lane_id() == 0) pc.hist[t >> 6] = (uint32_t)__popcll(eq);
            __syncthreads();
            uint32_t at = (uint32_t)__popcll(eq & lanemask_lt());
            for (uint32_t k = 0; k < (t >> 6); ++k) at += pc.hist[k];
            if (same && at == want) pc.rank = pos;
            __syncthreads();
            Te = uniform(pc.rank);
        }
    }
    __syncthreads();
    // the list: every edge read and checked, those up to the threshold kept;
    // the first round's minima in the same pass where they fit LDS
    uint64_t *r = reinterpret_cast<uint64_t *>(smem);
    uint32_t Ec = 0, err = 0;
    bool ready = 10 * (size_t)n + 16 <= S && m > persist_rq(NT) * NT;
    if (ready)
        for (uint32_t i = tid; i < n; i += NT) r[i] = KEY_INF;
    __syncthreads();
    {
        const uint32_t me = tile_item0<U>();
        int par = 0;
        int2 uv[U];
        uint32_t wn[U];
        if (m > 0) {
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const uint32_t e = min((me + 64u * q), m - 1);
                uv[q] = E[e];
                wn[q] = W[e];
            }
        }
        for (uint32_t base = 0; base < m; base += NT * U) {
            PEdge x[U];
            uint32_t pos[U], c = 0;
            bool keep[U];
            // edges of the threshold's weight up to the tile that holds the
            // last of them
            const uint32_t Tt = base <= Te ? T : T - 1, mt = base <= Te || T ? m : 0u;
#pragma unroll
            for (int q = 0; q < U; ++q)
                x[q] = PEdge{(uint32_t)uv[q].x, (uint32_t)uv[q].y, wn[q],
                             base + (me + 64u * q)};
            if (base + NT * U < m) {  // the next tile's loads in flight meanwhile
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const uint32_t e = min(base + NT * U + (me + 64u * q), m - 1);
                    uv[q] = E[e];
                    wn[q] = W[e];
                }
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                uint32_t bad = x[q].a >= n || x[q].b >= n ? ERR_ENDPOINT : 0u;
                if (WT == MSF_W_F32 && (x[q].w & 0x7FFFFFFFu) > 0x7F800000u) bad |= ERR_NAN;
                err |= bad;
                x[q].w = weight_key(x[q].w, WT);
                keep[q] = base + (me + 64u * q) < mt && !bad && x[q].a != x[q].b && x[q].w <= Tt;
                const uint64_t mask = __ballot(keep[q]);
                pos[q] = c + (uint32_t)__popcll(mask & lanemask_lt());
                c += (uint32_t)__popcll(mask);
            }
            uint32_t tot;
            const uint32_t first = Ec + wave_place<NT>(c, pc, par, &tot);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                pos[q] += first;
                if (keep[q]) list.put(pos[q], x[q]);
            }
            if (ready) lower_ends<PM_MIN, U>(PMinArgs{r, 0, 0}, x, keep, pos);
            Ec += tot;
            par ^= 1;
        }
    }
    if (err) atomicOr(&pc.gerr, err);
    __syncthreads();
    const bool bad = uniform(pc.gerr) != 0;
    uint32_t nrounds = 0;
    for (int ph = 0; ph < (two ? 2 : 1) && !bad; ++ph) {
        const bool trees = two && ph == 0;  // tree numbers wanted
        uint32_t L = n, off = 0;
        int lev = 0;
        if (ph == 1) {
            // a tree number per vertex (at the top of LDS where they fit): the
            // later levels' maps and tree numbers in LDS, as many as there is
            // room for, where a chain is followed without a barrier; the levels
            // before them one by one, each from the level after it (a level by
            // itself takes two dependent reads and a barrier, 3 us: a third of
            // the time of a graph of 1000 vertices)
            const bool lds = 2 * ((size_t)n + 8) <= S && n <= 65536u;
            uint16_t *c16 = reinterpret_cast<uint16_t *>(smem + S) - ((n + 7) & ~7u);
            uint32_t *lm = reinterpret_cast<uint32_t *>(smem);
            const int nl = (int)uniform(pc.bin);
            const uint32_t room = (uint32_t)((lds ? S - 2 * ((size_t)n + 8) : S) / 4);
            int k1 = 1;
            while (uniform(pc.off[nl]) - uniform(pc.off[k1]) > room) ++k1;
            const uint32_t base1 = uniform(pc.off[k1]);
            for (int k = k1; k < nl; ++k) {
                const uint32_t ok = uniform(pc.off[k]), o1 = uniform(pc.off[k + 1]);
                for (uint32_t i0 = ok + opaque_tid(); i0 < o1; i0 += PC_B * NT) {
                    uint32_t x[PC_B], d[PC_B];
#pragma unroll
                    for (int q = 0; q < PC_B; ++q) {
                        x[q] = mapg[min(i0 + q * NT, o1 - 1)];
                        d[q] = didg[min(i0 + q * NT, o1 - 1)];
                    }
#pragma unroll
                    for (int q = 0; q < PC_B; ++q)
                        if (i0 + q * NT < o1)
                            lm[i0 + q * NT - base1] =
                                x[q] == PC_MARK ? PC_TREE | d[q] : o1 - base1 + x[q];
                }
            }
            __syncthreads();
            for (int k = k1 - 1; k >= 0; --k) {
                const uint32_t ok = uniform(pc.off[k]), o1 = uniform(pc.off[k + 1]), Lk = o1 - ok;
                for (uint32_t i0 = opaque_tid(); i0 < Lk; i0 += PC_B * NT) {
                    uint32_t x[PC_B], d[PC_B];
#pragma unroll
                    for (int q = 0; q < PC_B; ++q) x[q] = mapg[ok + min(i0 + q * NT, Lk - 1)];
#pragma unroll
                    for (int q = 0; q < PC_B; ++q) {
                        const uint32_t i = min(i0 + q * NT, Lk - 1);
                        d[q] = x[q];
                        if (x[q] == PC_MARK || k < k1 - 1)
                            d[q] = didg[x[q] != PC_MARK ? o1 + x[q] : ok + i];
                    }
#pragma unroll
                    for (int q = 0; q < PC_B; ++q) {
                        const uint32_t i = i0 + q * NT;
                        if (i >= Lk) continue;
                        if (x[q] != PC_MARK && k == k1 - 1) {
                            uint32_t v = lm[x[q]];
                            while (!(v & PC_TREE)) v = lm[v];
                            d[q] = v & ~PC_TREE;
                        }
                        if (lds && k == 0) c16[i] = (uint16_t)d[q];
                        else if (x[q] != PC_MARK) didg[ok + i] = d[q];
                    }
                }
                __syncthreads();
            }
            L = uniform(pc.dead);
            // the edges between different trees, again in edge-id order
            ready = lds && 8 * (size_t)L + 2 * ((size_t)n + 8) <= S;
            if (ready)
                for (uint32_t i = tid; i < L; i += NT) r[i] = KEY_INF;
            __syncthreads();
            Ec = 0;
            const uint32_t me = tile_item0<U>();
            int par = 0;
            int2 uv[U];
            uint32_t wn[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const uint32_t e = min((me + 64u * q), m - 1);
                uv[q] = E[e];
                wn[q] = W[e];
            }
            for (uint32_t base = 0; base < m; base += NT * U) {
                PEdge x[U];
                uint32_t pos[U], c = 0;
                bool keep[U];
                if (lds) {
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        x[q].a = c16[uv[q].x];
                        x[q].b = c16[uv[q].y];
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        x[q].a = didg[uv[q].x];
                        x[q].b = didg[uv[q].y];
                    }
                }
#pragma unroll
                for (int q = 0; q < U; ++q) x[q].w = weight_key(wn[q], WT);
                if (base + NT * U < m) {
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        const uint32_t e = min(base + NT * U + (me + 64u * q), m - 1);
                        uv[q] = E[e];
                        wn[q] = W[e];
                    }
                }
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    x[q].e = base + (me + 64u * q);
                    keep[q] = x[q].e < m && x[q].a != x[q].b;
                    const uint64_t mask = __ballot(keep[q]);
                    pos[q] = c + (uint32_t)__popcll(mask & lanemask_lt());
                    c += (uint32_t)__popcll(mask);
                }
                uint32_t tot;
                const uint32_t first = Ec + wave_place<NT>(c, pc, par, &tot);
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    pos[q] += first;
                    if (keep[q]) list.put(pos[q], x[q]);
                }
                if (ready) lower_ends<PM_MINF, U>(PMinArgs{r, 0, 0}, x, keep, pos);
                Ec += tot;
                par ^= 1;
            }
            __syncthreads();
        }
        // ready: this round's minima were taken when the list was written
        for (uint32_t round = 0; L > 0 && (Ec > 0 || trees); ++round) {
            if (round >= PC_LEVELS - 1) {  // every round halves the vertices with an edge
                err |= ERR_CYCLE;
                break;
            }
            if (Ec <= persist_rq(NT) * NT && 10 * (size_t)L + 16 <= S) {
                if (tid == 0) pc.off[lev] = off;
                if (trees)
                    for (uint32_t i = tid; i < L; i += NT) mapg[off + i] = PC_MARK;
                list_rounds<NT>(list, Ec, L, smem, S, flags, trees ? didg + off : nullptr, pc,
                                A.round_hooks, nrounds);
                if (trees) off += L;
                ++lev;
                break;
            }
            if (10 * (size_t)L + 16 <= S) {
                // minima, targets, numbers and the map (2 L at the top) in LDS
                if (!ready) {
                    for (uint32_t i = tid; i < L; i += NT) r[i] = KEY_INF;
                    __syncthreads();
                    if (Ec)
                        list_pass<NT, U, false, PM_MINF, uint16_t>(list, Ec, nullptr,
                                                                   PMinArgs{r, 0, 0}, pc);
                }
                uint2 *lrec = reinterpret_cast<uint2 *>(smem);
                hook_records<NT, U>(list, Ec, r, 0, L, L);
                tie_and_chase<NT>(HRec{lrec}, lrec, L, flags, trees ? didg + off : nullptr, pc);
                uint16_t *map = reinterpret_cast<uint16_t *>(smem + S) - ((L + 7) & ~7u);
                for (uint32_t i = tid; i < L; i += NT) {
                    const uint32_t v = lrec[lrec[i].x].y;
                    map[i] = (uint16_t)v;
                    if (trees) mapg[off + i] = v;
                }
            } else {
                // minima by vertex ranges that fit LDS, hook records in the slot
                const uint32_t rs = (uint32_t)(S / 8);
                for (uint32_t lo = 0; lo < L; lo += rs) {
                    const uint32_t len = min(rs, L - lo);
                    for (uint32_t i = tid; i < len; i += NT) r[i] = KEY_INF;
                    __syncthreads();
                    if (Ec)
                        list_pass<NT, U, false, PM_RANGE, uint16_t>(list, Ec, nullptr,
                                                                    PMinArgs{r, lo, len}, pc);
                    hook_records<NT, U>(list, Ec, r, lo, len, L);
                    for (uint32_t i = tid; i < len; i += NT) {
                        const uint64_t v = r[i];
                        rec[lo + i] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                    }
                    __syncthreads();
                }
                if (2 * ((size_t)L + 8) <= S && L <= 65536u) {
                    uint16_t *map = reinterpret_cast<uint16_t *>(smem + S) - ((L + 7) & ~7u);
                    for (uint32_t i0 = opaque_tid(); i0 < L; i0 += PC_B * NT) {
                        uint32_t v[PC_B];
#pragma unroll
                        for (int q = 0; q < PC_B; ++q) v[q] = rec[min(i0 + q * NT, L - 1)].x;
#pragma unroll
                        for (int q = 0; q < PC_B; ++q)
                            if (i0 + q * NT < L) map[i0 + q * NT] = (uint16_t)v[q];
                    }
                    __syncthreads();
                    tie_and_chase<NT>(H16{map}, rec, L, flags, trees ? didg + off : nullptr, pc);
                    for (uint32_t i0 = opaque_tid(); i0 < L; i0 += PC_B * NT) {
                        uint32_t v[PC_B];
#pragma unroll
                        for (int q = 0; q < PC_B; ++q) v[q] = rec[map[min(i0 + q * NT, L - 1)]].y;
#pragma unroll
                        for (int q = 0; q < PC_B; ++q) {
                            const uint32_t i = i0 + q * NT;
                            if (i >= L) continue;
                            map[i] = (uint16_t)v[q];  // only its own thread reads it now
                            if (trees) mapg[off + i] = v[q];
                        }
                    }
                } else {
                    tie_and_chase<NT>(HRec{rec}, rec, L, flags, trees ? didg + off : nullptr, pc);
                    for (uint32_t i = tid; i < L; i += NT) mapg[off + i] = rec[rec[i].x].y;
                }
            }
            const uint32_t Ln = uniform(pc.live);
            if (A.round_hooks && tid == 0 && nrounds < 64) A.round_hooks[nrounds] = pc.hooks;
            ++nrounds;
            if (tid == 0) pc.off[lev] = off;
            ++lev;
            // the next round's list, and its minima where map and minima fit;
            // with few vertices left the pairs' minima instead, and the
            // remaining rounds on them
            const bool m16 = 2 * ((size_t)L + 8) <= S && L <= 65536u;
            const uint16_t *map = reinterpret_cast<uint16_t *>(smem + S) - ((L + 7) & ~7u);
            const uint32_t sh = Ln <= 32 ? 5u : Ln <= 64 ? 6u : 7u;
            const bool mat = m16 && Ln > 0 && Ln <= PC_MAT && Ln * (Ln - 1) <= 2 * persist_rq(NT) * NT &&
                             (8ull * Ln << sh) + 2 * ((size_t)L + 8) <= S;
            ready = m16 && 8 * (size_t)Ln + 2 * ((size_t)L + 8) <= S;
            __syncthreads();
            const uint32_t words = mat ? Ln << sh : ready ? Ln : 0u;
            for (uint32_t i = tid; i < words; i += NT) r[i] = KEY_INF;
            __syncthreads();
            if (mat) {
                if (Ec)
                    list_pass<NT, U, true, PM_MAT, uint16_t>(list, Ec, map, PMinArgs{r, sh, 0},
                                                             pc);
                if (trees) {
                    off += L;
                    if (tid == 0) pc.off[lev] = off;
                    for (uint32_t i = tid; i < Ln; i += NT) mapg[off + i] = PC_MARK;
                }
                Ec = matrix_list<NT>(r, Ln, sh, list, pc);
                list_rounds<NT>(list, Ec, Ln, smem, S, flags, trees ? didg + off : nullptr, pc,
                                A.round_hooks, nrounds);
                if (trees) off += Ln;
                ++lev;
                break;
            }
            if (Ec) {
                const PMinArgs M{r, 0, 0};
                if (ready && Ln >= 1024)
                    Ec = list_pass<NT, U, true, PM_MIN, uint16_t>(list, Ec, map, M, pc);
                else if (ready)
                    Ec = list_pass<NT, U, true, PM_MINF, uint16_t>(list, Ec, map, M, pc);
                else if (m16)
                    Ec = list_pass<NT, U, true, PM_NONE, uint16_t>(list, Ec, map, M, pc);
                else
                    Ec = list_pass<NT, U, true, PM_NONE, uint32_t>(list, Ec, mapg + off, M, pc);
            }
            if (trees) off += L;
            L = Ln;
        }
        if (tid == 0) {
            pc.off[lev] = off;
            pc.bin = (uint32_t)lev;  // levels of the first phase
        }
        __syncthreads();
        if (err & ERR_CYCLE) break;
    }
    if (A.round_hooks && tid == 0) {
        // the round that finds no edge left
        if (nrounds < 64) A.round_hooks[nrounds] = 0;
        A.round_hooks[64] = nrounds + 1;
    }

    // ---- output: ascending forest ids, count, totals ----------------------
    // a graph that failed validation writes no ids (the call fails); its
    // count is minus its error flags
    if (err) atomicOr(&pc.gerr, err);
    __syncthreads();
    const bool failed = uniform(pc.gerr) != 0;
    WSum ws;
    uint32_t pos = 0;
    int32_t *out = A.out + v0;
    // through LDS, so that the ids leave in whole lines and their weights'
    // loads go out together (each thread reading the weights of its 16 edges'
    // one after the other: 91 us for 1024 graphs of 40000 vertices and four
    // edges each, of 886 us in all)
    uint16_t *s_id = reinterpret_cast<uint16_t *>(smem);
    static_assert(16 * NT <= 65536, "places of a tile in 16 bits");
    uint4 f4 = make_uint4(0u, 0u, 0u, 0u);
    if (tid < nw && !failed) f4 = fw[tid];
    for (uint32_t base = 0; base < nw && !failed; base += NT) {
        const uint32_t f[4] = {f4.x, f4.y, f4.z, f4.w};
        f4 = make_uint4(0u, 0u, 0u, 0u);
        if (base + NT + tid < nw) f4 = fw[base + NT + tid];  // the next tile's, meanwhile
        const uint32_t c = __popc(f[0]) + __popc(f[1]) + __popc(f[2]) + __popc(f[3]);
        uint32_t total;
        uint32_t at = block_excl_sum<NT>(c, s_scan, &total);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (uint32_t bits = f[q]; bits; bits &= bits - 1)
                s_id[at++] = (uint16_t)(16 * tid + 4 * q + (__builtin_ctz(bits) >> 3));
        __syncthreads();
        for (uint32_t i0 = opaque_tid(); i0 < total; i0 += PC_B * NT) {
            uint32_t e[PC_B], w[PC_B];
#pragma unroll
            for (int q = 0; q < PC_B; ++q) e[q] = 16 * base + s_id[min(i0 + q * NT, total - 1)];
#pragma unroll
            for (int q = 0; q < PC_B; ++q) w[q] = W[e[q]];
#pragma unroll
            for (int q = 0; q < PC_B; ++q) {
                if (i0 + q * NT >= total) continue;
                out[pos + i0 + q * NT] = (int32_t)e[q];
                wsum_add<WT>(ws, weight_key(w[q], WT));
            }
        }
        pos += total;
        __syncthreads();
    }
    graph_results<NT, WT>(A, g, ws, failed, err, pos, pc, s_sum, s_tot);
}

// The forest of a graph whose edges fit the registers of the workgroup: all
// rounds on chip, the forest as bits in LDS.  (Through the list and the flags in the slot, a graph of a few
// hundred edges waits for a dozen dependent device accesses, 1 us each.)
template <int NT, int WT>
__device__ __forceinline__ void solve_registers(const PersistArgs &A, uint32_t g, uint8_t *smem,
                                                PCtl<NT> &pc, int64_t *s_sum, int64_t *s_tot,
                                                uint32_t *s_scan)
{
    const uint32_t tid = opaque_tid();
    const bool one = A.one_out != nullptr;
    const int64_t v0 = one ? 0 : uniform(A.vtx_off[g]);
    const uint32_t n = uniform((uint32_t)(one ? A.one_n : A.vtx_off[g + 1] - v0));
    const int64_t e0 = one ? 0 : uniform(A.edge_off[g]);
    const uint32_t m = uniform((uint32_t)(one ? A.one_m : A.edge_off[g + 1] - e0));
    const int2 *E = reinterpret_cast<const int2 *>(A.edges) + e0;
    const uint32_t *W = A.w + e0;
    const int qa = (int)uniform((m + NT - 1) / NT);
    int2 uv[persist_rq(NT)];
    uint32_t wb[persist_rq(NT)], ab[persist_rq(NT)];
    uint64_t key[persist_rq(NT)];
#pragma unroll
    for (int q = 0; q < persist_rq(NT); ++q) {
        if (q >= qa) continue;
        const uint32_t j = min(q * NT + tid, m - 1);
        uv[q] = E[j];
        wb[q] = W[j];
    }
    uint32_t *bits = reinterpret_cast<uint32_t *>(smem);
    constexpr uint32_t BYTES = persist_rq(NT) * NT / 8;
    for (uint32_t i = opaque_tid(); i < BYTES / 4; i += NT) bits[i] = 0;
    if (threadIdx.x == 0) {
        pc.gerr = 0;
        pc.dead = 0;
    }
    __syncthreads();
    uint32_t err = 0;
#pragma unroll
    for (int q = 0; q < persist_rq(NT); ++q) {
        key[q] = KEY_INF;
        ab[q] = 0;
        if (q >= qa) continue;
        const uint32_t j = q * NT + tid, a = (uint32_t)uv[q].x, b = (uint32_t)uv[q].y;
        uint32_t bad = a >= n || b >= n ? ERR_ENDPOINT : 0u;
        if (WT == MSF_W_F32 && (wb[q] & 0x7FFFFFFFu) > 0x7F800000u) bad |= ERR_NAN;
        err |= bad;
        if (j < m && !bad && a != b) {
            key[q] = ((uint64_t)weight_key(wb[q], WT) << 32) | j;
            ab[q] = a | (b << 16);
        }
    }
    if (err) {
        atomicOr(&pc.gerr, err);
        atomicOr(&pc.err, err);
    }
    __syncthreads();
    const bool failed = uniform(pc.gerr) != 0;
    uint32_t pos = 0, nrounds = 0;
    if (!failed)
        register_rounds<NT>(
            key, ab, qa, n, smem + BYTES, A.lds_bytes - BYTES,
            [&](uint64_t k) {
                const uint32_t e = (uint32_t)k;
                atomicOr(&bits[e >> 5], 1u << (e & 31));
            },
            nullptr, pc, A.round_hooks, nrounds);
    WSum ws;
    if (!failed) {
        // as many edges a thread (their weights once more, from the caches:
        // sums held through the rounds would not leave enough registers)
        const uint32_t j0 = persist_rq(NT) * opaque_tid();
        const uint32_t f = (bits[j0 >> 5] >> (j0 & 31)) & ((1u << persist_rq(NT)) - 1u);
        uint32_t w[persist_rq(NT)];
#pragma unroll
        for (int q = 0; q < persist_rq(NT); ++q) w[q] = (f >> q) & 1 ? W[j0 + q] : 0u;
        uint32_t at = block_excl_sum<NT>(__popc(f), s_scan, &pos);
        int32_t *out = A.out + v0;
#pragma unroll
        for (int q = 0; q < persist_rq(NT); ++q) {
            if (!((f >> q) & 1)) continue;
            out[at++] = (int32_t)(j0 + q);
            wsum_add<WT>(ws, weight_key(w[q], WT));
        }
    }
    if (A.round_hooks && threadIdx.x == 0) {
        // the round that finds no edge left
        if (nrounds < 64) A.round_hooks[nrounds] = 0;
        A.round_hooks[64] = nrounds + 1;
    }
    graph_results<NT, WT>(A, g, ws, failed, 0, pos, pc, s_sum, s_tot);
}

}  // namespace

template <int NT, int EPT, int WT>
__global__ __launch_bounds__(NT, 4) void k_persist(PersistArgs A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ PCtl<NT> pc;
    __shared__ int64_t s_sum[(NT / 64) * (ACC_DIGITS + 1)];
    __shared__ int64_t s_tot[WS_WORDS];
    __shared__ uint32_t s_scan[NT / 64 + 1];
    uint8_t *slot = A.scratch + (size_t)blockIdx.x * A.slot_bytes;
    const uint64_t t0 = wall_clock64();
    const bool one = A.one_out != nullptr;
    if (threadIdx.x == 0) pc.err = 0;
    for (bool first = true;; first = false) {
        if (threadIdx.x == 0) {
            const uint32_t k = one ? (first ? 0u : 1u) : atomicAdd(A.queue, 1u);
            pc.g = k < (uint32_t)A.G ? (!one && A.order ? A.order[k] : k) : NONE32;
        }
        __syncthreads();
        const uint32_t g = uniform(pc.g);
        if (g == NONE32) break;
        const uint32_t n = (uint32_t)(one ? A.one_n : A.vtx_off[g + 1] - A.vtx_off[g]);
        const uint32_t m = (uint32_t)(one ? A.one_m : A.edge_off[g + 1] - A.edge_off[g]);
        // vertex numbers of at most 16 bits: both ends of an edge in one word
        if (uniform((uint32_t)persist_in_registers(n, m, NT, A.lds_bytes)))
            solve_registers<NT, WT>(A, g, smem, pc, s_sum, s_tot, s_scan);
        else if (n <= 65536)
            solve_contracted<NT, EPT, WT, true>(A, g, smem, slot, pc, s_sum, s_tot, s_scan);
        else
            solve_contracted<NT, EPT, WT, false>(A, g, smem, slot, pc, s_sum, s_tot, s_scan);
    }
    if (one) {
        // (round_hooks was written before the last barriers)
        if (threadIdx.x < 65) A.one_out->hooks[threadIdx.x] = A.round_hooks[threadIdx.x];
        if (threadIdx.x == 0) {
            A.one_out->err = pc.err;
            A.one_out->clk = wall_clock64() - t0;
        }
    } else if (threadIdx.x == 0 && pc.err) {
        atomicOr(A.err, pc.err);
    }
}

// Queue counter and error word to zero (a kernel, not a memset, so the
// launch sequence can be captured into a graph).
__global__ void k_persist_reset(uint32_t *queue, uint32_t *err)
{
    if (threadIdx.x == 0) {
        *queue = 0;
        *err = 0;
    }
}

namespace {

template <int NT, int EPT>
hipError_t launch_cfg(hipStream_t s, const PersistArgs &A, int wt, unsigned grid)
{
    const size_t dyn = A.lds_bytes;
    if (wt == MSF_W_F32) {
        (void)hipFuncSetAttribute((const void *)k_persist<NT, EPT, MSF_W_F32>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
        k_persist<NT, EPT, MSF_W_F32><<<grid, NT, dyn, s>>>(A);
    } else {
        (void)hipFuncSetAttribute((const void *)k_persist<NT, EPT, MSF_W_U32>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
        k_persist<NT, EPT, MSF_W_U32><<<grid, NT, dyn, s>>>(A);
    }
    return hipGetLastError();
}

}  // namespace

int persist_blocks_per_cu(const PersistCfg &cfg, int wt)
{
    // one occupancy query per (device, configuration, weight type)
    static std::mutex mu;
    static std::map<std::tuple<int, int, int, uint32_t, int>, int> known;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const auto key = std::make_tuple(dev, cfg.nt, cfg.ept, (uint32_t)cfg.lds, wt);
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = known.find(key);
        if (it != known.end()) return it->second;
    }
    const void *f = nullptr;
#define MSF_PERSIST_FN(NT_, EPT_)                                                            \
    if (cfg.nt == NT_ && cfg.ept == EPT_)                                                   \
        f = wt == MSF_W_F32 ? (const void *)k_persist<NT_, EPT_, MSF_W_F32>                  \
                            : (const void *)k_persist<NT_, EPT_, MSF_W_U32>;
    MSF_PERSIST_FN(256, 4)
    MSF_PERSIST_FN(512, 2)
    MSF_PERSIST_FN(512, 4)
    MSF_PERSIST_FN(1024, 2)
    MSF_PERSIST_FN(1024, 4)
#undef MSF_PERSIST_FN
    if (!f) return 0;
    (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)cfg.lds);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, cfg.nt, cfg.lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    std::lock_guard<std::mutex> lk(mu);
    known[key] = nb;
    return nb;
}

const PersistCfg *persist_candidates(int *count)
{
    // threads per workgroup x edges per thread and load round x dynamic LDS
    // (which sets how many workgroups share a compute unit)
    static const PersistCfg c[] = {
        {256, 4, 32 << 10},  {512, 2, 32 << 10},  {512, 4, 64 << 10},  {512, 4, 32 << 10},
        {1024, 2, 64 << 10}, {1024, 4, 64 << 10}, {1024, 2, 150 << 10}, {1024, 4, 150 << 10},
    };
    *count = (int)(sizeof(c) / sizeof(c[0]));
    return c;
}

hipError_t launch_persist(hipStream_t s, const PersistArgs &A, const PersistCfg &cfg, int wt,
                          unsigned grid, bool reset)
{
    if (reset) k_persist_reset<<<1, 64, 0, s>>>(A.queue, A.err);
    if (cfg.nt == 256 && cfg.ept == 4) return launch_cfg<256, 4>(s, A, wt, grid);
    if (cfg.nt == 512 && cfg.ept == 2) return launch_cfg<512, 2>(s, A, wt, grid);
    if (cfg.nt == 512 && cfg.ept == 4) return launch_cfg<512, 4>(s, A, wt, grid);
    if (cfg.nt == 1024 && cfg.ept == 2) return launch_cfg<1024, 2>(s, A, wt, grid);
    if (cfg.nt == 1024 && cfg.ept == 4) return launch_cfg<1024, 4>(s, A, wt, grid);
    return hipErrorInvalidValue;
}

}  // namespace msf
