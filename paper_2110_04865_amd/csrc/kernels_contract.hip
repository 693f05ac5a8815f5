// Rounds of Algorithm 2 over an edge list whose ends are renumbered every
// round, light edges first.
//
// The forest is unique under the order of the keys (weight, edge id), so an
// edge that joins two vertices of one tree of the forest of all lighter
// edges is not in it (the cycle property).  From half a million edges on,
// phase 0 therefore takes only the lightest edges (about 0.4 n ln(4 m / n) of
// them, by a sampled threshold on the key) and builds their forest; one pass
// over the input then drops every edge inside a tree of it, and phase 1
// continues with the few edges left
// between the trees.  Each phase runs the rounds of Algorithm 2:
//   edges   the multilinear kernel of section 3.1 with the projection: every
//           edge {a, b} with key x lowers r[a] and r[b] to x.  After the
//           first round the pass first maps the ends to this round's
//           vertices and keeps only the edges between different ones, in
//           place;
//   hook    every vertex hooks onto the far end of its minimum edge;
//   tie     of two vertices that hooked onto each other the smaller stays;
//           the vertices that stay get the next round's numbers, those
//           without an edge (a finished tree) a tree number;
//   chase   complete shortcutting (section 4.2), giving every vertex the
//           number of its new tree (chains of hooks that it cannot follow
//           are left to launches of their own behind a host step, ct_far).
// So a round costs its live edges once and its vertices a few times, and
// both shrink; no adjacency matrix is built.
//
// Every wave owns one segment of the list, so the compaction is a ballot
// and an in-place store: no barrier and no counter.  Kernels take their
// sizes from the counters on the device and return at once when there is
// nothing to do, so a whole solve is enqueued without a host round trip (one
// follows if a phase needs more rounds, or a chain is given up).
// A round of at most CT_FINISH vertices needs only the edge pass: its last
// workgroup to finish does the rest of the round in LDS.
//
// Measured, us a solve over an adjacency matrix / over the list: R-MAT s16
// (0.91M edges) 672 / 188, grid 101^3 1671 / 459, R-MAT s22 (64M edges) 4436 /
// 1894, grid 256^3 (47.6M) 8735 / 3407.  Large rounds are bound by lookups
// (57-205 G/s by the table's size) and device-scope minima (27 G/s), small
// ones by chains of dependent accesses of 1 us each.
#include <algorithm>

#include "contract.hpp"
#include "exact_sum.hpp"
#include "wave.hpp"

namespace msf {

namespace {

constexpr int CE_NT = 1024;               // threads of the list kernels
constexpr int CE_WV = CE_NT / 64;
constexpr int CI_NT = 256;                // of the set-up
constexpr int TIE_NT = 512;               // of the hook
constexpr uint32_t CT_DEAD = 0x80000000u; // a finished tree's number
constexpr uint32_t CT_SAMPLES = 2048;

__device__ __forceinline__ uint32_t ct_wkey(uint32_t bits, int wt)
{
    return wt == MSF_W_F32 ? wkey_f32_bits(bits) : bits;
}

__device__ __forceinline__ bool ct_nan(uint32_t bits, int wt)
{
    return wt == MSF_W_F32 && (bits & 0x7FFFFFFFu) > 0x7F800000u;
}

// Round k >= 1's map starts here in maps: round j has at most n >> j vertices.
__host__ __device__ inline size_t ct_map_at(int32_t n, int k)
{
    size_t at = 0;
    for (int j = 1; j < k; ++j) at += (((size_t)n >> j) + 63) & ~(size_t)63;
    return at;
}

__device__ __forceinline__ uint32_t *ct_map(const CtArgs &A, int k)
{
    return k == 0 ? A.map0 : A.maps + ct_map_at(A.n, k);
}

__device__ __forceinline__ uint32_t ct_uniform(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// r[i] <- min(r[i], x), where a read of r[i] gave cur (r only falls, so a
// stale read can cost an atomic, never lose one).
__device__ __forceinline__ void lower_dev(uint64_t *r, uint32_t i, uint64_t cur, uint64_t x)
{
    if (x < cur) __hip_atomic_fetch_min(r + i, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void lower_lds(uint64_t *r, uint32_t i, uint64_t cur, uint64_t x)
{
    if (x < cur) __hip_atomic_fetch_min(r + i, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Workgroups of the largest round's hook, a slot of partial sums each.
__host__ __device__ inline uint32_t ct_wslots(int32_t n)
{
    const uint32_t g = ((uint32_t)n + 2 * TIE_NT - 1) / (2 * TIE_NT);
    return g < 1 ? 1 : g < CT_WSLOTS ? g : CT_WSLOTS;
}

unsigned grid_for(size_t n, unsigned block, unsigned cap)
{
    size_t g = (n + block - 1) / block;
    return (unsigned)std::max<size_t>(1, std::min<size_t>(g, cap));
}

}  // namespace

uint32_t ct_wslots_host(int32_t n) { return ct_wslots(n); }

size_t ct_maps_words(int32_t n) { return ct_map_at(n, 34) + 64; }

size_t ct_wpart_bytes() { return 8 * (size_t)CT_WSLOTS * WS_WORDS; }

// ----------------------------------------------------------------- set-up --

// The rank-th smallest key of a sample of CT_SAMPLES edges (one from each of
// as many equal stretches of the input, at a mixed place): the threshold of
// phase 0.  One workgroup beside those of the set-up (a launch of its own
// takes 6 us more), samples in registers, eight bits per step until
// the bin holds one sample (the second or third step, unless weights repeat).
__device__ void ct_threshold(const CtArgs &A, uint32_t rank)
{
    __shared__ uint32_t s_hist[256];
    __shared__ uint32_t s_bin, s_rank, s_num;
    constexpr int PER = CT_SAMPLES / CI_NT;
    uint64_t key[PER];
    const uint64_t m = (uint64_t)A.m;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t i = q * CI_NT + threadIdx.x;
        const uint64_t lo = m * i / CT_SAMPLES, hi = m * (i + 1) / CT_SAMPLES;
        uint32_t x = i * 0x9E3779B9u + 0x7F4A7C15u;
        x ^= x >> 15;
        x *= 0x2C1B3C6Du;
        x ^= x >> 12;
        uint64_t e = lo + (((hi - lo) * (uint64_t)x) >> 32);
        if (e >= m) e = m - 1;
        key[q] = ((uint64_t)ct_wkey(A.w[e], A.wt) << 32) | e;
    }
    uint64_t pre = 0;
    uint32_t want = rank;
    for (int sh = 56;; sh -= 8) {
        if (threadIdx.x < 256) s_hist[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (sh == 56 || (key[q] >> (sh + 8)) == pre)
                atomicAdd(&s_hist[(uint32_t)(key[q] >> sh) & 255u], 1u);
        __syncthreads();
        if (threadIdx.x < 64) {
            uint32_t c[4], t = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) t += c[q] = s_hist[threadIdx.x * 4 + q];
            uint32_t ex = wave_incl_sum(t) - t;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (want >= ex && want < ex + c[q]) {
                    s_bin = threadIdx.x * 4 + q;
                    s_rank = want - ex;
                    s_num = c[q];
                }
                ex += c[q];
            }
        }
        __syncthreads();
        pre = (pre << 8) | s_bin;
        want = s_rank;
        if (s_num == 1 || sh == 0) {
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if ((key[q] >> sh) == pre) A.cnt->ct.T = key[q];
            return;
        }
        __syncthreads();
    }
}

// rank: of the threshold in the sample, which one more workgroup takes, or
// NONE32 for every edge.
__global__ __launch_bounds__(CI_NT) void k_ct_init(CtArgs A, size_t flag_words, uint32_t rank)
{
    const uint32_t blocks = gridDim.x - (rank != NONE32);
    if (blockIdx.x == blocks) {
        ct_threshold(A, rank);
        return;
    }
    const size_t stride = (size_t)blocks * blockDim.x;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0) {
        uint32_t *c = reinterpret_cast<uint32_t *>(A.cnt);
        // (the threshold is set elsewhere, or to every key below)
        const uint32_t t = offsetof(Counters, ct.T) / 4;
        for (uint32_t i = threadIdx.x; i < sizeof(Counters) / 4; i += CI_NT)
            if (i != t && i != t + 1) c[i] = 0u;
        __syncthreads();
        if (threadIdx.x == 0) {
            A.cnt->ct.L[0][0] = (uint32_t)A.n;
            if (rank == NONE32) A.cnt->ct.T = KEY_INF;
            A.cnt->ct.clk[0] = wall_clock64();
        }
    }
    uint32_t *fl = reinterpret_cast<uint32_t *>(A.flags);
    for (size_t i = i0; i < (size_t)A.n; i += stride) A.r[0][i] = KEY_INF;
    for (size_t i = i0; i < flag_words; i += stride) fl[i] = 0u;
    const uint32_t slots = ct_wslots(A.n);
    for (size_t i = i0; i < (size_t)slots * WS_WORDS; i += stride)
        A.wpart[i / slots * CT_WSLOTS + i % slots] = 0;
    for (size_t i = i0; i < CT_PAIR * CT_PAIR; i += stride) A.mat[i] = KEY_INF;
}

void ct_init(hipStream_t s, const CtArgs &A, size_t flag_words, int64_t light)
{
    uint32_t rank = NONE32;
    if (light < A.m) {  // else every edge
        const double f = (double)light / (double)A.m;
        rank = std::min<uint32_t>((uint32_t)(f * CT_SAMPLES), CT_SAMPLES - 1);
    }
    const unsigned g = grid_for(std::max<size_t>((size_t)A.n, flag_words), CI_NT, 4096);
    k_ct_init<<<g + (rank != NONE32), CI_NT, 0, s>>>(A, flag_words, rank);
}

// ------------------------------------------------------- list of phase 0 --
// Every edge read once and checked; those up to the threshold (no loops) go
// to the wave's segment.  A wave takes every W-th tile, so the segments are
// even whatever the order of the input.

// A wave's tile t of the input (indices past the end clamped).
template <bool WEIGHTS>
__device__ __forceinline__ void ct_load(const CtArgs &A, int64_t t, int lane, int2 (&uv)[4],
                                        uint32_t (&wb)[4])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int64_t e = t * CT_TILE + q * 64 + lane;
        e = e < A.m ? e : A.m - 1;
        uv[q] = A.edges[e];
        if (WEIGHTS) wb[q] = A.w[e];
    }
}

__global__ __launch_bounds__(CE_NT) void k_ct_select(CtArgs A)
{
    __shared__ uint32_t s_cnt[CE_WV];
    const int lane = __lane_id();
    const uint32_t wv = ct_uniform(blockIdx.x * CE_WV + (threadIdx.x >> 6));
    const uint64_t T = A.cnt->ct.T;
    const int64_t tiles = (A.m + CT_TILE - 1) / CT_TILE;
    const uint32_t n = (uint32_t)A.n;
    CtEdge *seg = A.list + (size_t)wv * A.segcap;
    uint32_t out = 0, err = 0;
    int2 uv[4];
    uint32_t wb[4];
    ct_load<true>(A, wv, lane, uv, wb);
    for (int64_t t = wv; t < tiles; t += A.W) {
        int2 x[4];
        uint32_t y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[q] = uv[q];
            y[q] = wb[q];
        }
        // the next tile's loads are in flight meanwhile
        if (t + A.W < tiles) ct_load<true>(A, t + A.W, lane, uv, wb);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t e = t * CT_TILE + q * 64 + lane;
            const uint32_t a = (uint32_t)x[q].x, b = (uint32_t)x[q].y;
            uint32_t bad = a >= n || b >= n ? ERR_ENDPOINT : 0u;
            if (ct_nan(y[q], A.wt)) bad |= ERR_NAN;
            err |= bad;
            const uint64_t key = ((uint64_t)ct_wkey(y[q], A.wt) << 32) | (uint32_t)e;
            const bool sel = e < A.m && !bad && a != b && key <= T;
            const uint64_t mask = __ballot(sel);
            if (sel) seg[out + __popcll(mask & lanemask_lt())] = CtEdge{a, b, key};
            out += (uint32_t)__popcll(mask);
        }
    }
    if (err) atomicOr(&A.cnt->err, err);
    if (lane == 0) {
        A.cw[wv] = out;
        s_cnt[threadIdx.x >> 6] = out;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < CE_WV; ++i) t += s_cnt[i];
        if (t) atomicAdd(&A.cnt->ct.E0[0], t);
    }
}

void ct_select(hipStream_t s, const CtArgs &A) { k_ct_select<<<A.W / CE_WV, CE_NT, 0, s>>>(A); }

// ------------------------------------------------------------- edge pass --

namespace {

// The vertices of round k that the ends of U minimum edges lie in: through
// the maps of the rounds before it, and from the first small round (tl) on
// through one cumulative map.  Each step's loads are issued together.
template <int U>
__device__ __forceinline__ void ct_ends(const CtArgs &A, const uint64_t (&key)[U], int k, int tl,
                                        uint32_t (&a)[U], uint32_t (&b)[U])
{
    // every lane loads, from place 0 without an edge: loads behind a branch
    // would wait for each other
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int2 uv = A.edges[key[q] != KEY_INF ? (uint32_t)key[q] : 0u];
        a[q] = (uint32_t)uv.x;
        b[q] = (uint32_t)uv.y;
    }
    const int top = k < tl ? k : tl;
    for (int l = A.comp ? -1 : 0; l <= top; ++l) {
        if (l == top && k <= tl) break;
        const uint32_t *map = l < 0 ? A.comp : l < top ? ct_map(A, l) : A.cum;
        uint32_t x[U], y[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            x[q] = map[key[q] != KEY_INF ? a[q] : 0u];
            y[q] = map[key[q] != KEY_INF ? b[q] : 0u];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            a[q] = x[q];
            b[q] = y[q];
        }
    }
}

// What a small round's last workgroup needs from the counters, read before
// the pass (only that workgroup changes them).
struct CtSmall {
    uint32_t tl1;   // 1 + the phase's first small round, if there was one
    uint32_t L0;    // that round's vertices (else this one's)
    uint32_t dead;  // finished trees
    uint32_t wl;    // weight keys listed
};

// The rest of round k in one workgroup (at most CT_SMALL vertices): hook,
// tie break, shortcut and the next round's numbers, with the targets in LDS.
__device__ void ct_small_round(const CtArgs &A, int k, uint32_t L, const CtSmall &z,
                               uint32_t *s_h, uint32_t *s_nid, uint32_t *s_c)
{
    Counters *c = A.cnt;
    const uint32_t tid = threadIdx.x;
    const uint64_t *r = A.r[k & 1];
    const uint32_t tl1 = z.tl1, dead0 = z.dead, wl0 = z.wl;
    const int tl = tl1 ? (int)tl1 - 1 : k;
    constexpr int IT = (CT_SMALL + CE_NT - 1) / CE_NT;
    uint64_t key[IT];
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const uint32_t i = q * CE_NT + tid;
        key[q] = i < L ? load_relaxed_u64(r + i) : KEY_INF;
    }
    uint32_t a[IT], b[IT];
    ct_ends<IT>(A, key, k, tl, a, b);
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const uint32_t i = q * CE_NT + tid;
        if (i < L) s_h[i] = key[q] == KEY_INF ? i : (a[q] == i ? b[q] : a[q]);
    }
    if (tid < 4) s_c[tid] = 0;
    __syncthreads();
    // the larger of a mutual pair never reverts, whatever it reads
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const uint32_t i = q * CE_NT + tid;
        if (i >= L) continue;
        const uint32_t t = s_h[i];
        if (i < t && s_h[t] == i) s_h[i] = i;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        if (q * CE_NT >= L) break;
        const uint32_t i = q * CE_NT + tid;
        const bool in = i < L, live = in && key[q] != KEY_INF;
        const bool stay = live && s_h[i] == i, dead = in && !live, hook = live && !stay;
        const uint64_t ms = __ballot(stay), md = __ballot(dead), mh = __ballot(hook);
        uint32_t at[3] = {0, 0, 0};
        if (__lane_id() == 0) {
            if (ms) at[0] = atomicAdd(&s_c[0], (uint32_t)__popcll(ms));
            if (md) at[1] = atomicAdd(&s_c[1], (uint32_t)__popcll(md));
            if (mh) at[2] = atomicAdd(&s_c[2], (uint32_t)__popcll(mh));
        }
        const uint64_t lt = lanemask_lt();
        const uint32_t bs = __shfl(at[0], 0, 64), bd = __shfl(at[1], 0, 64),
                       bh = __shfl(at[2], 0, 64);
        if (stay) s_nid[i] = bs + __popcll(ms & lt);
        if (dead) s_nid[i] = CT_DEAD | (dead0 + bd + __popcll(md & lt));
        if (hook) {
            A.flags[(uint32_t)key[q]] = 1;
            A.wlist[wl0 + bh + __popcll(mh & lt)] = (uint32_t)(key[q] >> 32);
        }
    }
    // pointer jumping in place: a value read is always an ancestor
    for (;;) {
        if (tid == 0) s_c[3] = 0;
        __syncthreads();
        bool any = false;
        for (uint32_t i = tid; i < L; i += CE_NT) {
            const uint32_t x = s_h[i], y = s_h[x];
            if (x != y) {
                s_h[i] = y;
                any = true;
            }
        }
        if (any) s_c[3] = 1;
        __syncthreads();
        const uint32_t more = s_c[3];
        __syncthreads();
        if (!more) break;
    }
    const uint32_t Ln = s_c[0];
    uint32_t *map = ct_map(A, k);
    for (uint32_t i = tid; i < L; i += CE_NT) map[i] = s_nid[s_h[i]];
    // the first small round's vertices: what they are now (a single vertex
    // left has no edge: it is a finished tree)
    for (uint32_t i = tid; i < z.L0; i += CE_NT) {
        const uint32_t x = tl1 ? A.cum[i] : i;
        if (x & CT_DEAD) continue;
        const uint32_t v = s_nid[s_h[x]];
        A.cum[i] = Ln == 1 && !(v & CT_DEAD) ? CT_DEAD | (dead0 + s_c[1]) : v;
    }
    uint64_t *rn = A.r[(k + 1) & 1];
    for (uint32_t i = tid; i < Ln; i += CE_NT) rn[i] = KEY_INF;
    if (tid == 0) {
        if (!tl1) c->ct.tl[A.ph] = (uint32_t)k + 1;
        c->ct.L[A.ph][k + 1] = Ln == 1 ? 0 : Ln;
        c->ct.dead[A.ph] = dead0 + s_c[1] + (Ln == 1 ? 1 : 0);
        c->ct.hooks[A.ph][k] = s_c[2];
        c->ct.wl = wl0 + s_c[2];
        c->ct.done[A.ph][k] = 1;
        if (Ln <= 1) c->ct.phdone[A.ph] = 1;
    }
}

// The remaining rounds of a phase with L <= CT_PAIR vertices in one
// workgroup, on the minimum keys of their pairs (one pair a thread).
__device__ void ct_pair_rounds(const CtArgs &A, int k, uint32_t L, const CtSmall &z,
                               uint64_t *s_min, uint32_t *s_h, uint32_t *s_c)
{
    static_assert(CT_PAIR * CT_PAIR == CE_NT, "one pair a thread");
    Counters *c = A.cnt;
    const uint32_t tid = threadIdx.x, i = tid / CT_PAIR, j = tid % CT_PAIR;
    uint32_t *s_comp = s_h + CT_PAIR, *s_id = s_comp + CT_PAIR;
    const uint64_t key = load_relaxed_u64(A.mat + tid);
    const uint32_t tl1 = z.tl1, dead0 = z.dead;
    uint32_t wl = z.wl;
    if (tid < CT_PAIR) s_comp[tid] = tid;
    int rr = k;
    for (;; ++rr) {
        if (tid < CT_PAIR) s_min[tid] = KEY_INF;
        if (tid == 0) s_c[0] = 0;
        __syncthreads();
        const uint32_t a = s_comp[i], b = s_comp[j];
        const bool live = key != KEY_INF && a != b;
        if (live) {
            lower_lds(s_min, a, KEY_INF, key);
            lower_lds(s_min, b, KEY_INF, key);
        }
        __syncthreads();
        // keys are distinct: one pair has each minimum
        if (live && s_min[a] == key) s_h[a] = b;
        if (live && s_min[b] == key) s_h[b] = a;
        __syncthreads();
        if (tid < CT_PAIR) {  // lanes of one wave
            const bool root = s_comp[tid] == tid && s_min[tid] != KEY_INF;
            const uint32_t t = root ? s_h[tid] : tid;
            const bool stay = root && tid < t && s_h[t] == tid;
            const bool hook = root && !stay;
            const uint64_t mk = __ballot(hook);
            if (hook) {
                const uint64_t x = s_min[tid];
                A.flags[(uint32_t)x] = 1;
                A.wlist[wl + __popcll(mk & lanemask_lt())] = (uint32_t)(x >> 32);
            }
            s_h[tid] = hook ? t : tid;
            if (tid == 0) s_c[0] = (uint32_t)__popcll(mk);
        }
        __syncthreads();
        const uint32_t hooks = s_c[0];
        if (tid == 0 && rr < CT_ROUNDS - 1 && (hooks || rr == k)) {
            c->ct.hooks[A.ph][rr] = hooks;
            c->ct.done[A.ph][rr] = 1;
        }
        if (!hooks) break;
        wl += hooks;
        uint32_t x = 0;
        if (tid < CT_PAIR) {
            x = s_comp[tid];
            while (s_h[x] != x) x = s_h[x];
        }
        __syncthreads();
        if (tid < CT_PAIR) s_comp[tid] = x;
    }
    // every vertex is in a finished tree now: number them by their roots
    if (tid < CT_PAIR) {
        const uint64_t mk = __ballot(tid < L && s_comp[tid] == tid);
        s_id[tid] = dead0 + (uint32_t)__popcll(mk & lanemask_lt());
        if (tid == 0) s_c[1] = (uint32_t)__popcll(mk);
    }
    __syncthreads();
    for (uint32_t q = tid; q < z.L0; q += CE_NT) {
        const uint32_t x = tl1 ? A.cum[q] : q;
        if (!(x & CT_DEAD)) A.cum[q] = CT_DEAD | s_id[s_comp[x]];
    }
    if (tid == 0) {
        if (!tl1) c->ct.tl[A.ph] = (uint32_t)k + 1;
        c->ct.L[A.ph][k + 1] = 0;
        c->ct.dead[A.ph] = dead0 + s_c[1];
        c->ct.wl = wl;
        c->ct.phdone[A.ph] = 1;
    }
}

}  // namespace

// Hot vertices of an edge pass (a star's centre, the largest tree of phase 0)
// would take one atomic after another on one address, 3 ns each: the read
// in front of an atomic sees what its XCD's L2 holds, not the latest value.
// Each workgroup samples its edges, and the vertices with at least one in
// CT_HOT_SHARE of the live ones (and CT_HOT_MIN of them: with 4 the few edges
// of late rounds fill many slots by chance, grid 60^3 274 us a solve, 270 with
// 8) keep their minimum in LDS until the end of the pass.
constexpr uint32_t CT_HOT = 512, CT_HOT_MIN = 8, CT_HOT_SHARE = 64;
constexpr uint32_t CT_READ = 320;  // edges of a wave above which minima are read first

__device__ __forceinline__ uint32_t ct_hot_slot(uint32_t v) { return (v * 0x9E3779B1u) >> 23; }

enum { CT_MIN_LDS, CT_MIN_HOT, CT_MIN_DEV, CT_MIN_PAIR };
// Ends as they are (a phase's first round); through the last round's map,
// the edges between different vertices kept in place; through the cumulative
// map since the first small round, in LDS, the list left as it is (few edges
// become internal from there on, and a pass then only reads).
enum { CT_ENDS, CT_MAP, CT_CUM };

// m <- min(m, the m of the lane CTRL names) where that lane has the same a.
template <int CTRL>
__device__ __forceinline__ void run_min(uint32_t a, uint64_t &m)
{
    const uint32_t oa = dpp_u32<CTRL>(a, ~a);
    const uint64_t om = dpp_u64<CTRL>(m, KEY_INF);
    if (oa == a && om < m) m = om;
}

// One wave over a segment: map the ends and lower the minima (read: behind a
// read of them).  Returns the live edges.
template <int ENDS, int MODE>
__device__ __forceinline__ uint32_t ct_sweep(CtEdge *seg, uint32_t cnt,
                                             const uint32_t *__restrict__ map,
                                             const uint16_t *s_cum, uint64_t *r, uint64_t *s_r,
                                             const uint32_t *s_tag, bool read)
{
    constexpr int U = 4;
    const int lane = __lane_id();
    uint32_t out = 0;
    for (uint32_t j0 = 0; j0 < cnt; j0 += 64 * U) {
        CtEdge x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t j = j0 + q * 64 + lane;
            x[q] = seg[j < cnt ? j : cnt - 1];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (ENDS == CT_MAP) {
                x[q].a = map[x[q].a];
                x[q].b = map[x[q].b];
            } else if (ENDS == CT_CUM) {
                x[q].a = s_cum[x[q].a];
                x[q].b = s_cum[x[q].b];
            }
        }
        uint64_t ra[U], rb[U];
        uint32_t pr[U];
        bool ha[U], hb[U];  // the end is a hot vertex
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (MODE == CT_MIN_PAIR) {
                pr[q] = x[q].a != x[q].b ? min(x[q].a, x[q].b) * CT_PAIR + max(x[q].a, x[q].b) : 0u;
                ra[q] = s_r[pr[q]];
            } else if (ENDS == CT_CUM && x[q].a == x[q].b) {
                ra[q] = rb[q] = 0;  // internal (a finished tree's number is no index)
                ha[q] = hb[q] = false;
            } else if (MODE == CT_MIN_LDS) {
                ra[q] = s_r[x[q].a];
                rb[q] = s_r[x[q].b];
            } else {
                const uint32_t sa = ct_hot_slot(x[q].a), sb = ct_hot_slot(x[q].b);
                ha[q] = MODE == CT_MIN_HOT && s_tag[sa] == x[q].a;
                hb[q] = MODE == CT_MIN_HOT && s_tag[sb] == x[q].b;
                ra[q] = ha[q] ? s_r[sa] : read ? load_relaxed_u64(r + x[q].a) : KEY_INF;
                rb[q] = hb[q] ? s_r[sb] : read ? load_relaxed_u64(r + x[q].b) : KEY_INF;
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const bool live = j0 + q * 64 + lane < cnt && x[q].a != x[q].b;
            if (ENDS != CT_CUM && MODE != CT_MIN_LDS && MODE != CT_MIN_PAIR) {
                // the list is in the input's order, where edges often come in
                // runs of one first end: a run's minimum (within 16 lanes)
                // leaves from its last lane alone (first round of grid 256^3,
                // 16.4M light edges: 366 us, 522 us with one atomic per end;
                // random edges either way alike), and the runs of the input
                // stay runs while the ends are mapped (a solve with one atomic
                // per end / this: R-MAT s19 527 / 463 us, s20 860 / 737, grid
                // 101^3 480 / 455, 2^22 vertices and 2^24 random edges 2155 /
                // 2155)
                const uint32_t a = live ? x[q].a : NONE32;
                uint64_t m = live ? x[q].key : KEY_INF;
                run_min<DPP_ROW_SHR1>(a, m);
                run_min<DPP_ROW_SHR2>(a, m);
                run_min<DPP_ROW_SHR4>(a, m);
                run_min<DPP_ROW_SHR8>(a, m);
                const bool last = dpp_u32<DPP_ROW_SHL1>(a, ~a) != a;
                if (live) {
                    if (last) {
                        if (ha[q]) lower_lds(s_r, ct_hot_slot(x[q].a), ra[q], m);
                        else lower_dev(r, x[q].a, ra[q], m);
                    }
                    if (hb[q]) lower_lds(s_r, ct_hot_slot(x[q].b), rb[q], x[q].key);
                    else lower_dev(r, x[q].b, rb[q], x[q].key);
                }
            } else if (live && MODE == CT_MIN_PAIR) {
                lower_lds(s_r, pr[q], ra[q], x[q].key);
            } else if (live) {
                if (MODE == CT_MIN_LDS) lower_lds(s_r, x[q].a, ra[q], x[q].key);
                else if (ha[q]) lower_lds(s_r, ct_hot_slot(x[q].a), ra[q], x[q].key);
                else lower_dev(r, x[q].a, ra[q], x[q].key);
                if (MODE == CT_MIN_LDS) lower_lds(s_r, x[q].b, rb[q], x[q].key);
                else if (hb[q]) lower_lds(s_r, ct_hot_slot(x[q].b), rb[q], x[q].key);
                else lower_dev(r, x[q].b, rb[q], x[q].key);
            }
            const uint64_t mask = __ballot(live);
            if (ENDS == CT_MAP && live) seg[out + __popcll(mask & lanemask_lt())] = x[q];
            out += (uint32_t)__popcll(mask);
        }
    }
    return out;
}

// The pass of one workgroup: minima into LDS where the round's vertices (or
// their pairs) fit, lowering r (or the matrix) at the end; else into r
// directly, hot vertices in LDS.
template <int ENDS>
__device__ __forceinline__ uint32_t ct_pass(const CtArgs &A, int k, uint32_t L,
                                            const uint32_t *map, const uint16_t *s_cum,
                                            uint64_t *r, uint64_t *s_r, uint32_t *s_tag,
                                            uint32_t *s_num, uint32_t *s_c)
{
    // (a wave's numbers in scalar registers)
    const uint32_t tid = threadIdx.x, wv = ct_uniform(blockIdx.x * CE_WV + (tid >> 6));
    const int lane = __lane_id();
    uint32_t live = 0;
    // every wave over its segments, one sweep each
#define CT_SEGMENTS(MODE, READ)                                                               \
    for (uint32_t sg = wv; sg < A.W; sg += gridDim.x * CE_WV) {                               \
        const uint32_t cnt = ct_uniform(A.cw[sg]);                                            \
        const uint32_t out = ct_sweep<ENDS, MODE>(A.list + (size_t)sg * A.segcap, cnt, map,   \
                                                  s_cum, r, s_r, s_tag, READ);                \
        if (ENDS == CT_MAP && lane == 0) A.cw[sg] = out;                                      \
        live += out;                                                                          \
    }
    if (L <= CT_SMALL) {
        const bool pair = L <= CT_PAIR;
        const uint32_t cells = pair ? CT_PAIR * CT_PAIR : L;
        uint64_t *dst = pair ? A.mat : r;
        for (uint32_t i = tid; i < cells; i += CE_NT) s_r[i] = KEY_INF;
        __syncthreads();
        if (pair) {
            CT_SEGMENTS(CT_MIN_PAIR, true)
        } else {
            CT_SEGMENTS(CT_MIN_LDS, true)
        }
        __syncthreads();
        // behind a read only where every workgroup has most cells to lower
        if (tid == 0) s_c[0] = 0;
        __syncthreads();
        if (lane == 0) atomicAdd(&s_c[0], live);
        __syncthreads();
        const bool read = s_c[0] > cells;
        for (uint32_t i = tid; i < cells; i += CE_NT) {
            const uint64_t v = s_r[i];
            if (v != KEY_INF) lower_dev(dst, i, read ? load_relaxed_u64(dst + i) : KEY_INF, v);
        }
        __syncthreads();
        return live;
    }
    for (uint32_t i = tid; i < CT_HOT; i += CE_NT) {
        s_tag[i] = NONE32;
        s_num[i] = s_num[CT_HOT + i] = 0;
        s_r[i] = KEY_INF;
    }
    if (tid < 4) s_c[tid] = 0;
    __syncthreads();
    // the first edges of every wave are the sample
    const uint32_t cnt0 = ct_uniform(A.cw[wv]);
    uint32_t va = NONE32, vb = NONE32;
    if ((uint32_t)lane < cnt0) {
        const CtEdge *seg = A.list + (size_t)wv * A.segcap;
        va = seg[lane].a;
        vb = seg[lane].b;
        if (ENDS == CT_MAP) {
            va = map[va];
            vb = map[vb];
        } else if (ENDS == CT_CUM) {
            va = s_cum[va];
            vb = s_cum[vb];
        }
        if (va != vb) {
            atomicAdd(&s_num[ct_hot_slot(va)], 1u);
            atomicAdd(&s_num[ct_hot_slot(vb)], 1u);
        }
    }
    const uint64_t lv = __ballot(va != vb);
    if (lane == 0 && lv) atomicAdd(&s_c[1], (uint32_t)__popcll(lv));
    __syncthreads();
    const uint32_t hot = max(CT_HOT_MIN, s_c[1] / CT_HOT_SHARE);
    // the vertex of each slot with that many ends: any of them is proposed and
    // its own ends are counted, the next one if they are too few (a slot's
    // other vertices: with the last one written taken unseen, a hub lost its
    // slot to a leaf in one workgroup of ten: a star of 10^6 vertices 804 us a
    // solve, 146 us with the count; 2 * 10^6 edges of 3 hubs 1690 / 265 us)
    uint32_t *s_hit = s_num + CT_HOT;
    const uint32_t la = ct_hot_slot(va), lb = ct_hot_slot(vb);
    bool ca = va != vb && s_num[la] >= hot, cb = va != vb && s_num[lb] >= hot;
    if (ca || cb) s_c[0] = 1;
    for (int t = 0; t < 4; ++t) {
        if (ca) s_tag[la] = va;
        if (cb) s_tag[lb] = vb;
        __syncthreads();
        if (!s_c[0] || s_c[2] != (uint32_t)t) break;
        const uint32_t ta = ca ? s_tag[la] : NONE32, tb = cb ? s_tag[lb] : NONE32;
        if (ca && ta == va) atomicAdd(&s_hit[la], 1u);
        if (cb && tb == vb) atomicAdd(&s_hit[lb], 1u);
        __syncthreads();
        const bool ha = ca && s_hit[la] >= hot, hb = cb && s_hit[lb] >= hot;
        __syncthreads();
        if (ca && !ha && ta == va) {
            s_tag[la] = NONE32;
            s_hit[la] = 0;
        }
        if (cb && !hb && tb == vb) {
            s_tag[lb] = NONE32;
            s_hit[lb] = 0;
        }
        ca = ca && !ha && ta != va;
        cb = cb && !hb && tb != vb;
        if (ca || cb) s_c[2] = t + 1;
        if (ha || hb) s_c[3] = 1;
        __syncthreads();
    }
    // Whether minima are read before an atomic.  A wave with few edges sends
    // them all at once, before any read could show a minimum, and reading
    // lines that atomics change is slow (passes over 271 / 113 / 70 / 60 edges
    // a wave, 10^6 edges on 10^6 vertices and less: 81 / 82 / 51 / 56 us with
    // the read, 62 / 48 / 26 / 26 us without; over 1720 edges a
    // wave, the first two passes of R-MAT s22: 206 and 292 us with it, 372 and
    // 389 without).
    const bool read = cnt0 > CT_READ;
    if (s_c[3]) {
        CT_SEGMENTS(CT_MIN_HOT, read)
        __syncthreads();
        for (uint32_t i = tid; i < CT_HOT; i += CE_NT) {
            const uint64_t v = s_r[i];
            if (v != KEY_INF) lower_dev(r, s_tag[i], load_relaxed_u64(r + s_tag[i]), v);
        }
    } else {
        CT_SEGMENTS(CT_MIN_DEV, read)
    }
#undef CT_SEGMENTS
    return live;
}

// Whether the edge pass's last workgroup finishes a round of L vertices: from
// CT_SMALL down, as one compute unit's scattered reads (eight or so a vertex,
// one a cycle) are slower than two more launches above CT_FINISH, only if
// those launches follow (3000 vertices, grid 60^3: 26 us alone, 14 us by hook
// and chase; 1000: 11 us alone).  From a phase's first such round on all are
// (the maps since are composed into one).  A line at 1024 / 2048 / 3072, us a
// solve: R-MAT s16 194 / 190 / 199, R-MAT s19 423 / 412 / 414, grid 60^3 264 /
// 270 / 286.
__device__ __forceinline__ bool ct_one_finishes(uint32_t L, uint32_t tl1, bool big)
{
    return L <= (big && !tl1 ? CT_FINISH : CT_SMALL);
}

// (two workgroups on a compute unit: at most 64 registers)
template <bool FIRST>
__global__ __launch_bounds__(CE_NT, 8) void k_ct_edges(CtArgs A, int k, int big)
{
    // minima of a small round; then its targets and numbers
    __shared__ __align__(16) uint64_t s_r[CT_SMALL];
    // the cumulative map of a small round, or a larger one's hot vertices
    __shared__ __align__(16) uint16_t s_cum[CT_SMALL];
    __shared__ uint32_t s_cnt[CE_WV];
    __shared__ uint32_t s_c[4];
    static_assert(2 * (sizeof s_r + sizeof s_cum + 256) <= 160 << 10, "two workgroups a CU");
    static_assert(sizeof s_cum >= 12 * CT_HOT, "tags and counts in the map's place");
    Counters *c = A.cnt;
    if (A.ph == 0 && k <= 1 && blockIdx.x == 0 && threadIdx.x == 0 && !c->ct.clk[1 + k])
        c->ct.clk[1 + k] = wall_clock64();
    const uint32_t L = c->ct.L[A.ph][k];
    if (c->err || L == 0 || (L > CT_SMALL && !big)) return;
    if (k > 0 ? !c->ct.done[A.ph][k - 1] : (A.ph > 0 && !c->ct.phdone[A.ph - 1])) return;
    if (c->ct.done[A.ph][k]) return;
    const uint32_t tl1 = ct_uniform(c->ct.tl[A.ph]);
    // (in scalar registers)
    const CtSmall z{tl1, ct_uniform(tl1 ? c->ct.L[A.ph][tl1 - 1] : L),
                    ct_uniform(c->ct.dead[A.ph]), ct_uniform(c->ct.wl)};
    const bool finish = ct_one_finishes(L, tl1, big);
    const int lane = __lane_id();
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x == 0 && tid == 0) c->ct.ran[A.ph][k] = 1;
    uint64_t *r = A.r[k & 1];
    uint32_t *s_tag = reinterpret_cast<uint32_t *>(s_cum), *s_num = s_tag + CT_HOT;
    uint32_t out;
    if (FIRST) {
        out = ct_pass<CT_ENDS>(A, k, L, nullptr, nullptr, r, s_r, s_tag, s_num, s_c);
    } else if (tl1 && k >= (int)tl1) {
        for (uint32_t i = tid; i < z.L0; i += CE_NT) s_cum[i] = (uint16_t)min(A.cum[i], 0xFFFFu);
        __syncthreads();
        out = ct_pass<CT_CUM>(A, k, L, nullptr, s_cum, r, s_r, s_tag, s_num, s_c);
    } else {
        out = ct_pass<CT_MAP>(A, k, L, ct_map(A, k - 1), nullptr, r, s_r, s_tag, s_num, s_c);
    }
    if (lane == 0) s_cnt[tid >> 6] = out;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid < 64) {
        const uint32_t t = wave_sum(tid < CE_WV ? s_cnt[tid] : 0u);
        // live edges and the workgroups through, in one atomic; its answer is
        // waited for (13 ns each on one address) only where it is needed
        unsigned long long *tick = (unsigned long long *)&c->ct.tick[A.ph][k];
        const unsigned long long add = ((unsigned long long)t << 16) | 1u;
        if (!finish) {
            if (tid == 0) atomicAdd(tick, add);
        } else if (tid == 0) {
            s_c[1] = (uint32_t)(atomicAdd(tick, add) & 0xFFFFu);
        }
    }
    if (!finish) return;
    // The last workgroup of a small round finishes it.  It reads only r (or
    // the matrix), which is written by device-scope atomics alone: each wave
    // waits for its own before the ticket (a release fence would write back
    // the whole L2 in every workgroup, 70-220 us a pass), and the last one
    // drops what its L2 holds of r before reading.
    __syncthreads();
    if (s_c[1] != gridDim.x - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    if (L <= CT_PAIR)
        ct_pair_rounds(A, k, L, z, s_r, reinterpret_cast<uint32_t *>(s_cum), s_c);
    else
        ct_small_round(A, k, L, z, reinterpret_cast<uint32_t *>(s_r),
                       reinterpret_cast<uint32_t *>(s_r) + CT_SMALL, s_c);
}

// ------------------------------------------------ rounds of many vertices --

// Whether round k's kernels after the edge pass have work.
__device__ __forceinline__ bool ct_big_round(const CtArgs &A, int k, uint32_t L)
{
    const Counters *c = A.cnt;
    return !ct_one_finishes(L, c->ct.tl[A.ph], true) && !c->err && c->ct.ran[A.ph][k];
}

// Hook, tie break, forest flags, weights, and the numbers of the vertices
// that stay (dense from 0) and of the finished trees.  Two vertices hooked
// onto each other exactly when they have the same minimum (keys are
// distinct), so the tie break reads the target's minimum instead of waiting
// for its hook.  A tile is IT x 512 consecutive vertices; the numbers keep
// the vertices' order inside it (item-major, then wave, then lane) and each
// tile takes its range with one atomic, so neighbours stay neighbours.

template <int IT, int WT>
__device__ __forceinline__ uint32_t ct_hook_tiles(const CtArgs &A, int k, uint32_t L,
                                                  uint32_t (*s_off)[64], uint32_t *s_base,
                                                  WSum &ws)
{
    constexpr int NW = TIE_NT / 64;
    static_assert(IT * NW <= 64, "one count a lane");
    Counters *c = A.cnt;
    const uint64_t *r = A.r[k & 1];
    uint32_t *map = ct_map(A, k);
    const uint32_t w = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    const uint32_t tiles = (uint32_t)(((uint64_t)L + IT * TIE_NT - 1) / (IT * TIE_NT));
    uint32_t hooks = 0;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint64_t base = (uint64_t)tile * (IT * TIE_NT) + threadIdx.x;
        uint64_t key[IT];
        uint32_t a[IT], b[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            key[q] = i < L ? r[i] : KEY_INF;
        }
        ct_ends<IT>(A, key, k, k, a, b);
        uint64_t kt[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            a[q] = a[q] == (uint32_t)(base + q * TIE_NT) ? b[q] : a[q];  // the target
            kt[q] = r[key[q] != KEY_INF ? a[q] : 0u];
        }
        uint32_t stay = 0, dead = 0;
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            if (i >= L) continue;
            uint32_t t = (uint32_t)i;
            if (key[q] == KEY_INF) {
                dead |= 1u << q;
            } else if (kt[q] == key[q] && (uint32_t)i < a[q]) {
                stay |= 1u << q;
            } else {
                t = a[q];
                A.flags[(uint32_t)key[q]] = 1;
                wsum_add<WT>(ws, (uint32_t)(key[q] >> 32));
                ++hooks;
            }
            A.h[i] = t;
        }
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t ms = __ballot((stay >> q) & 1u), md = __ballot((dead >> q) & 1u);
            if (__lane_id() == 0) {
                s_off[0][q * NW + w] = (uint32_t)__popcll(ms);
                s_off[1][q * NW + w] = (uint32_t)__popcll(md);
            }
        }
        __syncthreads();
        if (w < 2) {
            // exclusive scan of one list's IT x NW counts by one wave
            const uint32_t l = __lane_id();
            const uint32_t c0 = l < IT * NW ? s_off[w][l] : 0u;
            const uint32_t inc = wave_incl_sum(c0);
            s_off[w][l] = inc - c0;
            if (l == 63)
                s_base[w] = inc ? atomicAdd(w ? &c->ct.dead[A.ph] : &c->ct.L[A.ph][k + 1], inc) : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            const bool st = (stay >> q) & 1u, de = (dead >> q) & 1u;
            const uint64_t ms = __ballot(st), md = __ballot(de);
            if (st) map[i] = s_base[0] + s_off[0][q * NW + w] + (uint32_t)__popcll(ms & lt);
            if (de) map[i] = CT_DEAD | (s_base[1] + s_off[1][q * NW + w] + (uint32_t)__popcll(md & lt));
        }
        __syncthreads();
    }
    return hooks;
}

template <int WT>
__global__ __launch_bounds__(TIE_NT) void k_ct_hook(CtArgs A, int k)
{
    constexpr int NW = TIE_NT / 64;
    __shared__ uint32_t s_off[2][64];
    __shared__ uint32_t s_base[2];
    __shared__ int64_t s_sum[NW * (ACC_DIGITS + 1)];
    __shared__ int64_t s_tot[WS_WORDS];
    __shared__ uint32_t s_hk[NW];
    Counters *c = A.cnt;
    const uint32_t L = c->ct.L[A.ph][k];
    if (!ct_big_round(A, k, L) || c->ct.done[A.ph][k]) return;
    const uint32_t w = threadIdx.x >> 6;
    WSum ws;
    // eight vertices a thread while there are many (one atomic, 13 ns on one
    // address, per 4096), two with fewer, to keep the compute units busy
    uint32_t hooks = L >= (1u << 20) ? ct_hook_tiles<8, WT>(A, k, L, s_off, s_base, ws)
                                     : ct_hook_tiles<2, WT>(A, k, L, s_off, s_base, ws);
    // this workgroup's weights into its slot, its hooks into the round's count
    hooks = wave_sum(hooks);
    if (__lane_id() == 0) s_hk[w] = hooks;
    wsum_block<TIE_NT, WT>(ws, s_sum, s_tot, 1);
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < NW; ++i) t += s_hk[i];
        if (t) {
            atomicAdd(&c->ct.hooks[A.ph][k], t);
            int64_t old[WS_WORDS];
#pragma unroll
            for (int j = 0; j < WS_WORDS; ++j) old[j] = A.wpart[(size_t)j * CT_WSLOTS + blockIdx.x];
#pragma unroll
            for (int j = 0; j < WS_WORDS; ++j)
                A.wpart[(size_t)j * CT_WSLOTS + blockIdx.x] = old[j] + s_tot[j];
        }
    }
}

// Every vertex that hooked follows its chain to the vertex that stays and
// takes its number; improvements are written back, so other chains get
// shorter (the hooks form no cycle after the tie break).  A thread takes at
// most CT_WALK steps for one of its vertices and comes back to those that
// are not there yet after all its others.  Where that does not end within
// A.sweeps visits, the solve stops (ERR_FAR) and goes on behind ct_far.
//
// Walked to the end at once, a chain that leads from early vertices to late
// ones, which nobody has shortened yet, takes a step per vertex: a path of 2 *
// 10^6 vertices with falling weights 1165 ms a solve, 0.26 ms with this (4 /
// 8 / 16 steps: 16 * 10^6 vertices 1.31 / 1.39 / 1.60 ms; R-MAT s22, grids and
// random graphs even).  All workgroups are on the chip together (CHASE_WG),
// which makes the chains shrink everywhere at once; but a compute die's L2 can
// hold a target as it was first read, so only the end of a launch is sure to
// show every improvement (with 16 unrolled steps the same path fell back to
// 157 ms at 4 * 10^6 vertices).  Giving up after 1 / 16 visits, us a solve:
// falling paths of 5 * 10^5 and 4 * 10^6 vertices 198 / 152 and 502 / 420.
constexpr int CT_WALK = 8;
constexpr unsigned CHASE_WG = 2048;

__global__ __launch_bounds__(256) void k_ct_chase(CtArgs A, int k)
{
    Counters *c = A.cnt;
    const uint32_t L = c->ct.L[A.ph][k];
    if (!ct_big_round(A, k, L)) return;
    const uint32_t Ln = c->ct.L[A.ph][k + 1];
    uint32_t *map = ct_map(A, k);
    uint64_t *rn = A.r[(k + 1) & 1];
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    const uint64_t i0 = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    uint64_t left = ~0ull;  // its vertices to look at (the last bit: all from the 64th on)
    for (uint32_t sweep = 0; left && sweep < A.sweeps; ++sweep) {
        uint64_t far = 0, bit = 1;
        for (uint64_t i = i0; i < L; i += stride) {
            if (left & bit) {
                uint32_t x = load_relaxed_u32(A.h + i);
                if (x != (uint32_t)i) {
                    bool there = false;
                    for (int q = 0; q < CT_WALK && !there; ++q) {
                        const uint32_t y = load_relaxed_u32(A.h + x);
                        there = y == x;
                        if (!there) store_relaxed_u32(A.h + i, y);
                        x = y;
                    }
                    if (there) map[i] = map[x];
                    else far |= bit;
                }
                if (sweep == 0 && i < Ln) rn[i] = KEY_INF;
            }
            if (bit << 1) bit <<= 1;
        }
        left = far;
    }
    if (__ballot(left != 0) && __lane_id() == 0) {
        c->ct.far = (uint32_t)(A.ph * CT_ROUNDS + k);
        if (!(load_relaxed_u32(&c->err) & ERR_FAR)) atomicOr(&c->err, ERR_FAR);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->ct.done[A.ph][k] = 1;
        if (Ln == 0) c->ct.phdone[A.ph] = 1;
    }
}

// CT_WALK steps along every chain of round k.  Each launch sees what the one
// before it wrote, so it leaves at most 1 / (CT_WALK + 1) of every chain.
__global__ __launch_bounds__(256) void k_ct_jump(CtArgs A, int k)
{
    const uint32_t L = A.cnt->ct.L[A.ph][k];
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += stride) {
        const uint32_t x0 = load_relaxed_u32(A.h + i);
        uint32_t x = x0;
        for (int q = 0; q < CT_WALK; ++q) {
            const uint32_t y = load_relaxed_u32(A.h + x);
            if (y == x) break;
            x = y;
        }
        if (x != x0) store_relaxed_u32(A.h + i, x);
    }
}

__global__ void k_ct_jumped(CtArgs A) { A.cnt->err = 0; }

void ct_far(hipStream_t s, CtArgs A, int k, uint32_t L)
{
    for (uint64_t len = L; len > 1; len = (len + CT_WALK) / (CT_WALK + 1))
        k_ct_jump<<<grid_for(L, 256, 8192), 256, 0, s>>>(A, k);
    k_ct_jumped<<<1, 1, 0, s>>>(A);
    A.sweeps = 1;
    k_ct_chase<<<grid_for(L, 256, CHASE_WG), 256, 0, s>>>(A, k);
}

void ct_round(hipStream_t s, const CtArgs &A, int k, bool big, uint32_t bound)
{
    const unsigned g = (A.ph ? A.W : A.pass_waves) / CE_WV;
    if (k == 0) k_ct_edges<true><<<g, CE_NT, 0, s>>>(A, k, big);
    else k_ct_edges<false><<<g, CE_NT, 0, s>>>(A, k, big);
    if (!big || bound <= CT_FINISH) return;
    const unsigned t = grid_for(bound, 2 * TIE_NT, CT_WSLOTS);
    if (A.wt == MSF_W_F32) k_ct_hook<MSF_W_F32><<<t, TIE_NT, 0, s>>>(A, k);
    else k_ct_hook<MSF_W_U32><<<t, TIE_NT, 0, s>>>(A, k);
    k_ct_chase<<<grid_for(bound, 256, CHASE_WG), 256, 0, s>>>(A, k);
}

// ------------------------------------------------------- between phases --

// comp[v] = number of v's tree after phase 0; phase 1's vertices are these
// numbers.
__global__ __launch_bounds__(256) void k_ct_compose(CtArgs A, uint32_t *comp)
{
    Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[0] || c->ct.ran[1][0]) return;
    const uint32_t tl1 = c->ct.tl[0];
    const int tl = tl1 ? (int)tl1 - 1 : 64;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x; v < (uint64_t)A.n; v += stride) {
        uint32_t x = (uint32_t)v;
        for (int l = 0; l < tl && !(x & CT_DEAD); ++l) x = ct_map(A, l)[x];
        if (!(x & CT_DEAD)) x = A.cum[x];
        comp[v] = x & ~CT_DEAD;
        A.r[0][v] = KEY_INF;
    }
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < CT_PAIR * CT_PAIR; i += 256) A.mat[i] = KEY_INF;
        if (threadIdx.x == 0) c->ct.L[1][0] = c->ct.dead[0];
    }
}

// The tree that most of 256 sampled edge ends lie in.
__global__ __launch_bounds__(256) void k_ct_giant(CtArgs A, const uint32_t *__restrict__ comp)
{
    __shared__ __align__(16) uint32_t s_v[256];
    __shared__ unsigned long long s_best;
    Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[0] || c->ct.ran[1][0]) return;
    const int64_t e = (int64_t)((uint64_t)A.m * threadIdx.x / 256);
    const int2 uv = A.edges[e];
    const uint32_t v = comp[(threadIdx.x & 1) ? uv.x : uv.y];
    s_v[threadIdx.x] = v;
    if (threadIdx.x == 0) s_best = 0;
    __syncthreads();
    uint32_t same = 0;
    const uint4 *s_v4 = reinterpret_cast<const uint4 *>(s_v);
#pragma unroll 16
    for (int i = 0; i < 64; ++i) {
        const uint4 x = s_v4[i];
        same += (x.x == v) + (x.y == v) + (x.z == v) + (x.w == v);
    }
    atomicMax(&s_best, ((unsigned long long)same << 32) | v);
    __syncthreads();
    if (threadIdx.x == 0) c->ct.giant = (uint32_t)s_best;
}

__global__ __launch_bounds__(256) void k_ct_bits(CtArgs A, const uint32_t *__restrict__ comp,
                                                 uint64_t *__restrict__ bits)
{
    const Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[0] || c->ct.ran[1][0]) return;
    const uint32_t g = c->ct.giant;
    const uint64_t words = ((uint64_t)A.n + 63) / 64, stride = (uint64_t)gridDim.x * 4;
    for (uint64_t i = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < words; i += stride) {
        const uint64_t v = i * 64 + __lane_id();
        const uint64_t mask = __ballot(v < (uint64_t)A.n && comp[v] == g);
        if (__lane_id() == 0) bits[i] = mask;
    }
}

// Every edge read once more: those between different trees of phase 0 go to
// the wave's segment with the trees as ends.  With many vertices an edge is
// first looked up in the bits of the largest tree (n / 8 bytes, which stay
// in every L2), where most edges have both ends.
template <bool BITS>
__global__ __launch_bounds__(CE_NT) void k_ct_between(CtArgs A, const uint32_t *__restrict__ comp,
                                                      const uint32_t *__restrict__ bits)
{
    __shared__ uint32_t s_cnt[CE_WV];
    Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[0] || c->ct.ran[1][0]) return;
    const int lane = __lane_id();
    const uint32_t wv = ct_uniform(blockIdx.x * CE_WV + (threadIdx.x >> 6));
    const int64_t tiles = (A.m + CT_TILE - 1) / CT_TILE;
    CtEdge *seg = A.list + (size_t)wv * A.segcap;
    uint32_t out = 0;
    int2 nx[4];
    uint32_t none[4];
    ct_load<false>(A, wv, lane, nx, none);
    for (int64_t t = wv; t < tiles; t += A.W) {
        int2 uv[4];
        bool go[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uv[q] = nx[q];
            go[q] = t * CT_TILE + q * 64 + lane < A.m;
        }
        // the next tile's loads are in flight meanwhile
        if (t + A.W < tiles) ct_load<false>(A, t + A.W, lane, nx, none);
        if (BITS) {
            uint32_t ba[4], bb[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ba[q] = bits[(uint32_t)uv[q].x >> 5];
                bb[q] = bits[(uint32_t)uv[q].y >> 5];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                go[q] = go[q] && !((ba[q] >> (uv[q].x & 31)) & (bb[q] >> (uv[q].y & 31)) & 1u);
        }
        uint32_t a[4], b[4], wb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = go[q] ? comp[uv[q].x] : 0u;
            b[q] = go[q] ? comp[uv[q].y] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t e = t * CT_TILE + q * 64 + lane;
            go[q] = go[q] && a[q] != b[q];
            wb[q] = go[q] ? A.w[e] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t e = t * CT_TILE + q * 64 + lane;
            const uint64_t mask = __ballot(go[q]);
            if (go[q])
                seg[out + __popcll(mask & lanemask_lt())] =
                    CtEdge{a[q], b[q], ((uint64_t)ct_wkey(wb[q], A.wt) << 32) | (uint32_t)e};
            out += (uint32_t)__popcll(mask);
        }
    }
    if (lane == 0) {
        A.cw[wv] = out;
        s_cnt[threadIdx.x >> 6] = out;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int i = 0; i < CE_WV; ++i) t += s_cnt[i];
        if (t) atomicAdd(&c->ct.E0[1], t);
    }
}

void ct_between(hipStream_t s, const CtArgs &A, uint32_t *comp, uint32_t *bits)
{
    k_ct_compose<<<grid_for((size_t)A.n, 256, 8192), 256, 0, s>>>(A, comp);
    // a table of 2^20 trees (4 MB) still fits an L2: 205 G lookups/s against
    // 76 at 2^22, where the bits give 259 (64M random lookups)
    if (A.n > (1 << 20)) {
        k_ct_giant<<<1, 256, 0, s>>>(A, comp);
        k_ct_bits<<<grid_for(((size_t)A.n + 63) / 64, 4, 4096), 256, 0, s>>>(
            A, comp, reinterpret_cast<uint64_t *>(bits));
        k_ct_between<true><<<A.W / CE_WV, CE_NT, 0, s>>>(A, comp, bits);
    } else {
        k_ct_between<false><<<A.W / CE_WV, CE_NT, 0, s>>>(A, comp, nullptr);
    }
}

}  // namespace msf
