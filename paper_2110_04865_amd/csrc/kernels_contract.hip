// Rounds of Algorithm 2 over an edge list whose ends are renumbered every
// round, light edges first.
//
// The forest is unique under the order of the keys (weight, edge id), so an
// edge that joins two vertices of one tree of the forest of all lighter
// edges is not in it (the cycle property).  Phase 0 therefore takes only the
// lightest edges (about n ln(4 m / n) / 2 of them, by a sampled threshold on
// the key) and builds their forest; one pass over the input then drops every
// edge inside a tree of it, and phase 1 continues with the few edges left
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
//           number of its new tree.
// So a round costs its live edges once and its vertices a few times, and
// both shrink; no adjacency matrix is built.
//
// Every wave owns one segment of the list, so the compaction is a ballot
// and an in-place store: no barrier and no counter.  Kernels take their
// sizes from the counters on the device and return at once when there is
// nothing to do, so a whole solve is enqueued without a host round trip.
// A round of at most CT_SMALL vertices needs only the edge pass: its last
// workgroup to finish does the rest of the round in LDS.
#include <algorithm>

#include "contract.hpp"
#include "exact_sum.hpp"
#include "wave.hpp"

namespace msf {

namespace {

constexpr int CE_NT = 1024;               // threads of the list kernels
constexpr int CE_WV = CE_NT / 64;
constexpr uint32_t CT_LDSR = 4096;        // minima kept in LDS up to this many vertices
constexpr uint32_t CT_DEAD = 0x80000000u; // a finished tree's number
constexpr uint32_t CT_SAMPLES = 8192;

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

unsigned grid_for(size_t n, unsigned block, unsigned cap)
{
    size_t g = (n + block - 1) / block;
    return (unsigned)std::max<size_t>(1, std::min<size_t>(g, cap));
}

}  // namespace

size_t ct_maps_words(int32_t n) { return ct_map_at(n, 34) + 64; }

size_t ct_wpart_bytes() { return 8 * (size_t)CT_WSLOTS * WS_WORDS; }

// ----------------------------------------------------------------- set-up --

__global__ __launch_bounds__(256) void k_ct_init(CtArgs A, size_t flag_words)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0) {
        uint32_t *c = reinterpret_cast<uint32_t *>(A.cnt);
        for (uint32_t i = threadIdx.x; i < sizeof(Counters) / 4; i += 256) c[i] = 0u;
        __syncthreads();
        if (threadIdx.x == 0) {
            A.cnt->ct.L[0][0] = (uint32_t)A.n;
            A.cnt->ct.T = KEY_INF;
        }
    }
    uint32_t *fl = reinterpret_cast<uint32_t *>(A.flags);
    for (size_t i = i0; i < (size_t)A.n; i += stride) A.r[0][i] = KEY_INF;
    for (size_t i = i0; i < flag_words; i += stride) fl[i] = 0u;
    for (size_t i = i0; i < (size_t)CT_WSLOTS * WS_WORDS; i += stride) A.wpart[i] = 0;
}

void ct_init(hipStream_t s, const CtArgs &A, size_t flag_words)
{
    k_ct_init<<<grid_for(std::max<size_t>((size_t)A.n, flag_words), 256, 4096), 256, 0, s>>>(
        A, flag_words);
}

// The rank-th smallest key of a sample of CT_SAMPLES edges (one from each of
// as many equal stretches of the input, at a mixed place): the threshold of
// phase 0.  One workgroup, samples in registers, eight bits per step.
__global__ __launch_bounds__(CE_NT) void k_ct_threshold(CtArgs A, uint32_t rank)
{
    __shared__ uint32_t s_hist[256];
    __shared__ uint32_t s_bin, s_rank;
    constexpr int PER = CT_SAMPLES / CE_NT;
    uint64_t key[PER];
    const uint64_t m = (uint64_t)A.m;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t i = q * CE_NT + threadIdx.x;
        const uint64_t lo = m * i / CT_SAMPLES, hi = m * (i + 1) / CT_SAMPLES;
        uint32_t x = i * 0x9E3779B9u + 0x7F4A7C15u;
        x ^= x >> 15;
        x *= 0x2C1B3C6Du;
        x ^= x >> 12;
        uint64_t e = lo + (hi > lo ? x % (hi - lo) : 0);
        if (e >= m) e = m - 1;
        key[q] = ((uint64_t)ct_wkey(A.w[e], A.wt) << 32) | e;
    }
    uint64_t pre = 0;
    uint32_t want = rank;
    for (int sh = 56; sh >= 0; sh -= 8) {
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
                }
                ex += c[q];
            }
        }
        __syncthreads();
        pre = (pre << 8) | s_bin;
        want = s_rank;
        __syncthreads();
    }
    if (threadIdx.x == 0) A.cnt->ct.T = pre;
}

void ct_threshold(hipStream_t s, const CtArgs &A, int64_t light)
{
    if (light >= A.m) return;  // every edge (the threshold starts at the largest key)
    const double f = (double)light / (double)A.m;
    const uint32_t rank = std::min<uint32_t>((uint32_t)(f * CT_SAMPLES), CT_SAMPLES - 1);
    k_ct_threshold<<<1, CE_NT, 0, s>>>(A, rank);
}

// ------------------------------------------------------- list of phase 0 --
// Every edge read once and checked; those up to the threshold (no loops) go
// to the wave's segment.  A wave takes every W-th tile, so the segments are
// even whatever the order of the input.
__global__ __launch_bounds__(CE_NT) void k_ct_select(CtArgs A)
{
    __shared__ uint32_t s_cnt[CE_WV];
    const int lane = __lane_id();
    const uint32_t wv = blockIdx.x * CE_WV + (threadIdx.x >> 6);
    const uint64_t T = A.cnt->ct.T;
    const int64_t tiles = (A.m + CT_TILE - 1) / CT_TILE;
    const uint32_t n = (uint32_t)A.n;
    CtEdge *seg = A.list + (size_t)wv * A.segcap;
    uint32_t out = 0, err = 0;
    for (int64_t t = wv; t < tiles; t += A.W) {
        int2 uv[4];
        uint32_t wb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int64_t e = t * CT_TILE + q * 64 + lane;
            e = e < A.m ? e : A.m - 1;
            uv[q] = A.edges[e];
            wb[q] = A.w[e];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t e = t * CT_TILE + q * 64 + lane;
            const uint32_t a = (uint32_t)uv[q].x, b = (uint32_t)uv[q].y;
            if (a >= n || b >= n) err |= ERR_ENDPOINT;
            if (ct_nan(wb[q], A.wt)) err |= ERR_NAN;
            const uint64_t key = ((uint64_t)ct_wkey(wb[q], A.wt) << 32) | (uint32_t)e;
            const bool sel = e < A.m && !err && a != b && key <= T;
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
        if (t) atomicAdd(&A.cnt->ct.E[0][0], t);
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
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int2 uv = key[q] != KEY_INF ? A.edges[(uint32_t)key[q]] : make_int2(0, 0);
        a[q] = (uint32_t)uv.x;
        b[q] = (uint32_t)uv.y;
    }
    const int top = k < tl ? k : tl;
    for (int l = A.comp ? -1 : 0; l <= top; ++l) {
        if (l == top && k <= tl) break;
        const uint32_t *map = l < 0 ? A.comp : l < top ? ct_map(A, l) : A.cum;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (key[q] != KEY_INF) {
                a[q] = map[a[q]];
                b[q] = map[b[q]];
            }
        }
    }
}

// The rest of round k in one workgroup (at most CT_SMALL vertices): hook,
// tie break, shortcut and the next round's numbers, with the targets in LDS.
__device__ void ct_small_round(const CtArgs &A, int k, uint32_t L, uint32_t *s_h, uint32_t *s_nid,
                               uint32_t *s_c)
{
    Counters *c = A.cnt;
    const uint32_t tid = threadIdx.x;
    const uint64_t *r = A.r[k & 1];
    const uint32_t tl1 = load_relaxed_u32(&c->ct.tl[A.ph]);
    const int tl = tl1 ? (int)tl1 - 1 : k;
    constexpr int IT = CT_SMALL / CE_NT;
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
    const uint32_t dead0 = load_relaxed_u32(&c->ct.dead[A.ph]);
    const uint32_t wl0 = load_relaxed_u32(&c->ct.wl);
#pragma unroll
    for (int q = 0; q < IT; ++q) {
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
    // the first small round's vertices: what they are now
    const uint32_t L0 = tl1 ? load_relaxed_u32(&c->ct.L[A.ph][tl]) : L;
    for (uint32_t i = tid; i < L0; i += CE_NT) {
        const uint32_t x = tl1 ? A.cum[i] : i;
        if (!(x & CT_DEAD)) A.cum[i] = s_nid[s_h[x]];
    }
    uint64_t *rn = A.r[(k + 1) & 1];
    for (uint32_t i = tid; i < Ln; i += CE_NT) rn[i] = KEY_INF;
    if (tid == 0) {
        if (!tl1) c->ct.tl[A.ph] = (uint32_t)k + 1;
        c->ct.L[A.ph][k + 1] = Ln;
        c->ct.dead[A.ph] = dead0 + s_c[1];
        c->ct.hooks[A.ph][k] = s_c[2];
        c->ct.wl = wl0 + s_c[2];
        c->ct.done[A.ph][k] = 1;
        if (Ln == 0) c->ct.phdone[A.ph] = 1;
    }
}

}  // namespace

// Hot vertices of an edge pass (a star's centre, the largest tree of phase 0)
// would take one atomic after another on one address, 3 ns each: the read
// in front of an atomic sees what its XCD's L2 holds, not the latest value.
// Each workgroup samples its edges, and the vertices it meets at least
// CT_HOT_MIN times keep their minimum in LDS until the end of the pass.
constexpr uint32_t CT_HOT = 512, CT_HOT_MIN = 16;

__device__ __forceinline__ uint32_t ct_hot_slot(uint32_t v) { return (v * 0x9E3779B1u) >> 23; }

enum { CT_MIN_LDS, CT_MIN_HOT, CT_MIN_DEV };

// One wave over its segment: map the ends, lower the minima, keep the edges
// between different vertices in place.  Returns how many it kept.
template <bool FIRST, int MODE>
__device__ __forceinline__ uint32_t ct_sweep(CtEdge *seg, uint32_t cnt,
                                             const uint32_t *__restrict__ map, uint64_t *r,
                                             uint64_t *s_r, const uint32_t *s_tag)
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
        if (!FIRST) {
#pragma unroll
            for (int q = 0; q < U; ++q) {
                x[q].a = map[x[q].a];
                x[q].b = map[x[q].b];
            }
        }
        uint64_t ra[U], rb[U];
        uint32_t ha[U], hb[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (MODE == CT_MIN_LDS) {
                ra[q] = s_r[x[q].a];
                rb[q] = s_r[x[q].b];
            } else {
                ha[q] = hb[q] = CT_HOT;
                if (MODE == CT_MIN_HOT) {
                    const uint32_t sa = ct_hot_slot(x[q].a), sb = ct_hot_slot(x[q].b);
                    if (s_tag[sa] == x[q].a) ha[q] = sa;
                    if (s_tag[sb] == x[q].b) hb[q] = sb;
                }
                ra[q] = ha[q] < CT_HOT ? s_r[ha[q]] : load_relaxed_u64(r + x[q].a);
                rb[q] = hb[q] < CT_HOT ? s_r[hb[q]] : load_relaxed_u64(r + x[q].b);
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const bool live = j0 + q * 64 + lane < cnt && x[q].a != x[q].b;
            if (live) {
                if (MODE == CT_MIN_LDS) lower_lds(s_r, x[q].a, ra[q], x[q].key);
                else if (ha[q] < CT_HOT) lower_lds(s_r, ha[q], ra[q], x[q].key);
                else lower_dev(r, x[q].a, ra[q], x[q].key);
                if (MODE == CT_MIN_LDS) lower_lds(s_r, x[q].b, rb[q], x[q].key);
                else if (hb[q] < CT_HOT) lower_lds(s_r, hb[q], rb[q], x[q].key);
                else lower_dev(r, x[q].b, rb[q], x[q].key);
            }
            if (!FIRST) {
                const uint64_t mask = __ballot(live);
                if (live) seg[out + __popcll(mask & lanemask_lt())] = x[q];
                out += (uint32_t)__popcll(mask);
            }
        }
    }
    return out;
}

template <bool FIRST>
__global__ __launch_bounds__(CE_NT) void k_ct_edges(CtArgs A, int k, int big)
{
    __shared__ __align__(16) uint64_t s_r[CT_LDSR];  // also the targets of a small round
    __shared__ uint32_t s_nid[CT_SMALL];             // also the hot vertices' tags and counts
    __shared__ uint32_t s_cnt[CE_WV];
    __shared__ uint32_t s_c[4];
    static_assert(sizeof(uint64_t) * CT_LDSR >= sizeof(uint32_t) * CT_SMALL, "targets alias minima");
    Counters *c = A.cnt;
    const uint32_t L = c->ct.L[A.ph][k];
    if (c->err || L == 0 || (L > CT_SMALL && !big)) return;
    if (k > 0 ? !c->ct.done[A.ph][k - 1] : (A.ph > 0 && !c->ct.phdone[A.ph - 1])) return;
    if (c->ct.done[A.ph][k]) return;
    const int lane = __lane_id();
    const uint32_t tid = threadIdx.x, wv = blockIdx.x * CE_WV + (tid >> 6);
    if (blockIdx.x == 0 && tid == 0) c->ct.ran[A.ph][k] = 1;
    uint64_t *r = A.r[k & 1];
    const uint32_t *map = FIRST ? nullptr : ct_map(A, k - 1);
    CtEdge *seg = A.list + (size_t)wv * A.segcap;
    const uint32_t cnt = A.cw[wv];
    const bool lds = L <= CT_LDSR;
    uint32_t out = 0;
    if (lds) {
        for (uint32_t i = tid; i < L; i += CE_NT) s_r[i] = KEY_INF;
        __syncthreads();
        out = ct_sweep<FIRST, CT_MIN_LDS>(seg, cnt, map, r, s_r, nullptr);
        __syncthreads();
        for (uint32_t i = tid; i < L; i += CE_NT) {
            const uint64_t v = s_r[i];
            if (v != KEY_INF) lower_dev(r, i, load_relaxed_u64(r + i), v);
        }
    } else {
        uint32_t *s_tag = s_nid, *s_num = s_nid + CT_HOT;
        for (uint32_t i = tid; i < CT_HOT; i += CE_NT) {
            s_tag[i] = NONE32;
            s_num[i] = 0;
            s_r[i] = KEY_INF;
        }
        if (tid == 0) s_c[0] = 0;
        __syncthreads();
        uint32_t va = NONE32, vb = NONE32;
        if ((uint32_t)lane < cnt) {
            va = seg[lane].a;
            vb = seg[lane].b;
            if (!FIRST) {
                va = map[va];
                vb = map[vb];
            }
            if (va != vb) {
                atomicAdd(&s_num[ct_hot_slot(va)], 1u);
                atomicAdd(&s_num[ct_hot_slot(vb)], 1u);
            }
        }
        __syncthreads();
        if (va != vb) {
            if (s_num[ct_hot_slot(va)] >= CT_HOT_MIN) {
                s_tag[ct_hot_slot(va)] = va;
                s_c[0] = 1;
            }
            if (s_num[ct_hot_slot(vb)] >= CT_HOT_MIN) {
                s_tag[ct_hot_slot(vb)] = vb;
                s_c[0] = 1;
            }
        }
        __syncthreads();
        if (s_c[0]) {
            out = ct_sweep<FIRST, CT_MIN_HOT>(seg, cnt, map, r, s_r, s_tag);
            __syncthreads();
            for (uint32_t i = tid; i < CT_HOT; i += CE_NT) {
                const uint64_t v = s_r[i];
                if (v != KEY_INF) lower_dev(r, s_tag[i], load_relaxed_u64(r + s_tag[i]), v);
            }
        } else {
            out = ct_sweep<FIRST, CT_MIN_DEV>(seg, cnt, map, r, s_r, s_tag);
        }
    }
    if (!FIRST) {
        if (lane == 0) {
            A.cw[wv] = out;
            s_cnt[tid >> 6] = out;
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t t = 0;
            for (int i = 0; i < CE_WV; ++i) t += s_cnt[i];
            if (t) atomicAdd(&c->ct.E[A.ph][k], t);
        }
    }
    if (L > CT_SMALL) return;
    // The last workgroup of a small round finishes it.  It reads only r,
    // which is written by device-scope atomics alone: each wave waits for
    // its own before the ticket (a release fence would write back the whole
    // L2 in every workgroup, 70-220 us a pass), and the last one drops what
    // its L2 holds of r before reading.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) s_c[1] = atomicAdd(&c->ct.tick[A.ph][k], 1u);
    __syncthreads();
    if (s_c[1] != gridDim.x - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    ct_small_round(A, k, L, reinterpret_cast<uint32_t *>(s_r), s_nid, s_c);
}

// ------------------------------------------------ rounds of many vertices --

// Whether round k's kernels after the edge pass have work.
__device__ __forceinline__ bool ct_big_round(const CtArgs &A, int k, uint32_t L)
{
    const Counters *c = A.cnt;
    return L > CT_SMALL && !c->err && c->ct.ran[A.ph][k];
}

__global__ __launch_bounds__(256) void k_ct_hook(CtArgs A, int k)
{
    const uint32_t L = A.cnt->ct.L[A.ph][k];
    if (!ct_big_round(A, k, L) || A.cnt->ct.done[A.ph][k]) return;
    const uint64_t *r = A.r[k & 1];
    constexpr int U = 4;
    for (uint64_t base = (uint64_t)blockIdx.x * (256 * U); base < L;
         base += (uint64_t)gridDim.x * (256 * U)) {
        uint64_t key[U];
        uint32_t a[U], b[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint64_t i = base + q * 256 + threadIdx.x;
            key[q] = i < L ? r[i] : KEY_INF;
        }
        ct_ends<U>(A, key, k, k, a, b);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint64_t i = base + q * 256 + threadIdx.x;
            if (i < L) A.h[i] = key[q] == KEY_INF ? (uint32_t)i : (a[q] == (uint32_t)i ? b[q] : a[q]);
        }
    }
}

// Tie break, forest flags, weights, and the numbers of the vertices that
// stay (dense from 0) and of the finished trees.  A tile is IT x 512
// consecutive vertices; the numbers keep the vertices' order inside it
// (item-major, then wave, then lane) and each tile takes its range with one
// atomic, so neighbours stay neighbours.
constexpr int TIE_NT = 512;

template <int IT, int WT>
__global__ __launch_bounds__(TIE_NT) void k_ct_tie(CtArgs A, int k)
{
    constexpr int NW = TIE_NT / 64;
    static_assert(IT * NW <= 128 && (IT * NW) % 2 == 0, "two counts a lane");
    __shared__ uint32_t s_off[2][128];
    __shared__ uint32_t s_base[2];
    __shared__ int64_t s_sum[NW * (ACC_DIGITS + 1)];
    __shared__ int64_t s_tot[WS_WORDS];
    __shared__ uint32_t s_hk[NW];
    Counters *c = A.cnt;
    const uint32_t L = c->ct.L[A.ph][k];
    if (!ct_big_round(A, k, L) || c->ct.done[A.ph][k]) return;
    const uint64_t *r = A.r[k & 1];
    uint32_t *map = ct_map(A, k);
    const uint32_t w = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    const uint32_t tiles = (uint32_t)(((uint64_t)L + IT * TIE_NT - 1) / (IT * TIE_NT));
    WSum ws;
    uint32_t hooks = 0;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint64_t base = (uint64_t)tile * (IT * TIE_NT) + threadIdx.x;
        uint32_t t[IT], back[IT];
        uint64_t key[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            t[q] = i < L ? load_relaxed_u32(A.h + i) : NONE32;
            key[q] = i < L ? r[i] : KEY_INF;
        }
#pragma unroll
        for (int q = 0; q < IT; ++q)
            back[q] = key[q] != KEY_INF ? load_relaxed_u32(A.h + t[q]) : NONE32;
        uint32_t stay = 0, dead = 0;
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            if (i >= L) continue;
            if (key[q] == KEY_INF) {
                dead |= 1u << q;
            } else if (back[q] == (uint32_t)i && (uint32_t)i < t[q]) {
                store_relaxed_u32(A.h + i, (uint32_t)i);
                stay |= 1u << q;
            } else {
                A.flags[(uint32_t)key[q]] = 1;
                wsum_add<WT>(ws, (uint32_t)(key[q] >> 32));
                ++hooks;
            }
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
            const uint32_t l2 = 2 * __lane_id();
            const uint32_t c0 = l2 < IT * NW ? s_off[w][l2] : 0u;
            const uint32_t c1 = l2 + 1 < IT * NW ? s_off[w][l2 + 1] : 0u;
            const uint32_t inc = wave_incl_sum(c0 + c1);
            if (l2 < IT * NW) {
                s_off[w][l2] = inc - c0 - c1;
                s_off[w][l2 + 1] = inc - c1;
            }
            if (__lane_id() == 63)
                s_base[w] = inc ? atomicAdd(w ? &c->ct.dead[A.ph] : &c->ct.L[A.ph][k + 1], inc) : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const uint64_t i = base + q * TIE_NT;
            const bool a = (stay >> q) & 1u, b = (dead >> q) & 1u;
            const uint64_t ms = __ballot(a), md = __ballot(b);
            if (a) map[i] = s_base[0] + s_off[0][q * NW + w] + (uint32_t)__popcll(ms & lt);
            if (b) map[i] = CT_DEAD | (s_base[1] + s_off[1][q * NW + w] + (uint32_t)__popcll(md & lt));
        }
        __syncthreads();
    }
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
// shorter (the hooks form no cycle after the tie break).
__global__ __launch_bounds__(256) void k_ct_chase(CtArgs A, int k)
{
    Counters *c = A.cnt;
    const uint32_t L = c->ct.L[A.ph][k];
    if (!ct_big_round(A, k, L)) return;
    const uint32_t Ln = c->ct.L[A.ph][k + 1];
    uint32_t *map = ct_map(A, k);
    uint64_t *rn = A.r[(k + 1) & 1];
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += stride) {
        uint32_t x = load_relaxed_u32(A.h + i);
        if (x != (uint32_t)i) {
            uint32_t steps = 0;
            for (;;) {
                const uint32_t y = load_relaxed_u32(A.h + x);
                if (y == x) break;
                x = y;
                store_relaxed_u32(A.h + i, x);
                if (++steps > L) {  // cannot happen: a cycle of hooks
                    atomicOr(&c->err, ERR_CYCLE);
                    break;
                }
            }
            map[i] = map[x];
        }
        if (i < Ln) rn[i] = KEY_INF;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->ct.done[A.ph][k] = 1;
        if (Ln == 0) c->ct.phdone[A.ph] = 1;
    }
}

void ct_round(hipStream_t s, const CtArgs &A, int k, bool big, uint32_t bound)
{
    const unsigned g = A.W / CE_WV;
    if (k == 0) k_ct_edges<true><<<g, CE_NT, 0, s>>>(A, k, big);
    else k_ct_edges<false><<<g, CE_NT, 0, s>>>(A, k, big);
    if (!big || bound <= CT_SMALL) return;
    k_ct_hook<<<grid_for(bound, 1024, 4096), 256, 0, s>>>(A, k);
    // 16 vertices a thread while there are many (one atomic per 8192), four
    // with fewer, to keep the compute units busy
    if (bound >= (1u << 22)) {
        const unsigned t = grid_for(bound, 16 * TIE_NT, CT_WSLOTS);
        if (A.wt == MSF_W_F32) k_ct_tie<16, MSF_W_F32><<<t, TIE_NT, 0, s>>>(A, k);
        else k_ct_tie<16, MSF_W_U32><<<t, TIE_NT, 0, s>>>(A, k);
    } else {
        const unsigned t = grid_for(bound, 4 * TIE_NT, CT_WSLOTS);
        if (A.wt == MSF_W_F32) k_ct_tie<4, MSF_W_F32><<<t, TIE_NT, 0, s>>>(A, k);
        else k_ct_tie<4, MSF_W_U32><<<t, TIE_NT, 0, s>>>(A, k);
    }
    k_ct_chase<<<grid_for(bound, 256, 8192), 256, 0, s>>>(A, k);
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
    if (blockIdx.x == 0 && threadIdx.x == 0) c->ct.L[1][0] = c->ct.dead[0];
}

// The tree that most of 1024 sampled edge ends lie in.
__global__ __launch_bounds__(CE_NT) void k_ct_giant(CtArgs A, const uint32_t *__restrict__ comp)
{
    __shared__ __align__(16) uint32_t s_v[CE_NT];
    __shared__ unsigned long long s_best;
    Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[0] || c->ct.ran[1][0]) return;
    const int64_t e = (int64_t)((uint64_t)A.m * threadIdx.x / CE_NT);
    const int2 uv = A.edges[e];
    const uint32_t v = comp[(threadIdx.x & 1) ? uv.x : uv.y];
    s_v[threadIdx.x] = v;
    if (threadIdx.x == 0) s_best = 0;
    __syncthreads();
    uint32_t same = 0;
    const uint4 *s_v4 = reinterpret_cast<const uint4 *>(s_v);
#pragma unroll 8
    for (int i = 0; i < CE_NT / 4; ++i) {
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
    const uint32_t wv = blockIdx.x * CE_WV + (threadIdx.x >> 6);
    const int64_t tiles = (A.m + CT_TILE - 1) / CT_TILE;
    CtEdge *seg = A.list + (size_t)wv * A.segcap;
    uint32_t out = 0;
    for (int64_t t = wv; t < tiles; t += A.W) {
        int2 uv[4];
        bool go[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t e = t * CT_TILE + q * 64 + lane;
            uv[q] = A.edges[e < A.m ? e : A.m - 1];
            go[q] = e < A.m;
        }
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
        if (t) atomicAdd(&c->ct.E[1][0], t);
    }
}

void ct_between(hipStream_t s, const CtArgs &A, uint32_t *comp, uint32_t *bits)
{
    k_ct_compose<<<grid_for((size_t)A.n, 256, 8192), 256, 0, s>>>(A, comp);
    // a table of 2^20 trees (4 MB) still fits an L2: 205 G lookups/s against
    // 76 at 2^22, where the bits give 259 (64M random lookups)
    if (A.n > (1 << 20)) {
        k_ct_giant<<<1, CE_NT, 0, s>>>(A, comp);
        k_ct_bits<<<grid_for(((size_t)A.n + 63) / 64, 4, 4096), 256, 0, s>>>(
            A, comp, reinterpret_cast<uint64_t *>(bits));
        k_ct_between<true><<<A.W / CE_WV, CE_NT, 0, s>>>(A, comp, bits);
    } else {
        k_ct_between<false><<<A.W / CE_WV, CE_NT, 0, s>>>(A, comp, nullptr);
    }
}

// ------------------------------------------------------------------ total --

template <int WT>
__global__ __launch_bounds__(CE_NT) void k_ct_total(CtArgs A, int last_phase)
{
    __shared__ int64_t s_sum[CE_WV * (ACC_DIGITS + 1)];
    __shared__ int64_t s_tot[WS_WORDS];
    Counters *c = A.cnt;
    if (c->err || !c->ct.phdone[last_phase]) return;
    WSum ws;
    for (uint32_t i = threadIdx.x; i < CT_WSLOTS; i += CE_NT) {
        if (WT == MSF_W_U32) {
            ws.su += (uint64_t)A.wpart[i];
        } else {
#pragma unroll
            for (int d = 0; d < ACC_DIGITS; ++d) ws.acc[d] += A.wpart[(size_t)(1 + d) * CT_WSLOTS + i];
            ws.pinf += (uint32_t)A.wpart[(size_t)(1 + ACC_DIGITS) * CT_WSLOTS + i];
            ws.ninf += (uint32_t)A.wpart[(size_t)(2 + ACC_DIGITS) * CT_WSLOTS + i];
        }
    }
    const uint32_t wl = c->ct.wl;
    for (uint32_t i = threadIdx.x; i < wl; i += CE_NT) wsum_add<WT>(ws, A.wlist[i]);
    wsum_block<CE_NT, WT>(ws, s_sum, s_tot, 1);
    if (threadIdx.x == 0) {
        c->total_u64 = WT == MSF_W_U32 ? (uint64_t)s_tot[0] : 0;
        c->total_f64 = exact_total_f64((uint64_t)s_tot[0], s_tot + 1,
                                       (uint32_t)s_tot[1 + ACC_DIGITS],
                                       (uint32_t)s_tot[2 + ACC_DIGITS], WT);
        c->ct.fin = 1;
    }
}

void ct_total(hipStream_t s, const CtArgs &A, int last_phase)
{
    if (A.wt == MSF_W_F32) k_ct_total<MSF_W_F32><<<1, CE_NT, 0, s>>>(A, last_phase);
    else k_ct_total<MSF_W_U32><<<1, CE_NT, 0, s>>>(A, last_phase);
}

}  // namespace msf
