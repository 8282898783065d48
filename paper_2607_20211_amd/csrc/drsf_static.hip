// Static rebuild of a rooted spanning forest (the baseline the dynamic update
// is measured against, Sec. V's static GPU BFS): connected components by
// linking, each rooted at its smallest vertex, then a breadth-first forest
// from all roots at once.  Kept apart from the update path; it shares only
// the small fill and grid helpers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <mutex>

#include "../../include/drsf.h"
#include "drsf_kernels.h"

namespace drsf {
namespace {

// position of this lane's entry in a list counted by *cnt, one atomic per
// wave (every lane of the wave calls it)
__device__ __forceinline__ int64_t wave_append(bool take, unsigned long long *cnt) {
    const uint64_t m = __ballot(take);
    if (!m) return 0;
    const int leader = __ffsll((unsigned long long)m) - 1;
    unsigned long long base = 0;
    if (lane_id() == leader) base = atomicAdd(cnt, (unsigned long long)__popcll(m));
    base = __shfl(base, leader);
    return (int64_t)base + __popcll(m & ((1ull << lane_id()) - 1ull));
}

// Frontier appends gathered per workgroup: claims go to an LDS buffer (one
// LDS atomic per wave and call) and the workgroup reserves its whole run of
// the next frontier with one global atomic at the end; claims beyond the
// buffer fall back to a global append per wave.  Every atomic on the one
// frontier counter costs a serialised round trip, so per-wave appends from
// thousands of waves were most of a level's time.
constexpr int APP_BUF = 4096;
// Threads of a workgroup that a wide level runs with: its atomics on the level
// counters (three a workgroup, on the same words) were most of its time (R-MAT
// 20's widest level, 524288 threads: 178 us in workgroups of 256, 92 of 512, 50
// of 1024).
constexpr int WIDE_BLOCK = 1024;
struct Appender {
    int32_t buf[APP_BUF];
    int n;
    unsigned long long base;
};
__device__ __forceinline__ void app_begin(Appender &a) {
    if (threadIdx.x == 0) a.n = 0;
    __syncthreads();
}
// every lane of the wave calls it
__device__ __forceinline__ void app_push(Appender &a, bool take, int32_t w, int32_t *next,
                                         unsigned long long *ncnt) {
    const uint64_t m = __ballot(take);
    if (!m) return;
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane_id() == leader) base = atomicAdd(&a.n, __popcll(m));
    base = __shfl(base, leader);
    const int pos = base + __popcll(m & ((1ull << lane_id()) - 1ull));
    const bool spill = take && pos >= APP_BUF;
    if (take && !spill) a.buf[pos] = w;
    if (base + __popcll(m) > APP_BUF) {  // wave-uniform
        const int64_t g = wave_append(spill, ncnt);
        if (spill) next[g] = w;
    }
}
// every thread of the workgroup calls it
template <int BS>
__device__ __forceinline__ void app_end(Appender &a, int32_t *next, unsigned long long *ncnt) {
    __syncthreads();
    const int k = a.n < APP_BUF ? a.n : APP_BUF;
    if (threadIdx.x == 0 && k > 0) a.base = atomicAdd(ncnt, (unsigned long long)k);
    __syncthreads();
    for (int i = threadIdx.x; i < k; i += BS) next[a.base + i] = a.buf[i];
}

// Row lengths of the vertices a workgroup claimed, into the next level's
// degree sum and maximum (stat[0] sum, stat[1] max): each thread accumulates
// over its whole grid-stride loop, then one atomic pair per workgroup (every
// thread calls it once, at the end of the kernel).
template <int BS>
__device__ __forceinline__ void block_degree(unsigned long long sum, unsigned long long mx,
                                             unsigned long long *stat) {
    __shared__ unsigned long long s_sum[BS / WAVE], s_max[BS / WAVE];
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        const unsigned long long y = __shfl_xor(mx, o);
        mx = y > mx ? y : mx;
    }
    if (lane_id() == 0) {
        s_sum[threadIdx.x / WAVE] = sum;
        s_max[threadIdx.x / WAVE] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0, m = 0;
        for (int w = 0; w < BS / WAVE; w++) {
            t += s_sum[w];
            m = s_max[w] > m ? s_max[w] : m;
        }
        if (t) {
            atomicAdd(&stat[0], t);
            if (stat[1] < m) atomicMax(&stat[1], m);
        }
    }
}
// Level counters: three groups of four words, level L's in group L % 3
// (frontier vertices with rows of up to LONG_ROW slots, listed from the
// frontier's front; row-length sum; longest row; frontier vertices with longer
// rows, listed from its end), then the depth word (the number of non-empty
// levels seen so far) and two words for the level reached: launch k reads the
// one of its parity and writes the other, so levels run back to back with no
// host step between them, whatever number of levels a launch does.  The kernel
// of level L reads group L % 3, fills group (L + 1) % 3 and clears group
// (L + 2) % 3 for the level after.
constexpr int CNT_DEPTH = 12, CNT_LEVEL = 13, CNT_WORDS = 15;
__device__ __forceinline__ unsigned long long *level_group(unsigned long long *g, int L) { return g + 4 * (L % 3); }
__device__ __forceinline__ void level_begin(unsigned long long *g, int L, int k, bool nonempty) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        unsigned long long *c = level_group(g, L + 2);
        c[0] = 0;
        c[1] = 0;
        c[2] = 0;
        c[3] = 0;
        if (nonempty) g[CNT_DEPTH] = (unsigned long long)(L + 1);
        g[CNT_LEVEL + ((k + 1) & 1)] = (unsigned long long)(L + (nonempty ? 1 : 0));
    }
}

// A claimed vertex (every lane of the wave calls it): its row length into the
// sums, itself into the next frontier.
constexpr int LONG_ROW = 1024;
__device__ __forceinline__ void claim_vertex(Appender &app, bool take, const int64_t *row_ptr, int32_t n, int32_t w,
                                             int32_t *next, unsigned long long *ng, unsigned long long &sum,
                                             unsigned long long &mx) {
    unsigned long long dg = 0;
    if (take) {
        dg = (unsigned long long)(row_ptr[w + 1] - row_ptr[w]);
        sum += dg;
        mx = dg > mx ? dg : mx;
        if (dg > LONG_ROW) next[n - 1 - (int64_t)atomicAdd(&ng[3], 1ull)] = w;
    }
    app_push(app, take && dg <= LONG_ROW, w, next, ng);
}

// ------------------------------------------------------------ components
//
// Every tree of comp[] is rooted at its smallest vertex: a root only ever
// hooks below a smaller one.  One pass that links the ends of every edge is
// enough (a link ends when both ends hang below one vertex), and most edges
// need not be looked at: after each vertex has been linked to its first two
// neighbours, nearly all of a large component hangs together, so its vertices
// skip the rest of their rows, which their neighbours outside it cover from
// their side (the sampling of Sutton, Ben-Nun and Barak's Afforest).  Bound by
// the gathers of the first two slots.  R-MAT 20 with 31.4e6 slots: 51 us for
// these kernels; three hooking rounds over every slot took 408 and the row of
// every slot, which they read, 326.

// A link only swaps roots, it does not shorten the path it walks.  Several
// threads halving one path store different ancestors into one word: a data
// race, so the stores have to be atomic, and those were slower than longer walks
// (G(1e6, 5e6), first links: 117 us without, 552 from the ninth step on).  Plain
// stores are no choice: on a 2048 x 2048 grid 1 to 7 vertices of each call kept a
// former ancestor as their label, with atomic stores or none no vertex did (how
// the plain ones lead there is not known: a kernel of such stores alone, read
// back from all XCDs, showed nothing).
__device__ __forceinline__ void st_link(int32_t *comp, int32_t u, int32_t v) {
    int32_t a = comp[u], b = comp[v];
    while (a != b) {
        const int32_t hi = a > b ? a : b, lo = a > b ? b : a;
        int32_t up = comp[hi];  // may be stale: an ancestor at most hi all the same
        if (up == hi) {
            up = atomicCAS(&comp[hi], hi, lo);
            if (up == hi) return;
        }
        a = up;  // below hi: every turn goes down in ids
        b = lo;
    }
}
// every vertex below its first neighbour if that is smaller, else a root (and
// the level counters cleared)
__global__ __launch_bounds__(BLOCK) void k_st_comp_init(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                                        int32_t *comp, unsigned long long *g) {
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    if (blockIdx.x == 0 && threadIdx.x < CNT_WORDS) g[threadIdx.x] = 0;
    for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n; v += stride) {
        const int64_t a = row_ptr[v];
        int32_t c = (int32_t)v;
        if (a < row_ptr[v + 1] && col[a] < c) c = col[a];
        comp[v] = c;
    }
}
__global__ __launch_bounds__(BLOCK) void k_st_link_first(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                                         int32_t *comp) {
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n; v += stride) {
        const int64_t a = row_ptr[v], b = row_ptr[v + 1];
        if (a < b && col[a] > v) st_link(comp, (int32_t)v, col[a]);
        if (a + 1 < b) st_link(comp, (int32_t)v, col[a + 1]);
    }
}
// pointer jumping to the roots, every step published (long chains of
// vertices walked at the same time shorten each other)
__global__ __launch_bounds__(BLOCK) void k_st_compress(int32_t n, int32_t *comp) {
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n; v += stride) {
        int32_t x = comp[v];
        for (int32_t y = comp[x]; y != x; y = comp[x]) {
            comp[v] = y;
            x = y;
        }
    }
}
// the label that most of a sample of the vertices carry
constexpr int SAMPLE = 1024;
__global__ __launch_bounds__(BLOCK) void k_st_sample(int32_t n, const int32_t *comp, int32_t *giant) {
    __shared__ int32_t s_id[SAMPLE * 2];
    __shared__ int s_cnt[SAMPLE * 2];
    __shared__ int s_best;
    for (int i = threadIdx.x; i < SAMPLE * 2; i += BLOCK) {
        s_id[i] = -1;
        s_cnt[i] = 0;
    }
    if (threadIdx.x == 0) s_best = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < SAMPLE; i += BLOCK) {
        const int32_t l = comp[hmix((uint64_t)i + 1) % (uint64_t)n];
        uint32_t h = (uint32_t)l * 2654435769u % (SAMPLE * 2);
        for (;;) {  // at most SAMPLE labels in twice as many places
            const int32_t was = atomicCAS(&s_id[h], -1, l);
            if (was == -1 || was == l) break;
            h = (h + 1) % (SAMPLE * 2);
        }
        atomicAdd(&s_cnt[h], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SAMPLE * 2; i += BLOCK)
        if (s_cnt[i]) atomicMax(&s_best, s_cnt[i] << 11 | i);
    __syncthreads();
    if (threadIdx.x == 0) *giant = s_id[s_best & (SAMPLE * 2 - 1)];
}
static_assert(SAMPLE * 2 == 1 << 11, "a place fits the low bits of the vote");
// the rest of the rows outside the sampled component: short ones by a lane,
// longer ones by the wave
__global__ __launch_bounds__(BLOCK) void k_st_link_rest(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                                        int32_t *comp, const int32_t *giant) {
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    const int32_t skip = *giant;
    for (int64_t base = (int64_t)blockIdx.x * BLOCK; base < n; base += stride) {
        const int64_t v = base + threadIdx.x;
        int64_t a = 0, b = 0;
        if (v < n && comp[v] != skip) {
            a = row_ptr[v] + 2;
            b = row_ptr[v + 1];
        }
        const bool big = b - a > 32;
        if (!big)
            for (int64_t s = a; s < b; s++) st_link(comp, (int32_t)v, col[s]);
        uint64_t m = __ballot(big);
        while (m) {
            const int l = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const int32_t bv = __shfl((int32_t)v, l);
            const int64_t ba = __shfl(a, l), bb = __shfl(b, l);
            for (int64_t s = ba + lane_id(); s < bb; s += WAVE) st_link(comp, bv, col[s]);
        }
    }
}

// --------------------------------------------------- breadth-first levels

// roots: level 0, their own parents, the first frontier (those with edges)
__global__ __launch_bounds__(WIDE_BLOCK) void k_st_bfs_init(int32_t n, const int64_t *row_ptr, const int32_t *comp,
                                                       int32_t *level, int32_t *parent, int32_t *front,
                                                       unsigned long long *g) {
    const int64_t stride = (int64_t)gridDim.x * WIDE_BLOCK;
    unsigned long long *fg = level_group(g, 0);
    __shared__ Appender app;
    app_begin(app);
    unsigned long long dsum = 0, dmax = 0;
    for (int64_t base = (int64_t)blockIdx.x * WIDE_BLOCK; base < n; base += stride) {
        const int64_t v = base + threadIdx.x;
        const bool root = v < n && comp[v] == (int32_t)v;
        if (v < n) {
            level[v] = root ? 0 : -1;
            parent[v] = root ? (int32_t)v : -1;
        }
        const bool start = root && row_ptr[v + 1] > row_ptr[v];
        claim_vertex(app, start, row_ptr, n, (int32_t)v, front, fg, dsum, dmax);
    }
    app_end<WIDE_BLOCK>(app, front, fg);
    block_degree<WIDE_BLOCK>(dsum, dmax, fg + 1);
}

// Top-down level: each unvisited neighbour of the frontier is claimed by a
// compare-and-swap on its level.  Rows of up to SHORT_ROW slots are walked by
// four lanes each (sixteen frontier vertices per wave, the wave looping to its
// longest such row), rows of up to LONG_ROW by the whole wave, and longer ones
// (a hub's) by the whole grid.
constexpr int SHORT_ROW = 32;
__device__ __forceinline__ bool td_claim(const int32_t *col, int32_t *level, int32_t *parent, int L, int32_t v,
                                         int64_t s, int32_t &w) {
    w = col[s];
    const bool claim = level[w] < 0 && atomicCAS(&level[w], -1, L + 1) == -1;
    if (claim) parent[w] = v;
    return claim;
}
template <int BS>
__device__ __forceinline__ void top_down(Appender &app, int32_t n, const int64_t *row_ptr, const int32_t *col,
                                         int32_t *level, int32_t *parent, int L, const int32_t *front,
                                         int32_t *next, unsigned long long *g, unsigned long long &dsum,
                                         unsigned long long &dmax) {
    const int64_t nf = (int64_t)level_group(g, L)[0], nlong = (int64_t)level_group(g, L)[3];
    unsigned long long *ng = level_group(g, L + 1);
    const int sub = lane_id() & 3;
    const int64_t step = (int64_t)gridDim.x * (BS / WAVE) * (WAVE / 4);
    for (int64_t f0 = ((int64_t)blockIdx.x * (BS / WAVE) + threadIdx.x / WAVE) * (WAVE / 4); f0 < nf;
         f0 += step) {
        const int64_t f = f0 + (lane_id() >> 2);
        int32_t v = 0;
        int64_t a = 0, b = 0;
        if (f < nf) {
            v = front[f];
            a = row_ptr[v];
            b = row_ptr[v + 1];
        }
        const bool big = b - a > SHORT_ROW;
        int rounds = big ? 0 : (int)((b - a + 3) >> 2);
        for (int o = WAVE / 2; o > 0; o >>= 1) {
            const int y = __shfl_xor(rounds, o);
            rounds = y > rounds ? y : rounds;
        }
        for (int r = 0; r < rounds; r++) {
            const int64_t sl = a + 4 * r + sub;
            bool claim = false;
            int32_t w = 0;
            if (!big && sl < b) claim = td_claim(col, level, parent, L, v, sl, w);
            claim_vertex(app, claim, row_ptr, n, w, next, ng, dsum, dmax);
        }
        uint64_t bm = __ballot(big && sub == 0);
        while (bm) {
            const int l = __ffsll((unsigned long long)bm) - 1;
            bm &= bm - 1;
            const int32_t bv = __shfl(v, l);
            const int64_t ba = __shfl(a, l), bb = __shfl(b, l);
            for (int64_t s0 = ba; s0 < bb; s0 += WAVE) {
                const int64_t sl = s0 + lane_id();
                bool claim = false;
                int32_t w = 0;
                if (sl < bb) claim = td_claim(col, level, parent, L, bv, sl, w);
                claim_vertex(app, claim, row_ptr, n, w, next, ng, dsum, dmax);
            }
        }
    }
    for (int64_t i = 0; i < nlong; i++) {
        const int32_t v = front[n - 1 - i];
        const int64_t a = row_ptr[v], b = row_ptr[v + 1];
        for (int64_t s0 = a + ((int64_t)blockIdx.x * BS + threadIdx.x) / WAVE * WAVE; s0 < b;
             s0 += (int64_t)gridDim.x * BS) {
            const int64_t sl = s0 + lane_id();
            bool claim = false;
            int32_t w = 0;
            if (sl < b) claim = td_claim(col, level, parent, L, v, sl, w);
            claim_vertex(app, claim, row_ptr, n, w, next, ng, dsum, dmax);
        }
    }
}

// Bottom-up level for a large frontier: every unvisited vertex looks along
// its row for a neighbour on level L and takes one that it meets as its
// parent (no atomics: a vertex writes only its own entries; the level L + 1
// it writes is never mistaken for L).  A row that has shown none in its first
// BU_LANE slots is walked on by the whole wave; looking at 2, 4 or 8 slots at
// once instead of one measured the same.
constexpr int BU_LANE = 64;
template <int BS>
__device__ __forceinline__ void bottom_up(Appender &app, int32_t n, const int64_t *row_ptr, const int32_t *col,
                                          int32_t *level, int32_t *parent, int L, int32_t *next,
                                          unsigned long long *g, unsigned long long &dsum,
                                          unsigned long long &dmax) {
    const int64_t stride = (int64_t)gridDim.x * BS;
    unsigned long long *ng = level_group(g, L + 1);
    for (int64_t base = (int64_t)blockIdx.x * BS; base < n; base += stride) {
        const int64_t v = base + threadIdx.x;
        int32_t p = -1;
        int64_t s = 0, b = 0;
        if (v < n && level[v] < 0) {
            s = row_ptr[v];
            b = row_ptr[v + 1];
            const int64_t e = b - s > BU_LANE ? s + BU_LANE : b;
            for (; s < e && p < 0; s++) {
                const int32_t u = col[s];
                if (level[u] == L) p = u;
            }
        }
        uint64_t m = __ballot(p < 0 && s < b);
        while (m) {
            const int lane = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const int64_t ws = __shfl(s, lane), wb = __shfl(b, lane);
            int32_t got = -1;
            uint64_t hit = 0;
            for (int64_t t0 = ws; t0 < wb && !hit; t0 += WAVE) {
                const int64_t t = t0 + lane_id();
                got = t < wb ? col[t] : -1;
                hit = __ballot(got >= 0 && level[got] == L);
            }
            if (hit) {
                got = __shfl(got, __ffsll((unsigned long long)hit) - 1);
                if (lane_id() == lane) p = got;
            }
        }
        if (p >= 0) {
            parent[v] = p;
            level[v] = L + 1;
        }
        claim_vertex(app, p >= 0, row_ptr, n, (int32_t)v, next, ng, dsum, dmax);
    }
}

// A frontier with few edges is expanded from its own rows, one with many
// bottom-up.
__host__ __device__ inline bool few_edges(uint64_t dsum, int64_t nnz) { return dsum * 16 < (uint64_t)nnz; }

// One level, top-down or as its counters say (choose): the levels can be
// queued without the host reading them in between.  k: the number of the
// launch (its parity); fronts are taken by the level's parity.
template <int BS>
__global__ __launch_bounds__(BS) void k_st_level(int32_t n, int64_t nnz, const int64_t *row_ptr, const int32_t *col,
                                                 int32_t *level, int32_t *parent, int k, int32_t *front0,
                                                 int32_t *front1, unsigned long long *g, int choose) {
    const int L = (int)g[CNT_LEVEL + (k & 1)];
    const unsigned long long *c = level_group(g, L);
    const bool nonempty = c[0] + c[3] > 0;
    level_begin(g, L, k, nonempty);
    if (!nonempty) return;
    const int32_t *front = L & 1 ? front1 : front0;
    int32_t *next = L & 1 ? front0 : front1;
    __shared__ Appender app;
    app_begin(app);
    unsigned long long dsum = 0, dmax = 0;
    if (!choose || few_edges(c[1], nnz))
        top_down<BS>(app, n, row_ptr, col, level, parent, L, front, next, g, dsum, dmax);
    else
        bottom_up<BS>(app, n, row_ptr, col, level, parent, L, next, g, dsum, dmax);
    app_end<BS>(app, next, level_group(g, L + 1));
    block_degree<BS>(dsum, dmax, level_group(g, L + 1) + 1);
}

// Levels with a small frontier and short rows, by one workgroup, until one is
// not or SOLO_LEVELS are done (so a launch ends in bounded time): a level's
// claims stay in LDS with their rows, which leaves it three dependent memory
// accesses (the slot, the neighbour's level, its row) and no launch.  Bound by
// them.  A path of 20000 vertices took 109 ms with a launch a level and takes
// 24; a 512 x 512 grid (frontiers up to 512) 7.0 and 3.6.  The workgroup walks
// 256 rows at once, so beyond SOLO_FRONTIER a launch over the chip is as fast:
// a 2048 x 2048 grid took 26.3, 25.3, 27.3 and 49.9 ms with bounds of 256, 512,
// 1024 and 2048, the 512 x 512 grid 4.7, 3.6, 3.5 and 3.6.
constexpr int SOLO_FRONTIER = 512, SOLO_ROW = 32, SOLO_LEVELS = 4096;
__global__ __launch_bounds__(WIDE_BLOCK) void k_st_solo(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                                        int32_t *level, int32_t *parent, int k, int32_t *front0,
                                                        int32_t *front1, unsigned long long *g) {
    __shared__ int32_t s_v[2][SOLO_FRONTIER], s_len[2][SOLO_FRONTIER];
    __shared__ int64_t s_row[2][SOLO_FRONTIER];
    __shared__ int s_n[2], s_long, s_wide;
    const int L0 = (int)g[CNT_LEVEL + (k & 1)];
    const unsigned long long *c0 = level_group(g, L0);
    const int64_t nf0 = (int64_t)c0[0];
    int L = L0;
    if (nf0 > 0 && nf0 <= SOLO_FRONTIER && c0[3] == 0 && c0[2] <= SOLO_ROW) {
        const int32_t *front = L & 1 ? front1 : front0;
        for (int i = threadIdx.x; i < nf0; i += WIDE_BLOCK) {
            const int32_t v = front[i];
            const int64_t a = row_ptr[v];
            s_v[L & 1][i] = v;
            s_row[L & 1][i] = a;
            s_len[L & 1][i] = (int32_t)(row_ptr[v + 1] - a);
        }
        if (threadIdx.x == 0) {
            s_n[L & 1] = (int)nf0;
            s_n[(L + 1) & 1] = 0;
            s_long = 0;
            s_wide = 0;
        }
        unsigned long long dsum, dmax;
        for (;;) {
            __syncthreads();
            const int b = L & 1, nf = s_n[b];
            int32_t *next = b ? front0 : front1;
            dsum = dmax = 0;
            for (int f = threadIdx.x >> 2; f < nf; f += WIDE_BLOCK / 4) {
                const int32_t v = s_v[b][f], len = s_len[b][f];
                const int64_t a = s_row[b][f];
                for (int r = threadIdx.x & 3; r < len; r += 4) {
                    const int32_t w = col[a + r];
                    if (level[w] >= 0 || atomicCAS(&level[w], -1, L + 1) != -1) continue;
                    parent[w] = v;
                    const int64_t wa = row_ptr[w], wl = row_ptr[w + 1] - wa;
                    dsum += (unsigned long long)wl;
                    dmax = (unsigned long long)wl > dmax ? (unsigned long long)wl : dmax;
                    if (wl > SOLO_ROW) s_wide = 1;
                    if (wl > LONG_ROW) {
                        next[n - 1 - (int64_t)atomicAdd(&s_long, 1)] = w;
                        continue;
                    }
                    const int p = atomicAdd(&s_n[b ^ 1], 1);
                    if (p < SOLO_FRONTIER) {
                        s_v[b ^ 1][p] = w;
                        s_row[b ^ 1][p] = wa;
                        s_len[b ^ 1][p] = (int32_t)wl;
                    } else {
                        next[p] = w;
                    }
                }
            }
            __syncthreads();
            L++;
            const int nn = s_n[b ^ 1];
            if (nn == 0 || nn > SOLO_FRONTIER || s_wide || L - L0 >= SOLO_LEVELS) break;
            if (threadIdx.x == 0) s_n[b] = 0;
        }
        // the frontier reached and its counters, as a level's kernel leaves them
        const int b = L & 1, nn = s_n[b];
        int32_t *front_out = b ? front1 : front0;
        for (int i = threadIdx.x; i < nn && i < SOLO_FRONTIER; i += WIDE_BLOCK) front_out[i] = s_v[b][i];
        unsigned long long *c = level_group(g, L);
        if (threadIdx.x < 12) g[threadIdx.x] = 0;
        __threadfence();
        __syncthreads();
        block_degree<WIDE_BLOCK>(dsum, dmax, c + 1);
        if (threadIdx.x == 0) {
            c[0] = (unsigned long long)nn;
            c[3] = (unsigned long long)s_long;
            g[CNT_DEPTH] = (unsigned long long)L;
        }
    }
    if (threadIdx.x == 0) g[CNT_LEVEL + ((k + 1) & 1)] = (unsigned long long)L;
}

}  // namespace
}  // namespace drsf

using namespace drsf;

namespace {

// Scratch of one static rebuild: breadth-first levels, two frontiers, the
// sampled component and the level counters, each 256-byte aligned in one
// block.
struct StaticScratch {
    int32_t *level, *front0, *front1, *giant;
    unsigned long long *cnt;
};
size_t aligned(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
size_t scratch_bytes(int32_t n) {
    return 3 * aligned(sizeof(int32_t) * (size_t)n) + aligned(sizeof(int32_t)) +
           aligned(CNT_WORDS * sizeof(unsigned long long));
}
StaticScratch carve(void *p, int32_t n) {
    unsigned char *b = static_cast<unsigned char *>(p);
    const size_t v = aligned(sizeof(int32_t) * (size_t)n);
    return StaticScratch{(int32_t *)b, (int32_t *)(b + v), (int32_t *)(b + 2 * v), (int32_t *)(b + 3 * v),
                         (unsigned long long *)(b + 3 * v + aligned(sizeof(int32_t)))};
}

// The rebuild on given scratch; h: host memory for CNT_WORDS counters
// (pinned or not: every read of it follows a stream synchronisation).
int static_forest_core(int32_t n, const int64_t *row_ptr, const int32_t *col, int64_t nnz, int32_t *parent_out,
                       int32_t *label_out, hipStream_t s, int32_t *levels_out, const StaticScratch &w,
                       unsigned long long *h) {
    int32_t *level = w.level;
    unsigned long long *cnt = w.cnt;
    int rc = DRSF_OK;
    auto ok = [&](hipError_t e) {
        if (e != hipSuccess && rc == DRSF_OK) rc = DRSF_E_DEVICE;
        return e == hipSuccess;
    };
    int32_t *comp = label_out;
    const int gv = grid_for(n, BLOCK);
    hipLaunchKernelGGL(k_st_comp_init, dim3(gv), dim3(BLOCK), 0, s, n, row_ptr, col, comp, cnt);
    if (nnz > 0) {
        hipLaunchKernelGGL(k_st_compress, dim3(gv), dim3(BLOCK), 0, s, n, comp);
        hipLaunchKernelGGL(k_st_link_first, dim3(gv), dim3(BLOCK), 0, s, n, row_ptr, col, comp);
        hipLaunchKernelGGL(k_st_compress, dim3(gv), dim3(BLOCK), 0, s, n, comp);
        hipLaunchKernelGGL(k_st_sample, dim3(1), dim3(BLOCK), 0, s, n, comp, w.giant);
        hipLaunchKernelGGL(k_st_link_rest, dim3(gv), dim3(BLOCK), 0, s, n, row_ptr, col, comp, w.giant);
        hipLaunchKernelGGL(k_st_compress, dim3(gv), dim3(BLOCK), 0, s, n, comp);
    }
    // breadth-first forest from the roots, a level at a time.  A launch takes
    // its level and frontier from the device, so launches are queued ahead of
    // the host's reads of the counters: first a run of small levels and
    // FIRST_LEVELS levels that pick their direction on the device (a power-law
    // graph is nearly done then).  After a read, small frontiers run on in one
    // workgroup, with levels over the chip behind for what it grows to.  While
    // the frontier's rows' sum is far below the switch point, up to BATCH_MAX
    // top-down levels are queued at once (the batch length doubles while this
    // keeps holding), so a deep graph pays one host read per batch instead of
    // per level; a batch that outgrows its estimate stays correct, only slower.
    constexpr int BATCH_MAX = 64, FIRST_LEVELS = 4, WIDE_CAP = GRID_CAP * BLOCK / WIDE_BLOCK;
    const int gl = grid_for(n, WIDE_BLOCK, WIDE_CAP);
    hipLaunchKernelGGL(k_st_bfs_init, dim3(gl), dim3(WIDE_BLOCK), 0, s, n, row_ptr, comp, level, parent_out,
                       w.front0, cnt);
    int launches = 0, batch = 1;
    auto solo = [&]() {
        hipLaunchKernelGGL(k_st_solo, dim3(1), dim3(WIDE_BLOCK), 0, s, n, row_ptr, col, level, parent_out,
                           launches++, w.front0, w.front1, cnt);
    };
    auto wide = [&]() {
        hipLaunchKernelGGL((k_st_level<WIDE_BLOCK>), dim3(gl), dim3(WIDE_BLOCK), 0, s, n, nnz, row_ptr, col, level,
                           parent_out, launches++, w.front0, w.front1, cnt, 1);
    };
    if (nnz > 0) {
        solo();
        for (int i = 0; i < FIRST_LEVELS; i++) wide();
    }
    while (rc == DRSF_OK) {
        if (!ok(hipMemcpyAsync(h, cnt, CNT_WORDS * sizeof(unsigned long long), hipMemcpyDeviceToHost, s)) ||
            !ok(hipStreamSynchronize(s)))
            break;
        const int64_t L = (int64_t)h[CNT_LEVEL + (launches & 1)];
        const unsigned long long *hg = h + 4 * (L % 3);
        const int64_t nf = (int64_t)(hg[0] + hg[3]);
        if (nf == 0) break;
        if (L > n) {  // more levels than vertices: the counters are wrong
            rc = DRSF_E_DEVICE;
            break;
        }
        if (nf <= SOLO_FRONTIER && hg[2] <= SOLO_ROW) {
            batch = 1;
            solo();
            wide();
        } else if (few_edges(hg[1], nnz)) {
            // room for twice the frontier in a batch; a long row takes the
            // whole grid
            const int k = hg[1] * 256 < (uint64_t)nnz ? batch : 1;
            const int64_t want = std::max<int64_t>(std::max<int64_t>(2 * nf, 64) * 4, hg[3] ? (int64_t)hg[2] : 0);
            const int g = grid_for(want, BLOCK);
            if (g > WIDE_CAP) {  // its workgroups' atomics would be most of its time
                batch = 1;
                wide();
                continue;
            }
            for (int i = 0; i < k; i++)
                hipLaunchKernelGGL((k_st_level<BLOCK>), dim3(g), dim3(BLOCK), 0, s, n, nnz, row_ptr, col, level,
                                   parent_out, launches++, w.front0, w.front1, cnt, 0);
            batch = k == batch ? std::min(2 * batch, BATCH_MAX) : 1;
        } else {
            batch = 1;
            wide();
        }
    }
    // a graph without edges has one level, its roots
    if (levels_out) *levels_out = rc == DRSF_OK ? std::max<int32_t>(1, (int32_t)h[CNT_DEPTH]) : 0;
    if (rc == DRSF_OK && !ok(hipStreamSynchronize(s))) rc = DRSF_E_DEVICE;
    return rc;
}

// Reads row_ptr[n] (the CSR's entry count) on the stream, through a word of h.
int read_nnz(int32_t n, const int64_t *row_ptr, hipStream_t s, unsigned long long *h, int64_t *nnz) {
    if (hipMemcpyAsync(h, row_ptr + n, sizeof *nnz, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        (void)hipGetLastError();
        return DRSF_E_DEVICE;
    }
    *nnz = (int64_t)h[0];
    return DRSF_OK;
}

// Pinned words for the level counters of calls in flight: a few slots kept
// until the process ends, one taken by each call and given back; a call that
// finds none free allocates its own.  A copy to pinned words and the wait for
// it take 12 us, to pageable ones 21, allocating pinned words on each call 27.
constexpr int PIN_SLOTS = 8;
std::mutex g_pin_mu;
unsigned long long *g_pin[PIN_SLOTS] = {};
bool g_pin_used[PIN_SLOTS] = {};
struct PinnedWords {
    unsigned long long *p = nullptr;
    int slot = -1;
    PinnedWords() {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        for (int k = 0; k < PIN_SLOTS && slot < 0; k++)
            if (!g_pin_used[k]) slot = k;
        unsigned long long *q = slot >= 0 ? g_pin[slot] : nullptr;
        if (!q && hipHostMalloc((void **)&q, CNT_WORDS * sizeof(unsigned long long), hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            slot = -1;
            return;
        }
        p = q;
        if (slot >= 0) {
            g_pin[slot] = q;
            g_pin_used[slot] = true;
        }
    }
    ~PinnedWords() {
        if (slot >= 0) {
            std::lock_guard<std::mutex> lk(g_pin_mu);
            g_pin_used[slot] = false;
        } else if (p) {
            (void)hipHostFree(p);
        }
    }
};

// Scratch of the allocation-free entry point: one array per device, held
// until the process ends.  In host code its name only stands for the
// symbol; kernels get the device address that hipGetSymbolAddress returns
// for the device that is current.
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES] = {};

// Device address of this device's scratch array, looked up once per device.
int scratch_address(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        return DRSF_E_DEVICE;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return DRSF_E_DEVICE;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DRSF_OK;
}

}  // namespace

extern "C" int drsf_static_forest(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                  int32_t *parent_out, int32_t *label_out, void *stream,
                                  int32_t *levels_out) {
    if (n < 0 || (n > 0 && (!row_ptr || !parent_out || !label_out))) return DRSF_E_ARG;
    if (n == 0) {
        if (levels_out) *levels_out = 0;
        return DRSF_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    PinnedWords h;
    if (!h.p) return DRSF_E_NOMEM;
    int64_t nnz = 0;
    int rc = read_nnz(n, row_ptr, s, h.p, &nnz);
    if (rc) return rc;
    if (nnz < 0 || (nnz > 0 && !col)) return DRSF_E_ARG;
    void *p = nullptr;
    if (hipMalloc(&p, scratch_bytes(n)) != hipSuccess) {
        (void)hipGetLastError();
        return DRSF_E_NOMEM;
    }
    rc = static_forest_core(n, row_ptr, col, nnz, parent_out, label_out, s, levels_out, carve(p, n), h.p);
    (void)hipStreamSynchronize(s);
    (void)hipFree(p);
    return rc;
}

extern "C" int drsf_static_forest_noalloc(int32_t n, const int64_t *row_ptr, const int32_t *col,
                                          int32_t *parent_out, int32_t *label_out, void *stream,
                                          int32_t *levels_out) {
    if (n < 0 || (n > 0 && (!row_ptr || !parent_out || !label_out))) return DRSF_E_ARG;
    if (n == 0) {
        if (levels_out) *levels_out = 0;
        return DRSF_OK;
    }
    void *base = nullptr;
    int rc = scratch_address(&base);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    int64_t nnz = 0;
    unsigned long long h[CNT_WORDS] = {};  // pageable: each read follows a stream synchronisation
    if ((rc = read_nnz(n, row_ptr, s, h, &nnz))) return rc;
    if (nnz < 0 || (nnz > 0 && !col)) return DRSF_E_ARG;
    if (nnz > ((int64_t)1 << 32)) return DRSF_E_CAPACITY;
    // the documented bound, whatever part of the array is used
    size_t total = 3 * aligned(sizeof(int32_t) * (size_t)n) + aligned(sizeof(int32_t) * (size_t)(nnz + 1)) +
                   aligned(sizeof(uint32_t) * (size_t)std::max<int64_t>(nnz, 1)) +
                   aligned(scan_tmp_bytes(nnz) + 64) + aligned(sizeof(int32_t)) +
                   aligned(CNT_WORDS * sizeof(unsigned long long));
    if (total > NOALLOC_SCRATCH_BYTES) return DRSF_E_CAPACITY;
    rc = static_forest_core(n, row_ptr, col, nnz, parent_out, label_out, s, levels_out, carve(base, n), h);
    (void)hipStreamSynchronize(s);
    return rc;
}
