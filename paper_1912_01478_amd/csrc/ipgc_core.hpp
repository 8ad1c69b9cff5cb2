// The last rounds of a coloring on one workgroup, everything in its shared memory.
//
// Once at most kCore nodes are uncolored, k_rounds leaves its loop and the remaining rounds run
// here.  Of the graph they need only the edges between uncolored nodes (a bit matrix) and, per
// node, the colors that committed neighbours already hold (a window of 128 colors from the node's
// tentative color on; first-fit colors never decrease).  On hub-heavy graphs the uncolored nodes
// are nearly a clique by then and commit a few at a time, so there are hundreds of such rounds.
//
// What bounds them: nothing but the length of a round.  In k_rounds a round of this size takes 26
// to 36 us (two or three grid barriers of 4 us and chains of dependent loads, whatever the number of
// nodes); here it takes three workgroup barriers and reads of shared memory, 1 to 2 us.
#pragma once

#include "ipgc_device.hpp"

namespace ipgc {

constexpr int kCore = 1024;                // nodes: a thread each
constexpr int kCoreWords = kCore / 64;     // words of a matrix row
constexpr int kCoreStride = kCore + 1;     // words per column of the matrix: rows and columns both free of bank conflicts
constexpr int kCoreBuckets = 64;           // tentative colors modulo 64

// What the core needs of one uncolored node (global memory, by rank: ascending id).
struct CoreNode {
    uint64_t lo, hi;   // bit k: a committed neighbour holds color t + k (hi: t + 64 + k)
    int32_t v;
    int32_t t;         // the node's last tentative color: no smaller color is free
    int32_t deg;
    int32_t pad;
};

// Global memory between the kernels of the core.
struct CoreMem {
    uint64_t *adj;     // [kCore][kCoreWords]: bit j of row i set iff nodes i > j (by rank) are neighbours
    CoreNode *node;    // [kCore]
    int32_t *rank;     // per node id: its rank (valid for the uncolored nodes only)
};

struct CoreShared {
    uint64_t adj[kCoreWords * kCoreStride];        // word w of row i at [w * kCoreStride + i]; symmetric
    uint64_t bucket[kCoreWords * kCoreBuckets];    // [w][h]: uncolored nodes of word w with tentative color h modulo 64
    uint64_t won[kCoreWords];                      // nodes that commit in this round
    int32_t t[kCore];
    uint16_t win[kCore];                           // the same as a list
    int nwin;
    unsigned long long wdeg;                       // degree sum of the nodes that commit
};
static_assert(sizeof(CoreShared) <= 160 * 1024, "one workgroup's shared memory");

// A thread's node: its state, and the colors its committed neighbours hold from base + 1 on.
struct CoreState {
    uint64_t lo = 0, hi = 0;   // bit k: color base + 1 + k
    int32_t v = -1, base = 0, t = 0, deg = 0;
};

// Committed neighbour with color x: into the window, or (a color past it) into the node's byte map,
// which this thread alone uses now.  Maps hold colors up to d + 1; a larger one never matters.
template <class D>
__device__ __forceinline__ void core_forbid(const D &d, CoreState &s, int32_t x) {
    const int32_t k = x - 1 - s.base;
    if (k < 0) return;
    if (k < 64) s.lo |= 1ull << k;
    else if (k < 128) s.hi |= 1ull << (k - 64);
    else {
        const MapRef fm = map_of(d, s.v, d.fshift(s.v));
        if ((uint32_t)x <= fm.size) d.F[fm.pos + x - 1] = 1;
    }
}

// The smallest color not forbidden.  A full window moves on by 128 colors (all above 64, so the byte
// map holds what is known of them).
template <class D>
__device__ __forceinline__ int32_t core_first_free(const D &d, CoreState &s) {
    while ((s.lo & s.hi) == ~0ull) {
        s.base += 128;
        s.lo = s.hi = 0;
        const MapRef fm = map_of(d, s.v, d.fshift(s.v));
        for (int k = 0; k < 128 && (uint32_t)(s.base + k) < fm.size; ++k) {
            if (!d.F[fm.pos + s.base + k]) continue;
            if (k < 64) s.lo |= 1ull << k;
            else s.hi |= 1ull << (k - 64);
        }
    }
    return s.base + (s.lo != ~0ull ? __ffsll((unsigned long long)~s.lo) : 64 + __ffsll((unsigned long long)~s.hi));
}

// Rounds r, r + 1, ... until every node of the core is colored, by the whole workgroup (kCore threads;
// thread i holds the node of rank i, s.v < 0 for none).  commit(s, round) stores a node's color;
// record(round, nodes, degree sum) is called by thread 0 at the start of every round with the uncolored
// nodes.  Returns the number of the last round; *sum_nodes: the uncolored nodes summed over the rounds.
//
// A node loses iff a smaller uncolored neighbour has the same tentative color.  Candidates are the
// neighbours whose color agrees modulo 64, found word by word from the bucket sets; each is compared
// exactly.  Losers then learn the colors committed by their neighbours: from the list of winners if
// it is short, else from their matrix row against the winners' set.
template <class D, class Commit, class Record>
__device__ __forceinline__ int32_t core_rounds(const D &d, CoreShared &sh, CoreState s, int32_t r, int nact, int64_t degsum,
                                               int64_t *sum_nodes, Commit &&commit, Record &&record) {
    const int i = threadIdx.x, w = i / kWave, lane = lane_id(), h0 = i;
    bool act = s.v >= 0;
    if (act) s.t = core_first_free(d, s);
    *sum_nodes = 0;
    for (; nact > 0; ++r) {
        if (i == 0) record(r, nact, degsum);
        *sum_nodes += nact;
        sh.bucket[h0] = 0;  // kCoreWords * kCoreBuckets words, one per thread
        if (act) sh.t[i] = s.t;
        __syncthreads();
        if (i == 0) {
            sh.nwin = 0;
            sh.wdeg = 0;
        }
        const int h = s.t & (kCoreBuckets - 1);
        const uint64_t am = __ballot(act);
        if (am) {  // the leading lane's color goes in at once (late in the run nearly all agree)
            const int lead = __ffsll((unsigned long long)am) - 1;
            const int hl = __shfl(h, lead);
            const uint64_t same = __ballot(act && h == hl);
            unsigned long long *col = (unsigned long long *)&sh.bucket[w * kCoreBuckets];
            if (lane == lead) atomicOr(&col[hl], (unsigned long long)same);
            if (act && h != hl) atomicOr(&col[h], 1ull << lane);
        }
        __syncthreads();
        bool lose = false;
        if (act) {
            for (int w0 = 0; w0 <= w && !lose; w0 += 4) {
                uint64_t x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {  // the four words' loads are in flight together
                    const int ww = w0 + q;
                    x[q] = ww <= w ? sh.adj[ww * kCoreStride + i] & sh.bucket[ww * kCoreBuckets + h] : 0;
                    if (ww == w) x[q] &= lanes_below();
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    while (x[q] && !lose) {
                        lose = sh.t[(w0 + q) * 64 + __ffsll((unsigned long long)x[q]) - 1] == s.t;
                        x[q] &= x[q] - 1;
                    }
                }
            }
        }
        const bool win = act && !lose;
        const uint64_t wm = __ballot(win);
        if (lane == 0) sh.won[w] = wm;
        if (wm) {
            int at = 0;
            const int64_t wd = wave_sum(win ? s.deg : 0);
            if (lane == 0) {
                at = atomicAdd(&sh.nwin, (int)__popcll(wm));
                atomicAdd(&sh.wdeg, (unsigned long long)wd);
            }
            at = __shfl(at, 0);
            if (win) {
                sh.win[at + __popcll(wm & lanes_below())] = (uint16_t)i;
                commit(s, r);
            }
        }
        __syncthreads();
        const int nwin = sh.nwin;
        degsum -= (int64_t)sh.wdeg;
        if (act && lose) {
            if (nwin <= kCoreWords) {
                for (int k = 0; k < nwin; ++k) {
                    const int j = sh.win[k];
                    if (sh.adj[(j >> 6) * kCoreStride + i] >> (j & 63) & 1) core_forbid(d, s, sh.t[j]);
                }
            } else {
                for (int ww = 0; ww < kCoreWords; ++ww) {
                    uint64_t x = sh.adj[ww * kCoreStride + i] & sh.won[ww];
                    while (x) {
                        core_forbid(d, s, sh.t[ww * 64 + __ffsll((unsigned long long)x) - 1]);
                        x &= x - 1;
                    }
                }
            }
            s.t = core_first_free(d, s);
        }
        act = act && lose;
        nact -= nwin;
        // the next round's first barrier comes before nwin, wdeg, won and win are written again, and
        // only losers write t before it
    }
    return r - 1;
}

// ------------------------------------------------------------------ the last rounds of a large graph

constexpr int kCoreRankGroups = 16;

// Ranks of the uncolored nodes by id: the worklist that k_rounds left for round ct->tail_round, at most
// kCore nodes.  Every workgroup reads the whole list and ranks its share, a wavefront per node.
template <class D>
__global__ __launch_bounds__(kCore) void k_core_rank(D d, CoreMem cm) {
    __shared__ int32_t pre[kNumClasses][kMaxRoundBlocks + 1];
    __shared__ int32_t id[kCore];
    const int32_t r = d.ct->tail_round;
    if (r == 0) return;
    const int nb = d.grid, src = r & 1;
    int x[kNumClasses], ex[kNumClasses], tot[kNumClasses];
    for (int k = 0; k < kNumClasses; ++k)
        x[k] = threadIdx.x < (unsigned)d.ct->tail_writers ? d.seg_cnt[src][k * nb + threadIdx.x] : 0;
    block_scan3(x, ex, tot);
    for (int k = 0; k < kNumClasses; ++k) {
        if (threadIdx.x < (unsigned)nb) pre[k][threadIdx.x] = ex[k];
        if (threadIdx.x == 0) pre[k][nb] = tot[k];
    }
    id[threadIdx.x] = INT32_MAX;
    __syncthreads();
    const int total = tot[0] + tot[1] + tot[2];
    int k = 0, i = threadIdx.x;
    if (i < total) {
        while (i >= tot[k]) i -= tot[k++];
        int lo = 0, hi = nb;  // segment lo with pre[lo] <= i < pre[lo + 1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[k][mid] <= i) lo = mid;
            else hi = mid;
        }
        id[threadIdx.x] = d.seg_list[src][d.ct->seg_off[k] + (int64_t)lo * d.ct->seg_cap[k] + (i - pre[k][lo])];
    }
    __syncthreads();
    const int lane = lane_id();
    for (int q = blockIdx.x * (kCore / kWave) + threadIdx.x / kWave; q < total; q += gridDim.x * (kCore / kWave)) {
        const int32_t v = id[q];
        int below = 0;
#pragma unroll
        for (int j = 0; j < kCore / kWave; ++j) below += id[j * kWave + lane] < v;
        below = (int)wave_sum(below);
        if (lane == 0) {
            cm.node[below].v = v;
            cm.rank[v] = below;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) d.ct->tail_nodes = total;
}

// Matrix row and color window of every node of the core, a workgroup each: the uncolored nodes among the
// node's smaller neighbours (class L: its row; W and M: its ring, which holds every smaller neighbour
// not yet seen committed), and which of the 128 colors from its last tentative color on are taken
// (color mask and byte map; class L when it pulls: its neighbours' colors).
template <class D>
__global__ __launch_bounds__(kCore) void k_core_build(D d, CoreMem cm) {
    __shared__ uint64_t row[kCoreWords];
    __shared__ uint64_t win[2];
    const int i = blockIdx.x;
    if (d.ct->tail_round == 0 || i >= d.ct->tail_nodes) return;
    if (threadIdx.x < kCoreWords) row[threadIdx.x] = 0;
    if (threadIdx.x < 2) win[threadIdx.x] = 0;
    __syncthreads();
    const int32_t v = cm.node[i].v;
    const int64_t b = d.rowptr[v], deg = d.rowptr[v + 1] - b;
    const int32_t t = max(1, -d.c[v]);
    const bool light = d.cls[v] == kL;
    const int32_t start = light ? 0 : d.lstart[v], len = light ? (int32_t)deg : d.llen[v];
    const int32_t gb = light ? d.base(v) : 0;  // rows hold ids local to the graph, rings global ones
    const bool pull = light && d.light_pull != kPushAll;
    const int32_t *list = light ? d.colidx : d.lower;
    constexpr int P = 4;
    for (int32_t k0 = 0; k0 < len; k0 += P * kCore) {
        int32_t u[P], cu[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int64_t k = (int64_t)k0 + j * kCore + threadIdx.x;
            int64_t p = start + k;
            if (p >= deg) p -= deg;
            u[j] = k < len ? list[b + p] + gb : -1;
        }
#pragma unroll
        for (int j = 0; j < P; ++j) cu[j] = u[j] >= 0 ? d.c[u[j]] : 1;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (u[j] < 0) continue;
            if (cu[j] <= 0) {
                if (u[j] >= v) continue;
                const int q = cm.rank[u[j]];
                atomicOr((unsigned long long *)&row[q >> 6], 1ull << (q & 63));
            } else if (pull && cu[j] >= t && cu[j] < t + 128) {
                atomicOr((unsigned long long *)&win[(cu[j] - t) >> 6], 1ull << ((cu[j] - t) & 63));
            }
        }
    }
    if (!pull && threadIdx.x < 128) {
        const int32_t x = t + (int32_t)threadIdx.x;
        bool taken = false;
        if (x <= kMaskColors) {
            taken = d.mask[v] >> (x - 1) & 1;
        } else {
            const MapRef fm = map_of(d, v, d.fshift(v));
            taken = (uint32_t)x <= fm.size && !light && d.F[fm.pos + x - 1];
        }
        const uint64_t tm = __ballot(taken);
        if (lane_id() == 0) win[threadIdx.x / kWave] = tm;
    }
    __syncthreads();
    if (threadIdx.x < kCoreWords) cm.adj[i * kCoreWords + threadIdx.x] = row[threadIdx.x];
    if (threadIdx.x == 0) {
        CoreNode nd;
        nd.lo = win[0];
        nd.hi = win[1];
        nd.v = v;
        nd.t = t;
        nd.deg = (int32_t)deg;
        nd.pad = 0;
        cm.node[i] = nd;
    }
}

// Upper half of the matrix from its lower half, 64 x 64 bits at a time: column b of the block whose rows
// a wavefront holds is one ballot.
__device__ __forceinline__ void core_mirror(CoreShared &sh, int words) {
    const int lane = lane_id();
    for (int blk = threadIdx.x / kWave; blk < words * words; blk += kCore / kWave) {
        const int wi = blk / words, wj = blk % words;  // rows 64 wi.., columns 64 wj..
        if (wj > wi) continue;
        const uint64_t x = sh.adj[wj * kCoreStride + wi * 64 + lane];
        uint64_t y = 0;
        for (int b = 0; b < 64; ++b) {
            const uint64_t col = __ballot(x >> b & 1);
            if (lane == b) y = col;
        }
        // row 64 wj + lane, word wi; a diagonal block keeps its lower half as well
        sh.adj[wi * kCoreStride + wj * 64 + lane] = wi == wj ? x | y : y;
    }
}

// The rounds themselves (one workgroup).
template <class D>
__global__ __launch_bounds__(kCore) void k_core_rounds(D d, CoreMem cm) {
    __shared__ CoreShared sh;
    const int32_t r0 = d.ct->tail_round;
    if (r0 == 0) return;
    const int i = threadIdx.x, n = d.ct->tail_nodes;
    const int words = (n + 63) / 64;
    CoreState s;
    if (i < n) {
        const CoreNode nd = cm.node[i];
        s.v = nd.v;
        s.lo = nd.lo;
        s.hi = nd.hi;
        s.base = nd.t - 1;
        s.deg = nd.deg;
    }
    for (int k = i; k < kCore * kCoreWords; k += kCore) {
        const int row = k / kCoreWords, w = k % kCoreWords;
        sh.adj[w * kCoreStride + row] = row < n ? cm.adj[k] : 0;
    }
    if (i == 0) sh.wdeg = 0;
    __syncthreads();
    const int64_t ds = wave_sum(s.deg);
    if (lane_id() == 0 && ds) atomicAdd(&sh.wdeg, (unsigned long long)ds);
    core_mirror(sh, words);
    __syncthreads();
    const int64_t degsum = (int64_t)sh.wdeg;
    __syncthreads();
    int64_t nodes = 0;
    const int32_t last = core_rounds(
        d, sh, s, r0, n, degsum, &nodes,
        [&](const CoreState &x, int32_t r) {
            d.c[x.v] = x.t;
            if (d.grounds) atomicMax(&d.grounds[d.gidx[x.v]], r);
        },
        [&](int32_t r, int32_t active, int64_t deg) {
            if (r - 1 < d.trace_cap) {
                d.trace[r - 1] = active;
                d.trace_deg[r - 1] = deg;
            }
            for (int q = 0; q < 3; ++q) tick(d, 3 * (int64_t)(r - 1) + q);
        });
    tick(d, 3 * (int64_t)last);
    if (i == 0) {
        d.ct->finished = 1;
        d.ct->rounds = last;
        d.units[kUAssignNodes * d.grid] += nodes;
        d.units[kUConflictNodes * d.grid] += nodes;
        d.units[kUCommits * d.grid] += n;
    }
}

}  // namespace ipgc
