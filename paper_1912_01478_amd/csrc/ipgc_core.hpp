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
// nodes); here it takes three workgroup barriers and reads of shared memory, 4 to 5 us (R-MAT of 65 536 nodes, 88 rounds).
#pragma once

#include "ipgc_device.hpp"

namespace ipgc {

constexpr int kCore = 1024;                // nodes: a thread each
constexpr int kCoreWords = kCore / 64;     // words of a matrix row
constexpr int kCoreStride = kCore + 1;     // words per column of the matrix: rows and columns both free of bank conflicts
constexpr int kCoreBuckets = 128;          // tentative colors modulo 128

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
    uint64_t *adj;     // [kCore][kCoreWords]: bit j of row i set iff node i's list names node j (by rank), j < i
                       // unless every node reads its own row (core_own_rows)
    CoreNode *node;    // [kCore]
    int32_t *rank;     // per node id: its rank (valid for the uncolored nodes only)
};

struct CoreShared {
    uint64_t adj[kCoreWords * kCoreStride];        // word w of row i at [w * kCoreStride + i]: the nodes that node i
                                                   // may lose to or learn colors from
    uint64_t bucket[kCoreWords * kCoreBuckets];    // [w][h]: uncolored nodes of word w with tentative color h modulo 128
    uint64_t won[kCoreWords];                      // nodes that commit in this round
    uint64_t done[kCoreWords];                     // nodes committed in earlier rounds (their colors stay in t)
    int32_t t[kCore];
    int cnt[kCoreWords];
    int nwin;
    unsigned long long wdeg;                       // degree sum of the nodes that commit
};
static_assert(sizeof(CoreShared) <= 160 * 1024, "one workgroup's shared memory");

// A thread's node: its state, and which colors from base + 1 on its committed neighbours hold.
struct CoreState {
    uint64_t lo = 0, hi = 0;   // bit k: color base + 1 + k (hi: base + 65 + k)
    int32_t v = -1, base = 0, t = 0, deg = 0;
    int32_t rank = 0;
};

// A neighbour has committed color x.  Colors past the window are found again when it moves on.
__device__ __forceinline__ void core_forbid(CoreState &s, int32_t x) {
    const uint32_t k = (uint32_t)(x - 1 - s.base);
    const uint64_t bit = 1ull << (k & 63);
    if (k < 64) s.lo |= bit;
    else if (k < 128) s.hi |= bit;
}

// What a node's byte map says of the 64 colors from x on, all above 64 (bit k: color x + k): the state that
// the rounds before the core left.
template <class D>
struct CoreMaps {
    const D &d;
    __device__ __forceinline__ uint64_t taken(const CoreState &s, int32_t x) const {
        const MapRef fm = map_of(d, s.v, d.fshift(s.v));
        uint64_t m = 0;
        for (int k = 0; k < 64 && (uint32_t)(x - 1 + k) < fm.size; ++k) m |= (uint64_t)(d.F[fm.pos + x - 1 + k] & 1) << k;
        return m;
    }
};

// Workgroup barrier for shared memory alone: stores to global memory stay in flight (nothing in the core
// reads them back), where __syncthreads would wait a microsecond for each round's colors to be written.
__device__ __forceinline__ void core_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The smallest color not forbidden, after round r.  A full first word moves the window on by 64 colors.  No
// color above r has been committed yet, so the word that comes in is empty unless the node is more than
// 64 colors behind the rounds; then it holds the colors taken before the core (by round r0 - 1) and
// those of the node's neighbours that the core has committed.
template <class Far>
__device__ __forceinline__ int32_t core_first_free(const Far &far, const CoreShared &sh, CoreState &s, int32_t r0, int32_t r) {
    while (s.lo == ~0ull) {
        s.base += 64;
        s.lo = s.hi;
        s.hi = 0;
        if (s.base + 64 >= r) continue;
        if (s.base + 64 < r0) s.hi = far.taken(s, s.base + 65);
        for (int w = 0; w < kCoreWords; ++w) {
            uint64_t x = sh.adj[w * kCoreStride + s.rank] & (sh.done[w] | sh.won[w]);
            for (; x; x &= x - 1) core_forbid(s, sh.t[w * 64 + __ffsll((unsigned long long)x) - 1]);
        }
    }
    return s.base + __ffsll((unsigned long long)~s.lo);
}

// The nodes still uncolored move to the first threads (nact of them, at most half of `span`), in rank order,
// so that the other wavefronts have nothing left to do.  Called by the whole workgroup.
__device__ __forceinline__ void core_compact(CoreShared &sh, CoreState &s, bool act, int nact) {
    const int i = threadIdx.x, w = i / kWave, lane = lane_id();
    const uint64_t am = __ballot(act);
    if (lane == 0) sh.cnt[w] = __popcll(am);
    core_sync();
    int at = __popcll(am & lanes_below());
    for (int q = 0; q < kCoreWords; ++q) at += q < w ? sh.cnt[q] : 0;
    uint64_t *stage = sh.bucket;  // all zero between rounds, at most kCore / 2 nodes
    static_assert(kCoreWords * kCoreBuckets >= kCore / 2, "staging area");
    const uint64_t in[5] = {s.lo, s.hi, (uint64_t)(uint32_t)s.v << 32 | (uint32_t)s.deg,
                            (uint64_t)(uint32_t)s.t << 32 | (uint32_t)s.base, (uint64_t)(uint32_t)s.rank};
    uint64_t out[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        if (act) stage[at] = in[f];
        core_sync();
        out[f] = i < nact ? stage[i] : 0;
        core_sync();
    }
    if (i < kCore / 2) stage[i] = 0;
    core_sync();
    s.lo = out[0];
    s.hi = out[1];
    s.v = i < nact ? (int32_t)(out[2] >> 32) : -1;
    s.deg = (int32_t)out[2];
    s.t = (int32_t)(out[3] >> 32);
    s.base = (int32_t)out[3];
    s.rank = (int32_t)out[4];
}

// Rounds r0, r0 + 1, ... until every node of the core is colored, by the whole workgroup (kCore threads;
// thread i holds the node of rank i, s.v < 0 for none).  commit(s, round) stores a node's color;
// record(round, nodes, degree sum) is called by thread 0 at the start of every round with the uncolored
// nodes (their degrees are summed only if `degrees`).  Returns the number of the last round; *sum_nodes: the uncolored nodes summed over the rounds.
//
// A node loses iff a smaller uncolored neighbour has the same tentative color.  Candidates are the
// neighbours whose color agrees modulo 128, found word by word from the bucket sets, and compared exactly.
// Losers then learn the colors committed by their neighbours, from their matrix row against the winners' set;
// the winners and their colors are the same for the whole wavefront, so they come from scalar registers.
template <class Far, class Commit, class Record>
__device__ __forceinline__ int32_t core_rounds(const Far &far, CoreShared &sh, CoreState s, int32_t r0, int nact,
                                               bool degrees, int64_t degsum, int64_t *sum_nodes, Commit &&commit, Record &&record) {
    const int i = threadIdx.x, w = i / kWave, lane = lane_id();
    bool act = s.v >= 0;
    int span = kCore;  // threads that may hold a node
    int32_t r = r0;
    s.rank = i;
    if (i < kCoreWords) sh.done[i] = sh.won[i] = 0;
    for (int k = i; k < kCoreWords * kCoreBuckets; k += kCore) sh.bucket[k] = 0;
    core_sync();
    if (act) s.t = core_first_free(far, sh, s, r0, r - 1);
    *sum_nodes = 0;
    for (; nact > 0; ++r) {
        if (i == 0) record(r, nact, degsum);
        *sum_nodes += nact;
        if (span > kWave && nact <= span / 2) {  // the same for the whole workgroup
            core_compact(sh, s, act, nact);
            act = s.v >= 0;
            while (span > kWave && nact <= span / 2) span /= 2;
        }
        const int rw = s.rank / 64, h = s.t & (kCoreBuckets - 1);
        const uint64_t rbit = 1ull << (s.rank & 63);
        unsigned long long *const mine = (unsigned long long *)&sh.bucket[rw * kCoreBuckets + h];
        if (act) sh.t[s.rank] = s.t;
        const uint64_t am = __ballot(act);
        if (am) {
            if (span == kCore) {  // a wavefront's nodes share a word: most of them go in at once
                const int lead = __ffsll((unsigned long long)am) - 1;
                const int hl = __builtin_amdgcn_readlane(h, lead);
                const uint64_t same = __ballot(act && h == hl);
                if (lane == lead) atomicOr(mine, (unsigned long long)same);
                if (act && h != hl) atomicOr(mine, (unsigned long long)rbit);
            } else if (act) {
                atomicOr(mine, (unsigned long long)rbit);
            }
        }
        core_sync();  // everyone has left the previous round
        if (i < kCoreWords) {
            sh.done[i] |= sh.won[i];
            sh.won[i] = 0;
        }
        if (i == 0) {
            sh.nwin = 0;
            sh.wdeg = 0;
        }
        bool lose = false;
        // all colors are at most r, so up to round 128 the buckets are exact
        if (act) {
            for (int w0 = 0; w0 <= rw && !lose; w0 += 4) {
                uint64_t x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {  // the four words' loads are in flight together
                    const int ww = w0 + q;  // past rw: smaller ranks only, so masked out below
                    x[q] = sh.adj[ww * kCoreStride + s.rank] & sh.bucket[ww * kCoreBuckets + h];
                    if (ww == rw) x[q] &= rbit - 1;
                    if (ww > rw) x[q] = 0;
                }
                if (r <= kCoreBuckets) {
                    lose = (x[0] | x[1] | x[2] | x[3]) != 0;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        for (; x[q] && !lose; x[q] &= x[q] - 1)
                            lose = sh.t[(w0 + q) * 64 + __ffsll((unsigned long long)x[q]) - 1] == s.t;
                }
            }
        }
        core_sync();
        const bool win = act && !lose;
        const uint64_t wm = __ballot(win);
        if (act) *mine = 0;
        if (wm) {
            if (lane == 0) atomicAdd(&sh.nwin, (int)__popcll(wm));
            if (span == kCore && lane == 0) sh.won[w] = wm;  // the wavefront's own word
            if (win) {
                if (span != kCore) atomicOr((unsigned long long *)&sh.won[rw], (unsigned long long)rbit);
                if (degrees) atomicAdd(&sh.wdeg, (unsigned long long)s.deg);
                commit(s, r);
            }
        }
        core_sync();
        nact -= sh.nwin;
        degsum -= (int64_t)sh.wdeg;
        act = act && lose;
        if (__ballot(act)) {
            const uint64_t wv = sh.won[lane & (kCoreWords - 1)];
            uint32_t nz = (uint32_t)__ballot(wv != 0) & ((1u << kCoreWords) - 1);  // words with winners
            while (nz) {  // two words at a time, their loads in flight together
                int at[2], tq[2];
                uint64_t m[2], a[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    at[q] = nz ? __ffs(nz) - 1 : 0;
                    m[q] = nz ? (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(wv >> 32), at[q]) << 32 |
                                    (uint32_t)__builtin_amdgcn_readlane((int)wv, at[q])
                              : 0;
                    nz &= nz - 1;
                    a[q] = act ? sh.adj[at[q] * kCoreStride + s.rank] & m[q] : 0;
                    tq[q] = sh.t[at[q] * 64 + lane];
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (!__ballot(a[q] != 0)) continue;
                    if (__popcll(m[q]) <= 8) {
                        for (uint64_t y = m[q]; y; y &= y - 1) {
                            const int b = __ffsll((unsigned long long)y) - 1;
                            if (a[q] >> b & 1) core_forbid(s, __builtin_amdgcn_readlane(tq[q], b));
                        }
                    } else {  // many winners: each lane takes its own neighbours among them
                        for (uint64_t y = a[q]; y; y &= y - 1)
                            core_forbid(s, sh.t[at[q] * 64 + __ffsll((unsigned long long)y) - 1]);
                    }
                }
            }
            if (act) s.t = core_first_free(far, sh, s, r0, r);
        }
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

// Graphs of class L alone: in every round a node reads its own row, so the matrix holds the rows as they are, and entries
// that are not named back count as in the definition.  The other lists (rings) hold smaller neighbours only, and the
// matrix is completed from its lower half.
template <class D>
__device__ __forceinline__ bool core_own_rows(const D &d) {
    return d.light_pull == kPullOnly;
}

// Matrix row and color window of every node of the core, a workgroup each: the uncolored nodes among the
// node's smaller neighbours (core_own_rows: all neighbours; class L: its row; W and M: its ring, which holds every smaller neighbour
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
    const int32_t t = max(1, -state_of(d, v));
    const bool light = deg <= d.light_max;
    const int32_t start = light ? 0 : d.lstart[v], len = light ? (int32_t)deg : d.llen[v];
    const int32_t gb = light ? d.base(v) : 0;  // rows hold ids local to the graph, rings global ones
    const bool pull = light && d.light_pull != kPushAll, own = core_own_rows(d);
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
        for (int j = 0; j < P; ++j) cu[j] = u[j] >= 0 ? d.tag[u[j]] : 0;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (u[j] < 0) continue;
            if (!(cu[j] & kDone)) {
                if (own ? u[j] == v : u[j] >= v) continue;
                const int q = cm.rank[u[j]];
                atomicOr((unsigned long long *)&row[q >> 6], 1ull << (q & 63));
            } else if (pull) {  // a node of class L needs no color above 33
                const int32_t x = (cu[j] & kTagMax) - t;
                if (x >= 0 && x < 64) atomicOr((unsigned long long *)&win[0], 1ull << x);
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

// The transpose of a 64 x 64 bit block (lane l holds row l), by exchanging half blocks of 32, 16, ... 1.
__device__ __forceinline__ uint64_t core_transpose(uint64_t x) {
    const int lane = lane_id();
    uint64_t mask = 0x00000000FFFFFFFFull;  // the columns of the lower half of each block of 2 j
#pragma unroll
    for (int j = 32; j > 0; j >>= 1) {
        const uint64_t y = (uint64_t)__shfl_xor((unsigned long long)x, j);
        x = lane & j ? (x & ~mask) | (y >> j & mask) : (x & mask) | (y << j & ~mask);
        mask ^= mask << (j >> 1);
    }
    return x;
}

// Upper half of the matrix from its lower half, 64 x 64 bits at a time.
__device__ __forceinline__ void core_mirror(CoreShared &sh, int words) {
    const int lane = lane_id();
    for (int blk = threadIdx.x / kWave; blk < words * words; blk += kCore / kWave) {
        const int wi = blk / words, wj = blk % words;  // rows 64 wi.., columns 64 wj..
        if (wj > wi) continue;
        const uint64_t x = sh.adj[wj * kCoreStride + wi * 64 + lane], y = core_transpose(x);
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
    uint64_t word[kCoreWords];
#pragma unroll
    for (int q = 0; q < kCoreWords; ++q) {  // all loads in flight
        const int k = q * kCore + i;
        word[q] = k / kCoreWords < n ? cm.adj[k] : 0;
    }
#pragma unroll
    for (int q = 0; q < kCoreWords; ++q) {
        const int k = q * kCore + i;
        sh.adj[k % kCoreWords * kCoreStride + k / kCoreWords] = word[q];
    }
    if (i == 0) sh.wdeg = 0;
    __syncthreads();
    const int64_t ds = wave_sum(s.deg);
    if (lane_id() == 0 && ds) atomicAdd(&sh.wdeg, (unsigned long long)ds);
    if (!core_own_rows(d)) core_mirror(sh, words);
    __syncthreads();
    const int64_t degsum = (int64_t)sh.wdeg;
    __syncthreads();
    int64_t nodes = 0;
    const int32_t last = core_rounds(
        CoreMaps<D>{d}, sh, s, r0, n, true, degsum, &nodes,
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
