// Small graphs: one workgroup colors a whole graph, its state in shared memory.
//
// The cooperative kernel spends 20 to 40 us on a round however small the graph is (grid barriers, chains of
// dependent loads from memory), and a call adds six launches and two host waits.  Here a graph of at most
// kSmallNodes nodes is checked and colored in one launch: while more than kCore nodes are uncolored, rounds
// walk a worklist with the colors, the forbidden-color masks and both lists in shared memory (only the
// rows come from memory, mostly the L2); then the uncolored nodes go on in the core (ipgc_core.hpp) or, in
// graphs without long rows, in the row rounds below.  Graphs of up to kCore (kRowsNodes) nodes start there.  A batch
// runs a workgroup per graph, largest first.
#pragma once

#include <cstddef>

#include "ipgc_core.hpp"

namespace ipgc {

// 14 bytes of shared memory a node: mask 8, color 2, two list entries 4.
constexpr int kSmallNodes = 10240;
// Rows up to this length take a thread each, longer ones 16 lanes or a wavefront.  A row stops at its first
// conflict or its first larger id, so a lane reads a few entries of most rows, and 64 rows overlap in a
// wavefront.  Whole calls at 32 / 64 / 128 / 256: uniform, 10^4 nodes of degree 32, 912 / 484 / 484 / 481 us;
// of degree 64, 2391 / 1736 / 1165 / 1158; R-MAT, 8192 nodes and 2.0e5 entries, 616 / 615 / 564 / 568; 4096
// nodes and 5.3e4 entries, 256 / 258 / 251 / 277.
constexpr int kSmallLight = 128;

// A node's state in the list rounds.  Conflict tests look at the nodes that were uncolored when the round began
// (tentative, or committed in this very round: kFresh): the smallest of them wins whatever its row says, so every
// round has a winner.  Nodes committed before (kPast) are in the masks of the nodes in their own rows; a row that
// names one of those without being named back (a one-way entry, which the default checks let through) must not
// lose to it round after round.
constexpr int kHeld = 0x3FFF;   // the color: at most 65 + kSmallNodes
constexpr int kFresh = 0x4000;
constexpr int kPast = 0x8000;

struct SmallLists {
    uint64_t mask[kSmallNodes];     // bit t - 1: a committed neighbour has color t (t <= 64); not with own rows
    uint16_t c[kSmallNodes];        // color, tentative or committed, and for committed nodes when (kFresh, kPast)
    uint16_t wl[2][kSmallNodes];    // worklists: short rows from the front, long rows from the back
};

// Sparse graphs (no row longer than kRowsDegree) leave the worklist for the row rounds instead of the core: the
// uncolored nodes' rows among themselves in shared memory, by rank.  A bit matrix of a sparse graph is mostly
// zeros: reading its rows took 8 us a round for 1000 nodes of degree 8, reading the lists takes 1 us.
constexpr int kRowsNodes = 4096;     // four a thread
constexpr int kRowsEntries = 40960;  // sum of the nodes' degrees
constexpr int kRowsDegree = 63;      // so that 64 color bits always have a free one

struct SmallRows {
    uint16_t adj[kRowsEntries];  // ranks of each node's uncolored neighbours, ascending if the rows are
    uint16_t c[kSmallNodes];     // the list rounds' colors stay in place until the rows are built
    int16_t s[kRowsNodes];       // > 0 committed in these rounds, -t tentative
    int left[2];                 // uncolored nodes after each round, by parity
};

static_assert(offsetof(SmallRows, c) == offsetof(SmallLists, c), "the colors stay in place");

struct SmallShared {
    union {
        SmallLists a;
        CoreShared core;
        SmallRows rows;
    };
    uint64_t bits[kSmallNodes / 64];  // uncolored nodes, when the core starts
    int32_t pre[kSmallNodes / 64];    // and the number of them before each word
    int nl[2], nw[2];                 // entries of each worklist, short and long rows
    int bad, descents, starts, maxdeg;
    unsigned long long deg;
};
static_assert(sizeof(SmallShared) <= 160 * 1024 - 1024, "one workgroup's shared memory");

struct SmallArgs {
    const int32_t *rowptr;     // one graph's CSR, or a packed batch's
    const int32_t *colidx;
    int32_t *out;
    int64_t n, m;              // one graph
    const int64_t *node_off;   // a batch: offsets of its graphs (null for one graph)
    const int64_t *edge_off;
    const int32_t *order;      // a batch: the graph of each workgroup
    int32_t *grounds;          // a batch: rounds per graph
    Counters *ct;              // verdicts; one graph: also finished, rounds and the CSR's ends
    int32_t *trace;            // one graph: per-round sizes and degree sums (null: not kept)
    int64_t *trace_deg;
    int64_t trace_cap;
    int32_t check;             // check the column ids
};

// The colors that the committed neighbours of a node hold among the 64 from x on (bit k: color x + k), from
// its row: for nodes whose mask says no more.
struct SmallRow {
    const int32_t *rp, *ci, *out;  // out: colors, 0 for nodes the core has not committed yet
    __device__ __forceinline__ uint64_t taken(const CoreState &s, int32_t x) const {
        uint64_t m = 0;
        for (int32_t k = rp[s.v]; k < rp[s.v + 1]; ++k) {
            const uint32_t q = (uint32_t)(out[ci[k]] - x);
            if (q < 64) m |= 1ull << q;
        }
        return m;
    }
};

// First free color above 64 of node v, whose mask is full.
__device__ __forceinline__ int32_t small_pull(const SmallShared &sh, const SmallArgs &, const int32_t *rp, const int32_t *ci, int v) {
    for (int32_t x = max(kMaskColors + 1, (int32_t)sh.a.c[v]);; x += 64) {
        uint64_t m = 0;
        for (int32_t k = rp[v]; k < rp[v + 1]; ++k) {
            const int c = sh.a.c[ci[k]];
            const uint32_t q = (uint32_t)((c & kHeld) - x);
            if ((c & (kFresh | kPast)) && q < 64) m |= 1ull << q;
        }
        if (m != ~0ull) return x + __ffsll((unsigned long long)~m) - 1;
    }
}

// Places for the flagged lanes of a wavefront after *count (shared): one atomic per wavefront.
__device__ __forceinline__ int wave_append(bool flag, int *count) {
    const uint64_t m = __ballot(flag);
    int at = 0;
    if (m) {
        if (lane_id() == 0) at = atomicAdd(count, (int)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
    }
    return at + __popcll(m & lanes_below());
}

// Graphs of class L alone (no row longer than this) learn the committed colors from the nodes' own rows, as the general
// path does and as the definition reads them: their colors are the definition's also where a row names a node that does
// not name it back, whose color no push brings.  Longer rows cost too much to read again in every round, and learn from
// the neighbours' pushes.  Whole calls with pushes for all / own rows here / own rows up to 63 entries: 10^4 nodes of
// degree 8 137 / 141 / 143 us, 1024 graphs of 10^3 to 10^4 nodes 1250 / 1264 / 1320.
constexpr int kOwnRows = 32;
static_assert(kCore * kOwnRows <= kRowsEntries, "they go on in the row rounds");

// Tentative colors of a round from the nodes' own rows, a lane per row.  Word: 32 bits while no committed color is above
// 32 (half the instructions of 64).
template <typename Word>
__device__ __forceinline__ void small_learn(SmallShared &sh, const int32_t *rp, const int32_t *ci, int32_t m, int p) {
    constexpr int C = 4;
    const int nl = sh.nl[p];
    for (int i = threadIdx.x; i < nl; i += kCore) {
        const int v = sh.a.wl[p][i];
        const Bounds<int32_t> row = row_of(rp, v);
        Word used = 0;  // bit x - 1: color x
        for (int k = row.b; k < row.e; k += C) {
            int u[C];
            load4(ci, k, m, 0, u);
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const uint32_t c = k + q < row.e ? sh.a.c[u[q]] : 0;
                used |= (Word)(c / kFresh & 1) << ((c - 1) % (8 * sizeof(Word)));
            }
        }
        sh.a.c[v] = (uint16_t)__ffsll((unsigned long long)~(uint64_t)used);
    }
}

// gone: degrees of the nodes this thread commits.
// One round's conflict tests, commits and pushes (Push) of the short rows, a lane each, two in flight per lane.
template <bool Push>
__device__ __forceinline__ void small_light(SmallShared &sh, const int32_t *rp, const int32_t *ci, int32_t m, int32_t *out,
                                            int p, bool sorted, int &gone) {
    constexpr int K = 2, C = 4;
    const int nl = sh.nl[p];
    const uint16_t *cur = sh.a.wl[p];
    uint16_t *nxt = sh.a.wl[p ^ 1];
    for (int i0 = 0; i0 < nl; i0 += K * kCore) {
        int v[K], t[K], b[K], e[K];
        uint32_t lose = 0, done = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = i0 + j * kCore + (int)threadIdx.x;
            v[j] = i < nl ? (int)cur[i] : -1;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            t[j] = v[j] >= 0 ? (int)sh.a.c[v[j]] : 0;
            const Bounds<int32_t> row = v[j] >= 0 ? row_of(rp, v[j]) : Bounds<int32_t>{0, 0};
            b[j] = row.b;
            e[j] = row.e;
            done |= (b[j] >= e[j] ? 1u : 0u) << j;
        }
        for (int q0 = 0; done != (1u << K) - 1; q0 += C) {
            int u[K][C];
#pragma unroll
            for (int j = 0; j < K; ++j)
            {
                if (!(done >> j & 1u)) load4(ci, b[j] + q0, m, INT32_MAX, u[j]);
#pragma unroll
                for (int q = 0; q < C; ++q)
                    if ((done >> j & 1u) || b[j] + q0 + q >= e[j]) u[j][q] = INT32_MAX;
            }
#pragma unroll
            for (int j = 0; j < K; ++j) {
                bool past = false;
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    if (u[j][q] >= v[j]) past |= sorted;
                    else if ((sh.a.c[u[j][q]] & ~kFresh) == t[j]) lose |= 1u << j;
                }
                if (past || (lose >> j & 1u) || b[j] + q0 + C >= e[j]) done |= 1u << j;
            }
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool l = v[j] >= 0 && (lose >> j & 1u);
            const int at = wave_append(l, &sh.nl[p ^ 1]);
            if (l) nxt[at] = (uint16_t)v[j];
            if (v[j] < 0 || l) continue;
            sh.a.c[v[j]] = (uint16_t)(t[j] | kFresh);
            out[v[j]] = t[j];
            gone += e[j] - b[j];
        }
        if (!Push) continue;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (v[j] < 0 || (lose >> j & 1u) || t[j] > kMaskColors) continue;
            const unsigned long long bit = 1ull << (t[j] - 1);
            for (int k = b[j]; k < e[j]; k += C) {
                int u[C];
                load4(ci, k, m, -1, u);
#pragma unroll
                for (int q = 0; q < C; ++q)
                    if (k + q < e[j]) atomicOr((unsigned long long *)&sh.a.mask[u[q]], bit);
            }
        }
    }
}

// The same for the long rows, by groups of S lanes (16, so that four rows overlap in a wavefront, or a
// wavefront when there are few of them).
__device__ __forceinline__ void small_wide(SmallShared &sh, const int32_t *rp, const int32_t *ci, int32_t *out, int p,
                                           bool sorted, int &gone) {
    constexpr int C = 4;
    const int nw = sh.nw[p], S = nw >= kCore / kWave * 4 ? 16 : kWave, per = kCore / S;
    const int lane = lane_id(), gl = threadIdx.x % S;
    const uint64_t gm = S == kWave ? ~0ull : 0xFFFFull << (lane - gl);
    const uint16_t *cur = sh.a.wl[p];
    uint16_t *nxt = sh.a.wl[p ^ 1];
    for (int i0 = 0; i0 < nw; i0 += per) {  // the same for the whole workgroup
        const int i = i0 + (int)threadIdx.x / S;
        const int v = i < nw ? (int)cur[kSmallNodes - 1 - i] : -1;
        const int t = v >= 0 ? (int)sh.a.c[v] : 0, b = v >= 0 ? rp[v] : 0, e = v >= 0 ? rp[v + 1] : 0;
        bool lose = false, more = b < e;
        for (int k0 = b; __ballot(more); k0 += C * S) {  // the same for the whole wavefront
            int u[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int k = k0 + q * S + gl;
                u[q] = more && k < e ? ci[k] : INT32_MAX;
            }
            bool hit = false, past = false;
#pragma unroll
            for (int q = 0; q < C; ++q) {
                if (u[q] >= v) past |= sorted;
                else hit |= (sh.a.c[u[q]] & ~kFresh) == t;
            }
            lose = lose || (__ballot(hit) & gm) != 0;
            more = more && !lose && !(__ballot(past) & gm) && k0 + C * S < e;
        }
        const bool l = v >= 0 && lose && gl == 0;
        const int at = wave_append(l, &sh.nw[p ^ 1]);
        if (l) nxt[kSmallNodes - 1 - at] = (uint16_t)v;
        if (v < 0 || lose) continue;
        if (gl == 0) {
            sh.a.c[v] = (uint16_t)(t | kFresh);
            out[v] = t;
            gone += e - b;
        }
        if (t > kMaskColors) continue;
        const unsigned long long bit = 1ull << (t - 1);
        for (int k0 = b + gl; k0 < e; k0 += C * S) {
            int u[C];
#pragma unroll
            for (int q = 0; q < C; ++q) u[q] = k0 + q * S < e ? ci[k0 + q * S] : -1;
#pragma unroll
            for (int q = 0; q < C; ++q)
                if (u[q] >= 0) atomicOr((unsigned long long *)&sh.a.mask[u[q]], bit);
        }
    }
}

// Row rounds: from round r on, `nact` uncolored nodes; fresh: all nodes of the graph, before any round, else those of
// worklist p.  Up to four nodes a thread, each with its rank, its row and the colors it may not take.  A round has
// two steps: conflict (a smaller neighbour with the same color in |s|; winners turn their s positive at once, which
// changes no test) and, for the losers, the colors that neighbours have committed, whose entries leave the row.
// Returns the number of the last round, 0 if the rounds did not end.
__device__ __forceinline__ int32_t small_rows(SmallShared &sh, const SmallArgs &a, const int32_t *rp, const int32_t *ci,
                                              int32_t n, int32_t m, int32_t *out, int p, int32_t r, int nact, bool fresh, bool sorted) {
    constexpr int K = kRowsNodes / kCore;
    const int tid = threadIdx.x, lane = lane_id();
    const bool keep = a.trace != nullptr;
    int64_t degsum = (int64_t)sh.deg;
    int v[K], b[K], len[K], rank[K], at[K], t[K];
    uint64_t mask[K];
    if (!fresh) {
        for (int k = tid; k < kSmallNodes / 64; k += kCore) sh.bits[k] = 0;
        __syncthreads();
    }
    int sum = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int i = j * kCore + tid;
        v[j] = i >= nact ? -1 : fresh ? i : (int)sh.a.wl[p][i];
        mask[j] = 0;
        const Bounds<int32_t> row = v[j] >= 0 ? row_of(rp, v[j]) : Bounds<int32_t>{0, 0};
        b[j] = row.b;
        len[j] = row.e - row.b;
        sum += len[j];
        if (v[j] >= 0 && !fresh) atomicOr((unsigned long long *)&sh.bits[v[j] >> 6], 1ull << (v[j] & 63));
    }
    __syncthreads();
    int total;
    if (!fresh) {
        const int pc = tid < kSmallNodes / 64 ? __popcll(sh.bits[tid]) : 0;
        const int ex = block_scan(pc, &total);
        if (tid < kSmallNodes / 64) sh.pre[tid] = ex;
    }
    int first = block_scan(sum, &total);  // (its barriers: the worklist's state has been read)
    __syncthreads();
    const auto rank_of = [&](int32_t u) {
        if (fresh) return u;
        const uint64_t word = sh.bits[u >> 6], bit = 1ull << (u & 63);
        return word & bit ? sh.pre[u >> 6] + (int)__popcll(word & (bit - 1)) : -1;
    };
#pragma unroll
    for (int j = 0; j < K; ++j) {
        at[j] = first;
        first += len[j];
        rank[j] = v[j] >= 0 ? rank_of(v[j]) : 0;
        int w = 0;
        for (int q0 = 0; q0 < len[j]; q0 += 4) {
            int32_t u[4];
            load4(ci, b[j] + q0, m, -1, u);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q0 + q >= len[j]) continue;
                const int x = rank_of(u[q]);
                if (x >= 0 && x != rank[j]) sh.rows.adj[at[j] + w++] = (uint16_t)x;
                if (x < 0) mask[j] |= 1ull << ((sh.rows.c[u[q]] & kHeld) - 1);  // committed in the list rounds
            }
        }
        if (keep && v[j] >= 0) b[j] = len[j];  // the degree, for the record
        len[j] = w;
        t[j] = __ffsll((unsigned long long)~mask[j]);
        if (v[j] >= 0) sh.rows.s[rank[j]] = (int16_t)-t[j];
    }
    if (tid == 0) sh.rows.left[r & 1] = 0;
    core_sync();
    uint32_t act = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) act |= (v[j] >= 0 ? 1u : 0u) << j;
    for (; nact > 0; ++r) {
        if (r > n) return 0;
        if (keep && tid == 0 && r - 1 < a.trace_cap) {
            a.trace[r - 1] = nact;
            a.trace_deg[r - 1] = degsum;
        }
        if (tid == 0) sh.rows.left[(r + 1) & 1] = 0;  // last read before the barrier that ended the round before
        uint32_t won = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (!(act >> j & 1u)) continue;
            bool lose = false;
            for (int q0 = 0; q0 < len[j] && !lose; q0 += 4) {
                int x[4], c[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = q0 + q < len[j] ? (int)sh.rows.adj[at[j] + q0 + q] : kRowsNodes;
#pragma unroll
                for (int q = 0; q < 4; ++q) c[q] = x[q] < rank[j] ? abs((int)sh.rows.s[x[q]]) : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) lose |= c[q] == t[j];
                if (sorted && x[3] > rank[j]) break;
            }
            if (lose) continue;
            won |= 1u << j;
            sh.rows.s[rank[j]] = (int16_t)t[j];
            out[v[j]] = t[j];
        }
        act &= ~won;
        int some = __popc(act);
        for (int o = 32; o > 0; o >>= 1) some += __shfl_xor(some, o);
        if (lane == 0 && some) atomicAdd(&sh.rows.left[r & 1], some);
        if (keep) {
            int gone = 0;
#pragma unroll
            for (int j = 0; j < K; ++j) gone += won >> j & 1u ? b[j] : 0;
            gone = (int)wave_sum(gone);
            if (lane == 0 && gone) atomicAdd(&sh.deg, 0ull - (unsigned long long)gone);
        }
        core_sync();
        nact = sh.rows.left[r & 1];
        degsum = (int64_t)sh.deg;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (!(act >> j & 1u)) continue;
            int w = 0;
            for (int q0 = 0; q0 < len[j]; q0 += 4) {
                int x[4], c[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = q0 + q < len[j] ? (int)sh.rows.adj[at[j] + q0 + q] : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q) c[q] = x[q] >= 0 ? (int)sh.rows.s[x[q]] : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (c[q] > 0 && c[q] <= kMaskColors) mask[j] |= 1ull << (c[q] - 1);
                    if (c[q] < 0) sh.rows.adj[at[j] + w++] = (uint16_t)x[q];
                }
            }
            len[j] = w;
            t[j] = __ffsll((unsigned long long)~mask[j]);
            sh.rows.s[rank[j]] = (int16_t)-t[j];
        }
        core_sync();
    }
    return r - 1;
}

// More rounds than nodes.  (One graph alone: the host finds `finished` unset.)
__device__ __forceinline__ void limit(const SmallArgs &a) {
    if (threadIdx.x == 0) a.ct->small_limit = 1;
}

static __global__ __launch_bounds__(kCore) void k_small(SmallArgs a) {
    __shared__ SmallShared sh;
    const int tid = threadIdx.x, lane = lane_id();
    const int32_t g = a.order ? a.order[blockIdx.x] : 0;
    const int64_t n0 = a.node_off ? a.node_off[g] : 0, e0 = a.node_off ? a.edge_off[g] : 0;
    const int32_t n = (int32_t)(a.node_off ? a.node_off[g + 1] - n0 : a.n);
    const int64_t m = a.node_off ? a.edge_off[g + 1] - e0 : a.m;
    const int32_t *rp = a.rowptr + n0 + g, *ci = a.colidx + e0;
    int32_t *out = a.out + n0;

    // Checks: the CSR's ends, row pointers non-decreasing inside [0, m], ids inside [0, n); and whether every
    // row is sorted: the entries not above their predecessor are then all first entries of rows.
    if (tid == 0) {
        sh.bad = sh.descents = sh.starts = sh.maxdeg = 0;
        sh.nl[0] = sh.nw[0] = 0;
    }
    __syncthreads();
    int bad = 0, starts = 0, descents = 0, maxdeg = 0;
    for (int v = tid; v < n; v += kCore) {
        const int64_t b = rp[v], e = rp[v + 1];
        if (b < 0 || e < b || e > m) bad |= 1;
        else if (b > 0 && b < e) starts += ci[b] <= ci[b - 1];
        maxdeg = max(maxdeg, (int)min<int64_t>(e - b, INT32_MAX));
    }
    if (tid == 0) {
        if (rp[0] != 0 || rp[n] != m) bad |= 4;
        if (!a.node_off) {
            a.ct->ends[0] = rp[0];
            a.ct->ends[1] = rp[n];
        }
    }
    constexpr int P = 8;
    for (int64_t k0 = tid; k0 < m; k0 += P * kCore) {
        int32_t u[P], w[P];
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int64_t k = k0 + q * kCore;
            u[q] = k < m ? ci[k] : 0;
            w[q] = k > 0 && k < m ? ci[k - 1] : INT32_MIN;
        }
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int64_t k = k0 + q * kCore;
            if (k >= m) continue;
            if (a.check && (uint32_t)u[q] >= (uint32_t)n) bad |= 2;
            descents += k > 0 && u[q] <= w[q];
        }
    }
    if (bad) atomicOr(&sh.bad, bad);
    starts = (int)wave_sum(starts);
    descents = (int)wave_sum(descents);
    if (lane == 0 && starts) atomicAdd(&sh.starts, starts);
    if (lane == 0 && descents) atomicAdd(&sh.descents, descents);
    for (int o = 32; o > 0; o >>= 1) maxdeg = max(maxdeg, __shfl_xor(maxdeg, o));
    if (lane == 0) atomicMax(&sh.maxdeg, maxdeg);
    __syncthreads();
    bad = sh.bad;
    const bool sorted = sh.starts == sh.descents;
    if (bad) {
        if (tid == 0) {
            if (bad & 4) {
                if (a.node_off) a.ct->bad_rows = 1;
                else a.ct->bad_ends = 1;
            }
            if (bad & 1) a.ct->bad_rows = 1;
            if (bad & 2) a.ct->bad_ids = 1;
        }
        return;
    }

    // Rounds over the worklist while more than kCore nodes are uncolored.
    int32_t r = 1;
    int nact = n, p = 0;
    int64_t deg = m;
    const bool keep = a.trace != nullptr;
    CoreState s;
    const bool sparse = sh.maxdeg <= kRowsDegree, own = sh.maxdeg <= kOwnRows;
    bool rows = sparse && n <= kRowsNodes && m <= kRowsEntries;
    if (rows) {
        sh.deg = (unsigned long long)m;
    } else if (n > kCore) {
        for (int v0 = 0; v0 < n; v0 += kCore) {
            const int v = v0 + tid;
            const bool has = v < n, wide = has && rp[v + 1] - rp[v] > kSmallLight;
            if (has) {
                if (!own) sh.a.mask[v] = 0;
                sh.a.c[v] = 1;
            }
            const int at = wave_append(has && !wide, &sh.nl[0]), aw = wave_append(wide, &sh.nw[0]);
            if (wide) sh.a.wl[0][kSmallNodes - 1 - aw] = (uint16_t)v;
            else if (has) sh.a.wl[0][at] = (uint16_t)v;
        }
        if (tid == 0) sh.deg = (unsigned long long)m;
        __syncthreads();
        int pl = 0, pw = 0;  // entries of the round before's lists
        while (nact > kCore) {
            if (keep && tid == 0 && r - 1 < a.trace_cap) {
                a.trace[r - 1] = nact;
                a.trace_deg[r - 1] = (int64_t)sh.deg;
            }
            const int nl = sh.nl[p], nw = sh.nw[p];
            if (r > n) {  // every round has a winner (unless ids that nobody checked lead outside the graph)
                limit(a);
                return;
            }
            if (r > 1 && own) {
                if (r <= 33) small_learn<uint32_t>(sh, rp, ci, (int32_t)m, p);  // committed in rounds 1 to 32
                else small_learn<uint64_t>(sh, rp, ci, (int32_t)m, p);
            } else if (r > 1) {  // round 1's tentative colors are all 1
                for (int i = tid; i < pl + pw; i += kCore) {  // the round before's list: its winners
                    const int v = i < pl ? sh.a.wl[p ^ 1][i] : sh.a.wl[p ^ 1][kSmallNodes - 1 - (i - pl)];
                    const int c = sh.a.c[v];
                    if (c & kFresh) sh.a.c[v] = (uint16_t)(c ^ (kFresh | kPast));
                }
                for (int i = tid; i < nl + nw; i += kCore) {
                    const int v = i < nl ? sh.a.wl[p][i] : sh.a.wl[p][kSmallNodes - 1 - (i - nl)];
                    const uint64_t free = ~sh.a.mask[v];
                    sh.a.c[v] = (uint16_t)(free ? __ffsll((unsigned long long)free) : small_pull(sh, a, rp, ci, v));
                }
            }
            if (tid == 0) sh.nl[p ^ 1] = sh.nw[p ^ 1] = 0;
            core_sync();
            int gone = 0;
            if (own) {
                small_light<false>(sh, rp, ci, (int32_t)m, out, p, sorted, gone);
            } else {
                small_wide(sh, rp, ci, out, p, sorted, gone);
                small_light<true>(sh, rp, ci, (int32_t)m, out, p, sorted, gone);
            }
            gone = (int)wave_sum(gone);
            if (lane == 0 && gone) atomicAdd(&sh.deg, 0ull - (unsigned long long)gone);
            core_sync();
            p ^= 1;
            pl = nl;
            pw = nw;
            ++r;
            nact = sh.nl[p] + sh.nw[p];
            core_sync();  // the counts are cleared in the next round, the degree sum read
            rows = sparse && nact <= kRowsNodes && sh.deg <= kRowsEntries;
            if (rows) break;
        }
        deg = (int64_t)sh.deg;
    }
    if (rows) {
        const int32_t last = small_rows(sh, a, rp, ci, n, (int32_t)m, out, p, r, nact, n <= kRowsNodes && r == 1, sorted);
        if (last == 0 && n > 0) {
            limit(a);
            return;
        }
        if (tid == 0) {
            if (a.grounds) a.grounds[g] = last;
            if (!a.node_off) {
                a.ct->rounds = last;
                a.ct->finished = 1;
            }
        }
        return;
    }
    if (n > kCore) {
        // hand over to the core: ranks from a bit per uncolored node, the nodes' state through shared memory
        for (int k = tid; k < kSmallNodes / 64; k += kCore) sh.bits[k] = 0;
        __syncthreads();
        const int nl = sh.nl[p];
        int v = -1;
        if (tid < nact) v = tid < nl ? sh.a.wl[p][tid] : sh.a.wl[p][kSmallNodes - 1 - (tid - nl)];
        const int32_t t = v >= 0 ? (int32_t)sh.a.c[v] : 0;
        const uint64_t mask = v >= 0 ? sh.a.mask[v] : 0;
        if (v >= 0) {
            atomicOr((unsigned long long *)&sh.bits[v >> 6], 1ull << (v & 63));
            out[v] = 0;  // not committed (read when a color window has to be filled from the row)
        }
        __syncthreads();
        int total;
        const int pc = tid < kSmallNodes / 64 ? __popcll(sh.bits[tid]) : 0;
        const int ex = block_scan(pc, &total);
        if (tid < kSmallNodes / 64) sh.pre[tid] = ex;
        __syncthreads();
        uint64_t *stage = sh.core.adj;  // 3 words a node
        if (v >= 0) {
            const int rank = sh.pre[v >> 6] + __popcll(sh.bits[v >> 6] & ((1ull << (v & 63)) - 1));
            stage[rank] = (uint64_t)(uint32_t)v;
            stage[kCore + rank] = (uint64_t)(uint32_t)t;
            stage[2 * kCore + rank] = mask;
        }
        __syncthreads();
        if (tid < nact) {
            s.v = (int32_t)stage[tid];
            s.base = (int32_t)stage[kCore + tid] - 1;
            const uint64_t mk = stage[2 * kCore + tid];
            s.lo = s.base < 64 ? mk >> s.base : 0;
            if (r > kMaskColors + 1) {  // colors above 64 may be committed: the row says which
                const SmallRow row{rp, ci, out};
                s.lo = row.taken(s, s.base + 1);
                s.hi = row.taken(s, s.base + 65);
            }
        }
    } else if (tid < n) {
        s.v = tid;
        out[tid] = 0;
    }
    __syncthreads();
    if (nact > 0) {  // false for a graph without nodes alone
        // The matrix: short rows by their thread, long ones by 16 lanes or a wavefront.
        for (int k = tid; k < kCoreWords * kCoreStride; k += kCore) sh.core.adj[k] = 0;
        if (tid == 0) sh.core.nwin = 0;
        __syncthreads();
        const bool direct = n <= kCore;
        const auto put = [&](int rank, int32_t u) {
            int q = u;
            if (!direct) {
                const uint64_t word = sh.bits[u >> 6], bit = 1ull << (u & 63);
                if (!(word & bit)) return;
                q = sh.pre[u >> 6] + __popcll(word & (bit - 1));
            }
            atomicOr((unsigned long long *)&sh.core.adj[(q >> 6) * kCoreStride + rank], 1ull << (q & 63));
        };
        const int b = s.v >= 0 ? rp[s.v] : 0, e = s.v >= 0 ? rp[s.v + 1] : 0;
        s.deg = e - b;
        const bool wide = s.deg > kSmallLight;
        const int at = wave_append(wide, &sh.core.nwin);
        if (wide) sh.core.t[at] = tid;
        else {
            for (int k = b; k < e; k += 4) {
                int32_t u[4];
                load4(ci, k, (int32_t)m, -1, u);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (k + q < e) put(tid, u[q]);
            }
        }
        int32_t *node = reinterpret_cast<int32_t *>(sh.core.bucket);  // node of each rank, until the rounds start
        if (tid < nact) node[tid] = s.v;
        __syncthreads();
        const int nw = sh.core.nwin, S = nw >= kCore / kWave * 4 ? 16 : kWave, gl = tid % S;
        for (int i = tid / S; i < nw; i += kCore / S) {
            const int rank = sh.core.t[i], v = node[rank];
            const int e2 = rp[v + 1];
            for (int k = rp[v] + gl; k < e2; k += 4 * S) {
                int32_t u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) u[q] = k + q * S < e2 ? ci[k + q * S] : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (u[q] >= 0) put(rank, u[q]);
            }
        }
        __syncthreads();
    }
    int64_t nodes = 0;
    const int32_t last = core_rounds(
        SmallRow{rp, ci, out}, sh.core, s, r, nact, keep, deg, &nodes,
        [&](const CoreState &x, int32_t) { out[x.v] = x.t; },
        [&](int32_t q, int32_t active, int64_t dsum) {
            if (keep && q - 1 < a.trace_cap) {
                a.trace[q - 1] = active;
                a.trace_deg[q - 1] = dsum;
            }
        });
    if (tid == 0) {
        if (a.grounds) a.grounds[g] = last;
        if (!a.node_off) {
            a.ct->rounds = last;
            a.ct->finished = 1;
        }
    }
}

}  // namespace ipgc
