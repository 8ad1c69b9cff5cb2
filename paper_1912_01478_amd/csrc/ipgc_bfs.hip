// Level-synchronous breadth-first search under the keep-the-worklist hybrid
// schedule (Section IV of Rai, M P, Pai, arXiv 1912.01478, applied to another
// worklist algorithm, as its conclusion proposes).  Level L expands the
// frontier (the nodes at distance L): a topology-driven level sweeps every node
// and expands those with dist == L; a data-driven level walks the worklist.
// Both kinds push every newly reached node onto the worklist of level L + 1, so
// the worklist is kept in every level, and a level is topology-driven iff the
// frontier holds more than H nodes.
//
// A neighbour u is claimed with one compare-and-swap on dist[u] (-1 -> L + 1),
// so each node enters exactly one frontier, once.  Nodes of degree up to 32
// expand with one thread, nodes up to kHubDeg entries with a wavefront of the
// same workgroup, and wider ones (hubs) by the whole grid in a second step of
// the level.  Pushes go to the workgroup's own segment (shared-memory counter,
// no global atomic); a segment that fills up spills into an overflow list
// through one atomicAdd per spilled node.  All levels run in one cooperative
// launch with the grid barrier of the coloring kernels, one barrier per level
// and one more in levels with hubs.  Small graphs run on one workgroup
// (k_bfs_one), with the same distances and levels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "ipgc.h"
#include "ipgc_device.hpp"
#include "ipgc_host.hpp"

namespace ipgc {
namespace bfs {

constexpr int kBlock = 1024;
constexpr int kLightDeg = 32;     // wider frontier nodes are expanded by a wavefront
constexpr int kHeavyPerBlock = 1024;
// Rows longer than this are spread over the grid.  A wavefront takes about 1.5 us per 256 entries
// (column id, distance, claim: three dependent trips to memory), so a row of this length keeps it for
// about 12 us, what the extra barrier and the staging of the hub step cost; the widest row of an
// R-MAT graph of 2^22 nodes (160 000 entries) kept one for 4 ms.
constexpr int kHubDeg = 2048;
// Graphs of at most so many nodes and entries are searched by one workgroup: a level takes 4 us there and 14 us
// over the grid, but one compute unit reads 256 entries a microsecond.  One workgroup / the grid, a search:
// 1000 nodes and 8 000 entries 52 / 129 us, 20 000 and 80 000 129 / 205 us, R-MAT 8192 and 204 000 151 / 169 us,
// R-MAT 16 384 and 228 000 190 / 186 us, 32 000 and 256 000 246 / 218 us.
constexpr int kOneNodes = 32768;
constexpr int64_t kOneEntries = 3 << 16;
constexpr int kOneHubDeg = 1024;  // there, rows longer than this are walked by all threads together
constexpr int kHubChunk = 4 * kWave;  // hub entries per wavefront step

// Control block of one call: cleared before it, read back after it.
struct BfsCtl {
    int32_t levels;       // non-empty levels
    int32_t done;         // the last level was empty (stays 0 if a grid-barrier wait gave up)
    int32_t bad;          // decreasing row pointers, or a column id out of range
    int32_t bad_ends;     // rowptr[0] != 0 or rowptr[n] != m
    int32_t ovf_cnt[3];   // three rotating overflow sizes: level L reads L % 3, fills (L + 1) % 3
    int32_t hubs[3];      // three rotating hub counts: level L uses L % 3
};

struct BfsDev {
    const int32_t *rowptr;
    const int32_t *colidx;
    int32_t *dist;
    int32_t *seg[2];      // frontier lists: grid segments of cap entries
    int32_t *seg_cnt[2];  // entries per segment (at most cap)
    int32_t *ovf[2];      // overflow lists
    int32_t *hub;         // hubs of the level (at most m / (kHubDeg + 1))
    int32_t *trace;       // frontier size per level
    int64_t trace_cap;
    int64_t n;
    int64_t m;
    int64_t threshold;    // topology-driven level iff |frontier| > threshold
    int32_t source;
    int32_t cap;
    BfsCtl *ctl;
    Barrier *bar;
    uint64_t bar_limit;   // wall-clock ticks a grid-barrier wait may last
};

// Prefix sums over the grid segments plus the overflow list (grid + 1 parts) in shared memory.
__device__ int32_t frontier_view(const BfsDev &d, int p, int lvl, int32_t *pre) {
    const int nb = gridDim.x;
    int x = 0;
    if (threadIdx.x < (unsigned)nb) x = d.seg_cnt[p][threadIdx.x];
    else if (threadIdx.x == (unsigned)nb) x = d.ctl->ovf_cnt[lvl % 3];
    int tot;
    const int ex = block_scan(x, &tot);
    if (threadIdx.x <= (unsigned)nb) pre[threadIdx.x] = ex;
    if (threadIdx.x == 0) pre[nb + 1] = tot;
    __syncthreads();
    return tot;
}

__device__ __forceinline__ int32_t frontier_at(const BfsDev &d, int p, const int32_t *pre, int32_t i) {
    int lo = 0, hi = gridDim.x + 1;  // part lo with pre[lo] <= i < pre[lo + 1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pre[mid] <= i) lo = mid;
        else hi = mid;
    }
    if (lo == (int)gridDim.x) return d.ovf[p][i - pre[lo]];
    return d.seg[p][(int64_t)lo * d.cap + (i - pre[lo])];
}

// Row entries k0, k0 + step, ... (P of them) below e: claims their unvisited nodes for level `next`.  The
// P loads of each kind are in flight together.  A first look at dist reads through the caches: a value
// other than -1 is final, a stale -1 only leads to the second look, which does not (most entries of a
// large level lead to nodes reached long before, and those are settled in the caches).  Without the second
// look (Twice) a stale -1 costs a failed claim instead of a trip to memory for all: the rows that one thread
// walks, whose level lasts as long as its longest chain of trips (sparse random graph of 100 003 nodes,
// with 16 entries in flight instead of 4: 347 -> 307 us a search with one look, 354 with two).
// Winners go to this workgroup's segment, or to the overflow list, whose places the lanes of a wavefront
// take together (80 ns for every atomic on one address).
template <int P, bool Twice = true>
__device__ __forceinline__ void visit(const BfsDev &d, int64_t k0, int32_t step, int64_t e, int32_t next, int dst,
                                      int *s_cnt) {
    int32_t u[P];
    bool open[P];
#pragma unroll
    for (int j = 0; j < P; ++j) u[j] = k0 + j * step < e ? d.colidx[k0 + j * step] : -1;
#pragma unroll
    for (int j = 0; j < P; ++j)
        open[j] = u[j] >= 0 && __hip_atomic_load(&d.dist[u[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == -1;
    if (Twice) {
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (open[j]) open[j] = __hip_atomic_load(&d.dist[u[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == -1;
    }
#pragma unroll
    for (int j = 0; j < P; ++j) open[j] = open[j] && atomicCAS(&d.dist[u[j]], -1, next) == -1;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        if (!open[j]) continue;
        const int p = atomicAdd(s_cnt, 1);
        if (p < d.cap) {
            d.seg[dst][(int64_t)blockIdx.x * d.cap + p] = u[j];
        } else {
            const uint64_t full = __ballot(1);  // the lanes that are here
            int at = 0;
            if ((full & lanes_below()) == 0) at = atomicAdd(&d.ctl->ovf_cnt[next % 3], (int)__popcll(full));
            d.ovf[dst][__builtin_amdgcn_readfirstlane(at) + __popcll(full & lanes_below())] = u[j];
        }
    }
}

// Hub step of a level: the rows of its `hubs` hubs in chunks of kHubChunk entries over every wavefront of
// the grid.  Each workgroup stages up to kBlock hubs at a time (row bounds, chunk prefix sums).
__device__ void expand_hubs(const BfsDev &d, int32_t hubs, int32_t next, int dst, int *s_cnt) {
    __shared__ int32_t s_b[kBlock], s_e[kBlock], s_pre[kBlock + 1];
    const int64_t gw = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gridDim.x * blockDim.x / kWave;
    for (int32_t h0 = 0; h0 < hubs; h0 += kBlock) {
        const int32_t h = h0 + threadIdx.x;
        int chunks = 0;
        if (h < hubs) {
            const int32_t v = d.hub[h];
            s_b[threadIdx.x] = d.rowptr[v];
            s_e[threadIdx.x] = d.rowptr[v + 1];
            chunks = (int)(((int64_t)s_e[threadIdx.x] - s_b[threadIdx.x] + kHubChunk - 1) / kHubChunk);
        }
        int total;
        s_pre[threadIdx.x] = block_scan(chunks, &total);
        if (threadIdx.x == 0) s_pre[kBlock] = total;
        __syncthreads();
        const int nh = min(kBlock, hubs - h0);
        for (int64_t g = gw; g < total; g += nw) {
            int lo = 0, hi = nh;  // hub lo with s_pre[lo] <= g < s_pre[lo + 1]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_pre[mid] <= g) lo = mid;
                else hi = mid;
            }
            const int64_t k0 = s_b[lo] + (g - s_pre[lo]) * kHubChunk;
            visit<kHubChunk / kWave>(d, k0 + lane_id(), kWave, s_e[lo], next, dst, s_cnt);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_bfs(BfsDev d) {
    __shared__ int32_t pre[kMaxRoundBlocks + 2];
    __shared__ int32_t heavy[kHeavyPerBlock];
    __shared__ int s_cnt, s_heavy, s_hubs;
    if (d.ctl->bad | d.ctl->bad_ends) return;  // every workgroup reads the same flags: no row is read
    GridBarrier gb;
    if (!gb.setup(d.bar, d.bar_limit)) return;
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    const int lane = lane_id(), w = threadIdx.x / kWave, nwv = blockDim.x / kWave;
    int32_t lvl = 0;
    for (;; ++lvl) {
        const int src = lvl & 1, dst = src ^ 1;
        const int32_t size = frontier_view(d, src, lvl, pre);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            if (lvl < d.trace_cap) d.trace[lvl] = size;
            if (size == 0) {
                d.ctl->levels = lvl;
                d.ctl->done = 1;
            }
            // counts of level lvl + 1: last read before the barrier that ended level lvl - 1
            d.ctl->ovf_cnt[(lvl + 2) % 3] = 0;
            d.ctl->hubs[(lvl + 1) % 3] = 0;
        }
        if (size == 0) break;
        const bool topo = (int64_t)size > d.threshold;
        const int64_t items = topo ? d.n : size;
        const int32_t next = lvl + 1;
        if (threadIdx.x == 0) {
            s_cnt = 0;
            s_heavy = 0;
        }
        __syncthreads();
        // No barrier here: this level fills the lists and counts of parity dst, last read in level
        // lvl - 1, which every workgroup has left.
        // A wavefront's 64 items are next to each other, a workgroup's wavefronts far apart: nodes reached from one
        // row, and the low ids of an R-MAT graph, are wide together, and 1024 neighbours in the list left one
        // workgroup with a million entries (R-MAT of 2^20 nodes: 1.88 -> 0.60 ms a search; 100 003 nodes: 282 -> 235 us).
        for (int64_t i0 = (int64_t)blockIdx.x * kWave; i0 < items; i0 += nt) {
            const int64_t i = i0 + (int64_t)w * gridDim.x * kWave + lane;
            int32_t v = -1;
            if (i < items) {
                if (topo) v = d.dist[i] == lvl ? (int32_t)i : -1;
                else v = frontier_at(d, src, pre, (int32_t)i);
            }
            if (v >= 0) {
                const int32_t b = d.rowptr[v], e = d.rowptr[v + 1];
                if (e - b > kHubDeg) d.hub[atomicAdd(&d.ctl->hubs[lvl % 3], 1)] = v;
                else if (e - b > kLightDeg) heavy[atomicAdd(&s_heavy, 1)] = v;  // at most a workgroup's threads
                else
                    for (int64_t k = b; k < e; k += 16) visit<16, false>(d, k, 1, e, next, dst, &s_cnt);
            }
            __syncthreads();
            const int nh = s_heavy;
            for (int h = w; h < nh; h += nwv) {
                const int32_t u = heavy[h];
                const int32_t b = d.rowptr[u], e = d.rowptr[u + 1];
                for (int64_t k = b; k < e; k += 4 * kWave) visit<4>(d, k + lane, kWave, e, next, dst, &s_cnt);
            }
            __syncthreads();
            if (threadIdx.x == 0) s_heavy = 0;
            __syncthreads();
        }
        if (threadIdx.x == 0) d.seg_cnt[dst][blockIdx.x] = min(s_cnt, d.cap);
        if (!gb.sync()) return;
        if (threadIdx.x == 0) s_hubs = (int32_t)ld_agent((unsigned *)&d.ctl->hubs[lvl % 3]);
        __syncthreads();
        const int32_t hubs = s_hubs;
        if (hubs > 0) {  // the same in every workgroup
            expand_hubs(d, hubs, next, dst, &s_cnt);
            if (threadIdx.x == 0) d.seg_cnt[dst][blockIdx.x] = min(s_cnt, d.cap);
            if (!gb.sync()) return;
        }
    }
}

// The whole search on one workgroup: frontiers and reached nodes in shared memory, so that a level is two trips to
// memory (row bounds, entries) and workgroup barriers.
struct OneShared {
    uint16_t list[2][kOneNodes];
    uint32_t seen[kOneNodes / 32];
    uint16_t wide[kBlock];  // of the frontier nodes at hand: wavefront rows from the front, rows for all from the back
    int cnt[2];
    int rows, hubs;
};

// visit() for one workgroup
template <int P>
__device__ __forceinline__ void visit_one(const BfsDev &d, OneShared &sh, int32_t k0, int32_t step, int32_t e, int32_t next,
                                          int dst) {
    int32_t u[P];
#pragma unroll
    for (int j = 0; j < P; ++j) u[j] = (int64_t)k0 + (int64_t)j * step < e ? d.colidx[k0 + j * step] : -1;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        if (u[j] < 0) continue;
        const uint32_t bit = 1u << (u[j] & 31);
        if ((sh.seen[u[j] >> 5] & bit) || (atomicOr(&sh.seen[u[j] >> 5], bit) & bit)) continue;
        sh.list[dst][atomicAdd(&sh.cnt[dst], 1)] = (uint16_t)u[j];
        d.dist[u[j]] = next;
    }
}

__global__ __launch_bounds__(kBlock) void k_bfs_one(BfsDev d) {
    __shared__ OneShared sh;
    if (d.ctl->bad | d.ctl->bad_ends) return;
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    for (int k = tid; k < kOneNodes / 32; k += kBlock) sh.seen[k] = 0;
    __syncthreads();
    if (tid == 0) {
        sh.list[0][0] = (uint16_t)d.source;
        sh.seen[d.source >> 5] = 1u << (d.source & 31);
        sh.cnt[0] = 1;
    }
    __syncthreads();
    for (int32_t lvl = 0;; ++lvl) {
        const int src = lvl & 1, dst = src ^ 1, size = sh.cnt[src];
        if (tid == 0) {
            if (lvl < d.trace_cap) d.trace[lvl] = size;
            if (size == 0) {
                d.ctl->levels = lvl;
                d.ctl->done = 1;
            }
            sh.cnt[dst] = sh.rows = sh.hubs = 0;
        }
        if (size == 0) return;
        __syncthreads();
        for (int i0 = 0; i0 < size; i0 += kBlock) {
            const int i = i0 + tid;
            if (i < size) {
                const int32_t v = sh.list[src][i];
                const int32_t b = d.rowptr[v], e = d.rowptr[v + 1];
                if (e - b > kOneHubDeg) sh.wide[kBlock - 1 - atomicAdd(&sh.hubs, 1)] = (uint16_t)v;
                else if (e - b > kLightDeg) sh.wide[atomicAdd(&sh.rows, 1)] = (uint16_t)v;
                else
                    for (int32_t k = b; k < e; k += 16) visit_one<16>(d, sh, k, 1, e, lvl + 1, dst);
            }
            __syncthreads();
            const int rows = sh.rows, hubs = sh.hubs;
            for (int h = w; h < rows; h += kBlock / kWave) {
                const int32_t v = sh.wide[h];
                const int32_t b = d.rowptr[v], e = d.rowptr[v + 1];
                for (int64_t k = b + lane; k < e; k += 8 * kWave) visit_one<8>(d, sh, (int32_t)k, kWave, e, lvl + 1, dst);
            }
            for (int h = 0; h < hubs; ++h) {
                const int32_t v = sh.wide[kBlock - 1 - h];
                const int32_t b = d.rowptr[v], e = d.rowptr[v + 1];
                for (int64_t k = b + tid; k < e; k += 4 * kBlock) visit_one<4>(d, sh, (int32_t)k, kBlock, e, lvl + 1, dst);
            }
            __syncthreads();
            if (tid == 0) sh.rows = sh.hubs = 0;
            __syncthreads();
        }
    }
}

// Buffers of one device, kept between calls (they only grow).
struct BfsWorkspace {
    DBuf<int32_t> seg0, seg1, cnt0, cnt1, ovf0, ovf1, hub, tr;
    DBuf<BfsCtl> ctl;
    DBuf<Barrier> bar;
    BfsCtl *host_ctl = nullptr;  // pinned
};
std::mutex g_bfs_mutex;
std::vector<BfsWorkspace> g_bfs_ws;

// Initial state (the source at distance 0 and alone in the frontier, every other node unreached) and the
// input checks: the CSR ends, row pointers non-decreasing inside [0, m] and, with `ids`, every entry's
// column id inside [0, n).  The rows cover exactly the m entries when the row pointers pass, so the
// entries are read as one array, coalesced, whatever the degrees; a lane per row kept one lane for the
// 160 000 entries of the widest row of an R-MAT graph of 2^22 nodes (16.5 ms).
__global__ __launch_bounds__(256) void k_bfs_prep(BfsDev d, int32_t ids) {
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    if (gt == 0) {
        d.seg[0][0] = d.source;
        if (d.rowptr[0] != 0 || d.rowptr[d.n] != d.m) d.ctl->bad_ends = 1;
    }
    for (int64_t i = gt; i < kMaxRoundBlocks; i += nt) {
        d.seg_cnt[0][i] = i == 0;
        d.seg_cnt[1][i] = 0;
    }
    int b = 0;
    for (int64_t v = gt; v < d.n; v += nt) {
        d.dist[v] = v == d.source ? 0 : -1;
        if (ids) {
            const int64_t a = d.rowptr[v], e = d.rowptr[v + 1];
            b |= a < 0 || e < a || e > d.m;
        }
    }
    if (ids) {
        const uint32_t n = (uint32_t)d.n;
        for (int64_t k = gt; k < d.m; k += 8 * nt) {
            uint32_t u[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) u[j] = k + j * nt < d.m ? (uint32_t)d.colidx[k + j * nt] : 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) b |= u[j] >= n;  // negative ids too
        }
    }
    if (__ballot(b) && lane_id() == 0) d.ctl->bad = 1;
}

}  // namespace bfs

void release_bfs_workspaces() {
    std::lock_guard<std::mutex> lock(bfs::g_bfs_mutex);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (size_t dv = 0; dv < bfs::g_bfs_ws.size(); ++dv) {
        if (hipSetDevice((int)dv) != hipSuccess) continue;
        bfs::BfsWorkspace &w = bfs::g_bfs_ws[dv];
        w.seg0.release(); w.seg1.release(); w.cnt0.release(); w.cnt1.release(); w.ovf0.release(); w.ovf1.release();
        w.hub.release(); w.tr.release(); w.ctl.release(); w.bar.release();
        if (w.host_ctl) (void)hipHostFree(w.host_ctl);
    }
    (void)hipSetDevice(cur);
    bfs::g_bfs_ws.clear();
}

namespace bfs {

int bfs_impl(const int32_t *rowptr, const int32_t *colidx, int64_t n, int64_t m, int64_t source, int mode,
             const ipgc_options *options, hipStream_t s, int32_t *out_dist, int32_t *out_levels, ipgc_trace *trace) {
    if (!out_levels) return fail(IPGC_EINVAL, "null out_levels");
    *out_levels = -1;
    if (n < 0 || m < 0) return fail(IPGC_EINVAL, "negative n or m");
    if (n >= INT32_MAX || m >= INT32_MAX) return fail(IPGC_ETOOBIG, "n or m does not fit the int32 CSR");
    if (mode == IPGC_MODE_REBUILD) return fail(IPGC_EINVAL, "BFS runs TOPOLOGY, DATA or HYBRID");
    Params P;
    TRY(parse_options(options, mode, &P));
    if (P.stepped || P.racy || P.prof) return fail(IPGC_EINVAL, "BFS takes no flags and no profile");
    if (trace) trace->recorded = 0;
    if (n == 0) {
        *out_levels = 0;
        g_err[0] = 0;
        return IPGC_OK;
    }
    if (source < 0 || source >= n) return fail(IPGC_EINVAL, "source %lld outside [0, n)", (long long)source);
    if (!rowptr || !out_dist || (m > 0 && !colidx)) return fail(IPGC_EINVAL, "null device pointer");
    int dev = 0, cus = 0, per_cu = 0, coop = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) return fail(IPGC_EHIP, "the device cannot launch cooperatively");
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(k_bfs), kBlock, 0));
    // the frontier view keeps one prefix entry per workgroup plus the overflow list in a block of kBlock threads
    const int cap_grid = std::max(1, std::min(std::min(kMaxRoundBlocks, kBlock) - 1, cus * std::max(1, per_cu)));
    // Two nodes or 16 entries a thread: more workgroups make the barriers dearer, fewer walk more rows one after the
    // other (sparse random graph of 100 003 nodes, with 25 / 50 / 100 / 200 workgroups: 260 / 233 / 235 / 245 us a search;
    // R-MAT graph of 65 536 nodes and 1.8 million entries, with 32 / 64 / 128: 304 / 248 / 231 us).
    const int64_t want = P.workgroups > 0 ? P.workgroups : std::max(n / (2 * kBlock), m / (16 * kBlock)) + 1;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(want, cap_grid));

    int64_t H;
    if (P.mode == IPGC_MODE_TOPOLOGY) H = -1;
    else if (P.mode == IPGC_MODE_DATA) H = INT64_MAX;
    else H = P.threshold > 0 ? P.threshold : (6 * n) / 10;

    std::lock_guard<std::mutex> lock(g_bfs_mutex);
    if ((int)g_bfs_ws.size() <= dev) g_bfs_ws.resize(dev + 1);
    BfsWorkspace &w = g_bfs_ws[dev];
    const int32_t cap = (int32_t)((n + grid - 1) / grid) + kBlock;
    const int64_t seg_len = (int64_t)grid * cap;
    TRY(w.seg0.reserve(seg_len));
    TRY(w.seg1.reserve(seg_len));
    TRY(w.cnt0.reserve(kMaxRoundBlocks));
    TRY(w.cnt1.reserve(kMaxRoundBlocks));
    TRY(w.ovf0.reserve(n));
    TRY(w.ovf1.reserve(n));
    TRY(w.hub.reserve(m / (kHubDeg + 1) + 1));
    TRY(w.tr.reserve(n + 1));
    TRY(w.ctl.reserve(1));
    TRY(w.bar.reserve(1));
    if (!w.host_ctl) HIP_TRY(hipHostMalloc(&w.host_ctl, sizeof(BfsCtl), hipHostMallocDefault));
    BfsDev d{};
    d.rowptr = rowptr;
    d.colidx = colidx;
    d.dist = out_dist;
    d.seg[0] = w.seg0.p;
    d.seg[1] = w.seg1.p;
    d.seg_cnt[0] = w.cnt0.p;
    d.seg_cnt[1] = w.cnt1.p;
    d.ovf[0] = w.ovf0.p;
    d.ovf[1] = w.ovf1.p;
    d.hub = w.hub.p;
    d.trace = w.tr.p;
    d.trace_cap = n + 1;
    d.n = n;
    d.m = m;
    d.threshold = H;
    d.source = (int32_t)source;
    d.cap = cap;
    d.ctl = w.ctl.p;
    d.bar = w.bar.p;
    TRY(barrier_limit_ticks(dev, P.barrier_ms, &d.bar_limit));
    TRY(clear(w.ctl.p, sizeof(BfsCtl), s));
    // sweeps over every node are what TOPOLOGY and a caller's own H ask for, and a wait limit of -1 gives up at the
    // first barrier
    const bool sweeps = P.mode == IPGC_MODE_TOPOLOGY || (P.threshold > 0 && H < n);
    const bool one = n <= kOneNodes && m <= kOneEntries && P.workgroups == 0 && !sweeps && P.barrier_ms >= 0;
    if (!one) TRY(clear(w.bar.p, sizeof(Barrier), s));
    // the search reads no row when the checks fail, so the host waits once, at the end
    const int64_t work = n + (P.check_ids ? m / 8 : 0);
    k_bfs_prep<<<(int)std::min<int64_t>(4096, (work + 255) / 256), 256, 0, s>>>(d, P.check_ids ? 1 : 0);
    HIP_TRY(hipGetLastError());
    if (one) {
        k_bfs_one<<<1, kBlock, 0, s>>>(d);
        HIP_TRY(hipGetLastError());
    } else {
        void *args[] = {&d};
        HIP_TRY(hipLaunchCooperativeKernel(reinterpret_cast<const void *>(k_bfs), dim3(grid), dim3(kBlock), args, 0, s));
    }
    HIP_TRY(hipMemcpyAsync(w.host_ctl, w.ctl.p, sizeof(BfsCtl), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    const BfsCtl h = *w.host_ctl;
    if (h.bad_ends) return fail(IPGC_EBADCSR, "rowptr[0] != 0 or rowptr[n] != m");
    if (h.bad) return fail(IPGC_EBADCSR, "decreasing rowptr or a column id outside [0, n)");
    if (!h.done)
        return fail(IPGC_EHIP, "a grid-barrier wait exceeded %d ms: not every workgroup of the cooperative launch ran "
                    "(%d workgroups)", P.barrier_ms, grid);
    if (trace) {
        const int64_t k = std::min<int64_t>(trace->capacity, h.levels);
        if (k > 0 && trace->wl_size)
            HIP_TRY(hipMemcpy(trace->wl_size, w.tr.p, sizeof(int32_t) * k, hipMemcpyDeviceToHost));
        if (k > 0 && trace->topology && trace->wl_size)
            for (int64_t i = 0; i < k; ++i) trace->topology[i] = (int8_t)((int64_t)trace->wl_size[i] > H);
        trace->recorded = k;
    }
    *out_levels = h.levels;
    g_err[0] = 0;
    return IPGC_OK;
}

}  // namespace bfs
}  // namespace ipgc

extern "C" int ipgc_bfs(const int32_t *rowptr, const int32_t *colidx, int64_t n, int64_t m, int64_t source, int mode,
                        const ipgc_options *options, void *stream, int32_t *out_dist, int32_t *out_levels,
                        ipgc_trace *trace) {
    IPGC_GUARD(ipgc::bfs::bfs_impl(rowptr, colidx, n, m, source, mode, options, (hipStream_t)stream, out_dist, out_levels,
                                   trace));
}
