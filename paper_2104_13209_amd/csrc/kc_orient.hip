// Orientation and CSR rebuild on the GPU (paper Sec. 3.1).
//
// Steps, all on one stream:
//   validate  (optional) sorted, simple, symmetric CSR check
//   key       degree order: key(v) = deg(v)
//             degeneracy order: key(v) = peeling round of v (k-core removal
//             order computed by level-synchronous peeling: one cooperative kernel until
//             few vertices are left, one workgroup for those)
//   sort      stable LSD radix sort of vertex ids by key: the position in the
//             sorted order is the new id, so (key, old id) order is the orientation
//   filter    per vertex, keep neighbours with a larger new id; out-degree
//             histogram, exclusive scan -> row_ptr (the paper's histogram + scan)
//   compact   gather each kept row, sort it by new id, write col and the COO src
#include <climits>

#include "kc_barrier.h"
#include "kc_internal.h"

namespace kc {
namespace {

constexpr int kBlock = 256;
constexpr int kItems = 8;                       // scan items per thread
constexpr int kTile = kBlock * kItems;          // 2048 elements per scan tile
constexpr int kRowCap = KC_MAX_DMAX;            // rows sorted in LDS up to this length

// Control words in the orientation workspace.
enum Ctl {
    CTL_BAD = 0,       // validation: a malformed row or a missing reverse entry
    CTL_MAXKEY = 1,    // largest sort key
    CTL_DMAX = 2,      // max out-degree
    CTL_DEGEN = 3,     // degeneracy (peel)
    CTL_ROUNDS = 4,    // peel rounds
    CTL_LONG = 5,      // a row longer than kRowCap exists
    CTL_TOTAL = 6,     // DAG edges
    CTL_SIZE0 = 8,     // peel frontier sizes, ring of 3 (8, 9, 10)
    CTL_MIN = 11,      // peel level minimum
    CTL_LEVEL = 12,    // peel: current level
    CTL_CORE = 13,     // peel: vertices left for the one-workgroup rounds
    CTL_CORE_AT = 15,  // peel: entries of the compacted rows
    CTL_CL_SIZE0 = 8,  // colouring: light frontier sizes, ring of 3 (8, 9, 10; not used with the peel)
    CTL_CL_HSIZE0 = 12,// colouring: heavy frontier sizes, ring of 3 (12, 13, 14)
    CTL_AD_LIVE = 16,  // approximate degeneracy: vertices left
    CTL_AD_SUM = 18,   // approximate degeneracy: their degree sum (u64 over words 18, 19)
    CTL_BAR = 32,      // peel: barrier arrivals, on a cache line of their own
    CTL_UP = 34,       // validation: entries to longer rows less those to shorter ones (at most nnz < 2^31)
    CTL_STALL = 36,    // peel: barrier waits that ran out (kStall* bits)
    CTL_WORDS = 64
};

// A launch's first barrier is passed when all its blocks run, for which they may have to wait
// for other streams' work: the peel is launched again.  Later ones wait for nothing else.
constexpr int kStallStart = 1, kStallLater = 2;

// ------------------------------------------------------------ validation

// Kernels over rows: a block of 16 wavefronts takes 16 * per rows in runs of `run`
// consecutive ones (a power of two up to 16 * per).  Short runs spread the hubs, with
// which vertices ordered by degree or by peeling round end, over the blocks; longer ones
// share more cache lines where ids are near their neighbours' (runs of 1 / 4 / 8 / 16, us:
// k_outdeg and k_fill on the 1M-vertex power-law graph 764 / 712 / 751 / 859, on 3M vertices of
// mean degree 8 1,159 / 965 / 935 / 920; k_validate on a ring of 200,000 vertices with 80 nearest
// neighbours 310 / 150 / 150 / 142, on a clique of 5,000 among 100,000 1,466 / 2,016 / 2,281 /
// 2,667).  A batch's
// graphs, each with its own hubs, stay together (run = 16 * per: their rows and ranks
// share cache lines, k_fill 4.6 -> 3.3 ms on the batch of 10,000).  Each wavefront loads the bounds of its `per` rows a lane each
// and walks rows of up to kLongRow entries four at a time, 16 lanes each: an average
// row has some 32 entries, and a wavefront per row waits on one chain of loads for
// each.  Longer rows go to a list in LDS: those of up to kBlockRow entries are taken by a
// wavefront each, the others by the whole block (all of them by the block: graphs of
// 100,000 vertices and mean degree 300 took 1,340 us from sort to rows, with a wavefront
// per row before 911).
constexpr int kRowBlock = 1024;
constexpr int kLongRow = 256;
constexpr int kBlockRow = 2048;
constexpr int kMaxPer = 64;
constexpr int kRowRun = 8;        // k_outdeg, k_fill
constexpr int kCheckRun = 4;      // k_validate

struct LongRows {
    int n;
    int row[16 * kMaxPer];
};

// The row of this lane, or -1.
__device__ __forceinline__ int block_row(int n, int per, int run) {
    const int lane = threadIdx.x & 63;
    const int k = (threadIdx.x >> 6) * per + lane;
    const long long i = (static_cast<long long>(k / run) * gridDim.x + blockIdx.x) * run + k % run;
    return lane < per && i < n ? static_cast<int>(i) : -1;
}

// step(lane that holds the row's bounds, first entry of the row, entry, in range), called by all
// lanes together, for this wavefront's short rows.
template <class Step>
__device__ __forceinline__ void short_rows(int b, int e, int per, int lane, Step step) {
    const int shown = e - b > kLongRow ? b : e;
    for (int q = 0; 4 * q < per; q++) {
        const int from = 4 * q + (lane >> 4);
        const int gb = __shfl(b, from), ge = __shfl(shown, from);
        const int span = wave_max(ge - gb);
        for (int t = 0; t < span; t += 16) step(from, gb, gb + t + (lane & 15), gb + t + (lane & 15) < ge);
    }
}

// Sorted, simple, symmetric?  Every index is clamped before use so that the check
// is memory-safe on any input.  Symmetry: an entry (v, w) points down when w's row
// is shorter (ties: smaller id).  Every down entry must find v in w's row, the
// shorter one of the two; rows hold no entry twice, so if also as many entries point
// up as down, every up entry is the reverse of one of them.  That halves the
// searches of testing every entry and keeps them out of the hubs' rows: 2,870 us on
// the 1M-vertex power-law graph before, 1,280 so.  Down entries are gathered in LDS until
// a wavefront has 64 of them, for half the lanes would idle in the search loops, and
// searched with three probes a step: 1,170 us, bound by the gathers (16M rows of some
// two lines each).
__global__ void __launch_bounds__(kRowBlock) k_validate(int n, int nnz, int per, int run, const int* __restrict__ row_ptr,
                                                       const int* __restrict__ col, int* ctl) {
    __shared__ int s_up;
    __shared__ int s_bad;
    __shared__ LongRows longs;
    __shared__ int s_find[kRowBlock / 64][3][128];    // searches put off until 64 are there: id, row's begin and end
    const int lane = threadIdx.x & 63;
    int (*find)[128] = s_find[threadIdx.x >> 6];
    if (threadIdx.x == 0) {
        s_up = 0;
        s_bad = 0;
        longs.n = 0;
    }
    __syncthreads();
    int bad = 0;
    int up = 0;                                       // entries that point up, less those that point down
    const int row = block_row(n, per, run);
    int b = 0, e = 0;
    if (row >= 0) {
        b = row_ptr[row];
        e = row_ptr[row + 1];
        if ((row == 0 && b != 0) || (row == n - 1 && e != nnz)) bad = 1;
        if (b < 0 || e < b || e > nnz) {
            bad = 1;
            b = e = 0;
        }
        if (e - b > kLongRow) longs.row[atomicAdd(&longs.n, 1)] = row;
    }
    int left = 0;                                     // searches put off, below 64
    auto search = [&](int at, bool in) {
        int v = 0, lo = 0, hi = 0;
        if (in) {
            v = find[0][at];
            lo = find[1][at];
            hi = find[2][at];
        }
        bool hit = !in;
        while (lo < hi) {                             // three probes a step: fewer loads in a chain
            const int len = hi - lo;
            const int p0 = lo + (len >> 2), p1 = lo + (len >> 1), p2 = p1 + (len >> 2);
            const int x0 = col[p0], x1 = col[p1], x2 = col[p2];
            hit |= x0 == v || x1 == v || x2 == v;
            hi = x0 >= v ? p0 : x1 >= v ? p1 : x2 >= v ? p2 : hi;
            lo = x2 < v ? p2 + 1 : x1 < v ? p1 + 1 : x0 < v ? p0 + 1 : lo;
            if (hit) break;
        }
        if (!hit) bad = 1;
    };
    // all lanes of the wavefront together
    auto check = [&](int v, int dv, int first, int j, bool in) {
        int lo = 0, hi = 0;
        bool down = false;
        if (in) {
            const int w = col[j];
            if (w < 0 || w >= n || w == v) {
                bad = 1;
            } else {
                if (j > first && col[j - 1] >= w) bad = 1;
                lo = row_ptr[w];
                hi = row_ptr[w + 1];
                lo = lo < 0 ? 0 : (lo > nnz ? nnz : lo);
                hi = hi < lo ? lo : (hi > nnz ? nnz : hi);
                const int dw = hi - lo;
                down = !(dw > dv || (dw == dv && w > v));
                up += down ? -1 : 1;
            }
        }
        const unsigned long long m = __ballot(down);
        if (down) {
            const int at = left + __popcll(m & lanemask_lt());
            find[0][at] = v;
            find[1][at] = lo;
            find[2][at] = hi;
        }
        left += __popcll(m);
        if (left >= 64) {
            wave_sync_lds();
            left -= 64;
            search(left + lane, true);
            wave_sync_lds();
        }
    };
    short_rows(b, e, per, lane, [&](int from, int first, int j, bool in) {
        check(__shfl(row, from), __shfl(e - b, from), first, j, in);
    });
    __syncthreads();
    for (int l = 0; l < longs.n; l++) {
        // 64 entries a wavefront; the next row starts eleven wavefronts on, as rows of this list may be short of 16 slices
        const int v = longs.row[l], first = row_ptr[v], last = row_ptr[v + 1];
        for (int j = first + 64 * (((threadIdx.x >> 6) + 11 * l) & 15); j < last; j += kRowBlock)
            check(v, last - first, first, j + lane, j + lane < last);
    }
    wave_sync_lds();
    search(lane, lane < left);
    up = wave_sum(up);
    if (lane == 0 && up) atomicAdd(&s_up, up);
    if (bad) s_bad = 1;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_up) atomicAdd(&ctl[CTL_UP], s_up);
        if (s_bad) atomicOr(&ctl[CTL_BAD], 1);
    }
}

// An invalid graph: nothing after the validation may follow its indices.  A peel that was
// given up: nothing after it may follow keys and ids that were not written.
__device__ __forceinline__ bool rejected(const int* ctl) {
    return ctl[CTL_BAD] != 0 || ctl[CTL_UP] != 0 || ctl[CTL_STALL] != 0;
}

// --------------------------------------------------------------- keys

// Largest value of a block into *out, one atomic per block (an atomic per wavefront
// on the one address took 181 us of a 1M-vertex degree pass).
__device__ __forceinline__ void block_max_to(int x, int* sh, int* out) {
    if (threadIdx.x == 0) *sh = 0;
    __syncthreads();
    x = wave_max(x);
    if ((threadIdx.x & 63) == 0 && x > 0) atomicMax(sh, x);
    __syncthreads();
    if (threadIdx.x == 0 && *sh > 0) atomicMax(out, *sh);
}

// key = degree, or with `voff` (batches) graph * key_span + degree, so that every
// graph's vertices stay together.
__global__ void __launch_bounds__(kBlock) k_degree_key(int n, const int* __restrict__ row_ptr, int* key, int* val,
                                                      int* ctl, const int* __restrict__ voff, int ngraphs,
                                                      int key_span) {
    __shared__ int sh;
    if (rejected(ctl)) return;
    int mx = 0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        int d = row_ptr[v + 1] - row_ptr[v];
        if (voff) {
            int lo = 0, hi = ngraphs;                        // voff[lo] <= v < voff[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (voff[mid] <= v) lo = mid; else hi = mid;
            }
            d += lo * key_span;
        }
        key[v] = d;
        val[v] = v;
        mx = d > mx ? d : mx;
    }
    block_max_to(mx, &sh, &ctl[CTL_MAXKEY]);
}

// --------------------------------------------------- degeneracy order (peeling)
//
// Level-synchronous peeling (the paper only states that its k-core decomposition
// runs on the GPU; this schedule is ours).  Level c starts when no live vertex has
// degree <= c - 1; its first frontier is every live vertex of degree <= c.  Each
// round removes the whole frontier (key = round) and decrements its neighbours; a
// neighbour whose degree falls from c + 1 to c joins the next frontier.  When a
// round leaves an empty frontier the next level is the minimum live degree.  A
// vertex removed in round r at level c had at most c live neighbours at the start of
// round r, and its out-neighbours under the (round, id) order are among them, so
// the out-degree is bounded by the degeneracy (the largest level).
//
// No liveness check is needed anywhere: degrees of removed vertices never exceed
// the level at which they left, so they never fall "from c + 1", and between
// levels the live vertices are exactly those of degree > c.
//
// The rounds are serial (1,941 of them on a 1M-vertex power-law graph of
// degeneracy 286) and bound by latency: a barrier and a chain of dependent accesses
// each.  All but the first few hundred of them happen when few vertices are left, so
// the work is split there: k_peel removes vertices with the whole device until at
// most kCoreCap are left, the rows among those are compacted to 16-bit local ids
// (k_core_list, k_core_rows), and k_core_peel finishes in one workgroup
// with the degrees and the queue in LDS, where a round costs a block barrier and
// one row read.  Measured on that graph (orientation without validation, us): 35,100
// with every round behind a cooperative-groups grid barrier, of which the barriers
// alone are 8.7 us each at 61 blocks (their fences write back and invalidate
// every L2).

constexpr int kPeelBlock = 1024;
constexpr int kCoreCap = 26000;   // 6 bytes of LDS each, of 160 KB
constexpr int kCoreFront = 96;
constexpr int kCoreSmall = 4000;  // up to here the one workgroup does all rounds
constexpr int kCoreLds = 6 * kCoreCap + 8;
constexpr int kPeelSpins = 1 << 22;       // polls of the first barrier: seconds
constexpr int kPeelLaterSpins = 1 << 26;  // of a later one: a minute, far more than a block's longest round

template <class T>
__device__ __forceinline__ void st_agent(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid barrier of a cooperative launch (all blocks co-resident) for data that
// blocks exchange only through agent-scope atomic loads, stores and updates: those
// are served past the XCDs' L2s, so it is enough that they have been performed
// (s_waitcnt) when the block arrives; no cache is written back or invalidated.
// 1.3 us at 64 blocks (cooperative groups: 8.7).  False once a wait ran out, after
// which every block leaves, and CTL_STALL says so; blocks look at it now and then while
// they wait.
__device__ __forceinline__ bool peel_barrier(int* ctl, unsigned int& epoch, int* shared_ok) {
    int* bar = ctl + CTL_BAR;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    epoch++;
    if (threadIdx.x == 0) {
        const unsigned int want = epoch * gridDim.x;
        __hip_atomic_fetch_add(bar, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int limit = epoch == 1 ? kPeelSpins : kPeelLaterSpins;
        int spins = 0;
        while (arrivals_missing(static_cast<unsigned int>(ld_acquire(bar)), want) && ++spins < limit) {
            __builtin_amdgcn_s_sleep(1);
            if ((spins & 1023) == 0 && ld_acquire(&ctl[CTL_STALL]) != 0) spins = limit - 1;
        }
        *shared_ok = spins < limit;
        if (spins >= limit) atomicOr(&ctl[CTL_STALL], epoch == 1 ? kStallStart : kStallLater);
    }
    __syncthreads();
    return *shared_ok != 0;
}

// The next frontier as one block gathers it: vertices go to an LDS buffer and reach
// the global list by one atomic per block and round (peel_flush).  An atomic per
// appending wavefront on the list's size bound the whole kernel: some 700,000 of
// them at 11.6 ns, 8.6 ms.  What the buffer cannot hold is appended directly.
constexpr int kPeelBuf = 16384;

struct PeelNext {
    int* list;    // global list and its size
    int* size;
    int* buf;     // LDS
    int* count;
};

__device__ __forceinline__ void peel_push(bool flag, int v, const PeelNext& nx, int lane) {
    const unsigned long long m = __ballot(flag);
    if (m == 0ull) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(nx.count, __popcll(m));
    at = __shfl(at, 0) + __popcll(m & lanemask_lt());
    if (flag && at < kPeelBuf) nx.buf[at] = v;
    if (flag && at >= kPeelBuf) st_agent(&nx.list[atomicAdd(nx.size, 1)], v);
}

// Moves the block's buffer to the global list and empties it; all threads call it.
__device__ __forceinline__ void peel_flush(const PeelNext& nx, int* base) {
    __syncthreads();
    const int cnt = *nx.count < kPeelBuf ? *nx.count : kPeelBuf;
    if (cnt == 0) return;
    if (threadIdx.x == 0) *base = atomicAdd(nx.size, cnt);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) st_agent(&nx.list[*base + i], nx.buf[i]);
    if (threadIdx.x == 0) *nx.count = 0;
}

constexpr int kPeelLongRow = 128;

// Row entries j, j + stride, ... below e lose one degree each; those that reach the
// level c join the next frontier.  The wavefront makes as many steps as its longest
// share: `span` entries of 0, or from `first` to e.  Four loads, then four updates,
// are in flight per lane.
__device__ __forceinline__ void peel_row(int j, int first, int e, int stride, int c, const int* __restrict__ col,
                                         int* deg, const PeelNext& nx, int lane, int span = -1) {
    const int len = span >= 0 ? span : e - first;
    for (int t = 0; t < len; t += 4 * stride, j += 4 * stride) {
        int w[4], old[4];
#pragma unroll
        for (int q = 0; q < 4; q++) w[q] = j + q * stride < e ? col[j + q * stride] : -1;
#pragma unroll
        for (int q = 0; q < 4; q++) old[q] = w[q] >= 0 ? atomicSub(&deg[w[q]], 1) : 0;
#pragma unroll
        for (int q = 0; q < 4; q++) peel_push(w[q] >= 0 && old[q] == c + 1, w[q], nx, lane);
    }
}

// The whole-device rounds: until at most `keep` vertices are left and frontiers are
// small (kCoreFront vertices on a running average).  Graphs without a skewed core peel
// in wide fronts to the end, which one compute unit is slow at: G(26000, 20 / n) takes
// 1,390 us with all of it in one workgroup.  A frontier of
// f vertices gets the nwaves / f wavefronts (at most 64) that there are for each,
// so that the hubs' long rows are shared while frontiers are small.  Leaves the
// level in CTL_LEVEL, the rounds so far in CTL_ROUNDS, the degrees of the vertices
// left (their live neighbours) in deg[], and key[v] = -1 for those.
__global__ void __launch_bounds__(kPeelBlock) k_peel(int n, int keep, const int* __restrict__ row_ptr,
                                                    const int* __restrict__ col, int* deg, int* key, int* fr0,
                                                    int* fr1, int* val, int* ctl) {
    __shared__ int ok, count, base, least;
    __shared__ int buf[kPeelBuf];
    const int tid = blockIdx.x * kPeelBlock + threadIdx.x;
    const int nth = gridDim.x * kPeelBlock;
    const int lane = threadIdx.x & 63;
    const int wave = tid >> 6;
    const int nwaves = nth >> 6;
    unsigned int epoch = 0;
    if (rejected(ctl)) return;

    for (int v = tid; v < n; v += nth) {
        st_agent(&deg[v], row_ptr[v + 1] - row_ptr[v]);
        st_agent(&key[v], -1);   // written again from another XCD: no copy may stay in this one's L2
        val[v] = v;
    }
    if (tid == 0) st_agent(&ctl[CTL_MIN], INT_MAX);
    if (threadIdx.x == 0) {
        count = 0;
        least = INT_MAX;
    }
    if (!peel_barrier(ctl, epoch, &ok)) return;

    int removed = 0, r = 0, c = -1, degen = 0;
    int recent = n;                                  // goes to 32 times the frontier size of late
    while (n - removed > keep || (recent > 32 * kCoreFront && removed < n)) {
        const int* cur = (r & 1) ? fr1 : fr0;
        const PeelNext nx{(r & 1) ? fr0 : fr1, &ctl[CTL_SIZE0 + (r + 1) % 3], buf, &count};
        const int fsize = ld_acquire(&ctl[CTL_SIZE0 + r % 3]);
        if (tid == 0) st_agent(&ctl[CTL_SIZE0 + (r + 2) % 3], 0);   // only the finished round r - 1 read it
        if (fsize == 0) {
            // Level change, as an empty round r: one pass takes the live vertices of
            // degree c + 1 and the minimum live degree; a second one runs only when
            // no live vertex has that degree.
            int mn = INT_MAX;
            for (int b0 = tid - lane; b0 < n; b0 += 4 * nth) {
                int d[4];
#pragma unroll
                for (int q = 0; q < 4; q++) d[q] = b0 + q * nth + lane < n ? ld_acquire(&deg[b0 + q * nth + lane]) : -1;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    if (d[q] > c) mn = d[q] < mn ? d[q] : mn;
                    peel_push(d[q] == c + 1, b0 + q * nth + lane, nx, lane);
                }
            }
            mn = wave_min(mn);
            if (lane == 0 && mn != INT_MAX) atomicMin(&least, mn);
            peel_flush(nx, &base);
            if (threadIdx.x == 0) {
                if (least != INT_MAX) atomicMin(&ctl[CTL_MIN], least);
                least = INT_MAX;
            }
            if (!peel_barrier(ctl, epoch, &ok)) return;
            const int old = c;
            c = ld_acquire(&ctl[CTL_MIN]);
            if (c != old + 1) {
                for (int b0 = tid - lane; b0 < n; b0 += nth) {
                    const int v = b0 + lane;
                    peel_push(v < n && ld_acquire(&deg[v]) == c, v, nx, lane);
                }
            }
            if (c != old + 1) peel_flush(nx, &base);
            if (!peel_barrier(ctl, epoch, &ok)) return;
            if (tid == 0) st_agent(&ctl[CTL_MIN], INT_MAX);   // every read of it is behind the last barrier
            degen = c > degen ? c : degen;
            r++;
            continue;
        }
        if (fsize <= nwaves) {
            int parts = nwaves / fsize;
            parts = parts > 64 ? 64 : parts;
            const int units = fsize * parts;
            for (int q = wave; q < units; q += nwaves) {
                const int part = q / fsize;
                const int v = ld_acquire(&cur[q - part * fsize]);
                if (part == 0 && lane == 0) st_agent(&key[v], r);
                const int b = row_ptr[v], e = row_ptr[v + 1];
                peel_row(b + part * 64 + lane, b + part * 64, e, parts * 64, c, col, deg, nx, lane);
            }
        } else {
            // more vertices than wavefronts: a wavefront takes up to 64 at a time (their
            // row bounds in one load each) and walks eight short rows at once, eight
            // lanes each; rows beyond kPeelLongRow entries then get all its lanes
            int per = (fsize + nwaves - 1) / nwaves;
            per = per > 64 ? 64 : (per + 7) & ~7;
            for (int f0 = wave * per; f0 < fsize; f0 += nwaves * per) {
                int v = 0, b = 0, e = 0;
                if (lane < per && f0 + lane < fsize) {
                    v = ld_acquire(&cur[f0 + lane]);
                    st_agent(&key[v], r);
                    b = row_ptr[v];
                    e = row_ptr[v + 1];
                }
                const bool is_long = e - b > kPeelLongRow;
                const unsigned long long longs = __ballot(is_long);
                for (int g = 0; g < per; g += 8) {
                    const int from = g + (lane >> 3);
                    const int gb = __shfl(b, from), ge = __shfl(is_long ? b : e, from);
                    const int len = wave_max(ge - gb);
                    peel_row(gb + (lane & 7), 0, ge, 8, c, col, deg, nx, lane, len);
                }
                for (unsigned long long m = longs; m; m &= m - 1ull) {
                    const int from = __ffsll(static_cast<long long>(m)) - 1;
                    const int gb = __shfl(b, from), ge = __shfl(e, from);
                    peel_row(gb + lane, gb, ge, 64, c, col, deg, nx, lane);
                }
            }
        }
        peel_flush(nx, &base);
        removed += fsize;
        recent += fsize - recent / 32;
        r++;
        if (!peel_barrier(ctl, epoch, &ok)) return;
    }
    if (tid == 0) {
        ctl[CTL_DEGEN] = degen;
        ctl[CTL_LEVEL] = c;
        ctl[CTL_ROUNDS] = r;
        ctl[CTL_MAXKEY] = r > 0 ? r - 1 : 0;
    }
}

// Graphs of at most kCoreSmall vertices start in the one-workgroup peel.
__global__ void __launch_bounds__(kBlock) k_peel_init(int n, const int* __restrict__ row_ptr, int* deg, int* key,
                                                     int* val, int* ctl) {
    if (rejected(ctl)) return;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        deg[v] = row_ptr[v + 1] - row_ptr[v];
        key[v] = -1;
        val[v] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl[CTL_LEVEL] = -1;
}

// Local ids of the vertices left (cid[v], -1 for the others; list[id] = v) and
// where their rows start among the compacted ones.  Ids and rows are handed out
// block by block in any order: only the queue's order depends on it, and the keys
// do not.  span[id] = {start, live degree}.  Both are read eight bytes at a time, but as
// pairs of words: a caller's workspace need only be aligned to words.
struct CoreSpan {
    int at, degree;
};
struct CoreIds {
    unsigned int ab, cd;   // four 16-bit ids
};

__global__ void __launch_bounds__(kPeelBlock) k_core_list(int n, const int* __restrict__ key,
                                                         const int* __restrict__ deg, int* cid, int* list, CoreSpan* span,
                                                         int* ctl) {
    __shared__ int cnt[kPeelBlock / 64], sum[kPeelBlock / 64];
    __shared__ int base_id, base_at;
    if (rejected(ctl)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int v = blockIdx.x * kPeelBlock + threadIdx.x;
    const bool live = v < n && key[v] < 0;
    const int d = live && deg[v] > 0 ? deg[v] : 0;
    const int room = (d + 3) & ~3;               // four ids a load
    const unsigned long long m = __ballot(live);
    int inc = room;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    if (lane == 63) {
        cnt[w] = __popcll(m);
        sum[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0, at = 0;
        for (int i = 0; i < kPeelBlock / 64; i++) {
            const int t = cnt[i], u = sum[i];
            cnt[i] = run;
            sum[i] = at;
            run += t;
            at += u;
        }
        base_id = run ? atomicAdd(&ctl[CTL_CORE], run) : 0;
        base_at = at ? atomicAdd(&ctl[CTL_CORE_AT], at) : 0;
    }
    __syncthreads();
    int id = -1;
    if (live) {
        id = base_id + cnt[w] + __popcll(m & lanemask_lt());
        if (id < kCoreCap) {
            list[id] = v;
            span[id] = CoreSpan{base_at + sum[w] + inc - room, d};
        } else {
            id = -1;
        }
    }
    if (v < n) cid[v] = id;
}

// One wavefront per vertex left: its neighbours among those left, as local ids,
// filled up to a multiple of four with the id kCoreCap, which stands for no vertex.
__global__ void __launch_bounds__(kBlock) k_core_rows(const int* __restrict__ row_ptr,
                                                     const int* __restrict__ col, const int* __restrict__ cid,
                                                     const int* __restrict__ list, const CoreSpan* __restrict__ span,
                                                     unsigned short* rows, const int* ctl) {
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * blockDim.x) >> 6;
    const int L = ctl[CTL_CORE] < kCoreCap ? ctl[CTL_CORE] : kCoreCap;
    for (int i = wave; i < L; i += nwaves) {
        const int v = list[i];
        const int b = row_ptr[v], e = row_ptr[v + 1];
        int pos = span[i].at;
        const int end = pos + ((span[i].degree + 3) & ~3);
        for (int j0 = b; j0 < e; j0 += 256) {
            int x[4], id[4];
#pragma unroll
            for (int q = 0; q < 4; q++) x[q] = j0 + 64 * q + lane < e ? col[j0 + 64 * q + lane] : -1;
#pragma unroll
            for (int q = 0; q < 4; q++) id[q] = x[q] >= 0 ? cid[x[q]] : -1;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const unsigned long long m = __ballot(id[q] >= 0);
                const int at = pos + __popcll(m & lanemask_lt());
                if (id[q] >= 0 && at < end) rows[at] = static_cast<unsigned short>(id[q]);
                pos += __popcll(m);
            }
        }
        // at most three slots on a symmetric graph; one that lacks reverse entries (and was not
        // validated) can leave any number of them without a neighbour
        for (int at = pos + lane; at < end; at += 64) rows[at] = static_cast<unsigned short>(kCoreCap);
    }
}

// The remaining rounds by one workgroup: degrees and the queue (every vertex once, in
// order of removal; a round is the segment [head, tail)) are in LDS.  A round has some
// 28 rows of 300 entries; its latency and the conflicts of its atomics bound it (2.6 ms on
// the 1M-vertex graph: wavefronts wait on 76% of their cycles, 91% of the LDS cycles
// are conflicts, 0.28 vector instructions issued per cycle).  Degrees are whole words and rows
// are padded: an entry costs about five instructions instead of 14 with 16-bit degrees, bounds
// tests and an early exit each (which took 5.7 ms although they held half as many vertices
// again).
__global__ void __launch_bounds__(kPeelBlock) k_core_peel(const CoreSpan* __restrict__ span,
                                                         const unsigned short* __restrict__ rows,
                                                         const int* __restrict__ list, int* round_of, int* key,
                                                         int* ctl) {
    extern __shared__ int core_lds[];
    __shared__ int s_tail, s_min;
    int* deg = core_lds;                                                       // kCoreCap + 1
    unsigned short* queue = reinterpret_cast<unsigned short*>(core_lds + kCoreCap + 1);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int NW = kPeelBlock / 64;
    const int L = ctl[CTL_CORE] < kCoreCap ? ctl[CTL_CORE] : kCoreCap;
    for (int i = t; i < L; i += kPeelBlock) deg[i] = span[i].degree;
    int c = ctl[CTL_LEVEL], r = ctl[CTL_ROUNDS], degen = ctl[CTL_DEGEN];
    if (t == 0) {
        deg[kCoreCap] = INT_MAX;   // the padding: never falls to a level
        s_tail = 0;
        s_min = INT_MAX;
    }
    __syncthreads();
    // every vertex is queued once: its degree falls to the level once, and starts a level
    // at it once.  The bound costs nothing and does not rest on that.
    auto push = [&](int v) {
        const int at = atomicAdd(&s_tail, 1);
        if (at < kCoreCap) queue[at] = static_cast<unsigned short>(v);
    };
    auto queued = [&] { return s_tail < L ? s_tail : L; };
    // appends the vertices of degree d: lo < d <= hi; returns this thread's minimum degree above hi
    auto collect = [&](int lo, int hi) {
        int mn = INT_MAX;
        for (int v = t; v < L; v += kPeelBlock) {
            const int d = deg[v];
            if (d > hi) mn = d < mn ? d : mn;
            else if (d > lo) push(v);
        }
        return mn;
    };
    // four neighbours lose one degree each
    auto update = [&](const CoreIds& x) {
        const int i0 = x.ab & 0xffffu, i1 = x.ab >> 16, i2 = x.cd & 0xffffu, i3 = x.cd >> 16;
        const int o0 = atomicSub(&deg[i0], 1), o1 = atomicSub(&deg[i1], 1);
        const int o2 = atomicSub(&deg[i2], 1), o3 = atomicSub(&deg[i3], 1);
        if (o0 == c + 1 || o1 == c + 1 || o2 == c + 1 || o3 == c + 1) {
            if (o0 == c + 1) push(i0);
            if (o1 == c + 1) push(i1);
            if (o2 == c + 1) push(i2);
            if (o3 == c + 1) push(i3);
        }
    };
    // the frontier that the whole-device rounds left behind (none at a level change)
    collect(-1, c);
    __syncthreads();
    int head = 0, tail = queued();
    __syncthreads();
    while (head < L) {
        if (head == tail) {
            // the next level is almost always c + 1; otherwise the smallest live degree
            const int mn = wave_min(collect(c, c + 1));
            if (lane == 0 && mn != INT_MAX) atomicMin(&s_min, mn);
            __syncthreads();
            const bool found = queued() > head;
            const int next = found ? c + 1 : s_min;
            __syncthreads();   // the second pass appends: every thread has read the tail by now
            if (!found) collect(c, next);
            c = next;
            __syncthreads();
            degen = c > degen ? c : degen;
            tail = queued();
            __syncthreads();
            if (t == 0) s_min = INT_MAX;
            if (tail == head) break;   // cannot happen: a live vertex has the minimum degree
            r++;
            continue;
        }
        for (int i = head + t; i < tail; i += kPeelBlock) round_of[i] = r;
        for (int i = head + wave; i < tail; i += NW) {
            const CoreSpan sp = span[queue[i]];
            const int b = __builtin_amdgcn_readfirstlane(sp.at);
            const int e = b + ((__builtin_amdgcn_readfirstlane(sp.degree) + 3) & ~3);
            for (int j0 = b; j0 < e; j0 += 512) {
                const int j = j0 + 4 * lane;
                const bool two = j0 + 256 < e;
                CoreIds x0{}, x1{};
                if (j < e) x0 = *reinterpret_cast<const CoreIds*>(rows + j);
                if (two && j + 256 < e) x1 = *reinterpret_cast<const CoreIds*>(rows + j + 256);
                if (j < e) update(x0);
                if (two && j + 256 < e) update(x1);
            }
        }
        __syncthreads();
        head = tail;
        tail = queued();
        r++;
        __syncthreads();
    }
    for (int i = t; i < tail; i += kPeelBlock) key[list[queue[i]]] = round_of[i];
    if (t == 0) {
        ctl[CTL_DEGEN] = degen;
        ctl[CTL_ROUNDS] = r;
        ctl[CTL_MAXKEY] = r > 0 ? r - 1 : 0;
    }
}

// ------------------------------------------------------- block-level scan

// Exclusive scan of one int per thread across the block; returns the block total
// through *total.  All threads of the block must call it.
__device__ int block_exclusive_scan(int x, int* total, int* sh /* >= kBlock/64 + 1 */) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int i = 0; i < kBlock / 64; i++) {
            int t = sh[i];
            sh[i] = run;
            run += t;
        }
        sh[kBlock / 64] = run;
    }
    __syncthreads();
    int res = inc - x + sh[w];
    *total = sh[kBlock / 64];
    __syncthreads();
    return res;
}

// ------------------------------------------- approximate degeneracy order

// A relaxation of k-core peeling (an orientation criterion named in Sec. 2;
// the approximate peeling of ARB-COUNT with eps = 1/10): in rounds r = 0, 1,
// ..., with L vertices left of total current degree D, every remaining vertex
// of degree at most 1.1 D / L (10 deg L <= 11 D, exact in integers) leaves in
// round r; afterwards its remaining neighbours lose one degree each.  The round
// is the sort key, ties by id.  Rounds end when no vertex is left (each removes
// at least one: the smallest degree is at most the average, unless missing reverse
// entries have made the average negative).

__global__ void __launch_bounds__(kBlock) k_ad_init(int n, const int* __restrict__ row_ptr, int* deg, int* rnd,
                                                   int* val) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        deg[v] = row_ptr[v + 1] - row_ptr[v];
        rnd[v] = -1;
        val[v] = v;
    }
}

// L and D of the vertices still present.
__global__ void __launch_bounds__(kBlock) k_ad_sum(int n, const int* __restrict__ deg, const int* __restrict__ rnd,
                                                  int* ctl) {
    const int lane = threadIdx.x & 63;
    int live = 0;
    unsigned long long dsum = 0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        if (rnd[v] < 0) {
            live++;
            dsum += static_cast<unsigned long long>(deg[v]);
        }
    }
    live = wave_sum(live);
    dsum = wave_sum(dsum);
    if (lane == 0 && live) {
        atomicAdd(&ctl[CTL_AD_LIVE], live);
        atomicAdd(reinterpret_cast<unsigned long long*>(ctl + CTL_AD_SUM), dsum);
    }
}

__global__ void __launch_bounds__(kBlock) k_ad_mark(int n, int r, const int* __restrict__ deg, int* rnd,
                                                   const int* __restrict__ ctl) {
    const long long L = ctl[CTL_AD_LIVE];
    const long long D = static_cast<long long>(*reinterpret_cast<const unsigned long long*>(ctl + CTL_AD_SUM));
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
        if (rnd[v] < 0 && 10 * static_cast<long long>(deg[v]) * L <= 11 * D) rnd[v] = r;
}

// One wavefront per vertex that left in round r: its remaining neighbours lose
// one degree each.
__global__ void __launch_bounds__(kBlock) k_ad_dec(int n, int r, const int* __restrict__ row_ptr,
                                                  const int* __restrict__ col, int* deg,
                                                  const int* __restrict__ rnd) {
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * blockDim.x) >> 6;
    for (int v = wave; v < n; v += nwaves) {
        if (rnd[v] != r) continue;
        for (int j = row_ptr[v] + lane; j < row_ptr[v + 1]; j += 64) {
            const int w = col[j];
            if (rnd[w] < 0) atomicSub(&deg[w], 1);
        }
    }
}

// ---------------------------------------------------------- colouring order

// Graph colouring as an orientation criterion (Sec. 2 names it): vertices get
// the greedy first-fit colour in decreasing order of a pseudo-random priority
// (SplitMix64's output for the vertex id; the output function is a bijection, so
// priorities never tie), and the order is (colour, id); adjacent vertices differ
// in colour, so every edge goes from its lower colour to its higher one.
//
// The sequential greedy colouring is reproduced in Jones-Plassmann rounds kept
// as a countdown: hp[v] counts v's neighbours of higher priority that are not
// coloured yet, a vertex is coloured in the round after its count reaches zero
// (the first round for counts that start at zero), and then decrements its
// lower-priority neighbours.  Each vertex's colour depends only on its
// higher-priority neighbours, all coloured in earlier rounds, so the result is
// the greedy one and the total work is O(m) over however many rounds (the
// longest decreasing-priority path: 943 on the 1M-vertex power-law graph).

__device__ __forceinline__ unsigned long long colour_priority(int v) {
    unsigned long long z = static_cast<unsigned long long>(v) + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Frontiers are split by degree: a light vertex (degree <= kClHeavy) is coloured
// by one wavefront, a heavy one by a whole block, because the rounds are serial
// and almost every one of them holds a hub of thousands of neighbours.
constexpr int kClHeavy = 512;

struct ClFront {
    int* light;        // this round's light vertices
    int* heavy;        // and heavy ones
    int* next_light;   // the next round's
    int* next_heavy;
};

__device__ __forceinline__ void cl_append(int u, const int* row_ptr, const ClFront& f, int* ctl, int r) {
    if (row_ptr[u + 1] - row_ptr[u] > kClHeavy)
        f.next_heavy[atomicAdd(&ctl[CTL_CL_HSIZE0 + (r + 1) % 3], 1)] = u;
    else
        f.next_light[atomicAdd(&ctl[CTL_CL_SIZE0 + (r + 1) % 3], 1)] = u;
}

// One wavefront per vertex: hp[v] = higher-priority neighbours; the vertices
// with none form round 0's frontier (sizes in ring slot 0).
__global__ void __launch_bounds__(kBlock) k_cl_init(int n, const int* __restrict__ row_ptr,
                                                   const int* __restrict__ col, int* hp, int* val, ClFront f,
                                                   int* ctl) {
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * blockDim.x) >> 6;
    for (int v = wave; v < n; v += nwaves) {
        const unsigned long long pv = colour_priority(v);
        int c = 0;
        for (int j = row_ptr[v] + lane; j < row_ptr[v + 1]; j += 64)
            c += colour_priority(col[j]) > pv;
        c = wave_sum(c);
        if (lane == 0) {
            hp[v] = c;
            val[v] = v;
            if (c == 0) cl_append(v, row_ptr, f, ctl, -1);
        }
    }
}

// Colour v with the T threads of a wavefront (T = 64, sync = wave_sync_lds) or a
// block (T = kBlock, sync = __syncthreads), t = the thread's index among them:
// first fit over the colours of v's higher-priority neighbours in windows of
// 1024 (an LDS bitmap; every wavefront reads the whole bitmap, so all of them
// find the same colour), then count down the lower-priority neighbours.  The
// neighbour loops keep four loads in flight per thread.
template <int T, typename Sync>
__device__ __forceinline__ int cl_colour_vertex(int v, int t, unsigned int* used, const int* __restrict__ row_ptr,
                                                const int* __restrict__ col, int* hp, int* colour, const ClFront& f,
                                                int* ctl, int r, Sync sync) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63;
    const unsigned long long pv = colour_priority(v);
    const int b = row_ptr[v], e = row_ptr[v + 1];
    int c = -1;
    for (int base = 0; c < 0; base += 1024) {
        if (t < 32) used[t] = 0u;
        sync();
        for (int j0 = b + t; j0 < e; j0 += U * T) {
            int u[U];
#pragma unroll
            for (int q = 0; q < U; q++) u[q] = j0 + q * T < e ? col[j0 + q * T] : -1;
            int cu[U];
#pragma unroll
            for (int q = 0; q < U; q++) cu[q] = u[q] >= 0 && colour_priority(u[q]) > pv ? colour[u[q]] - base : -1;
#pragma unroll
            for (int q = 0; q < U; q++)
                if (cu[q] >= 0 && cu[q] < 1024) atomicOr(&used[cu[q] >> 5], 1u << (cu[q] & 31));
        }
        sync();
        const unsigned int free_bits = lane < 32 ? ~used[lane] : 0u;
        const unsigned long long m = __ballot(free_bits != 0u);
        if (m) {
            const int w = __ffsll(static_cast<long long>(m)) - 1;
            const unsigned int fw =
                static_cast<unsigned int>(__builtin_amdgcn_readlane(static_cast<int>(free_bits), w));
            c = base + 32 * w + __ffs(static_cast<int>(fw)) - 1;
        }
        sync();
    }
    if (t == 0) colour[v] = c;
    for (int j0 = b + t; j0 < e; j0 += U * T) {
        int u[U];
#pragma unroll
        for (int q = 0; q < U; q++) u[q] = j0 + q * T < e ? col[j0 + q * T] : -1;
        bool z[U];
#pragma unroll
        for (int q = 0; q < U; q++) z[q] = u[q] >= 0 && colour_priority(u[q]) < pv && atomicSub(&hp[u[q]], 1) == 1;
#pragma unroll
        for (int q = 0; q < U; q++)
            if (z[q]) cl_append(u[q], row_ptr, f, ctl, r);
    }
    return c;
}

// Round r: colour this round's frontier and build the next one.  Sizes live in
// rings of three slots (light: CTL_CL_SIZE0, heavy: CTL_CL_HSIZE0): this round
// reads slot r % 3, appends to slot (r + 1) % 3 (cleared by round r - 1) and
// clears slot (r + 2) % 3, which only the finished round r - 1 read.  A fixed
// grid strides over the frontier (blocks over the heavy list, then wavefronts
// over the light one), so the host launches rounds without reading sizes back.
__global__ void __launch_bounds__(kBlock) k_cl_round(int r, ClFront f, const int* __restrict__ row_ptr,
                                                    const int* __restrict__ col, int* hp, int* colour, int* ctl) {
    __shared__ unsigned int used_all[kBlock / 64][32];
    const int lane = threadIdx.x & 63;
    const int count = ctl[CTL_CL_SIZE0 + r % 3];
    const int hcount = ctl[CTL_CL_HSIZE0 + r % 3];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl[CTL_CL_SIZE0 + (r + 2) % 3] = ctl[CTL_CL_HSIZE0 + (r + 2) % 3] = 0;
        if (count + hcount > 0) atomicMax(&ctl[CTL_ROUNDS], r + 1);
    }
    int mx = 0;
    for (int h = blockIdx.x; h < hcount; h += gridDim.x) {
        const int c = cl_colour_vertex<kBlock>(f.heavy[h], threadIdx.x, used_all[0], row_ptr, col, hp, colour, f,
                                               ctl, r, [] { __syncthreads(); });
        mx = c > mx ? c : mx;
    }
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * blockDim.x) >> 6;
    for (int i = wave; i < count; i += nwaves) {
        const int c = cl_colour_vertex<64>(f.light[i], lane, used_all[threadIdx.x >> 6], row_ptr, col, hp, colour, f,
                                           ctl, r, [] { wave_sync_lds(); });
        mx = c > mx ? c : mx;
    }
    if (lane == 0 && mx > 0) atomicMax(&ctl[CTL_MAXKEY], mx);
}

// --------------------------------------------------------- exclusive scan

// Exclusive scan of a non-negative array, out[count] = total, and its maximum into
// *top; arrays of up to kScanOne entries by one block, others in three passes.
constexpr int kScanOne = 8192;

__global__ void __launch_bounds__(1024) k_scan_one(int count, const int* __restrict__ in, int* out, int* top,
                                                  int* ctl) {
    __shared__ int sums[16], s_top;
    if (rejected(ctl)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int per = (count + 1023) / 1024, b = threadIdx.x * per;
    int v[kScanOne / 1024];
    int s = 0, mx = 0;
#pragma unroll
    for (int i = 0; i < kScanOne / 1024; i++) {
        v[i] = i < per && b + i < count ? in[b + i] : 0;
        s += v[i];
        mx = v[i] > mx ? v[i] : mx;
    }
    int inc = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    if (lane == 63) sums[w] = inc;
    block_max_to(mx, &s_top, top);
    int run = inc - s;
    for (int i = 0; i < w; i++) run += sums[i];
#pragma unroll
    for (int i = 0; i < kScanOne / 1024; i++) {
        if (i < per && b + i < count) out[b + i] = run;
        run += v[i];
    }
    if (threadIdx.x == 1023) {
        out[count] = run;
        ctl[CTL_TOTAL] = run;
    }
}

// Pass 1: per-tile sums, and the maximum.
__global__ void __launch_bounds__(kBlock) k_tile_sum(int count, const int* __restrict__ in, int* tile_sum, int* top,
                                                    const int* ctl) {
    __shared__ int sh[kBlock / 64 + 1], s_top;
    if (rejected(ctl)) return;
    const int base = blockIdx.x * kTile + threadIdx.x * kItems;
    int s = 0, mx = 0;
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const int x = base + i < count ? in[base + i] : 0;
        s += x;
        mx = x > mx ? x : mx;
    }
    int tot;
    block_exclusive_scan(s, &tot, sh);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
    block_max_to(mx, &s_top, top);
}

// Pass 2: exclusive scan of the tile sums by one block; the total to CTL_TOTAL.
__global__ void __launch_bounds__(kBlock) k_scan_tiles(int ntiles, int* tile_sum, int* ctl) {
    __shared__ int sh[kBlock / 64 + 1];
    if (rejected(ctl)) return;
    int carry = 0;
    for (int base = 0; base < ntiles; base += kBlock) {
        int idx = base + threadIdx.x;
        int x = idx < ntiles ? tile_sum[idx] : 0;
        int tot;
        int ex = block_exclusive_scan(x, &tot, sh);
        if (idx < ntiles) tile_sum[idx] = ex + carry;
        carry += tot;
    }
    if (threadIdx.x == 0) ctl[CTL_TOTAL] = carry;
}

// Pass 3: out[i] = exclusive prefix of in[]; out[count] = total.
__global__ void __launch_bounds__(kBlock) k_scan_apply(int count, const int* __restrict__ in,
                                                      const int* __restrict__ tile_off, int* out, const int* ctl) {
    __shared__ int sh[kBlock / 64 + 1];
    if (rejected(ctl)) return;
    const int base = blockIdx.x * kTile + threadIdx.x * kItems;
    int v[kItems];
    int s = 0;
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        int idx = base + i;
        v[i] = idx < count ? in[idx] : 0;
        s += v[i];
    }
    int tot;
    int run = block_exclusive_scan(s, &tot, sh) + tile_off[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        int idx = base + i;
        if (idx < count) out[idx] = run;
        run += v[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[count] = ctl[CTL_TOTAL];
}

// Stable LSD radix sort of (key, id), eight bits a pass over tiles of 2048 entries:
// per-tile digit counts, a scan of each digit's counts over the tiles, and a
// scatter in which every wavefront ranks 512 consecutive entries by matching
// digits with eight ballots.  A pass whose digit is zero in every key (they are known
// on the device only) does nothing, so the sorted data is in buffer A after an even
// number of working passes and in B after an odd one (radix_passes).  One bit a pass,
// as before, took 36 launches and 240 us for 1M vertices of degree < 2^12, and 24
// launches and 70 us for 2,000 vertices.
__device__ __forceinline__ int radix_passes(const int* ctl) {
    const unsigned int mk = static_cast<unsigned int>(ctl[CTL_MAXKEY]);
    return mk == 0u ? 0 : (39 - __clz(static_cast<int>(mk))) >> 3;
}

struct RadixBuf {
    int *key_a, *val_a, *key_b, *val_b;
};

__global__ void __launch_bounds__(kBlock) k_radix_hist(int count, int pass, RadixBuf rb, int* hist, const int* ctl) {
    __shared__ int cnt[256];
    if (rejected(ctl) || pass >= radix_passes(ctl)) return;
    const int* key = (pass & 1) ? rb.key_b : rb.key_a;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * kTile;
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const int idx = base + i * kBlock + threadIdx.x;
        if (idx < count) atomicAdd(&cnt[(static_cast<unsigned int>(key[idx]) >> (8 * pass)) & 255u], 1);
    }
    __syncthreads();
    hist[threadIdx.x * gridDim.x + blockIdx.x] = cnt[threadIdx.x];
}

// Block d: exclusive scan of digit d's counts over the tiles; its total to dtot[d].
__global__ void __launch_bounds__(kBlock) k_radix_scan(int ntiles, int pass, int* hist, int* dtot, const int* ctl) {
    __shared__ int sh[kBlock / 64 + 1];
    if (rejected(ctl) || pass >= radix_passes(ctl)) return;
    int* h = hist + blockIdx.x * ntiles;
    int carry = 0;
    for (int base = 0; base < ntiles; base += kBlock) {
        const int idx = base + threadIdx.x;
        const int x = idx < ntiles ? h[idx] : 0;
        int tot;
        const int ex = block_exclusive_scan(x, &tot, sh);
        if (idx < ntiles) h[idx] = ex + carry;
        carry += tot;
    }
    if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

__global__ void __launch_bounds__(kBlock) k_radix_scatter(int count, int pass, RadixBuf rb, const int* __restrict__ hist,
                                                         const int* __restrict__ dtot, const int* ctl) {
    constexpr int NW = kBlock / 64;
    __shared__ int sh[NW + 1];
    __shared__ int at[NW][256];
    if (rejected(ctl) || pass >= radix_passes(ctl)) return;
    const int* kin = (pass & 1) ? rb.key_b : rb.key_a;
    const int* vin = (pass & 1) ? rb.val_b : rb.val_a;
    int* kout = (pass & 1) ? rb.key_a : rb.key_b;
    int* vout = (pass & 1) ? rb.val_a : rb.val_b;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < NW * 256; i += kBlock) at[i >> 8][i & 255] = 0;
    __syncthreads();
    const int base = blockIdx.x * kTile + w * (kTile / NW);
    int key[kItems], rank[kItems];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const int idx = base + i * 64 + lane;
        key[i] = idx < count ? kin[idx] : 0;
    }
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const bool in = base + i * 64 + lane < count;
        const unsigned int d = (static_cast<unsigned int>(key[i]) >> (8 * pass)) & 255u;
        unsigned long long same = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 8; bit++) {
            const unsigned long long m = __ballot((d >> bit) & 1u);
            same &= ((d >> bit) & 1u) ? m : ~m;
        }
        const int before = __popcll(same & lanemask_lt());
        const int seen = at[w][d];
        rank[i] = seen + before;
        wave_sync_lds();
        if (in && before == 0) at[w][d] = seen + __popcll(same);
        wave_sync_lds();
    }
    __syncthreads();
    // digit threadIdx.x: where this tile's entries of it start, wavefront by wavefront
    int tot;
    int run = block_exclusive_scan(dtot[threadIdx.x], &tot, sh) + hist[threadIdx.x * gridDim.x + blockIdx.x];
#pragma unroll
    for (int i = 0; i < NW; i++) {
        const int x = at[i][threadIdx.x];
        at[i][threadIdx.x] = run;
        run += x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const int idx = base + i * 64 + lane;
        if (idx < count) {
            const int pos = at[w][(static_cast<unsigned int>(key[i]) >> (8 * pass)) & 255u] + rank[i];
            kout[pos] = key[i];
            vout[pos] = vin[idx];
        }
    }
}

// --------------------------------------------------------- filter, compact

// perm = the sorted ids, rank = its inverse.  `passes` were launched: fewer than the largest
// key has digits where the caller's bound on the degrees is too low, and then that many ran.
__global__ void __launch_bounds__(kBlock) k_rank(int n, int passes, RadixBuf rb, int* perm, int* rank, const int* ctl) {
    if (rejected(ctl)) return;
    const int ran = radix_passes(ctl) < passes ? radix_passes(ctl) : passes;
    const int* val = (ran & 1) ? rb.val_b : rb.val_a;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int v = val[i];
        perm[i] = v;
        rank[v] = i;
    }
}

// Out-degree of new vertex i: neighbours of perm[i] with a larger new id.
__global__ void __launch_bounds__(kRowBlock) k_outdeg(int n, int per, int run, const int* __restrict__ row_ptr,
                                                     const int* __restrict__ col, const int* __restrict__ perm,
                                                     const int* __restrict__ rank, int* outdeg, const int* ctl) {
    __shared__ int cnt_all[kRowBlock / 64][64];
    __shared__ LongRows longs;
    if (rejected(ctl)) return;
    const int lane = threadIdx.x & 63;
    int* cnt = cnt_all[threadIdx.x >> 6];
    if (threadIdx.x == 0) longs.n = 0;
    __syncthreads();
    const int i = block_row(n, per, run);
    int b = 0, e = 0;
    if (i >= 0) {
        const int v = perm[i];
        b = row_ptr[v];
        e = row_ptr[v + 1];
        if (e - b > kLongRow) longs.row[atomicAdd(&longs.n, 1)] = i;
    }
    const int len = e - b > kLongRow ? 0 : e - b;
    for (int q = 0; 4 * q < per; q++) {
        const int from = 4 * q + (lane >> 4);
        const int gb = __shfl(b, from) + (lane & 15), row = __shfl(i, from), span = wave_max(__shfl(len, from));
        const int ge = gb - (lane & 15) + __shfl(len, from);
        int c = 0;
        for (int t = 0; t < span; t += 64) {
            int r[4];
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = gb + t + 16 * u < ge ? col[gb + t + 16 * u] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = r[u] >= 0 ? rank[r[u]] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) c += r[u] > row;
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
        if ((lane & 15) == 0) cnt[from] = c;
    }
    wave_sync_lds();
    if (i >= 0 && e - b <= kLongRow) outdeg[i] = cnt[lane];
    __syncthreads();
    for (int l = threadIdx.x >> 6; l < longs.n; l += kRowBlock / 64) {
        const int row = longs.row[l], v = perm[row];
        const int first = row_ptr[v], last = row_ptr[v + 1];
        if (last - first > kBlockRow) continue;
        int c = 0;
        for (int j0 = first; j0 < last; j0 += 256) {
            int r[4];
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = j0 + 64 * u + lane < last ? col[j0 + 64 * u + lane] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = r[u] >= 0 ? rank[r[u]] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) c += r[u] > row;
        }
        c = wave_sum(c);
        if (lane == 0) outdeg[row] = c;
    }
    for (int l = 0; l < longs.n; l++) {
        const int row = longs.row[l], v = perm[row];
        const int last = row_ptr[v + 1];
        if (last - row_ptr[v] <= kBlockRow) continue;
        if (threadIdx.x == 0) cnt_all[0][0] = 0;
        __syncthreads();
        int c = 0;
        for (int j = row_ptr[v] + threadIdx.x; j < last; j += kRowBlock) c += rank[col[j]] > row;
        c = wave_sum(c);
        if (lane == 0 && c) atomicAdd(&cnt_all[0][0], c);
        __syncthreads();
        if (threadIdx.x == 0) outdeg[row] = cnt_all[0][0];
        __syncthreads();
    }
}

// Gathers row i's kept neighbours (as new ids) into LDS, then places each at its
// rank within the row (count of smaller entries): col[] rows come out sorted.  Rows
// of up to kLongRow neighbours of which at most kGroupRow are kept are handled by 16
// lanes, those of up to kBlockRow of which at most kWaveRow are kept by a wavefront, the
// others by the whole block.  Rows of more than kRowCap kept neighbours
// go to tmp[] unsorted and are finished by k_sort_long_rows.  Bound by the gathers of ranks.
// Nothing is written when the rows hold more than `room` entries, which happens only on a
// graph that lacks reverse entries (and was not validated).
constexpr int kGroupRow = 64;
constexpr int kWaveRow = 4 * (kGroupRow + 16) - 4;   // the buffers of a wavefront's four groups, less the filling

__global__ void __launch_bounds__(kRowBlock) k_fill(int n, int per, int run, const int* __restrict__ row_ptr,
                                                   const int* __restrict__ col, const int* __restrict__ perm,
                                                   const int* __restrict__ rank,
                                                   const int* __restrict__ dag_ptr, int* dag_col, int* dag_src,
                                                   int* tmp, int room, int* ctl) {
    // a group's rows lie 16 words further apart than they are long, so that the four
    // broadcasts of a step use different banks
    __shared__ __align__(16) int groups[kRowBlock / 16][kGroupRow + 16];
    __shared__ __align__(16) int big_row[kRowCap + 4];
    __shared__ LongRows longs;
    __shared__ int s_pos;
    if (rejected(ctl) || ctl[CTL_TOTAL] > room) return;
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, gl = lane & 15;
    int* grow = groups[threadIdx.x >> 4];
    const unsigned int glt = (1u << gl) - 1u;
    if (threadIdx.x == 0) longs.n = 0;
    __syncthreads();
    const int row = block_row(n, per, run);
    int at = 0, len = 0, b = 0, e = 0;
    if (row >= 0) {
        at = dag_ptr[row];
        len = dag_ptr[row + 1] - at;
        if (len > 0) {
            const int v = perm[row];
            b = row_ptr[v];
            e = row_ptr[v + 1];
            if (e - b > kLongRow || len > kGroupRow) {
                longs.row[atomicAdd(&longs.n, 1)] = row;
                len = 0;
            }
        }
    }
    for (int q = 0; 4 * q < per; q++) {
        const int from = 4 * q + g;
        const int rlen = __shfl(len, from);
        if (__ballot(rlen > 0) == 0ull) continue;
        const int rat = __shfl(at, from), rb = __shfl(b, from), rend = __shfl(e, from), i = __shfl(row, from);
        const int re = rlen > 0 ? rend : rb;
        const int span = wave_max(re - rb);
        int pos = 0;
        for (int t = 0; t < span; t += 64) {
            int r[4];
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = rb + t + 16 * u + gl < re ? col[rb + t + 16 * u + gl] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = r[u] >= 0 ? rank[r[u]] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const unsigned int m = static_cast<unsigned int>(__ballot(r[u] > i) >> (16 * g)) & 0xffffu;
                if (r[u] > i) grow[pos + __popc(m & glt)] = r[u];
                pos += __popc(m);
            }
        }
        if (gl < 4) grow[pos + gl] = INT_MAX;        // fills the last four
        wave_sync_lds();
        const int longest = wave_max(rlen);
        for (int t = 0; t < longest; t += 16) {
            const int x = t + gl < rlen ? grow[t + gl] : INT_MAX;
            int below = 0;
            for (int u = 0; u < rlen; u += 4) {
                const int4 y = *reinterpret_cast<const int4*>(grow + u);
                below += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
            }
            if (t + gl < rlen) {
                dag_col[rat + below] = x;
                dag_src[rat + t + gl] = i;
            }
        }
        wave_sync_lds();
    }
    __syncthreads();
    int* wrow = groups[(threadIdx.x >> 6) * 4];
    for (int l = threadIdx.x >> 6; l < longs.n; l += kRowBlock / 64) {
        const int i = longs.row[l], v = perm[i];
        const int base = dag_ptr[i], rlen = dag_ptr[i + 1] - base;
        const int first = row_ptr[v], last = row_ptr[v + 1];
        if (rlen > kWaveRow || last - first > kBlockRow) continue;
        int pos = 0;
        for (int j0 = first; j0 < last; j0 += 256) {
            int r[4];
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = j0 + 64 * u + lane < last ? col[j0 + 64 * u + lane] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = r[u] >= 0 ? rank[r[u]] : -1;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const unsigned long long m = __ballot(r[u] > i);
                const int p = pos + __popcll(m & lanemask_lt());
                if (r[u] > i && p < rlen) wrow[p] = r[u];
                pos += __popcll(m);
            }
        }
        if (lane < 4) wrow[rlen + lane] = INT_MAX;
        wave_sync_lds();
        for (int t = lane; t < rlen; t += 64) {
            const int x = wrow[t];
            int below = 0;
            for (int u = 0; u < rlen; u += 4) {
                const int4 y = *reinterpret_cast<const int4*>(wrow + u);
                below += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
            }
            dag_col[base + below] = x;
            dag_src[base + t] = i;
        }
        wave_sync_lds();
    }
    for (int l = 0; l < longs.n; l++) {
        const int i = longs.row[l], v = perm[i];
        const int base = dag_ptr[i], rlen = dag_ptr[i + 1] - base;
        const int last = row_ptr[v + 1];
        if (rlen <= kWaveRow && last - row_ptr[v] <= kBlockRow) continue;
        const bool in_lds = rlen <= kRowCap;
        int* dst = in_lds ? big_row : tmp + base;
        if (threadIdx.x == 0) {
            s_pos = 0;
            if (!in_lds) atomicOr(&ctl[CTL_LONG], 1);
        }
        __syncthreads();
        for (int j0 = row_ptr[v]; j0 < last; j0 += kRowBlock) {
            const int j = j0 + threadIdx.x;
            const int r = j < last ? rank[col[j]] : -1;
            const unsigned long long m = __ballot(r > i);
            int p = 0;
            if (lane == 0 && m) p = atomicAdd(&s_pos, __popcll(m));
            p = __shfl(p, 0) + __popcll(m & lanemask_lt());
            if (r > i && p < rlen) dst[p] = r;      // any order: the row is sorted afterwards
        }
        __syncthreads();
        if (in_lds) {
            if (threadIdx.x < 4) big_row[rlen + threadIdx.x] = INT_MAX;   // fills the last four
            __syncthreads();
            if (static_cast<int>(threadIdx.x) < rlen) {
                const int x = big_row[threadIdx.x];
                int below = 0;
                for (int u = 0; u < rlen; u += 4) {
                    const int4 y = *reinterpret_cast<const int4*>(big_row + u);
                    below += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
                }
                dag_col[base + below] = x;
                dag_src[base + threadIdx.x] = i;
            }
            __syncthreads();
        }
    }
}

// One block per row longer than kRowCap: rows up to kLongSortCap entries are
// bitonic-sorted in LDS (entries are distinct new ids; the padding is INT_MAX);
// longer ones place each entry at its rank, counted over the row in global memory.
constexpr int kLongSortCap = 8192;

__global__ void __launch_bounds__(kBlock) k_sort_long_rows(int n, const int* __restrict__ dag_ptr,
                                                          const int* __restrict__ tmp, int* dag_col,
                                                          int* dag_src, const int* ctl) {
    __shared__ int buf[kLongSortCap];
    if (rejected(ctl) || !ctl[CTL_LONG]) return;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int base = dag_ptr[i];
        const int len = dag_ptr[i + 1] - base;
        if (len <= kRowCap) continue;
        const int* row = tmp + base;
        if (len <= kLongSortCap) {
            int p = 1;
            while (p < len) p <<= 1;
            for (int t = threadIdx.x; t < p; t += kBlock) buf[t] = t < len ? row[t] : INT_MAX;
            __syncthreads();
            for (int k = 2; k <= p; k <<= 1) {
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int t = threadIdx.x; t < p; t += kBlock) {
                        const int o = t ^ j;
                        if (o > t) {
                            const int x = buf[t], y = buf[o];
                            if ((x > y) == ((t & k) == 0)) {
                                buf[t] = y;
                                buf[o] = x;
                            }
                        }
                    }
                    __syncthreads();
                }
            }
            for (int t = threadIdx.x; t < len; t += kBlock) {
                dag_col[base + t] = buf[t];
                dag_src[base + t] = i;
            }
            __syncthreads();
        } else {
            for (int t = threadIdx.x; t < len; t += kBlock) {
                const int x = row[t];
                int below = 0;
                for (int q = 0; q < len; q++) below += row[q] < x;
                dag_col[base + below] = x;
                dag_src[base + below] = i;
            }
        }
    }
}

struct OrientWs {
    int *ctl, *key_a, *val_a, *key_b, *val_b, *rank, *outdeg, *tiles, *rnd, *fr0, *fr1, *hf0, *hf1, *tmp;
};

OrientWs carve(void* ws, int n, int nnz, size_t* bytes) {
    Carver c(ws);
    OrientWs w;
    size_t nn = static_cast<size_t>(n > 0 ? n : 1);
    size_t m = static_cast<size_t>(nnz / 2 > 0 ? nnz / 2 : 1);
    int ntiles = div_up(static_cast<long long>(n) + 1, kTile) + 1;
    w.ctl = c.take<int>(CTL_WORDS);
    w.key_a = c.take<int>(nn);
    w.val_a = c.take<int>(nn);
    w.key_b = c.take<int>(nn);
    w.val_b = c.take<int>(nn);
    // from tiles on, everything is idle during the radix sort, whose digit counts
    // (256 per tile of 2048 vertices, and 256 totals) start there: 512 ints for the
    // smallest graphs (eight slices of 64), 0.13 n + 256 of 7 n for large ones
    w.tiles = c.take<int>(static_cast<size_t>(ntiles));
    w.rank = c.take<int>(nn);
    w.fr0 = c.take<int>(nn);
    w.fr1 = c.take<int>(nn);
    w.hf0 = c.take<int>(nn);
    w.hf1 = c.take<int>(nn);
    // outdeg, rnd and tmp together hold the peel's compacted rows (nnz + 3 n 16-bit ids)
    w.outdeg = c.take<int>(nn + 1);
    w.rnd = c.take<int>(nn);
    w.tmp = c.take<int>(m);
    *bytes = c.bytes();
    return w;
}

int grid_for_waves(long long items_per_wave_units) {
    long long blocks = (items_per_wave_units + (kBlock / 64) - 1) / (kBlock / 64);
    long long cap = static_cast<long long>(device_cus()) * 16;
    if (blocks > cap) blocks = cap;
    return static_cast<int>(blocks < 1 ? 1 : blocks);
}

// Rows per wavefront of the row kernels: about four blocks per CU, 4 (one per group
// of 16 lanes) to 64 rows, a power of two.  One where most rows are long: the groups have
// little to do then, and few blocks would share the rows (every vertex of 4,000 joined to
// half of the others: 63 blocks, k_validate 1,070 us; 250, 290; 339 with a wavefront per row).
int rows_per_wave(int n, int nnz) {
    if (nnz / n > kLongRow) return 1;
    const int per = n / (16 * 4 * device_cus());
    int p = 4;
    while (p < kMaxPer && 2 * p <= per) p *= 2;
    return p;
}

int grid_for_threads(long long n) {
    long long blocks = (n + kBlock - 1) / kBlock;
    long long cap = static_cast<long long>(device_cus()) * 16;
    if (blocks > cap) blocks = cap;
    return static_cast<int>(blocks < 1 ? 1 : blocks);
}

// One atomic per block on the largest key: at most two blocks per CU.
int grid_for_keys(long long n) {
    const int g = grid_for_threads(n), cap = device_cus() * 2;
    return g < cap ? g : cap;
}

// out[0..count] = exclusive prefix sums of in[0..count) with out[count] = total (also
// in CTL_TOTAL); the largest entry to CTL_DMAX.
int exclusive_scan(int count, const int* in, int* out, int* tiles, int* ctl, hipStream_t s) {
    if (count <= kScanOne) {
        k_scan_one<<<1, 1024, 0, s>>>(count, in, out, ctl + CTL_DMAX, ctl);
    } else {
        const int ntiles = div_up(count, kTile);
        k_tile_sum<<<ntiles, kBlock, 0, s>>>(count, in, tiles, ctl + CTL_DMAX, ctl);
        k_scan_tiles<<<1, kBlock, 0, s>>>(ntiles, tiles, ctl);
        k_scan_apply<<<ntiles, kBlock, 0, s>>>(count, in, tiles, out, ctl);
    }
    KC_CHECK(hipGetLastError());
    return KC_OK;
}

// Sort by key (key_a / val_a hold the keys and ids, CTL_MAXKEY the largest key, which
// is at most `bound`), then out: perm, rank, and the DAG's rows, of at most `room` entries.
// Nothing is read on the host.
int build_dag(const OrientWs& w, int n, int nnz, const int* row_ptr, const int* col, long long bound, bool grouped,
              int room, int* out_row_ptr, int* out_col, int* out_src, int* out_perm, hipStream_t s) {
    const int ntiles = div_up(n, kTile);
    const RadixBuf rb{w.key_a, w.val_a, w.key_b, w.val_b};
    const int per = rows_per_wave(n, nnz), rows_grid = div_up(n, 16 * per);
    const int run = grouped ? 16 * per : kRowRun;
    int *dtot = w.tiles, *hist = w.tiles + 256;
    int pass = 0;
    for (; pass < 4 && (bound >> (8 * pass)) != 0; pass++) {
        k_radix_hist<<<ntiles, kBlock, 0, s>>>(n, pass, rb, hist, w.ctl);
        k_radix_scan<<<256, kBlock, 0, s>>>(ntiles, pass, hist, dtot, w.ctl);
        k_radix_scatter<<<ntiles, kBlock, 0, s>>>(n, pass, rb, hist, dtot, w.ctl);
    }
    k_rank<<<grid_for_threads(n), kBlock, 0, s>>>(n, pass, rb, out_perm, w.rank, w.ctl);
    k_outdeg<<<rows_grid, kRowBlock, 0, s>>>(n, per, run, row_ptr, col, out_perm, w.rank, w.outdeg, w.ctl);
    KC_CHECK(hipGetLastError());
    const int st = exclusive_scan(n, w.outdeg, out_row_ptr, w.tiles, w.ctl, s);
    if (st != KC_OK) return st;
    if (nnz > 0) {
        k_fill<<<rows_grid, kRowBlock, 0, s>>>(n, per, run, row_ptr, col, out_perm, w.rank, out_row_ptr, out_col, out_src,
                                              w.tmp, room, w.ctl);
        KC_CHECK(hipGetLastError());
    }
    return KC_OK;
}

// Degeneracy order: the peel's keys (rounds) and ids, and its control words.
int launch_peel(const OrientWs& w, int n, const int* row_ptr, const int* col, hipStream_t s) {
    int* deg = w.key_b;   // scratch until the sort
    if (n > kCoreSmall) {
        // one block per 16k vertices, between 16 and 64 (a barrier costs 0.8 us at
        // 16 blocks, 1.3 at 64, 3.7 at 256, whatever the block size)
        int occ = 0;
        KC_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_peel, kPeelBlock, 0));
        if (occ < 1) return KC_EDEVICE;
        int blocks = n / 16384;
        if (blocks > 64) blocks = 64;
        if (blocks < 16) blocks = 16;
        if (blocks > occ * device_cus()) blocks = occ * device_cus();   // all blocks co-resident
        int n_ = n, keep = kCoreCap;
        const int* rp = row_ptr;
        const int* cl = col;
        OrientWs ws = w;
        void* args[] = {&n_, &keep, &rp, &cl, &deg, &ws.key_a, &ws.fr0, &ws.fr1, &ws.val_a, &ws.ctl};
        KC_CHECK(hipLaunchCooperativeKernel(reinterpret_cast<void*>(k_peel), dim3(blocks), dim3(kPeelBlock),
                                            args, 0, s));
    } else {
        k_peel_init<<<grid_for_threads(n), kBlock, 0, s>>>(n, row_ptr, deg, w.key_a, w.val_a, w.ctl);
    }
    unsigned short* rows = reinterpret_cast<unsigned short*>(w.outdeg);   // outdeg, rnd, tmp: nnz + 4 n entries
    CoreSpan* span = reinterpret_cast<CoreSpan*>(w.hf0);   // hf0 and hf1 are adjacent: 2 n ints and more
    k_core_list<<<div_up(n, kPeelBlock), kPeelBlock, 0, s>>>(n, w.key_a, deg, w.rank, w.fr0, span, w.ctl);
    k_core_rows<<<grid_for_waves(n < kCoreCap ? n : kCoreCap), kBlock, 0, s>>>(
        row_ptr, col, w.rank, w.fr0, span, rows, w.ctl);
    const int lds = kCoreLds;
    KC_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_core_peel),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    k_core_peel<<<1, kPeelBlock, lds, s>>>(span, rows, w.fr0, w.fr1, w.key_a, w.ctl);
    KC_CHECK(hipGetLastError());
    return KC_OK;
}

__global__ void __launch_bounds__(kBlock) k_zero(int* p, int count) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) p[i] = 0;
}

}  // namespace

size_t orient_async_workspace(int n, int nnz) {
    size_t bytes = 0;
    carve(nullptr, n, nnz, &bytes);
    return bytes;
}

// Degree-order orientation of a batch's disjoint union with no host synchronisation,
// so it can be captured in a HIP graph.  The vertices of a graph stay together (their
// rows, ranks and roots share cache lines), ordered by (degree, id) inside it, unless
// graph and degree do not fit one 31-bit key: then the union is ordered by degree.
// Writes row_ptr, col, src, perm.  The order is a permutation whatever max_degree says; one
// that is too low lets graphs' ids mix, so the graph of an id is that of perm[id].
int orient_degree_async(int n, int nnz, const int* row_ptr, const int* col, const int* voff, int ngraphs,
                        int max_degree, int* out_row_ptr, int* out_col, int* out_src, int* out_perm, void* ws,
                        hipStream_t s) {
    size_t need = 0;
    OrientWs w = carve(ws, n, nnz, &need);
    if (n <= 0) return KC_EINVAL;
    const long long span = static_cast<long long>(max_degree) + 1;
    const long long keys = span * ngraphs;
    const bool grouped = keys <= INT_MAX;
    k_zero<<<1, kBlock, 0, s>>>(w.ctl, CTL_WORDS);
    k_degree_key<<<grid_for_keys(n), kBlock, 0, s>>>(n, row_ptr, w.key_a, w.val_a, w.ctl, grouped ? voff : nullptr,
                                                    ngraphs, static_cast<int>(span));
    int st = build_dag(w, n, nnz, row_ptr, col, grouped ? keys - 1 : span - 1, grouped, INT_MAX, out_row_ptr,
                       out_col, out_src, out_perm, s);
    if (st != KC_OK) return st;
    if (nnz > 0) {
        k_sort_long_rows<<<grid_for_threads(n), kBlock, 0, s>>>(n, out_row_ptr, w.tmp, out_col, out_src, w.ctl);
        KC_CHECK(hipGetLastError());
    }
    return KC_OK;
}

}  // namespace kc

using namespace kc;

extern "C" KC_API size_t kc_orient_workspace(int32_t n, int32_t nnz, int32_t order) {
    (void)order;
    if (n < 0 || nnz < 0) return 0;
    size_t bytes = 0;
    carve(nullptr, n, nnz, &bytes);
    return bytes;
}

namespace {
bool invalid(const int* hctl) { return hctl[CTL_BAD] != 0 || hctl[CTL_UP] != 0; }
}  // namespace

extern "C" KC_API int32_t kc_orient(const kc_csr* g, int32_t order, kc_dag* out, void* ws,
                                    size_t ws_bytes, int32_t validate, void* stream) {
    if (!g || !out) return KC_EINVAL;
    if (order != KC_ORDER_DEGREE && order != KC_ORDER_DEGENERACY && order != KC_ORDER_APPROX_DEGENERACY &&
        order != KC_ORDER_COLOR)
        return KC_EINVAL;
    const int n = g->n, nnz = g->nnz;
    if (n < 0 || nnz < 0 || (nnz & 1)) return KC_EINVAL;
    if (!g->row_ptr || !out->row_ptr || (n > 0 && !out->perm)) return KC_EINVAL;
    if (nnz > 0 && (!g->col || !out->col || !out->src)) return KC_EINVAL;
    size_t need = 0;
    OrientWs w = carve(ws, n, nnz, &need);
    if (!ws || ws_bytes < need) return KC_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int m = nnz / 2;

    out->n = n;
    out->m = m;
    out->order = order;
    out->d_max = 0;
    out->degeneracy = order == KC_ORDER_DEGENERACY ? 0 : -1;
    KC_CHECK(hipMemsetAsync(w.ctl, 0, CTL_WORDS * sizeof(int), s));
    if (n == 0) {
        if (nnz != 0) return KC_EINVAL;
        KC_CHECK(hipMemsetAsync(out->row_ptr, 0, sizeof(int), s));
        KC_CHECK(hipStreamSynchronize(s));
        return KC_OK;
    }

    // Rejected graphs stop every later kernel on the device; the orders that read back
    // on the way look at the verdict first.
    if (validate) {
        const int per = rows_per_wave(n, nnz);
        k_validate<<<div_up(n, 16 * per), kRowBlock, 0, s>>>(n, nnz, per, kCheckRun, g->row_ptr, g->col, w.ctl);
        KC_CHECK(hipGetLastError());
    }
    int hctl[CTL_WORDS];
    if (validate && (order == KC_ORDER_COLOR || order == KC_ORDER_APPROX_DEGENERACY)) {
        KC_CHECK(hipMemcpyAsync(hctl, w.ctl, sizeof(hctl), hipMemcpyDeviceToHost, s));
        KC_CHECK(hipStreamSynchronize(s));
        if (invalid(hctl)) return KC_EINVAL;
    }

    // 1. sort keys
    if (order == KC_ORDER_DEGREE) {
        k_degree_key<<<grid_for_keys(n), kBlock, 0, s>>>(n, g->row_ptr, w.key_a, w.val_a, w.ctl, nullptr, 0, 0);
        KC_CHECK(hipGetLastError());
    } else if (order == KC_ORDER_COLOR) {
        // the colours go straight into the sort keys; rounds are launched in
        // batches of 4, 8, ... 64, and the host reads the frontier size after each
        k_cl_init<<<grid_for_waves(n), kBlock, 0, s>>>(n, g->row_ptr, g->col, w.rnd, w.val_a,
                                                       ClFront{nullptr, nullptr, w.fr0, w.hf0}, w.ctl);
        KC_CHECK(hipGetLastError());
        const int grid = device_cus() * 4;
        int r = 0;
        for (int batch = 4;; batch = batch < 64 ? 2 * batch : 64) {
            for (int i = 0; i < batch; i++, r++) {
                const ClFront f = (r & 1) ? ClFront{w.fr1, w.hf1, w.fr0, w.hf0} : ClFront{w.fr0, w.hf0, w.fr1, w.hf1};
                k_cl_round<<<grid, kBlock, 0, s>>>(r, f, g->row_ptr, g->col, w.rnd, w.key_a, w.ctl);
            }
            KC_CHECK(hipGetLastError());
            int left[2] = {0, 0};
            KC_CHECK(hipMemcpyAsync(&left[0], w.ctl + CTL_CL_SIZE0 + r % 3, sizeof(int), hipMemcpyDeviceToHost, s));
            KC_CHECK(hipMemcpyAsync(&left[1], w.ctl + CTL_CL_HSIZE0 + r % 3, sizeof(int), hipMemcpyDeviceToHost, s));
            KC_CHECK(hipStreamSynchronize(s));
            if (left[0] + left[1] == 0) break;
            if (r > n) return KC_EDEVICE;   // cannot happen: every round colours at least one vertex
        }
    } else if (order == KC_ORDER_APPROX_DEGENERACY) {
        // host-driven rounds: the live count decides when to stop
        int* deg = w.key_b;   // scratch until the sort
        k_ad_init<<<grid_for_threads(n), kBlock, 0, s>>>(n, g->row_ptr, deg, w.rnd, w.val_a);
        KC_CHECK(hipGetLastError());
        int r = 0, before = -1;
        for (;; r++) {
            KC_CHECK(hipMemsetAsync(w.ctl + CTL_AD_LIVE, 0, 4 * sizeof(int), s));
            k_ad_sum<<<grid_for_threads(n), kBlock, 0, s>>>(n, deg, w.rnd, w.ctl);
            KC_CHECK(hipGetLastError());
            int live = 0;
            KC_CHECK(hipMemcpyAsync(&live, w.ctl + CTL_AD_LIVE, sizeof(int), hipMemcpyDeviceToHost, s));
            KC_CHECK(hipStreamSynchronize(s));
            if (live == 0) break;
            if (live == before) return KC_EINVAL;   // not symmetric (only possible without validation)
            before = live;
            k_ad_mark<<<grid_for_threads(n), kBlock, 0, s>>>(n, r, deg, w.rnd, w.ctl);
            k_ad_dec<<<grid_for_waves(n), kBlock, 0, s>>>(n, r, g->row_ptr, g->col, deg, w.rnd);
            KC_CHECK(hipGetLastError());
        }
        const int maxkey = r > 0 ? r - 1 : 0;
        KC_CHECK(hipMemcpyAsync(w.ctl + CTL_MAXKEY, &maxkey, sizeof(int), hipMemcpyHostToDevice, s));
        KC_CHECK(hipMemcpyAsync(w.ctl + CTL_ROUNDS, &r, sizeof(int), hipMemcpyHostToDevice, s));
        KC_CHECK(hipMemcpyAsync(w.key_a, w.rnd, sizeof(int) * n, hipMemcpyDeviceToDevice, s));
    }
    // 2. stable radix sort (key, id) -> position = new id; 3. filter: out-degrees and
    // their scan -> row_ptr; 4. compact + per-row sort.  Degrees and colours are below
    // n; the peel's rounds below 2 n, as a level change counts as one.
    for (;;) {
        if (order == KC_ORDER_DEGENERACY) {
            const int st = launch_peel(w, n, g->row_ptr, g->col, s);
            if (st != KC_OK) return st;
        }
        const int st = build_dag(w, n, nnz, g->row_ptr, g->col, order == KC_ORDER_DEGENERACY ? 2LL * n : n, false, m,
                                 out->row_ptr, out->col, out->src, out->perm, s);
        if (st != KC_OK) return st;
        KC_CHECK(hipMemcpyAsync(hctl, w.ctl, sizeof(hctl), hipMemcpyDeviceToHost, s));
        KC_CHECK(hipStreamSynchronize(s));
        if (invalid(hctl)) return KC_EINVAL;
        if (!(hctl[CTL_STALL] & kStallStart)) break;
        // other streams' work held the compute units for all of the first barrier's wait
        // (seconds): wait on
        KC_CHECK(hipMemsetAsync(w.ctl, 0, CTL_WORDS * sizeof(int), s));
    }
    if (hctl[CTL_STALL]) return KC_EDEVICE;   // a later barrier's wait ran out
    if (hctl[CTL_LONG]) {
        k_sort_long_rows<<<grid_for_threads(n), kBlock, 0, s>>>(n, out->row_ptr, w.tmp, out->col, out->src, w.ctl);
        KC_CHECK(hipGetLastError());
        KC_CHECK(hipStreamSynchronize(s));
    }
    if (hctl[CTL_TOTAL] != m) return KC_EINVAL;   // not symmetric (only possible without validation)
    out->d_max = hctl[CTL_DMAX];
    out->degeneracy = order == KC_ORDER_DEGENERACY ? hctl[CTL_DEGEN] : -1;
    return KC_OK;
}
