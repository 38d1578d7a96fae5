// Host-side layout shared by the counting sources (not part of the ABI).
#pragma once

#include "kc_internal.h"

namespace kc {

constexpr int kLightCap = 64;          // |S| bound of the light root list
constexpr int kMidCap = 128;           // and of the pivot's middle list

// Pivot leaf counters: leaves with nh holds among t = holds + pivots vertices.
constexpr __host__ __device__ int leaf_index(int t, int nh) { return t * (t + 1) / 2 + nh; }
constexpr int kPivBlocksPerCU = 8;     // grid cap of the heavy pivot kernel (sizes its stacks)
constexpr int kLaneWavesPerCU = 32;    // grid cap of the lane-walk kernel (sizes its registry)
constexpr int kListBlocks = 512;        // blocks that write the width lists
constexpr int kWidthLists = 6;         // root lists by bitset words per row: 1, 2, 4, 8, 16, 32
constexpr int kQueueCap = 16384;        // lane walk: ring slots for subtrees handed between wavefronts (power of 2)
constexpr int kItemWords = 36;          // queue item: root slot, path length, 2 spare, 32 words of R
// The lane walk's list 0 has no pair tasks and so no queue; list j >= 1 uses queue
// j - 1; the pivot launches use queues 0 (light), 1 (heavy) and 2 (middle).
constexpr int kQueueLists = kWidthLists - 1;
constexpr int queue_of(int list) { return list > 0 ? list - 1 : 0; }
constexpr int kQueueCtlWords = 8;       // per width list: head, tail, pending, rooting, hungry
// subtree queue control words, and its bounds
constexpr int Q_HEAD = 0, Q_TAIL = 1, Q_PENDING = 2, Q_ROOTING = 3, Q_HUNGRY = 4;
constexpr int kMaxWaiters = 256;                            // lane walk: wavefronts that wait for handed-over work
constexpr unsigned long long kStallTicks = 2000000000ull;   // 20 s at 100 MHz without queue progress
constexpr int kReadySpins = 1 << 22;                        // wait for a reserved item's sequence word
constexpr int kQueueCtlTotal = 3 * 8 * 32;   // the most any path uses: three sharded pivot queues
// bits of the CC_FLAGS control word
constexpr int kFlagBigBinom = 1;    // a binomial beyond 128 bits was used
constexpr int kFlagStalled = 2;     // a work queue stopped making progress (no valid count)
constexpr int kFlagCanceled = 4;    // the caller's cancel flag was seen (no valid count)
constexpr int kFlagLocalOverflow = 8;   // a per-vertex count passed 2^64
// handoff thresholds (defaults; kc_opts may lower them for tests)
constexpr int kLaneStealEvery = 16;    // lane walk: wavefront rounds between looks at the subtree queue
constexpr int kLaneStealAfter = 256;   // lane walk: rounds on the current root or subtree before it may hand over
// pivot: tree nodes between looks at the frame queue, and nodes of the current
// root or frame before it may hand over.  A consumer re-extracts the frame's
// root, so only long trees should give work away.
constexpr int kPivStealEvery = 64;
constexpr int kPivStealAfter = 8192;
// Pivot walks are latency-bound (one wavefront per tree, chains of dependent LDS
// and global accesses), so more wavefronts may wait for handed-over frames than
// in the lane walk: 4 per CU.  Dense-core count-all with a 4096-node first
// handoff (VC / EC, ms): 1500 / 800 with 256 waiters in all, 1110 / 713 at 2 per
// CU, 930 / 665 at 4, 1240 / 775 at 8, 3000 / 1390 at 16 (handoffs and queue
// traffic then outweigh the overlap); 810 / 650 at 4 per CU with 8192.
constexpr int kPivWaitersPerCU = 4;
// Pivot walks in registers: independent frame queues, 128 bytes between their control
// words; nodes between looks and before the first handoff; waiting wavefronts.
constexpr int kRegShards = 8;
constexpr int kShardLine = 32;
constexpr int kRegStealEvery = 256;
constexpr int kRegStealAfter = 1024;
constexpr int kRegWaitersPerCU = 32;
constexpr int kCancelEvery = 32;       // wavefront rounds (lane walk) or nodes (pivot) between cancel polls
// count lo/hi, light/heavy stats, per width list: nodes, words, iterations,
// expansions, busy, start, end; helper timing (3); per width list: counted
// cliques weighted by row words
constexpr int kAccWords = 9 + 8 * kWidthLists;
constexpr int kAccCwords = 9 + 7 * kWidthLists;
// Final counts of the traversal wavefronts: kAccSlots {lo, hi} pairs on cache
// lines of their own, after the words above; the host adds them up.  Atomics on
// one address are served one after the other (11.6 ns each, measured), so 8192
// wavefronts adding to a single pair took 95 us.
constexpr int kAccSlots = 32;
constexpr int kAccSlotStride = 16;                                   // u64 words: 128 bytes
constexpr int kAccSlotBase = ((kAccWords + 15) / 16) * 16;
constexpr int kAccTotal = kAccSlotBase + kAccSlots * kAccSlotStride;

enum CountCtl {
    CC_LIGHT_N = 0,      // light root count
    CC_HEAVY_N = 1,      // heavy root count
    CC_LIGHT_HEAD = 2,   // light queue head
    CC_HEAVY_HEAD = 3,   // heavy queue head
    CC_FLAGS = 4,        // kFlag* bits
    CC_WIDE_N = 5,       // wide root count
    CC_WIDE_HEAD = 6,    // wide queue head
    CC_MID_N = 7,        // pivot: middle root count
    CC_MID_HEAD = 14,    // pivot: middle queue head
    CC_WN0 = 8,          // width lists: root counts (8..13)
    CC_WH0 = 24,         // width lists: queue heads (24..29)
    CC_WORDS = 32
};

constexpr int kOptShareShift = 16;   // kc_opts.flags, set by the server: PivLaunch::share in two bits

constexpr size_t kAccAfterCtl = 256;   // bytes from the control words to the accumulators

// Saved levels a depth-first walk starting at path length `first` may need:
// the last two levels of a path are counted in registers (a node one level
// above the leaves adds the edge count of its candidate set), so levels are
// saved only while the path is shorter than k - 3.
inline int k_levels(int k, int first) {
    const int lv = k - 3 - first;
    return lv < 1 ? 1 : lv;
}

__host__ __device__ constexpr int b_stride_of(int maxw) { return (maxw > 1 && (maxw % 2) == 0) ? maxw + 1 : maxw; }

// Row stride (words) of the lane walk's bitset rows.  Rows of up to 4 words keep
// an odd stride and 32-bit reads (row starts spread over all banks); wider rows
// are padded to a multiple of 4 words and read with 128-bit loads (6 -> 8).
__host__ __device__ constexpr int lane_stride(int w) { return w <= 4 ? b_stride_of(w) : ((w + 3) & ~3); }

// Bitset words per row used for a DAG of this d_max (rows of at most 32 * maxw bits).
inline int maxw_for(int d_max) {
    if (d_max <= 64) return 2;
    if (d_max <= 128) return 4;
    if (d_max <= 256) return 8;
    if (d_max <= 512) return 16;
    return 32;
}

// The on-chip kernels see at most KC_MAX_DMAX out-neighbours per root: longer
// out-rows make their roots wide (kc_wide.hip) and the others skip them.
inline int bit_dmax(int d_max) { return d_max < KC_MAX_DMAX ? d_max : KC_MAX_DMAX; }

// Wide roots: candidate slots and row words (padded to 4) of one wavefront's slab,
// and the slab's words: rows, then per stack level the candidate and branch sets,
// then 4 words of level scalars.
inline int wide_s_cap(int d_max) { return ((d_max + 31) / 32) * 32; }
inline int wide_wcap(int d_max) { return ((wide_s_cap(d_max) / 32) + 3) & ~3; }
inline size_t wide_slab_words(int d_max) {
    const size_t s = static_cast<size_t>(wide_s_cap(d_max)), w = static_cast<size_t>(wide_wcap(d_max));
    return s * w + (s + 2) * (2 * w + 4);
}
constexpr size_t kWideSlabBudget = static_cast<size_t>(2) << 30;   // bytes of wide slabs at most

inline int s_cap_for(int d_max) { return ((d_max + 31) / 32) * 32 > kLightCap ? ((d_max + 31) / 32) * 32 : kLightCap; }

// Words of one pivot stack level: I, P_orig, P_remaining (maxw each) + p, np, nh, pad.
inline int piv_level_words(int maxw) { return 3 * maxw + 4; }

// A wavefront's claims on a launch's roots (0 .. nroots - 1, in list order): chunks
// of two thirds of its even share, at most `cap`.  The first chunk is fixed by the
// wavefront's index; later ones come from the queue head, whose atomics are served
// one after the other, 11.6 ns each: one per wavefront was 95 us of a launch over
// 2000 roots, one per root 2.3 ms of a count over 198,000.  Two thirds leave at most
// half a claim per wavefront (48 us) where a list is short, and the cap leaves many
// where it is long.  The head is not looked at before it is claimed from: plain loads
// of the contended line wait in the same queue (batch of 10,000 graphs: 37 -> 52 ms).
// A wavefront that is not running yet, as other streams' work holds its compute unit,
// keeps its first chunk: no other can take it, and the launch ends after it has run.  With
// four counts at a time (graphs of 100,000 vertices, a thread and a stream each) that costs less
// than it saves: k = 4 4.9 ms with every root from the head, 1.5 so; pivoting k = 8, 77 and 26.
//
// The roots of a chunk lie a chunk count apart.  Lists end with the dense core's
// roots and batches hold a graph's roots together, so neighbours are heavy together:
// chunks of neighbours took the per-vertex counts of a 200k-vertex power-law graph
// from 5.2 to 23 ms and a batch of 665 graphs at k = 7 from 9.5 to 11.5.
struct RootClaims {
    int next = 0, left = 0;         // claimed, unprocessed roots
    int step = 1;                   // distance between the roots of a chunk
    bool started = false;
};

// Claims the next chunk (roots c.next, c.next + c.step, ..., c.left of them;
// wave-uniform); false when no root is left.  `head` is zero at launch; every lane
// calls this.
__device__ __forceinline__ bool claim_chunk(RootClaims& c, int* head, int nroots, int wave, int nwaves, int cap) {
    const long long share = (2LL * nroots + 3LL * nwaves - 1) / (3LL * nwaves);
    const int size = share < 1 ? 1 : share > cap ? cap : static_cast<int>(share);
    const int chunks = (nroots + size - 1) / size;
    int q = wave;
    if (c.started) {
        if (nwaves >= chunks) return false;
        q = 0;
        if (__lane_id() == 0) q = atomicAdd(head, 1);
        q = nwaves + __shfl(q, 0);
    }
    c.started = true;
    if (q >= chunks) return false;
    c.next = q;
    c.step = chunks;
    c.left = (nroots - q + chunks - 1) / chunks;
    return true;
}

// The next root of this wavefront (wave-uniform), or -1 when none is left.
__device__ __forceinline__ int claim_root(RootClaims& c, int* head, int nroots, int wave, int nwaves, int cap) {
    if (c.left == 0 && !claim_chunk(c, head, nroots, wave, nwaves, cap)) return -1;
    const int r = c.next;
    c.next += c.step;
    c.left--;
    return r;
}

struct CountWs {
    int* ctl;
    unsigned long long* acc;      // [lo, hi, light nodes, words, heavy nodes, words, then per width list nodes, words]
    int* light;
    int* heavy;                   // pivot: the middle list grows down from its end
    int nroots_cap;               // entries of light and of heavy
    unsigned long long* leaves;   // pivot: leaf counters, and how many
    int leaf_count;
    unsigned long long* counts;   // count_all: (binom_n + 1) x {lo, hi}
    unsigned long long* binom;    // (binom_n + 1)^2 x {lo, hi}: C(i, j) at [i * (binom_n + 1) + j]
    unsigned char* big;           // same shape: 1 if C(i, j) needs more than 128 bits
    unsigned int* gstack;         // heavy pivot stacks, one slab per resident wavefront
    int* task_ctr;                // lane walk, pair tasks: claimed tasks per root
    int* task_tot;                // lane walk, pair tasks: total tasks + 1 per root (0 = unpublished)
    int* active;                  // lane walk: root slot owned by each wavefront (-1 = none), main + side
    int* bcnt;                    // width lists: roots per list and block
    int* qctl;                    // lane walk, subtree queue: kQueueCtlWords per width list
    int* qready;                  // subtree queue: slot sequence words, kQueueCap per queue (see queue_of)
    unsigned int* qitems;         // lane walk, subtree queue: kItemWords per slot, main + side
    int* wide;                    // wide roots (d_max > KC_MAX_DMAX only)
    unsigned int* wslabs;         // wide roots: one slab per wavefront
    size_t wslab_words;
    int nwslabs;
    int nactive;
    int binom_n;
    int counts_len;               // entries of counts (sizes 0 .. counts_len - 1)
    size_t slab_words;
    int slabs;
};

inline CountWs carve_count(void* ws, const kc_dag* d, bool pivot, size_t* bytes) {
    Carver c(ws);
    CountWs w{};
    const int nr = d->m > d->n ? d->m : d->n;
    w.ctl = c.take<int>(CC_WORDS);
    w.acc = c.take<unsigned long long>(kAccTotal);      // kAccAfterCtl bytes after ctl
    w.light = c.take<int>(static_cast<size_t>(nr > 0 ? nr : 1));
    w.heavy = c.take<int>(static_cast<size_t>(nr > 0 ? nr : 1));
    w.nroots_cap = nr > 0 ? nr : 1;
    w.task_ctr = c.take<int>(static_cast<size_t>(nr > 0 ? nr : 1));
    w.task_tot = c.take<int>(static_cast<size_t>(nr > 0 ? nr : 1));
    w.nactive = device_cus() * kLaneWavesPerCU;
    w.active = c.take<int>(2 * static_cast<size_t>(w.nactive));    // main and side stream
    w.bcnt = c.take<int>(kWidthLists * kListBlocks);
    w.qctl = c.take<int>(kQueueCtlTotal);
    w.qready = c.take<int>(static_cast<size_t>(kQueueCap) * kQueueLists);
    w.qitems = c.take<unsigned int>(2 * static_cast<size_t>(kQueueCap) * kItemWords);   // main and side stream
    const int dm = bit_dmax(d->d_max);
    if (pivot) {
        const int s_cap = s_cap_for(dm);
        w.binom_n = s_cap + 2;
        w.counts_len = w.binom_n + 1;
        if (d->d_max > KC_MAX_DMAX && d->d_max + 3 > w.counts_len) w.counts_len = d->d_max + 3;
        const size_t cells = static_cast<size_t>(w.binom_n + 1) * (w.binom_n + 1);
        w.counts = c.take<unsigned long long>(2 * static_cast<size_t>(w.counts_len));
        w.binom = c.take<unsigned long long>(2 * cells);
        w.big = c.take<unsigned char>(cells);
        w.leaf_count = leaf_index((dm < kMidCap ? dm : kMidCap) + 3, 0);
        w.leaves = c.take<unsigned long long>(static_cast<size_t>(w.leaf_count));
        if (dm > kMidCap) {   // smaller roots keep their stacks on chip
            const int maxw = maxw_for(dm);
            w.slab_words = static_cast<size_t>(s_cap + 2) * piv_level_words(maxw);
            w.slabs = device_cus() * kPivBlocksPerCU * 4;
            w.gstack = c.take<unsigned int>(w.slab_words * w.slabs);
        }
    }
    if (d->d_max > KC_MAX_DMAX && d->d_max <= KC_MAX_DMAX_WIDE) {
        w.wide = c.take<int>(static_cast<size_t>(d->n > 0 ? d->n : 1));
        w.wslab_words = wide_slab_words(d->d_max);
        size_t slabs = kWideSlabBudget / (4 * w.wslab_words);
        const size_t most = static_cast<size_t>(device_cus()) * 2;
        if (slabs > most) slabs = most;
        if (slabs < 1) slabs = 1;
        w.nwslabs = static_cast<int>(slabs);
        w.wslabs = c.take<unsigned int>(w.wslab_words * slabs);
    }
    *bytes = c.bytes();
    return w;
}

// Wide roots (kc_wide.hip): counts the cliques whose lowest vertex has more
// than KC_MAX_DMAX out-neighbours, one vertex root per such vertex (the other
// kernels skip these vertices' vertex and edge roots).  mode 0: graph
// orientation with target k (adds to w.acc); 1: pivoting with target k (w.acc);
// 2: pivoting, every size (w.counts).
int wide_launch(const kc_dag* d, int k, int mode, const CountWs& w, const int* cancel, hipStream_t s);

// Launch description for the pivot kernels (kc_pivot.hip).
struct PivLaunch {
    int k;                // clique size (ignored when all)
    bool all;             // count every size
    bool ec;              // edge roots
    bool stats;
    bool steal;           // hand saved frames to idle wavefronts
    int share = 0;        // 0: the whole device; a server's query, 1: alone, 2: beside others
    int steal_every = 0;                   // 0: the default (kPivStealEvery)
    int steal_after = 0;                   // 0: the default of the root list and scheme
    const int* cancel = nullptr;   // caller's cancel flag (null: none)
    unsigned long long* local = nullptr;   // per-vertex counts of size k (input ids); null: totals
    const int* perm = nullptr;             // DAG id -> input id (local counts)
    int d_max;
    const int* row_ptr;
    const int* col;
    const int* src;
    CountWs w;
};

int pivot_binom_table(const CountWs& w, hipStream_t s);
int pivot_launch(const PivLaunch& L, bool heavy, hipStream_t s);

// Roots of at most kLightCap (light) or kMidCap (mid) candidates with the search state
// in registers (kc_pivot_reg.hip): leaves go to w.leaves, which the last launch
// turns into counts.
int pivot_reg_launch(const PivLaunch& L, bool mid, hipStream_t s);
int pivot_leaves_launch(const PivLaunch& L, hipStream_t s);
// LDS bytes per wavefront of such a launch (its share of the block's leaf counters among
// them), and the wavefronts that fit the device's compute units by LDS.
size_t pivot_reg_lds(bool mid, int share, int cu_lds, int* waves);

// Launch description for the lane-walk graph-orientation kernel (kc_lane.hip).
struct LaneLaunch {
    int k;
    bool ec;
    bool pair;            // pair tasks from a global per-root counter + helping
    bool stats;
    int maxw;             // bitset words per row of this list
    int list;             // list index (0..kWidthLists-1)
    const int* row_ptr;
    const int* col;
    const int* src;
    const int* lists;     // all width lists back to back
    const int* counts;    // ctl + CC_WN0
    int* head;            // ctl + CC_WH0 + list
    int* task_ctr;
    int* task_tot;
    int* active;
    bool steal = false;   // hand subtrees to idle wavefronts through a global queue (pair mode)
    bool helper = false;  // join a running launch of this list: help and take queued subtrees only
    int* qctl = nullptr;  // this list's queue control words (zero at launch)
    int* qready = nullptr;  // this list's ring slot sequence words (zero at launch)
    unsigned int* qitems = nullptr;
    int* flags = nullptr;   // CC_FLAGS word: kFlagStalled, kFlagCanceled
    int steal_every = kLaneStealEvery;
    int steal_after = kLaneStealAfter;
    const int* cancel = nullptr;   // caller's cancel flag (null: none)
    unsigned long long* acc;
    unsigned long long* stats_ptr;
    unsigned long long* iters_ptr = nullptr;
    unsigned long long* timing_ptr = nullptr;
    unsigned long long* cwords_ptr = nullptr;   // stats: counted cliques x root row words
    int* grid_out = nullptr;              // receives the launched grid (wavefronts)
    unsigned long long* gacc = nullptr;   // batched: per-graph counters
    const int* gid = nullptr;             // batched: graph of each DAG vertex
};

int lane_launch(const LaneLaunch& L, hipStream_t s);

// On-chip memory a kc_count call keeps resident while it runs (an estimate for
// admission): the LDS bytes of one wavefront of its dominant traversal kernel
// (the widest width list's lane walk, or the largest of the pivot launches, the middle
// and the heavy one together) times the wavefronts that kernel launches (at most one per
// root), capped at the device's LDS (kc_count.hip).  share: see PivLaunch.
size_t count_lds_demand(const kc_dag* d, int k, int pivot, int share);
size_t device_lds_bytes();

// Sub-wavefront group walk (k_go, Sec. 3.5) over one width list of a batched
// call, adding each root's count to its graph's counter (kc_count.hip).
struct GoBatchLaunch {
    int k;
    bool ec;
    int list;                  // width list index (bitset words per row = 2^list)
    int group;                 // lanes per group (2 .. 32)
    const int* row_ptr;
    const int* col;
    const int* src;
    const int* lists;          // all width lists back to back
    const int* list_counts;    // ctl + CC_WN0
    int* head;                 // ctl + CC_WH0 + list
    unsigned long long* acc;   // scratch counters of the launch
    int* flags;                // CC_FLAGS word
    unsigned long long* gacc;  // per-graph {lo, hi}
    const int* gid;            // graph of each DAG vertex
};

int go_batch_launch(const GoBatchLaunch& B, hipStream_t s);

// Graph orientation over sorted candidate lists and binary-search
// intersections instead of bitsets (kc_lists.hip; KC_OPT_NO_BITSETS).
int lists_launch(const kc_dag* d, int k, bool ec, const CountWs& w, const int* cancel, hipStream_t s);

// Per-vertex counts by graph orientation (kc_local.hip): zeroes `local` (n
// entries, input ids) and adds every vertex's k-clique count; w.ctl is zero at launch.
int local_orient_launch(const kc_dag* d, int k, bool ec, unsigned long long* local, const CountWs& w,
                        const int* cancel, hipStream_t s);

// k-clique listing by graph orientation (kc_local.hip): writes up to `cap` rows
// of k input ids into `list` and counts every k-clique into *listed (device,
// zero at launch); w.ctl is zero at launch.
int list_orient_launch(const kc_dag* d, int k, bool ec, int* list, long long cap, unsigned long long* listed,
                       const CountWs& w, const int* cancel, hipStream_t s);

// Capture-safe degree orientation (kc_orient.hip).
size_t orient_async_workspace(int n, int nnz);
int orient_degree_async(int n, int nnz, const int* row_ptr, const int* col, const int* voff, int ngraphs,
                        int max_degree, int* out_row_ptr, int* out_col, int* out_src, int* out_perm, void* ws,
                        hipStream_t s);

// Whether a width list runs by pair tasks: trees four levels deep from the second
// vertex task on (shallower ones are counted from vertex tasks), except that roots of
// at most 64 candidates are walked by vertex tasks at the least of these depths: their
// trees are too small to pay for the pair counters (list 1 of k = 7 with edge roots on a
// 1M-vertex power-law graph: 21 ms by pairs, 14.5 by vertices; at k = 8, 23.6 and 26.2).
inline bool pair_list(int k, bool ec, int list) {
    const int deep = (ec ? 3 : 2) + 4;
    return list >= 2 ? k >= deep : list == 1 && k > deep;
}

// LDS bytes one lane-walk wavefront needs for a list of `maxw` words per row.
inline size_t lane_lds_bytes(int maxw, int k, bool ec, bool pair) {
    const int s_cap = 32 * maxw;
    const int slot = maxw + 1;
    const int first = (ec ? 3 : 2) + (pair ? 1 : 0);
    const int words = 16 + s_cap + s_cap * lane_stride(maxw) + (pair ? s_cap + 1 : 0) + 64 * slot +
                      k_levels(k, first) * slot * 64;
    return static_cast<size_t>(words) * 4;
}

}  // namespace kc
