// Pivoting traversal (paper Sec. 2.3 Fig. 3, as described in kc_pivot.hip) for roots of
// at most 128 candidates, with the whole search state in registers.
//
// A root's undirected rows fit the wavefront: lane l holds the row of vertex l (and of
// vertex l + 64), and every set of the search is a wave-uniform 64- or 128-bit mask
// in scalar registers.  Scoring the pivots is one AND + popcount per lane and a
// lane-move maximum; a child's candidates are a v_readlane of the branch vertex's row and
// a scalar AND; the stack is an array over lanes (level = lane), written by a
// conditional move and read with v_readlane.  So a node touches no memory: the version with
// LDS rows, LDS member lists and LDS or global-memory frames spent its time on chains of
// dependent accesses (VALU issue on 21-45% of the cycles).
//
// Leaves are counted, not evaluated: a leaf with nh holds and np pivots adds one to
// an LDS counter of its block (np + nh, nh), and a final kernel weighs the counters
// with the binomials.  That keeps the 128-bit table reads and additions out of the
// walk (np + 1 of them per leaf when every size is counted).
//
// Work distribution, the queue of handed-over frames and its termination are those
// of kc_pivot.hip, but the queue is split in kRegShards independent ones, each of the blocks
// of one XCD: every access to a queue's control words waits for the others' (11.6 ns
// each), and thousands of wavefronts look at them.  A wavefront hands over only
// frames of at least kRegMinFrame candidates.  Frames whose last branch vertex has been taken are not saved, and
// a set of vertices adjacent to all others of the node (each would be the only
// branch of its node) becomes that many pivots at once.
//
// Count-all of the dense-core graph (500k vertices, 50 communities of 60-80 vertices at
// density 0.9; 6.0e8 nodes under light roots, 2.1e8 under larger ones), vertex roots,
// ms: 561 with the LDS rows; 685 with registers and the one queue of before, whose
// control words bound it; 430 looking at it every 1024 nodes; 136 with eight queues and
// the smallest frame, looking every 256.  Light roots (260 SIMD cycles a node) are bound by
// scalar issue, 72% of the cycles with vertex roots and 86% with edge roots; larger
// ones (600) issue vector instructions on 56% and scalar ones on 36%, with 11 of 16 possible wavefronts per
// CU: each waits for its own chain.
// Sweep of (nodes between looks, before the first handoff) -> light + heavy ms:
// (128, 1024) 67 + 88, (256, 1024) 71 + 62, (256, 4096) 64 + 87, (256, 16384) 94 + 145,
// (1024, 1024) 63 + 74.
#include "kc_count_impl.h"
#include "kc_extract.h"

namespace kc {
namespace {

// Most roots claimed at once: light roots (at most 64 candidates), larger ones.
constexpr int kRegRootChunkLight = 4, kRegRootChunkMid = 1;

// A consumer extracts the frame's root again (tens of microseconds), and a frame of few
// candidates holds few nodes.
constexpr int kRegMinFrame = 32;
constexpr int kShardCap = kQueueCap / kRegShards;

struct PivRegParams {
    int k;
    int steal_every, steal_after, max_waiters;
    bool steal;
    const int* __restrict__ row_ptr;
    const int* __restrict__ col;
    const int* __restrict__ src;
    const int* __restrict__ roots;
    int root_step;                           // 1, or -1: the list grows downwards from `roots`
    const int* __restrict__ nroots;
    int* head;
    int* flags;
    unsigned long long* hist;                // leaf counters (see leaf_index)
    unsigned long long* stats;               // [nodes, words]
    int* qctl;
    int* qready;
    unsigned int* qitems;
    const int* cancel;
};

__device__ __forceinline__ unsigned int rdl(unsigned int v, int l) {
    return static_cast<unsigned int>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ unsigned long long rdl64(unsigned int lo, unsigned int hi, int l) {
    return static_cast<unsigned long long>(rdl(lo, l)) | (static_cast<unsigned long long>(rdl(hi, l)) << 32);
}
// v with lane l's word replaced by x.
__device__ __forceinline__ unsigned int wrl(unsigned int v, unsigned int x, int l) {
    return static_cast<int>(__lane_id()) == l ? x : v;
}

// A wave-uniform vertex set of H * 64 bits.
template <int H>
struct Set {
    unsigned long long w[H];
    __device__ __forceinline__ bool any() const {
        unsigned long long x = w[0];
#pragma unroll
        for (int h = 1; h < H; h++) x |= w[h];
        return x != 0ull;
    }
    __device__ __forceinline__ int size() const {
        int n = 0;
#pragma unroll
        for (int h = 0; h < H; h++) n += __popcll(w[h]);
        return n;
    }
    // lowest member, removed (not empty)
    __device__ __forceinline__ int take() {
        if (H == 1 || w[0]) {
            const int v = __ffsll(static_cast<long long>(w[0])) - 1;
            w[0] &= w[0] - 1ull;
            return v;
        }
        const int v = __ffsll(static_cast<long long>(w[H - 1])) - 1;
        w[H - 1] &= w[H - 1] - 1ull;
        return 64 * (H - 1) + v;
    }
    __device__ __forceinline__ void drop(int v) {
        if (H == 1 || v < 64) w[0] &= ~(1ull << (v & 63));
        else w[H - 1] &= ~(1ull << (v & 63));
    }
};

// Rows of the lane's vertices: r[i][h], words of vertex 64 i + lane.
template <int H>
struct Rows {
    unsigned int lo[H][H], hi[H][H];
    __device__ __forceinline__ Set<H> of(int v) const {
        Set<H> s;
#pragma unroll
        for (int h = 0; h < H; h++) {
            if (H == 1 || v < 64) s.w[h] = rdl64(lo[0][h], hi[0][h], v & 63);
            else s.w[h] = rdl64(lo[H - 1][h], hi[H - 1][h], v & 63);
        }
        return s;
    }
};

// Saved frames, one per lane and bank: I without the branch vertices already taken,
// the branch vertices left, and pivot | pivots << 8 | holds << 16.
template <int H>
struct Frames {
    unsigned int i_lo[H][H], i_hi[H][H], p_lo[H][H], p_hi[H][H], meta[H];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int b = 0; b < H; b++) {
            meta[b] = 0u;
#pragma unroll
            for (int h = 0; h < H; h++) i_lo[b][h] = i_hi[b][h] = p_lo[b][h] = p_hi[b][h] = 0u;
        }
    }
    template <int B>
    __device__ __forceinline__ void save_bank(int l, const Set<H>& I, const Set<H>& Pr, unsigned int m) {
#pragma unroll
        for (int h = 0; h < H; h++) {
            i_lo[B][h] = wrl(i_lo[B][h], static_cast<unsigned int>(I.w[h]), l);
            i_hi[B][h] = wrl(i_hi[B][h], static_cast<unsigned int>(I.w[h] >> 32), l);
            p_lo[B][h] = wrl(p_lo[B][h], static_cast<unsigned int>(Pr.w[h]), l);
            p_hi[B][h] = wrl(p_hi[B][h], static_cast<unsigned int>(Pr.w[h] >> 32), l);
        }
        meta[B] = wrl(meta[B], m, l);
    }
    template <int B>
    __device__ __forceinline__ void load_bank(int l, Set<H>& I, Set<H>& Pr, unsigned int& m) const {
#pragma unroll
        for (int h = 0; h < H; h++) {
            I.w[h] = rdl64(i_lo[B][h], i_hi[B][h], l);
            Pr.w[h] = rdl64(p_lo[B][h], p_hi[B][h], l);
        }
        m = rdl(meta[B], l);
    }
    __device__ __forceinline__ void save(int level, const Set<H>& I, const Set<H>& Pr, unsigned int m) {
        if (H == 1 || level < 64) save_bank<0>(level & 63, I, Pr, m);
        else save_bank<H - 1>(level & 63, I, Pr, m);
    }
    __device__ __forceinline__ void load(int level, Set<H>& I, Set<H>& Pr, unsigned int& m) const {
        if (H == 1 || level < 64) load_bank<0>(level & 63, I, Pr, m);
        else load_bank<H - 1>(level & 63, I, Pr, m);
    }
    // shallowest frame below `level` with branch vertices and enough candidates left, or -1
    __device__ __forceinline__ int shallowest(int level, int lane) const {
#pragma unroll
        for (int b = 0; b < H; b++) {
            unsigned int x = 0u;
            int n = 0;
#pragma unroll
            for (int h = 0; h < H; h++) {
                x |= p_lo[b][h] | p_hi[b][h];
                n += __popc(i_lo[b][h]) + __popc(i_hi[b][h]);
            }
            const unsigned long long m = __ballot(x != 0u && n >= kRegMinFrame && 64 * b + lane < level);
            if (m) return 64 * b + __ffsll(static_cast<long long>(m)) - 1;
        }
        return -1;
    }
};

// LDS words of one wavefront: control, S, rows.
template <int H>
constexpr int reg_wave_words() {
    return 8 + 64 * H + 64 * H * b_stride_of(2 * H);
}

// H: 64-bit words per set; EC: edge roots; ALL: every size (else size k); WPB:
// wavefronts per block, which share the leaf counters.
template <int H, bool EC, bool ALL, int WPB, bool STATS>
__global__ void __launch_bounds__(64 * WPB) k_piv_reg(PivRegParams P) {
    constexpr int CAP = 64 * H;                       // candidates
    constexpr int LEAVES = leaf_index(CAP + 2, 0) + CAP + 3;
    constexpr int STRIDE = b_stride_of(2 * H);
    extern __shared__ __align__(16) unsigned int lds_piv[];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    unsigned long long* hist = reinterpret_cast<unsigned long long*>(lds_piv);
    unsigned int* base = lds_piv + 2 * LEAVES + wv * reg_wave_words<H>();
    int* ctl = reinterpret_cast<int*>(base);
    int* S = reinterpret_cast<int*>(base + 8);
    unsigned int* A = base + 8 + CAP;
    const int k = P.k;
    const int nroots = *P.nroots;
    const int nh_root = EC ? 2 : 1;
    const int shard = blockIdx.x % kRegShards;
    int* q = P.qctl + shard * kShardLine;
    int* qready = P.qready + shard * kShardCap;
    unsigned int* qitems = P.qitems + static_cast<size_t>(shard) * kShardCap * kItemWords;

    for (int i = threadIdx.x; i < LEAVES; i += 64 * WPB) hist[i] = 0ull;
    __syncthreads();
    // an earlier launch of the call stalled or was canceled: no work here
    int stop = 0;
    if (lane == 0) {
        stop = (ld_acquire(P.flags) & (kFlagStalled | kFlagCanceled)) != 0;
        if (!stop && cancel_requested(P.cancel)) {
            atomicOr(P.flags, kFlagCanceled);
            stop = 1;
        }
    }
    stop = __builtin_amdgcn_readfirstlane(stop);

    const bool steal = P.steal;
    unsigned long long nodes = 0, words_done = 0;
    if (!stop && steal && lane == 0) atomicAdd(&q[Q_ROOTING], 1);
    RootClaims rc;
    bool roots_done = false, hungry = false;
    int cur = -1, chk = 0, cpoll = 0;                 // root whose rows are in the registers
    Rows<H> R;
    Frames<H> F;
    F.clear();

    auto leaf = [&](int np, int nh) {
        if (!ALL && (nh > k || nh + np < k)) return;
        if (lane == 0) atomicAdd(&hist[leaf_index(nh + np, nh)], 1ull);
    };

    while (!stop) {
        int slot = -1;
        bool from_item = false;
        Set<H> I, Pr;
#pragma unroll
        for (int h = 0; h < H; h++) I.w[h] = Pr.w[h] = 0ull;
        int np = 0, nh = nh_root, level = 0, p = 0;
        if (!roots_done) {
            slot = __builtin_amdgcn_readfirstlane(claim_root(rc, P.head, nroots, blockIdx.x * WPB + wv,
                                                             gridDim.x * WPB, H == 1 ? kRegRootChunkLight : kRegRootChunkMid));
            if (slot < 0) {
                roots_done = true;
                if (!steal) break;
                int stay = 1;
                if (lane == 0) {
                    __hip_atomic_fetch_add(&q[Q_ROOTING], -1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                    if (atomicAdd(&q[Q_HUNGRY], 1) >= P.max_waiters) {
                        atomicAdd(&q[Q_HUNGRY], -1);
                        stay = 0;
                    }
                }
                if (!__builtin_amdgcn_readfirstlane(stay)) break;
                hungry = true;
                continue;
            }
        } else {
            // wait for a queued frame, or for the end of all work
            int idx = -1, state = 0, backoff = 0;
            unsigned long long sig = ~0ull, t_sig = 0;
            for (;;) {
                // all control words in one request: they are on one line, where every
                // access waits for the others'.  The end is taken from a second look,
                // whose loads are ordered (rooting before pending).
                const int qw = lane < kQueueCtlWords ? ld_acquire(&q[lane]) : 0;
                const int h = __builtin_amdgcn_readlane(qw, Q_HEAD), t = __builtin_amdgcn_readlane(qw, Q_TAIL);
                if (lane == 0) {
                    if (h < t) {
                        if (atomicCAS(&q[Q_HEAD], h, h + 1) == h) idx = h;
                    } else {
                        int rooting = __builtin_amdgcn_readlane(qw, Q_ROOTING);
                        int pend = __builtin_amdgcn_readlane(qw, Q_PENDING);
                        if (rooting == 0 && pend == 0) {
                            rooting = __hip_atomic_load(&q[Q_ROOTING], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                            pend = __hip_atomic_load(&q[Q_PENDING], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        const unsigned long long now = __builtin_amdgcn_s_memrealtime();
                        const unsigned long long sg = (static_cast<unsigned long long>(static_cast<unsigned int>(t)) << 40) ^
                                                      (static_cast<unsigned long long>(static_cast<unsigned int>(pend)) << 20) ^
                                                      static_cast<unsigned int>(rooting);
                        if (sg != sig) { sig = sg; t_sig = now; }
                        if ((rooting == 0 && pend == 0) || (ld_acquire(P.flags) & (kFlagStalled | kFlagCanceled))) state = 1;
                        else if (now - t_sig > kStallTicks) state = 2;
                    }
                }
                idx = __builtin_amdgcn_readfirstlane(idx);
                state = __builtin_amdgcn_readfirstlane(state);
                if (idx >= 0 || state != 0) break;
                if (backoff < 4) backoff++;
                for (int i = 0; i < (1 << backoff); i++) __builtin_amdgcn_s_sleep(127);
            }
            if (idx < 0) {
                if (state == 2 && lane == 0) atomicOr(P.flags, kFlagStalled);
                break;
            }
            if (hungry && lane == 0) atomicAdd(&q[Q_HUNGRY], -1);
            hungry = false;
            const int qs = idx & (kShardCap - 1);
            const int gen = idx - qs;
            const unsigned int* it = qitems + static_cast<size_t>(qs) * kItemWords;
            int ok = 1;
            if (lane == 0) {
                int spins = 0;
                while (__hip_atomic_load(&qready[qs], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != gen + 1) {
                    if (++spins > kReadySpins) { ok = 0; break; }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
            if (!__builtin_amdgcn_readfirstlane(ok)) {
                if (lane == 0) atomicOr(P.flags, kFlagStalled);
                break;
            }
            const unsigned int x = lane < 2 + 4 * H ? ld_acquire(&it[lane]) : 0u;
            slot = static_cast<int>(rdl(x, 0));
            const unsigned int m = rdl(x, 1);
            p = m & 0xff;
            np = (m >> 8) & 0xff;
            nh = (m >> 16) & 0xff;
#pragma unroll
            for (int h = 0; h < H; h++) {
                I.w[h] = rdl(x, 2 + 2 * h) | (static_cast<unsigned long long>(rdl(x, 3 + 2 * h)) << 32);
                Pr.w[h] = rdl(x, 2 + 2 * H + 2 * h) | (static_cast<unsigned long long>(rdl(x, 3 + 2 * H + 2 * h)) << 32);
            }
            if (lane == 0)   // the wavefront's loads are done: the slot is free for the next generation
                __hip_atomic_store(&qready[qs], gen + kShardCap, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            from_item = true;
        }
        // the root's rows (kept when the next frame is of the same root)
        if (slot != cur) {
            extract_set<1, EC>(P.roots[P.root_step * slot], P.row_ptr, P.col, P.src, lane, S, &ctl[1]);
            extract_rows<1, true>(ctl[1], P.row_ptr, P.col, lane, S, A, STRIDE);
            const int n = ctl[1];
#pragma unroll
            for (int i = 0; i < H; i++) {
                const bool in = 64 * i + lane < n;
#pragma unroll
                for (int h = 0; h < H; h++) {
                    R.lo[i][h] = in ? A[(64 * i + lane) * STRIDE + 2 * h] : 0u;
                    R.hi[i][h] = in ? A[(64 * i + lane) * STRIDE + 2 * h + 1] : 0u;
                }
            }
            cur = slot;
        }
        const int s = __builtin_amdgcn_readfirstlane(ctl[1]);
        const unsigned long long W = static_cast<unsigned long long>((s + 31) >> 5);
        bool entering = !from_item;                   // a pivot is still to be chosen
        if (!from_item) {
#pragma unroll
            for (int h = 0; h < H; h++) {
                const int left = s - 64 * h;
                I.w[h] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1ull : 0ull;
            }
            if (s == 0) {
                leaf(0, nh_root);
                wave_sync_lds();
                continue;
            }
        }
        int run_nodes = 0;
        for (;;) {
            if (entering) {
                entering = false;
                // score every candidate: the lane's rows against I
                unsigned int best = 0u, sc[H];
                bool in[H];
#pragma unroll
                for (int i = 0; i < H; i++) {
                    in[i] = (I.w[i] >> lane) & 1ull;
                    sc[i] = 0u;
#pragma unroll
                    for (int h = 0; h < H; h++)
                        sc[i] += __popc(R.lo[i][h] & static_cast<unsigned int>(I.w[h])) +
                                 __popc(R.hi[i][h] & static_cast<unsigned int>(I.w[h] >> 32));
                    const unsigned int key = ((sc[i] + 1u) << 8) | static_cast<unsigned int>(255 - 64 * i - lane);
                    best = in[i] && key > best ? key : best;
                }
                best = wave_max_dpp(best);
                const int m = I.size();
                p = 255 - static_cast<int>(best & 255u);
                if (static_cast<int>(best >> 8) == m) {
                    // vertices adjacent to all others: one pivot level each, without branches
                    int d = 0;
#pragma unroll
                    for (int i = 0; i < H; i++) {
                        const unsigned long long dm = __ballot(in[i] && static_cast<int>(sc[i]) == m - 1);
                        d += __popcll(dm);
                        I.w[i] &= ~dm;
                    }
                    np += d;
                    if (STATS) {
                        nodes += static_cast<unsigned long long>(d);
                        for (int i = 0; i < d; i++) words_done += static_cast<unsigned long long>(m - i + 2) * W;
                    }
                    if (I.any()) entering = true;
                    else leaf(np, nh);
                } else {
                    const Set<H> ap = R.of(p);
#pragma unroll
                    for (int h = 0; h < H; h++) Pr.w[h] = I.w[h] & ~ap.w[h];
                    // scoring reads |I| rows of W words; P one more
                    if (STATS) words_done += static_cast<unsigned long long>(m + 1) * W;
                }
                if (entering) continue;
            }
            // cancellation: abandon the tree (the call's result is discarded)
            if (P.cancel && ++cpoll == kCancelEvery) {
                cpoll = 0;
                int c = 0;
                if (lane == 0 && (cancel_requested(P.cancel) || (ld_acquire(P.flags) & kFlagCanceled))) {
                    atomicOr(P.flags, kFlagCanceled);
                    c = 1;
                }
                if (__builtin_amdgcn_readfirstlane(c)) {
                    stop = 1;
                    break;
                }
            }
            if (steal && ++chk >= P.steal_every) {
                run_nodes += chk;
                chk = 0;
                if (run_nodes >= P.steal_after) {
                    const int qw = lane < kQueueCtlWords ? ld_acquire(&q[lane]) : 0;
                    const int want = __builtin_amdgcn_readlane(qw, Q_HUNGRY) -
                                     (__builtin_amdgcn_readlane(qw, Q_TAIL) - __builtin_amdgcn_readlane(qw, Q_HEAD));
                    const int fl = want > 0 ? F.shallowest(level, lane) : -1;
                    if (fl >= 0) {
                        int t0 = -1;
                        if (lane == 0) {
                            const int h = ld_acquire(&q[Q_HEAD]);
                            int t = ld_acquire(&q[Q_TAIL]);
                            for (;;) {
                                if (t + 1 - h > kShardCap) { t = -1; break; }
                                const int prev = atomicCAS(&q[Q_TAIL], t, t + 1);
                                if (prev == t) break;
                                t = prev;
                            }
                            if (t >= 0) atomicAdd(&q[Q_PENDING], 1);
                            t0 = t;
                        }
                        t0 = __builtin_amdgcn_readfirstlane(t0);
                        if (t0 >= 0) {
                            const int qs = t0 & (kShardCap - 1);
                            const int gen = t0 - qs;
                            unsigned int* it = qitems + static_cast<size_t>(qs) * kItemWords;
                            int ok = 1;
                            if (lane == 0) {
                                int spins = 0;
                                while (__hip_atomic_load(&qready[qs], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != gen) {
                                    if (++spins > kReadySpins) { ok = 0; break; }
                                    __builtin_amdgcn_s_sleep(2);
                                }
                            }
                            ok = __builtin_amdgcn_readfirstlane(ok);
                            if (!ok) {
                                if (lane == 0) atomicOr(P.flags, kFlagStalled);
                            } else {
                                Set<H> fi, fp, none;
                                unsigned int m;
                                F.load(fl, fi, fp, m);
                                if (lane == 0) {
                                    it[0] = static_cast<unsigned int>(slot);
                                    it[1] = m;
#pragma unroll
                                    for (int h = 0; h < H; h++) {
                                        it[2 + 2 * h] = static_cast<unsigned int>(fi.w[h]);
                                        it[3 + 2 * h] = static_cast<unsigned int>(fi.w[h] >> 32);
                                        it[2 + 2 * H + 2 * h] = static_cast<unsigned int>(fp.w[h]);
                                        it[3 + 2 * H + 2 * h] = static_cast<unsigned int>(fp.w[h] >> 32);
                                    }
                                    __hip_atomic_store(&qready[qs], gen + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                                }
                                // the frame's remaining branches now belong to the item
#pragma unroll
                                for (int h = 0; h < H; h++) none.w[h] = 0ull;
                                F.save(fl, fi, none, m);
                            }
                        }
                    }
                }
            }
            if (!Pr.any()) {
                if (level == 0) break;
                level--;
                unsigned int m;
                F.load(level, I, Pr, m);
                p = m & 0xff;
                np = (m >> 8) & 0xff;
                nh = m >> 16;
                continue;
            }
            const int v = Pr.take();
            const int np2 = np + (v == p ? 1 : 0);
            const int nh2 = nh + (v != p ? 1 : 0);
            Set<H> Y = R.of(v);
#pragma unroll
            for (int h = 0; h < H; h++) Y.w[h] &= I.w[h];
            I.drop(v);                                  // later branches exclude v
            if (!ALL && nh2 > k) continue;              // stopping criterion: holds <= k
            if (STATS) {
                nodes += 1;
                words_done += W;
            }
            if (!Y.any()) {
                leaf(np2, nh2);
                continue;
            }
            // no leaf below reaches size k with too few vertices left
            if (!ALL && nh2 + np2 + Y.size() < k) continue;
            if (Pr.any()) {
                F.save(level, I, Pr, static_cast<unsigned int>(p | (np << 8) | (nh << 16)));
                level++;
            }
            I = Y;
#pragma unroll
            for (int h = 0; h < H; h++) Pr.w[h] = 0ull;
            np = np2;
            nh = nh2;
            entering = true;
        }
        wave_sync_lds();
        if (stop) break;   // waiting wavefronts leave on the flag
        if (from_item) {
            if (lane == 0) {
                __hip_atomic_fetch_add(&q[Q_PENDING], -1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                atomicAdd(&q[Q_HUNGRY], 1);             // back to waiting for frames
            }
            hungry = true;
        }
    }
    if (hungry && lane == 0) atomicAdd(&q[Q_HUNGRY], -1);

    __syncthreads();
    for (int i = threadIdx.x; i < LEAVES; i += 64 * WPB) {
        const unsigned long long x = hist[i];
        if (x) atomicAdd(&P.hist[i], x);
    }
    if (STATS && lane == 0) {
        atomicAdd(P.stats, nodes);
        atomicAdd(P.stats + 1, words_done);
    }
}

// Block b adds the leaves' contributions to size `first` + b: a leaf with nh holds and np
// pivots stands for C(np, size - nh) cliques of that size (Sec. 2.3).
__global__ void __launch_bounds__(256) k_piv_leaves(int first, int most, int binom_n,
                                                   const unsigned long long* __restrict__ hist,
                                                   const unsigned long long* __restrict__ binom,
                                                   const unsigned char* __restrict__ big, unsigned long long* out,
                                                   int out_step, int* flags) {
    const int size = first + blockIdx.x;
    const int N1 = binom_n + 1;
    unsigned __int128 sum = 0;
    int ovf = 0;
    for (int t = size; t <= most; t++) {
        for (int nh = threadIdx.x; nh <= size && nh <= t; nh += blockDim.x) {
            const unsigned long long c = hist[leaf_index(t, nh)];
            if (c == 0ull) continue;
            const size_t ix = static_cast<size_t>(t - nh) * N1 + (size - nh);
            ovf |= big[ix];
            const unsigned __int128 hi = static_cast<unsigned __int128>(binom[2 * ix + 1]) * c;
            const unsigned __int128 lo = static_cast<unsigned __int128>(binom[2 * ix]) * c;
            ovf |= (hi >> 64) != 0;
            const unsigned __int128 x = lo + (hi << 64);
            ovf |= x < lo;
            const unsigned __int128 y = sum + x;
            ovf |= y < sum;
            sum = y;
        }
    }
    if (sum && atomic_add_u128(out + static_cast<size_t>(out_step) * blockIdx.x,
                               out + static_cast<size_t>(out_step) * blockIdx.x + 1,
                               static_cast<unsigned long long>(sum), static_cast<unsigned long long>(sum >> 64)))
        ovf = 1;
    if (ovf) atomicOr(flags, kFlagBigBinom);
}

// LDS bytes of a block: leaf counters, then the wavefronts' regions.
template <int H, int WPB>
constexpr size_t reg_block_lds() {
    return (2 * static_cast<size_t>(leaf_index(64 * H + 2, 0) + 64 * H + 3) + static_cast<size_t>(WPB) * reg_wave_words<H>()) * 4;
}

// Wavefronts per block of the light and of the middle launch.
constexpr int kRegLightWaves = 4, kRegMidWaves = 16;

// One block in this many of those that fit the device is launched, by PivLaunch::share: a
// block keeps its LDS until its longest root is done, and the server admits queries by LDS.  48
// mixed queries over 8 graphs of 30,000 vertices: 25.7 ms with all blocks (one pivot query
// at a time), 20.9 with a half of either launch, 18.9 with a quarter of the light one's
// (19.9 with a quarter of both); 67, 38, 26 and 26 ms where all are pivot queries.  A query
// that is alone loses little by the half (k = 3 on 1M vertices 3.7 -> 4.2 ms, most
// nothing), and others can join it.
constexpr int kRegLightShare[3] = {1, 2, 4}, kRegMidShare[3] = {1, 2, 2};

template <int H, bool EC, bool ALL, int WPB>
int launch_reg(const PivRegParams& P, bool stats, int share, hipStream_t s) {
    constexpr size_t lds = reg_block_lds<H, WPB>();
    auto kern = stats ? k_piv_reg<H, EC, ALL, WPB, true> : k_piv_reg<H, EC, ALL, WPB, false>;
    if (lds > 64 * 1024)
        KC_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     static_cast<int>(lds)));
    int occ = 0;
    KC_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 64 * WPB, lds));
    if (occ < 1) return KC_EUNSUPPORTED;
    kern<<<div_up(device_cus() * occ, share), 64 * WPB, lds, s>>>(P);
    KC_CHECK(hipGetLastError());
    return KC_OK;
}

}  // namespace

int pivot_reg_launch(const PivLaunch& L, bool mid, hipStream_t s) {
    const CountWs& w = L.w;
    const int queue = mid ? 2 : 0;
    PivRegParams P;
    P.k = L.k;
    P.steal_every = L.steal_every > 0 ? L.steal_every : kRegStealEvery;
    P.steal_after = L.steal_after > 0 ? L.steal_after : kRegStealAfter;
    P.max_waiters = kRegWaitersPerCU * device_cus() / kRegShards;
    P.steal = L.steal;
    P.row_ptr = L.row_ptr;
    P.col = L.col;
    P.src = L.src;
    P.roots = mid ? w.heavy + w.nroots_cap - 1 : w.light;
    P.root_step = mid ? -1 : 1;
    P.nroots = w.ctl + (mid ? CC_MID_N : CC_LIGHT_N);
    P.head = w.ctl + (mid ? CC_MID_HEAD : CC_LIGHT_HEAD);
    P.flags = w.ctl + CC_FLAGS;
    P.hist = w.leaves;
    P.stats = w.acc + (mid ? 4 : 2);
    P.qctl = w.qctl + kShardLine * kRegShards * queue;
    P.qready = w.qready + static_cast<size_t>(kQueueCap) * queue;
    P.qitems = w.qitems;   // the light launch has ended when the middle one begins; the heavy one has the other region
    P.cancel = L.cancel;
    constexpr int LW = kRegLightWaves, MW = kRegMidWaves;
    const int share = mid ? kRegMidShare[L.share] : kRegLightShare[L.share];
    if (mid) {
        if (L.ec) return L.all ? launch_reg<2, true, true, MW>(P, L.stats, share, s) : launch_reg<2, true, false, MW>(P, L.stats, share, s);
        return L.all ? launch_reg<2, false, true, MW>(P, L.stats, share, s) : launch_reg<2, false, false, MW>(P, L.stats, share, s);
    }
    if (L.ec) return L.all ? launch_reg<1, true, true, LW>(P, L.stats, share, s) : launch_reg<1, true, false, LW>(P, L.stats, share, s);
    return L.all ? launch_reg<1, false, true, LW>(P, L.stats, share, s) : launch_reg<1, false, false, LW>(P, L.stats, share, s);
}

size_t pivot_reg_lds(bool mid, int share, int cu_lds, int* waves) {
    const size_t block = mid ? reg_block_lds<2, kRegMidWaves>() : reg_block_lds<1, kRegLightWaves>();
    const int wpb = mid ? kRegMidWaves : kRegLightWaves;
    const int fit = device_cus() * static_cast<int>(static_cast<size_t>(cu_lds) / block);
    *waves = div_up(fit, mid ? kRegMidShare[share] : kRegLightShare[share]) * wpb;
    return block / wpb;
}

int pivot_leaves_launch(const PivLaunch& L, hipStream_t s) {
    const CountWs& w = L.w;
    const int cand = L.d_max < kMidCap ? L.d_max : kMidCap;
    const int most = cand + 2 < w.binom_n ? cand + 2 : w.binom_n;
    if (L.all) k_piv_leaves<<<most + 1, 256, 0, s>>>(0, most, w.binom_n, w.leaves, w.binom, w.big, w.counts, 2, w.ctl + CC_FLAGS);
    else if (L.k <= most)
        k_piv_leaves<<<1, 256, 0, s>>>(L.k, most, w.binom_n, w.leaves, w.binom, w.big, w.acc, 2, w.ctl + CC_FLAGS);
    KC_CHECK(hipGetLastError());
    return KC_OK;
}

}  // namespace kc
