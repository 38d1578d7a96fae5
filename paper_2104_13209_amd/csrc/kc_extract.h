// Induced sub-graph extraction into LDS bitsets (paper Sec. 2.4, 3.4), shared by
// the graph-orientation and pivoting traversals.
#pragma once

#include <climits>

#include "kc_internal.h"

namespace kc {

// A team is TEAM_LANES consecutive threads (one wavefront or a whole workgroup)
// that extracts one root's sub-graph together; tl is the thread's index in it.
template <int TW>
__device__ __forceinline__ void team_sync() {
    if (TW == 1) wave_sync_lds();
    else __syncthreads();
}

// Where x stands in the ascending y of the lanes (entries below x; at most 2 * STEP - 1).
template <int STEP>
__device__ __forceinline__ int lane_lower_bound(int y, int x) {
    int lo = 0;
#pragma unroll
    for (int step = STEP; step >= 1; step >>= 1) lo += __shfl(y, lo + step - 1, 64) < x ? step : 0;
    return lo;
}

// Candidate set S of a root, sorted ascending, into S[]; returns |S| through
// ctl_s (written by team lane 0) after a team sync.
//   VC root u:    S = N+(u)
//   EC root u->v: S = N+(u) cap N+(v), all of it past v in the row of u (one
//                 wavefront: 64 entries of N+(v) at a time, searched in 64 entries of
//                 N+(u) held a lane each, compacted in order with a ballot)
template <int TW, bool EC>
__device__ __forceinline__ void extract_set(int rid, const int* __restrict__ row_ptr, const int* __restrict__ col,
                                            const int* __restrict__ src, int tl, int* S, int* ctl_s) {
    constexpr int TEAM_LANES = 64 * TW;
    if (!EC) {
        const int b = row_ptr[rid], e = row_ptr[rid + 1];
        for (int j = tl; j < e - b; j += TEAM_LANES) S[j] = col[b + j];
        if (tl == 0) *ctl_s = e - b;
    } else if (tl < 64) {
        const int lane = tl;
        const int u = src[rid], v = col[rid];
        const int ub = rid + 1, ue = row_ptr[u + 1];
        const int vb = row_ptr[v], ve = row_ptr[v + 1];
        const int y0 = ub + lane < ue ? col[ub + lane] : INT_MAX;
        int cnt = 0;
        for (int j0 = vb; j0 < ve; j0 += 64) {
            const int x = j0 + lane < ve ? col[j0 + lane] : INT_MAX;
            const int first = __builtin_amdgcn_readfirstlane(x);
            const int last = __builtin_amdgcn_readlane(x, (ve - j0 < 64 ? ve - j0 : 64) - 1);
            bool hit = false;
            for (int t0 = ub; t0 < ue; t0 += 64) {
                const int y = t0 == ub ? y0 : t0 + lane < ue ? col[t0 + lane] : INT_MAX;
                if (__builtin_amdgcn_readfirstlane(y) > last) break;
                if (__builtin_amdgcn_readlane(y, 63) < first) continue;
                hit |= __shfl(y, lane_lower_bound<32>(y, x), 64) == x && x != INT_MAX;
            }
            const unsigned long long mk = __ballot(hit);
            if (hit) S[cnt + __popcll(mk & lanemask_lt())] = x;
            cnt += __popcll(mk);
        }
        if (lane == 0) *ctl_s = cnt;
    }
    team_sync<TW>();
}

// Bitset rows over S (row stride `stride` words, rows 0..s-1 zeroed first):
//   directed (UND = false): bit j of row i  <=>  S[j] in N+(S[i])  (j > i only)
//   undirected (UND = true): additionally bit i of row j for every such pair.
// Bits come from binary searches of each out-neighbour of S[i] in S[i+1..s),
// 16 lanes per row; rows are sorted, so the scan of N+(S[i]) stops past max S.
//
// extract_rows_small: the same for one wavefront and s <= 64.  S is held a lane each and
// searched with lane moves, and the rows' bounds are loaded a lane each: small roots are
// bound by instruction issue (some 1,500 wavefront instructions per root of up to 32
// candidates, two thirds of them here), and a lane-move search takes about half the
// instructions of a loop over LDS.
template <bool UND>
__device__ __forceinline__ void extract_rows_small(int s, const int* __restrict__ row_ptr, const int* __restrict__ col,
                                                   const int* S, unsigned int* B, int stride) {
    const int lane = __lane_id(), gl = lane & 15;
    for (int w = lane; w < s * stride; w += 64) B[w] = 0u;
    const int mine = lane < s ? S[lane] : INT_MAX;
    int b = 0, e = 0;
    if (lane + 1 < s) {                               // the last row has no out-neighbour in S
        b = row_ptr[mine];
        e = row_ptr[mine + 1];
    }
    const int smax = s > 0 ? __builtin_amdgcn_readlane(mine, s - 1) : 0;
    wave_sync_lds();
    for (int q = 0; q + 1 < s; q += 4) {
        const int i = q + (lane >> 4);
        const int ge = __shfl(e, i, 64);
        int j = __shfl(b, i, 64) + gl;
        int next = j < ge ? col[j] : INT_MAX;
        for (;;) {
            const int x = next;
            j += 16;
            next = j < ge ? col[j] : INT_MAX;
            const int lo = s <= 32 ? lane_lower_bound<16>(mine, x) : lane_lower_bound<32>(mine, x);
            if (__shfl(mine, lo, 64) == x && x != INT_MAX) {
                atomicOr(&B[i * stride + (lo >> 5)], 1u << (lo & 31));
                if (UND) atomicOr(&B[lo * stride + (i >> 5)], 1u << (i & 31));
            }
            if (__ballot(x < smax) == 0ull) break;    // every row is past its end or S's
        }
    }
    wave_sync_lds();
}

template <int TW, bool UND>
__device__ __forceinline__ void extract_rows(int s, const int* __restrict__ row_ptr, const int* __restrict__ col,
                                             int tl, const int* S, unsigned int* B, int stride) {
    constexpr int TEAM_LANES = 64 * TW;
    constexpr int XG = 16;
    if (TW == 1 && __builtin_amdgcn_readfirstlane(s) <= 64) {
        extract_rows_small<UND>(__builtin_amdgcn_readfirstlane(s), row_ptr, col, S, B, stride);
        return;
    }
    for (int w = tl; w < s * stride; w += TEAM_LANES) B[w] = 0u;
    team_sync<TW>();
    const int smax = s > 0 ? S[s - 1] : 0;
    for (int i = tl / XG; i < s; i += TEAM_LANES / XG) {
        const int w = S[i];
        const int b = row_ptr[w], e = row_ptr[w + 1];
        for (int j = b + (tl % XG); j < e; j += XG) {
            const int x = col[j];
            if (x > smax) break;
            int lo = i + 1, hi = s;
            while (lo < hi) {
                int mid = (lo + hi) >> 1;
                if (S[mid] < x) lo = mid + 1; else hi = mid;
            }
            if (lo < s && S[lo] == x) {
                atomicOr(&B[i * stride + (lo >> 5)], 1u << (lo & 31));
                if (UND) atomicOr(&B[lo * stride + (i >> 5)], 1u << (i & 31));
            }
        }
    }
    team_sync<TW>();
}

}  // namespace kc
