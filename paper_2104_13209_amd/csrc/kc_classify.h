// Width lists: root r goes to list j when its |S| needs 2^j words per bitset row (1, 2,
// 4, 8, 16 or 32), or to none.  Two launches over fixed shares of the roots: one counts
// every block's roots per list, the other adds up the counts before its own and writes
// the lists back to back, in increasing root order.  No atomics: one per wavefront and list
// on the list sizes (11.6 ns each, one line) took 4.3 ms of a batch of 10.5 million
// vertices, two passes of 360 us of 1M vertex roots, and 1.1 ms of 16M edge roots.
#pragma once

#include "kc_count_impl.h"

namespace kc {

constexpr int kListThreads = 256;
constexpr int kListUnroll = 4;

__device__ __forceinline__ int width_list(int bound) {
    return bound <= 32 ? 0 : bound <= 64 ? 1 : bound <= 128 ? 2 : bound <= 256 ? 3 : bound <= 512 ? 4 : 5;
}

// Roots of one block's share (a multiple of the roots of one step), and the blocks that
// have any: the 2,000 roots of a small count are two blocks, not 512 that all add up
// 512 counts per list.
__host__ __device__ __forceinline__ long long list_per_block(int nroots) {
    const long long step = kListThreads * kListUnroll;
    return ((static_cast<long long>(nroots) + kListBlocks - 1) / kListBlocks + step - 1) / step * step;
}

inline int list_blocks(int nroots) {
    const long long per = list_per_block(nroots);
    return nroots > 0 ? static_cast<int>((nroots + per - 1) / per) : 1;
}

// First root of block b's share.
__device__ __forceinline__ long long list_share(int nroots, int b) {
    const long long at = list_per_block(nroots) * b;
    return at < nroots ? at : nroots;
}

// list_of(r): the list of root r, -1 for none.
template <class ListOf>
__global__ void __launch_bounds__(kListThreads) k_lists_count(ListOf list_of, int nroots, int* bcnt) {
    __shared__ int tot[kWidthLists];
    if (threadIdx.x < kWidthLists) tot[threadIdx.x] = 0;
    __syncthreads();
    int cnt[kWidthLists];
#pragma unroll
    for (int j = 0; j < kWidthLists; j++) cnt[j] = 0;
    const long long end = list_share(nroots, blockIdx.x + 1);
    for (long long r = list_share(nroots, blockIdx.x) + threadIdx.x; r < end; r += kListThreads) {
        const int l = list_of(static_cast<int>(r));
#pragma unroll
        for (int j = 0; j < kWidthLists; j++) cnt[j] += l == j;
    }
#pragma unroll
    for (int j = 0; j < kWidthLists; j++) {
        const int c = wave_sum_dpp(cnt[j]);
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(&tot[j], c);
    }
    __syncthreads();
    if (threadIdx.x < kWidthLists) bcnt[threadIdx.x * kListBlocks + blockIdx.x] = tot[threadIdx.x];
}

template <class ListOf>
__global__ void __launch_bounds__(kListThreads) k_lists_fill(ListOf list_of, int nroots, const int* __restrict__ bcnt,
                                                            int* lists, int* ctl) {
    constexpr int NW = kListThreads / 64;
    __shared__ int sums[2 * kWidthLists];
    __shared__ int wcnt[kListUnroll * NW][kWidthLists];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < 2 * kWidthLists) sums[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kWidthLists; j++) {
        int before = 0, all = 0;
        for (int b = threadIdx.x; b < static_cast<int>(gridDim.x); b += kListThreads) {
            const int x = bcnt[j * kListBlocks + b];
            all += x;
            before += b < static_cast<int>(blockIdx.x) ? x : 0;
        }
        before = wave_sum_dpp(before);
        all = wave_sum_dpp(all);
        if (lane == 0) {
            atomicAdd(&sums[j], before);
            atomicAdd(&sums[kWidthLists + j], all);
        }
    }
    __syncthreads();
    int at[kWidthLists];
    int run = 0;
#pragma unroll
    for (int j = 0; j < kWidthLists; j++) {
        at[j] = run + sums[j];
        run += sums[kWidthLists + j];
    }
    if (blockIdx.x == 0 && threadIdx.x < kWidthLists) ctl[CC_WN0 + threadIdx.x] = sums[kWidthLists + threadIdx.x];
    const long long end = list_share(nroots, blockIdx.x + 1);
    for (long long base = list_share(nroots, blockIdx.x); base < end; base += kListThreads * kListUnroll) {
        int l[kListUnroll];
#pragma unroll
        for (int u = 0; u < kListUnroll; u++) {
            const long long r = base + u * kListThreads + threadIdx.x;
            l[u] = r < end ? list_of(static_cast<int>(r)) : -1;
#pragma unroll
            for (int j = 0; j < kWidthLists; j++) {
                const int c = __popcll(__ballot(l[u] == j));
                if (lane == 0) wcnt[u * NW + wave][j] = c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kWidthLists; j++) {
            int pos = at[j];
#pragma unroll
            for (int u = 0; u < kListUnroll; u++) {
#pragma unroll
                for (int w = 0; w < NW; w++) {
                    const unsigned long long m = __ballot(l[u] == j);
                    if (w == wave && l[u] == j)
                        lists[pos + __popcll(m & lanemask_lt())] =
                            static_cast<int>(base + u * kListThreads + threadIdx.x);
                    pos += wcnt[u * NW + w][j];
                }
            }
            at[j] = pos;
        }
        __syncthreads();
    }
}

template <class ListOf>
int lists_launch_widths(const ListOf& list_of, int nroots, int* bcnt, int* lists, int* ctl, hipStream_t s) {
    k_lists_count<<<list_blocks(nroots), kListThreads, 0, s>>>(list_of, nroots, bcnt);
    k_lists_fill<<<list_blocks(nroots), kListThreads, 0, s>>>(list_of, nroots, bcnt, lists, ctl);
    KC_CHECK(hipGetLastError());
    return KC_OK;
}

}  // namespace kc
