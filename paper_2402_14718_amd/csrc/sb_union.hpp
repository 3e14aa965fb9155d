// Walk of the union of R consecutive rows' columns, a lane per row, for the
// lists that the blocked streaming steps make once per solve.
//
// The walk is a chain (smallest next column, advance the rows that hold it),
// so it is bound by latency and wants many groups in flight: with a lane per
// row, 208710 rows make 3261 waves, and the rows of a wave (consecutive, so
// one run of memory) come through LDS, where they fit.  The matrix-core lists
// of 208710 rows of 55 couplings took 5.2 ms with a thread per block, 0.82
// with a lane per row and the entries from memory, and take 0.80; the quads'
// 2.6, 0.53 and 0.46 (the densest rows set the time: unions of 1253 columns).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sbt {

namespace {

constexpr int kNoColumn = INT32_MAX;

template <int CTRL>
__device__ __forceinline__ int min_dpp(int v) {
    return min(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false));
}

// The smallest value of each aligned group of R = 4 or 16 lanes.
template <int R>
__device__ __forceinline__ int group_min(int v) {
    static_assert(R == 4 || R == 16, "groups are quads or rows of lanes");
    v = min_dpp<0xB1>(v);  // quad_perm 1 0 3 2
    v = min_dpp<0x4E>(v);  // quad_perm 2 3 0 1
    if constexpr (R == 16) {
        v = min_dpp<0x141>(v);  // row_half_mirror
        v = min_dpp<0x140>(v);  // row_mirror
    }
    return v;
}

// Columns of a wave's rows in LDS, at most kWalkWords of them: the 64 rows of
// a workgroup of one wave.
constexpr int kWalkThreads = 64;
constexpr int kWalkWords = 5120;

// A row (padded CSR; its own column marks the padding) in column order, read
// from LDS where the wave's rows fit there.
struct RowWalk {
    const int *col, *lds;
    int pos, end, head, next, base;  // head: column at pos; next: the one after it; base: the wave's first entry
    bool staged;

    // every lane of the wave; i: this lane's row, consecutive over the wave
    __device__ __forceinline__ RowWalk(int n, const int *prow, const int *pcol, int i, int *words)
        : col(pcol), lds(words) {
        const int i0 = __builtin_amdgcn_readfirstlane(i);
        base = prow[min(i0, n)];
        const int size = prow[min(i0 + 64, n)] - base;
        staged = size <= kWalkWords;
        if (staged)
            for (int p = threadIdx.x; p < size; p += 4 * kWalkThreads) {
                int v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = pcol[base + min(p + u * kWalkThreads, size - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (p + u * kWalkThreads < size) words[p + u * kWalkThreads] = v[u];
            }
        __syncthreads();
        pos = i < n ? prow[i] : 0;
        end = i < n ? prow[i + 1] : 0;
        while (pos < end && at(end - 1) == i) --end;  // drop the padding
        head = pos < end ? at(pos) : kNoColumn;
        next = pos + 1 < end ? at(pos + 1) : kNoColumn;
    }
    __device__ __forceinline__ int at(int p) const { return staged ? lds[p - base] : col[p]; }
    // The row's entry for column c, the smallest head of the group, or -1.
    __device__ __forceinline__ int take(int c) {
        const bool mine = head == c && c != kNoColumn;
        const int entry = mine ? pos : -1;
        if (mine) {
            ++pos;
            head = next;
            next = pos + 1 < end ? at(pos + 1) : kNoColumn;
        }
        return entry;
    }
};

// Distinct columns of the group (every lane of the wave calls it).
template <int R>
__device__ __forceinline__ int union_size(RowWalk w) {
    int d = 0;
    while (true) {
        const int c = group_min<R>(w.head);
        if (!__any(c != kNoColumn)) return d;
        d += c != kNoColumn ? 1 : 0;
        (void)w.take(c);
    }
}

}  // namespace

}  // namespace sbt
