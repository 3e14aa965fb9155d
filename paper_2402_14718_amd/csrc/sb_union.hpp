// Walk of the union of R consecutive rows' columns, a lane per row, for the
// lists that the blocked streaming steps make once per solve.
//
// The walk is a chain (smallest next column, advance the rows that hold it),
// so it is bound by latency and wants many groups in flight: with a lane per
// row and the next entry of every row loaded a step ahead, 208710 rows make
// 3261 waves.  One thread per group, 204 waves in blocks of 16 rows, took
// 5.2 ms at 208710 rows for the matrix-core lists and 2.6 ms for the quads.
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

// A row (padded CSR; its own column marks the padding) in column order.
struct RowWalk {
    const int *col;
    int pos, end, head, next;  // head: column at pos, next: the one after it

    __device__ __forceinline__ RowWalk(int n, const int *prow, const int *pcol, int i) : col(pcol) {
        pos = i < n ? prow[i] : 0;
        end = i < n ? prow[i + 1] : 0;
        while (pos < end && pcol[end - 1] == i) --end;  // drop the padding
        head = pos < end ? pcol[pos] : kNoColumn;
        next = pos + 1 < end ? pcol[pos + 1] : kNoColumn;
    }
    // The row's entry for column c, the smallest head of the group, or -1.
    __device__ __forceinline__ int take(int c) {
        const bool mine = head == c && c != kNoColumn;
        const int at = mine ? pos : -1;
        if (mine) {
            ++pos;
            head = next;
            next = pos + 1 < end ? col[pos + 1] : kNoColumn;
        }
        return at;
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
