// Batched SB over many events (gfx950): per-event preparation, the work
// counters, best-agent selection, and the dispatch to the step kernel of
// each mode, coupling format and workgroup shape (sb_batch_step.hpp,
// instantiated once per triple by sb_batch_mode.hip).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cstdint>

#include "sb_device.hpp"
#include "sb_kernels.hpp"

namespace sbt {

constexpr int kLenBins = 64;  // row lengths 0..62 and "63 or more"

// perm[0..n) = spins by decreasing min(row length, 63), ascending id within a
// length; rank its inverse.  One workgroup (whole waves); bins: kLenBins
// ints per wave.  Each wave counts and then places one run of consecutive
// spins, so the order does not depend on timing.
__device__ __forceinline__ void rank_rows(int n, const int *row_ptr, int *perm, int *rank, int *bins) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, nw = static_cast<int>(blockDim.x) >> 6;
    const int run = ((n + nw - 1) / nw + 63) / 64 * 64;  // spins per wave
    const int i0 = min(n, wave * run), i1 = min(n, i0 + run);
    int *mine = bins + wave * kLenBins;
    mine[lane] = 0;
    auto bin_of = [&](int i) { return kLenBins - 1 - min(row_ptr[i + 1] - row_ptr[i], kLenBins - 1); };
    __syncthreads();
    for (int i = i0 + lane; i < i1; i += 64) atomicAdd(mine + bin_of(i), 1);
    __syncthreads();
    // exclusive prefix sums over (bin, wave); lane b of wave 0 takes bin b
    if (wave == 0) {
        int tot = 0;
        for (int w = 0; w < nw; ++w) tot += bins[w * kLenBins + lane];
        int at = tot;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(at, off, 64);
            if (lane >= off) at += v;
        }
        at -= tot;
        for (int w = 0; w < nw; ++w) {
            const int c = bins[w * kLenBins + lane];
            bins[w * kLenBins + lane] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int g = i0; g < i1; g += 64) {
        const int i = g + lane;
        const bool in = i < i1;
        const int b = in ? bin_of(i) : 0;
        uint64_t same = __ballot(in);  // this group's spins of the same length
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const uint64_t has = __ballot(in && ((b >> k) & 1));
            same &= ((b >> k) & 1) ? has : ~has;
        }
        const int below = __popcll(same & ((uint64_t(1) << lane) - 1));
        const int base = in ? mine[b] : 0;
        __builtin_amdgcn_wave_barrier();
        if (in) {
            if (below == 0) mine[b] = base + __popcll(same);
            perm[base + below] = i;
            rank[i] = base + below;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
}

// A column as its rank, bit 15: it is above the row.
__device__ __forceinline__ uint16_t column_rank(const int *rank, int row, int col) {
    return static_cast<uint16_t>(rank[col] | (col > row ? 0x8000 : 0));
}

// The largest of the workgroup's values (each at least 0), in thread 0; red:
// one double per wave.
__device__ __forceinline__ double block_max(double v, double *red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (unsigned w = 1; w < blockDim.x >> 6; ++w) v = fmax(v, red[w]);
    __syncthreads();
    return v;
}

// Per-event preparation, one workgroup per event: FP32 field h, 16-bit
// couplings J = -b/4, c0 and the Ising offset C (FP64, fixed order), and
// the spin order by decreasing row length.
__global__ __launch_bounds__(256) void batch_prep(BatchArgs B, int jprec) {
    __shared__ double red[4];
    __shared__ int bins[4 * kLenBins];
    const int e = blockIdx.x;
    const BatchEvent E = B.ev[e];
    const int t = threadIdx.x;
    double sj = 0.0, sj2 = 0.0, sup = 0.0, sa = 0.0, top = 0.0;
    int other = 0;  // a BF16 coupling that is no normal FP16 value
    for (int i = t; i < E.n; i += 256) {
        const int r0 = B.row_ptr[E.rp_off + i], r1 = B.row_ptr[E.rp_off + i + 1];
        double rs = 0.0, most = __builtin_fabs(B.a[E.row_off + i]);
        for (int p = r0; p < r1; ++p) {
            const double bv = B.b[E.nz_off + p];
            const double jv = -0.25 * bv;
            uint16_t bits;
            if (jprec == kJFp16) {
                bits = __half_as_ushort(static_cast<__half>(static_cast<_Float16>(jv)));
            } else {  // BF16: FP32 first, then round to nearest even on the upper half
                const uint32_t u = __float_as_uint(static_cast<float>(jv));
                bits = static_cast<uint16_t>((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
                const float f = __uint_as_float(static_cast<uint32_t>(bits) << 16);
                const bool normal = f == 0.0f || (__builtin_fabsf(f) >= 0x1p-14f && __builtin_fabsf(f) < 65536.0f);
                other |= normal && __half2float(__float2half_rn(f)) == f ? 0 : 1;
            }
            B.J16[E.nz_off + p] = bits;
            rs += bv;
            most += __builtin_fabs(bv);
            sj += jv;
            sj2 += jv * jv;
            if (B.col[E.nz_off + p] > i) sup += bv;
        }
        B.h[E.row_off + i] = static_cast<float>(-(0.5 * B.a[E.row_off + i] + 0.25 * rs));
        sa += B.a[E.row_off + i];
        top = most < INFINITY ? fmax(top, most) : top;
    }
    top = block_max(top, red);
    other = __syncthreads_or(other);
    const double t0 = block_sum(sj, red);
    const double t1 = block_sum(sj2, red);
    const double t2 = block_sum(sup, red);
    const double t3 = block_sum(sa, red);
    if (t == 0) {
        B.halves[e] = other == 0;
        // at most 2^14 spins of terms below 2^at: see rows_item's agent_energy
        const int at = top > 0.0 ? min(max(ilogb(top) + 1, -900), 1000) : 0;
        B.split_at[e] = ldexp(1.5, at + 14);
        const double n2 = static_cast<double>(E.n) * E.n;
        const double mean = t0 / n2;
        const double var = t1 / n2 - mean * mean;
        const double sd = var > 0.0 ? sqrt(var) : 0.0;
        double c0 = B.c0_fixed > 0.0 ? B.c0_fixed
                                     : (sd == 0.0 ? 0.5 / sqrt(static_cast<double>(E.n))
                                                  : 0.5 / (sqrt(static_cast<double>(E.n)) * sd));
        B.c0[e] = static_cast<float>(c0 * static_cast<double>(E.c0_scale));
        B.offset[e] = 0.5 * t3 + 0.25 * t2;
    }
    if (B.energy_apart)
        for (int m = t; m < 2 * B.M; m += 256) B.esum[static_cast<size_t>(e) * B.M * 2 + m] = 0.0;
    if (E.n > kBatchSlots) return;  // (a gang: it needs no spin order)
    rank_rows(E.n, B.row_ptr + E.rp_off, B.perm + E.row_off, B.rank + E.row_off, bins);
    if (E.n > kBatchSlotsSmall) {
        // (a list entry's place has 5 bits for a row's length: see rows_item)
        int rest = 0, longest = 0;
        for (int q = t; q < E.n; q += 256) {
            const int i = B.perm[E.row_off + q];
            const int past = max(0, B.row_ptr[E.rp_off + i + 1] - B.row_ptr[E.rp_off + i] - kHeldCaps[1][q / kBatchTPB]);
            rest += past;
            longest = max(longest, past);
        }
        (void)block_exclusive_scan(rest, bins, rest);
        const int list = __syncthreads_or(longest > 31) ? INT32_MAX : rest;
        if (t == 0) B.long_rows[e] = list > B.list_room;
    }
    // columns as ranks, for the step kernel's LDS addresses
    for (int i = t; i < E.n; i += 256)
        for (int p = B.row_ptr[E.rp_off + i]; p < B.row_ptr[E.rp_off + i + 1]; ++p)
            B.colr[E.nz_off + p] = column_rank(B.rank + E.row_off, i, B.col[E.nz_off + p]);
}

__global__ __launch_bounds__(1024) void rank_spins(int n, const int *__restrict__ row_ptr,
                                                   int *__restrict__ perm, int *__restrict__ rank) {
    __shared__ int bins[16 * kLenBins];
    rank_rows(n, row_ptr, perm, rank, bins);
}

__global__ __launch_bounds__(256) void rank_columns(int n, const int *__restrict__ row_ptr,
                                                    const int *__restrict__ col,
                                                    const int *__restrict__ rank,
                                                    uint16_t *__restrict__ colr) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    for (int p = row_ptr[i]; p < row_ptr[i + 1]; ++p) colr[p] = column_rank(rank, i, col[p]);
}

__global__ void batch_reset(int *counters, int n) {
    if (static_cast<int>(threadIdx.x) < n) counters[threadIdx.x] = 0;
}

// Final FP64 O(T) of every agent (Eq. 13), from the assignments: a workgroup
// sums kEnergyChunk rows of one event for 64 agents, one lane each, in the exact
// parts of add_split, so the atomic sums are the step kernel's energies to the
// bit.  Where a workgroup of the step kernel takes many items, their energies
// there cost it a chain of loads per slot and item (40 events of 5000 spins x
// 128 agents, 1 step: 1.05 -> 0.88 ms); of few this launch costs more than it
// saves.
// Four rows of a wave are in flight together: each is a chain of loads.
__global__ __launch_bounds__(1024) void batch_energy(BatchArgs B) {
    constexpr int kWaves = 16, kPer = kEnergyChunk / kWaves, R = 4;
    __shared__ double sum[2][kWaves][64];
    const int lanes = (B.M + 63) / 64, chunk = blockIdx.x / lanes, e = B.chunk_event[chunk];
    const BatchEvent E = B.ev[e];
    const int lo = (chunk - E.chunk0) * kEnergyChunk;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = (blockIdx.x % lanes) * 64 + lane, mc = min(m, B.M - 1);
    const int8_t *T = B.T + static_cast<size_t>(E.row_off) * B.M + mc;
    const int *rp = B.row_ptr + E.rp_off, *col = B.col + E.nz_off;
    const double *a = B.a + E.row_off, *b = B.b + E.nz_off, at = B.split_at[e];
    double v[2] = {0.0, 0.0};
    for (int u = 0; u < kPer; u += R) {
        double er[R];
        int p[R], q[R];
        bool on[R];
        int most = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = lo + wave * kPer + u + r, ic = min(i, E.n - 1);
            p[r] = rp[ic];
            q[r] = i < E.n ? rp[ic + 1] : p[r];
            er[r] = a[ic];
            on[r] = i < E.n && T[static_cast<size_t>(ic) * B.M] != 0;
            most = max(most, q[r] - p[r]);
        }
        for (int k = 0; k < most; ++k) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (k >= q[r] - p[r]) continue;  // (uniform: a row is a wave's)
                const int i = lo + wave * kPer + u + r, c = col[p[r] + k];
                const double bv = b[p[r] + k];
                if (c > i && T[static_cast<size_t>(c) * B.M] != 0) er[r] += bv;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) add_split(on[r] ? er[r] : 0.0, at, v[0], v[1]);
    }
    sum[0][wave][lane] = v[0];
    sum[1][wave][lane] = v[1];
    __syncthreads();
    if (wave < 2 && m < B.M) {
        double tot = 0.0;
        for (int w = 0; w < kWaves; ++w) tot += sum[wave][w][lane];
        atomicAdd(B.esum + (static_cast<size_t>(e) * B.M + m) * 2 + wave, tot);
    }
}

constexpr int kSelect = 256;

// Per event: best agent (minimum energy, lowest index on ties), its T,
// and the best-so-far trace over checkpoints.
__global__ __launch_bounds__(kSelect) void batch_select(BatchArgs B) {
    __shared__ double se[kSelect];
    __shared__ int sm[kSelect];
    const int e = blockIdx.x, t = threadIdx.x;
    const BatchEvent E = B.ev[e];
    double be = INFINITY;
    int bm = 0x7fffffff;
    for (int m = t; m < B.M; m += kSelect) {
        const size_t at = static_cast<size_t>(e) * B.M + m;
        if (B.energy_apart && !E.gang) B.energy[at] = B.esum[2 * at] + B.esum[2 * at + 1];
        const double v = B.energy[at];
        if (v < be || (v == be && m < bm)) {
            be = v;
            bm = m;
        }
    }
    se[t] = be;
    sm[t] = bm;
    __syncthreads();
    for (int w = kSelect / 2; w >= 1; w >>= 1) {
        if (t < w && (se[t + w] < se[t] || (se[t + w] == se[t] && sm[t + w] < sm[t]))) {
            se[t] = se[t + w];
            sm[t] = sm[t + w];
        }
        __syncthreads();
    }
    const int best = sm[0];
    if (t == 0) {
        B.best_energy[e] = se[0];
        B.best_agent[e] = best;
    }
    if (best >= 0 && best < B.M)
        for (int i = t; i < E.n; i += kSelect)
            B.best_T[E.row_off + i] = B.T[(static_cast<size_t>(E.row_off) + i) * B.M + best];
    if (B.trace && B.n_ckpt > 0) {
        double bsf = INFINITY;
        for (int c = 0; c < B.n_ckpt; ++c) {
            double v = INFINITY;
            for (int m = t; m < B.M; m += kSelect)
                v = fmin(v, B.etrace[(static_cast<size_t>(e) * B.n_ckpt + c) * B.M + m]);
            se[t] = v;
            __syncthreads();
            for (int w = kSelect / 2; w >= 1; w >>= 1) {
                if (t < w) se[t] = fmin(se[t], se[t + w]);
                __syncthreads();
            }
            bsf = fmin(bsf, se[0]);
            if (t == 0) B.trace[static_cast<size_t>(e) * B.n_ckpt + c] = bsf;
            __syncthreads();
        }
    }
}

hipError_t launch_batch_prep(int jprec, const BatchArgs &B, hipStream_t st) {
    batch_prep<<<B.E, 256, 0, st>>>(B, jprec);
    return hipGetLastError();
}

hipError_t launch_rank_spins(int n, const int *row_ptr, const int *col, int *perm, int *rank,
                             uint16_t *colr, hipStream_t st) {
    rank_spins<<<1, 1024, 0, st>>>(n, row_ptr, perm, rank);
    rank_columns<<<(n + 255) / 256, 256, 0, st>>>(n, row_ptr, col, rank, colr);
    return hipGetLastError();
}

hipError_t launch_resident_rows(int mode, const BatchArgs &B, const RowsShape &R, hipStream_t st) {
    if (mode == kASB) return launch_resident_rows_tu<kASB>(B, R, st);
    return mode == kDSB ? launch_resident_rows_tu<kDSB>(B, R, st) : launch_resident_rows_tu<kBSB>(B, R, st);
}

hipError_t launch_batch_reset(int *counters, int n, hipStream_t st) {
    batch_reset<<<1, 64, 0, st>>>(counters, n);
    return hipGetLastError();
}

template <int TPB>
static hipError_t steps_of_shape(int mode, int jprec, bool long_rows, const BatchArgs &B, hipStream_t st) {
    const bool f16 = jprec == kJFp16;
    if (mode == kDSB)
        return f16 ? launch_batch_steps_tu<kDSB, kJFp16, TPB>(B, long_rows, st)
                   : launch_batch_steps_tu<kDSB, kJBf16, TPB>(B, long_rows, st);
    if (mode == kASB)
        return f16 ? launch_batch_steps_tu<kASB, kJFp16, TPB>(B, long_rows, st)
                   : launch_batch_steps_tu<kASB, kJBf16, TPB>(B, long_rows, st);
    return f16 ? launch_batch_steps_tu<kBSB, kJFp16, TPB>(B, long_rows, st)
               : launch_batch_steps_tu<kBSB, kJBf16, TPB>(B, long_rows, st);
}

hipError_t launch_batch_steps(int mode, int jprec, int tpb, bool long_rows, const BatchArgs &B, hipStream_t st) {
    if (tpb == kBatchTPBSmall) return steps_of_shape<kBatchTPBSmall>(mode, jprec, long_rows, B, st);
    if (tpb == kBatchTPB) return steps_of_shape<kBatchTPB>(mode, jprec, long_rows, B, st);
    return hipErrorInvalidValue;
}

hipError_t launch_batch_energy(const BatchArgs &B, hipStream_t st) {
    if (B.n_chunks > 0) batch_energy<<<static_cast<unsigned>(B.n_chunks) * ((B.M + 63) / 64), 1024, 0, st>>>(B);
    return hipGetLastError();
}

hipError_t launch_batch_select(const BatchArgs &B, hipStream_t st) {
    batch_select<<<B.E, kSelect, 0, st>>>(B);
    return hipGetLastError();
}

}  // namespace sbt
