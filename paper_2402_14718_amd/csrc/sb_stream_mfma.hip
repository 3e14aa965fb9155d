// dSB streaming step on the matrix cores (gfx950).
//
// Paper section "Simulated Bifurcation", Eq. 9-12: the dSB coupling term
// of row i for agent a is h_i + sum_j J_ij sgn(x_j(a)).  Over a block of
// 16 consecutive rows, the listed columns of the block and a group of 16
// agents, that sum is a matrix product: couplings (16 rows x listed
// columns) times signs (listed columns x 16 agents).  sgn(x) = +-1 is exact
// in any operand type, so with couplings whose stored form is itself an
// operand type the products are exact and only the order of the FP32
// additions differs from the CSR step:
//   FP8 (e4m3, one scale per row): the codes are the operand and the row's
//     scale multiplies the row's sum once, F_i = h_i + s_i sum_j q_ij sgn_j;
//   BF16 hi + lo: two products on the same signs, F_i = h_i + sum hi sgn +
//     sum lo sgn;
//   FP32: each coupling split exactly into three BF16 terms (8 significant
//     bits each), three products on the same signs; FP8 with a scale per
//     block of 8 couplings: the FP32 value scale x code, split the same way;
//   BF16 or FP16 (the FP32 coupling rounded once): one product.
// The positions x and momenta y update in place as in the CSR step
// (sb_update); the signs live in this step's own records (16 bytes per row
// and group of 128 agents, bit t of byte c = agent 16 t + c of the group).
//
// In the azimuth spin order the couplings fill about 0.16 of a block's
// rows x listed columns on the stress event and 0.09 on the sparse events,
// so the matrix cores do 6-11 x the arithmetic of the couplings themselves,
// cheaply; what a K-step costs is one sign byte per listed column and lane
// and a few shifts per tile to spread it into the +-1 operand.
//
// One wave = one block x one group of 128 agents (8 tiles of 16).  Per
// K-step of 32 listed columns lane (g = lane / 16, c = lane % 16) holds,
// for each tile t, the signs of agent 16 t + c on listed columns 8 g ..
// 8 g + 7 (bit t of the lane's 8 sign bytes; the first operand, agents x
// columns) and row c's couplings on the same columns (the second operand,
// columns x rows), so the instruction pairs them; the 16 x 16 result of
// tile t (agents x rows) holds, in lane (g, c), agents 16 t + 4 g .. + 3 of
// row c: four consecutive agents, one 16-byte access of x and of y, and
// the lane's 32 new signs of row c are dword g of the row's record.  x and
// y are kept in this step's own tiled layout (mfma_state_floats), where a
// wave's accesses for one t are one contiguous 1 KB run: in the spin-major
// layout they touch 16 rows x 64 bytes and the step ran 1.4 x slower.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "sb_device.hpp"
#include "sb_kernels.hpp"
#include "sb_scan.hpp"
#include "sb_stream_kernels.hpp"
#include "sb_stream_chunk.hpp"
#include "sb_stream_mfma.hpp"
#include "sb_union.hpp"

namespace sbt {

namespace {

constexpr int kBR = kMfmaRows;
constexpr int kBK = kMfmaK;
constexpr int kChunkSteps = 4;   // K-steps whose sign records are staged in LDS at once
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kWalkThreads) void mfma_count(int n, int nb, const int *__restrict__ prow,
                                                  const int *__restrict__ pcol, int *__restrict__ cnt) {
    __shared__ int words[kWalkWords];
    const int i = blockIdx.x * kWalkThreads + threadIdx.x, b = i / kBR;
    const int d = union_size<kBR>(RowWalk(n, prow, pcol, i, words));
    if (i % kBR == 0 && b < nb) cnt[b] = (d + kBK - 1) / kBK;
}

__global__ __launch_bounds__(kScanThreads) void mfma_scan(int nb, int range, const int *__restrict__ cnt,
                                                          int *__restrict__ off) {
    scan_lengths(nb, range, [&](int b) { return cnt[b]; }, off);
}

// FP32 -> BF16, round to nearest even (finite values).
__device__ __forceinline__ uint32_t bf16_bits(float v) {
    const uint32_t u = __float_as_uint(v);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// An FP32 coupling as BF16 terms hi + mid + lo, exactly: each residual is
// exact in FP32 (Sterbenz), the last one has at most 8 significant bits.
__device__ __forceinline__ void bf16_triple(float v, uint32_t (&t)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        t[k] = bf16_bits(v);
        v -= __uint_as_float(t[k] << 16);
    }
}

// Lists block b's columns and writes every operand word of its K-steps:
// listed column u (0-based in the block) of row r is element u % 8 of lane
// 16 ((u % 32) / 8) + r in K-step u / 32 (FP8: byte e of the lane's word;
// BF16 terms: term k in words 2 k and 2 k + 1, 16 bits per element); zeros
// where a row has no coupling and in the padding, whose column repeats the
// last listed one.  A lane is a row of the block: it assembles its words over
// 8 consecutive listed columns and stores them whole, next to the 15 others'.
template <int JP>
__global__ __launch_bounds__(kWalkThreads) void mfma_fill(int nb, StreamArgs A, const int *__restrict__ koff,
                                                 int *__restrict__ kcol, uint64_t *__restrict__ kA) {
    constexpr int W = mfma_words(JP);
    __shared__ int words[kWalkWords];
    const int i = blockIdx.x * kWalkThreads + threadIdx.x, b = i / kBR, r = i % kBR;
    RowWalk walk(A.n, A.row_ptr, A.col, i, words);
    const int ks0 = b < nb ? koff[b] : 0, u1 = b < nb ? (koff[b + 1] - ks0) * kBK : 0;
    int last = 0;
    for (int u = 0; __any(u < u1); u += 8) {
        int at[8], mine = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = group_min<kBR>(walk.head);
            at[e] = walk.take(c);
            last = c == kNoColumn ? last : c;
            mine = e == r ? last : mine;
        }
        if (u >= u1) continue;
        uint64_t buf[W] = {};
        if constexpr (JP == kJFp8) {
            uint64_t code[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) code[e] = at[e] >= 0 ? A.J8[at[e]] : 0u;
#pragma unroll
            for (int e = 0; e < 8; ++e) buf[0] |= code[e] << (8 * e);
        } else {
            float v[8];      // the coupling, or of BF16 pairs
            uint32_t v2[8];  // both terms
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool there = at[e] >= 0;
                if constexpr (JP == kJBf16x2)
                    v2[e] = there ? A.J2[at[e]] : 0u;
                else if constexpr (JP == kJFp8Blk)  // the CSR step's decoded value
                    v[e] = there ? A.blkscale[at[e] / kStreamChunk] * e4m3_to_f32<0>(A.J8[at[e]]) : 0.0f;
                else
                    v[e] = there ? A.J[at[e]] : 0.0f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t term[3] = {0u, 0u, 0u};
                if constexpr (JP == kJBf16x2) {
                    term[0] = v2[e] >> 16;
                    term[1] = v2[e] & 0xFFFFu;
                } else if constexpr (JP == kJBf16) {
                    term[0] = bf16_bits(v[e]);
                } else if constexpr (JP == kJFp16) {
                    term[0] = __builtin_bit_cast(uint16_t, static_cast<_Float16>(v[e]));
                } else {
                    bf16_triple(v[e], term);
                }
                const int sh = 16 * (e % 4);
#pragma unroll
                for (int k = 0; k < W / 2; ++k)
                    buf[2 * k + e / 4] |= static_cast<uint64_t>(at[e] >= 0 ? term[k] : 0u) << sh;
            }
        }
        if (r < 8) kcol[static_cast<size_t>(ks0) * kBK + u + r] = mine;
        const size_t lane = static_cast<size_t>(ks0 + u / kBK) * 64 + 16 * ((u % kBK) / 8) + r;
#pragma unroll
        for (int w = 0; w < W; ++w) kA[lane * W + w] = buf[w];
    }
}

// Workgroup id -> (group of 4 blocks, agent group), XCD-contiguous: each
// XCD sweeps one contiguous range of blocks, all agent groups of a block
// next to each other, so the block's operand tiles and listed columns are
// reused from that XCD's L2 and the sign records its blocks read (all
// agent groups of a column share a line) stay there.
__device__ __forceinline__ bool mfma_block(int ngb, int nab, int &gb, int &ab) {
    const int total = ngb * nab;
    const int per_xcd = (total + 7) / 8;
    const int v = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (v >= total) return false;
    ab = v % nab;
    gb = v / nab;
    return true;
}

// The start state (init_state's draws) of one tile, by a wave; put(at, word)
// takes its sign words.
template <class Put>
__device__ __forceinline__ void mfma_draw(int n, int M, uint32_t k0, uint32_t k1, uint32_t event, int b, int ab, int R,
                                          int lane, float *x, float *y, Put put) {
    const int g = lane >> 4, c = lane & 15, i = b * kBR + c;
    const size_t tile = (static_cast<size_t>(b) * R + ab) * (kBR * kMfmaGroup) + 4 * lane;
    uint32_t word = 0;  // byte r, bit t: agent 16 t + 4 g + r
    for (int t = 0; t < kMfmaGroup / 16; ++t) {
        f32x4 xv = {0.0f, 0.0f, 0.0f, 0.0f}, yv = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = kMfmaGroup * ab + 16 * t + 4 * g + r;
            if (i < n && m < M) {
                const Philox4 d = philox4x32_10(static_cast<uint32_t>(i), static_cast<uint32_t>(m), event, 0u, k0, k1);
                xv[r] = philox_word_to_unit(d.v[0]);
                yv[r] = philox_word_to_unit(d.v[1]);
                word |= xv[r] >= 0.0f ? 1u << (8 * r + t) : 0u;
            }
        }
        *reinterpret_cast<f32x4 *>(x + tile + 256 * t) = xv;
        *reinterpret_cast<f32x4 *>(y + tile + 256 * t) = yv;
    }
    if (i < n) put((static_cast<size_t>(i) * R + ab) * 4 + g, word);
}

// The start state in the step's tiles and its sign records; a wave per tile.
__global__ __launch_bounds__(256) void mfma_init(int n, int M, uint32_t k0, uint32_t k1, uint32_t event,
                                                 float *__restrict__ x, float *__restrict__ y,
                                                 uint8_t *__restrict__ S) {
    const int R = mfma_groups(M), nb = (n + kBR - 1) / kBR;
    const int64_t id = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (id >= static_cast<int64_t>(nb) * R) return;
    mfma_draw(n, M, k0, k1, event, static_cast<int>(id / R), static_cast<int>(id % R), R, threadIdx.x & 63, x, y,
              [&](size_t at, uint32_t word) { reinterpret_cast<uint32_t *>(S)[at] = word; });
}

// A tile (layout of mfma_state_floats) -> spin-major x[i M + m], by a
// workgroup.  The tile's runs of 16 bytes go round the rows, so they pass
// through LDS and a row is written as one run of 512 bytes (208710 x 512,
// 0.33 -> 0.16 ms against a thread per run).
constexpr int kStateThreads = 256;
constexpr int kRuns = kMfmaGroup / 4;  // of a row
typedef f32x4 StateRows[kBR][kRuns + 1];
__device__ __forceinline__ void tile_state(int n, int M, int b, int ab, const float *src, float *dst, StateRows &rows) {
    const size_t at = static_cast<size_t>(b) * mfma_groups(M) + ab;
    const f32x4 *tile = reinterpret_cast<const f32x4 *>(src) + at * (kBR * kRuns);
#pragma unroll
    for (int u = 0; u < kBR * kRuns / kStateThreads; ++u) {
        const int q = u * kStateThreads + threadIdx.x, lane = q % 64;
        rows[lane & 15][4 * (q / 64) + (lane >> 4)] = tile[q];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kBR * kRuns / kStateThreads; ++u) {
        const int q = u * kStateThreads + threadIdx.x, c = q / kRuns, i = b * kBR + c;
        const int m = kMfmaGroup * ab + 4 * (q % kRuns);
        if (i >= n) continue;
        const f32x4 v = rows[c][q % kRuns];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (m + r < M) dst[static_cast<size_t>(i) * M + m + r] = v[r];
    }
}

__global__ __launch_bounds__(kStateThreads) void mfma_state(int n, int M, const float *__restrict__ src,
                                                            float *__restrict__ dst) {
    __shared__ StateRows rows;
    const int R = mfma_groups(M);
    tile_state(n, M, blockIdx.x / R, blockIdx.x % R, src, dst, rows);
}

// One K-step of a tile: acc[t] += (-sgn of 8 columns, agents of tile t) x
// (the row's couplings on them).
template <int JP>
__device__ __forceinline__ void mfma_kstep(const uint32_t (&s8)[8], const uint64_t (&a8)[mfma_words(JP)],
                                           f32x4 (&acc)[kMfmaGroup / 16]) {
    constexpr int T = kMfmaGroup / 16, W = mfma_words(JP);
    // -sgn(x_j): a set sign bit (x >= 0) gives -1
    if constexpr (JP != kJFp8) {
        // 16-bit operands: +-1 is 0x3F80 | sign in BF16, 0x3C00 | sign in FP16
        constexpr uint32_t kOne = JP == kJFp16 ? 0x3C003C00u : 0x3F803F80u;
        uint32_t yq[4];  // columns 2q, 2q+1 at bits 0 and 16
#pragma unroll
        for (int q = 0; q < 4; ++q) yq[q] = s8[2 * q] | (s8[2 * q + 1] << 16);
        u32x4 aop[W / 2];  // the terms, largest first
#pragma unroll
        for (int k = 0; k < W / 2; ++k)
            aop[k] = u32x4{static_cast<uint32_t>(a8[2 * k]), static_cast<uint32_t>(a8[2 * k] >> 32),
                           static_cast<uint32_t>(a8[2 * k + 1]), static_cast<uint32_t>(a8[2 * k + 1] >> 32)};
#pragma unroll
        for (int t = 0; t < T; ++t) {
            u32x4 bv;
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[q] = ((yq[q] << (15 - t)) & 0x80008000u) | kOne;
#pragma unroll
            for (int k = 0; k < W / 2; ++k) {
                if constexpr (JP == kJFp16)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        __builtin_bit_cast(f16x8, bv), __builtin_bit_cast(f16x8, aop[k]), acc[t], 0, 0, 0);
                else
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, bv), __builtin_bit_cast(bf16x8, aop[k]), acc[t], 0, 0, 0);
            }
        }
    } else {
        // byte e of xl / xh: the sign byte of column e / e + 4
        const uint32_t xl = s8[0] | (s8[1] << 8) | (s8[2] << 16) | (s8[3] << 24);
        const uint32_t xh = s8[4] | (s8[5] << 8) | (s8[6] << 16) | (s8[7] << 24);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t lo = ((xl << (7 - t)) & 0x80808080u) | 0x38383838u;  // e4m3 +-1
            const uint32_t hi = ((xh << (7 - t)) & 0x80808080u) | 0x38383838u;
            const long bop = static_cast<long>((static_cast<uint64_t>(hi) << 32) | lo);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(bop, static_cast<long>(a8[0]),
                                                                acc[t], 0, 0, 0);
        }
    }
}

}  // namespace

// One dSB step: a wave = one block of 16 rows x one group of 128 agents.
template <int JP, bool NT>
__global__ __launch_bounds__(256) void sb_stream_mfma(StreamArgs A, int k, const int *__restrict__ koff,
                                                      const int *__restrict__ kcol,
                                                      const uint64_t *__restrict__ kA,
                                                      const float *__restrict__ h,
                                                      const float *__restrict__ rowscale,
                                                      float *__restrict__ x, float *__restrict__ y,
                                                      const uint8_t *__restrict__ Sin,
                                                      uint8_t *__restrict__ Sout) {
    constexpr int T = kMfmaGroup / 16;    // tiles of 16 agents
    constexpr int W = mfma_words(JP);     // operand words per lane and K-step
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int M = A.M, R = mfma_groups(M);
    const int nb = (A.n + kBR - 1) / kBR;
    // When the state streams from HBM (NT), operands wider than one word per
    // lane (the 16-bit forms) are shared: a workgroup takes one block and up
    // to four agent groups (one per wave) and stages each chunk's operand
    // tiles in LDS once for all of them (measured on the stress event: BF16
    // pairs 0.452 -> 0.400 ms, FP32 0.490 -> 0.434).  Otherwise workgroups
    // take four blocks of one agent group, with no barriers and a third wave
    // per SIMD (cache-resident precision event, FP32: 23.6 against 27.8 us
    // with sharing).
    constexpr bool kShare = W > 1 && NT;
    int b, ab;
    bool active = true;   // the wave has an agent group (shared form: ab < R)
    if constexpr (kShare) {
        int ac;
        if (!mfma_block(nb, (R + 3) / 4, b, ac)) return;
        b = __builtin_amdgcn_readfirstlane(b);
        ab = __builtin_amdgcn_readfirstlane(ac * 4 + wave);
        active = ab < R;
    } else {
        int gb;
        if (!mfma_block((nb + 3) / 4, R, gb, ab)) return;
        b = __builtin_amdgcn_readfirstlane(gb * 4 + wave);
        if (b >= nb) return;
    }
    const int g = lane >> 4, c = lane & 15;
    f32x4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // The lane's x, y (row 16 b + c, agents 128 ab + 16 t + 4 g + r: 16
    // bytes at tile + 256 t, padding included) are loaded before the
    // coupling sums, so their latency hides behind them.
    const size_t tile = (static_cast<size_t>(b) * R + ab) * (kBR * kMfmaGroup) + 4 * lane;
    f32x4 xp[T], yp[T];
    if (active) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            xp[t] = ld_stream<NT>(reinterpret_cast<const f32x4 *>(x + tile + 256 * t));
            yp[t] = ld_stream<NT>(reinterpret_cast<const f32x4 *>(y + tile + 256 * t));
        }
    }

    // The block's sign records pass through LDS, kChunkSteps K-steps at a
    // time: each lane fetches two listed columns' whole 16-byte records
    // (two loads instead of eight per K-step on the texture path, whose
    // cost is per instruction), and the K-steps read their sign bytes from
    // LDS.  A 16-byte pad after every 8 slots puts the four lane groups'
    // records on different banks.  Columns are fetched two chunks ahead,
    // records one chunk ahead; FP8 operands one K-step ahead, shared
    // operands one chunk ahead (wave w fetches K-step w of the chunk).
    constexpr int kSlots = kChunkSteps * kBK;
    __shared__ uint4 rec_lds[4][kSlots + kSlots / 8];
    uint4 *lds = rec_lds[wave];
    const int ks0 = koff[b], ks1 = koff[b + 1];
    const int nk = ks1 - ks0, nch = (nk + kChunkSteps - 1) / kChunkSteps;
    int cn[2];
    uint4 rn[2];
    uint64_t an[W];
    __shared__ uint64_t op_lds[kShare ? kChunkSteps * 64 * W : 1];
    auto load_cols = [&](int j) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int u = j * kSlots + lane + 64 * hh;  // block-relative listed column
            cn[hh] = u < nk * kBK ? kcol[static_cast<size_t>(ks0) * kBK + u] : -1;
        }
    };
    auto load_recs = [&]() {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
            rn[hh] = cn[hh] >= 0
                         ? *reinterpret_cast<const uint4 *>(Sin + (static_cast<size_t>(cn[hh]) * R + ab) * 16)
                         : uint4{0u, 0u, 0u, 0u};
    };
    auto load_operand = [&](int ks) {
#pragma unroll
        for (int w = 0; w < W; ++w) an[w] = kA[(static_cast<size_t>(ks) * 64 + lane) * W + w];
    };
    // shared forms: this wave's K-step of chunk j (kept in `an` until stored)
    auto load_chunk_operand = [&](int j) {
        if (j * kChunkSteps + wave < nk) load_operand(ks0 + j * kChunkSteps + wave);
    };
    if (nch > 0) {
        if (active) {
            load_cols(0);
            load_recs();
            if (nch > 1) load_cols(1);
        }
        if constexpr (kShare)
            load_chunk_operand(0);
        else
            load_operand(ks0);
    }
    for (int j = 0; j < nch; ++j) {
        __builtin_amdgcn_wave_barrier();    // the previous chunk's LDS reads come first
        if (active) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int sl = lane + 64 * hh;
                lds[sl + sl / 8] = rn[hh];
            }
        }
        if constexpr (kShare) {
            __syncthreads();                // every wave is done with the previous chunk's operands
            if (j * kChunkSteps + wave < nk) {
#pragma unroll
                for (int w = 0; w < W; ++w) op_lds[(wave * 64 + lane) * W + w] = an[w];
            }
            __syncthreads();
        }
        __builtin_amdgcn_wave_barrier();
        if (j + 1 < nch) {
            if (active) {
                load_recs();
                if (j + 2 < nch) load_cols(j + 2);
            }
            if constexpr (kShare) load_chunk_operand(j + 1);
        }
        if (!active) continue;
        const int kend = min(kChunkSteps, nk - j * kChunkSteps);
        for (int kk = 0; kk < kend; ++kk) {
            const int ks = ks0 + j * kChunkSteps + kk;
            uint32_t s8[8];
            uint64_t a8[W];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int sl = kk * kBK + 8 * g + e;
                s8[e] = reinterpret_cast<const uint8_t *>(lds + sl + sl / 8)[c];
            }
            if constexpr (kShare) {
#pragma unroll
                for (int w = 0; w < W; ++w) a8[w] = op_lds[(kk * 64 + lane) * W + w];
            } else {
#pragma unroll
                for (int w = 0; w < W; ++w) a8[w] = an[w];
                if (ks + 1 < ks1) load_operand(ks + 1);
            }
            mfma_kstep<JP>(s8, a8, acc);
        }
    }

    // acc[t][r] = -(sum over the block's columns) for row 16 b + c, agent
    // 128 ab + 16 t + 4 g + r (agents past M are padding: updated, never
    // read back, their sign bits 0)
    const int i = b * kBR + c;
    if (!active || i >= A.n) return;
    const float c0 = static_cast<float>(A.scal[0]);
    const float gk = A.sched[k];
    const float hv = h[i];
    const float sc = JP == kJFp8 ? rowscale[i] : 1.0f;
    uint32_t word = 0;             // byte r, bit t: agent 16 t + 4 g + r
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int m = kMfmaGroup * ab + 16 * t + 4 * g;
        f32x4 xv = xp[t], yv = yp[t];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float xr = xv[r], yr = yv[r];
            sb_update(xr, yr, __builtin_fmaf(-sc, acc[t][r], hv), c0, gk, A.dt, A.dta0);
            xv[r] = xr;
            yv[r] = yr;
            if (m + r < M && xr >= 0.0f) word |= 1u << (8 * r + t);
        }
        st_stream<NT>(xv, reinterpret_cast<f32x4 *>(x + tile + 256 * t));
        st_stream<NT>(yv, reinterpret_cast<f32x4 *>(y + tile + 256 * t));
    }
    reinterpret_cast<uint32_t *>(Sout)[(static_cast<size_t>(i) * R + ab) * 4 + g] = word;
}

// ------------------------------------------------------- steps on the chip
//
// A streamed step moves 16 bytes of x and y per spin and agent, and a state
// of 70 to 100 MB misses the XCDs' L2s, so the step above is bound by the
// Infinity Cache and by its launch (8484 x 1024, FP32: 24 us, 134 MB).  The
// registers and LDS of the chip hold such a state.  sb_mfma_gang keeps it
// there for a run of steps: a gang is one group of 128 agents over all rows,
// its blocks are spread over `bands` workgroups of eight waves, a wave holds
// up to three tiles (two in registers, one in LDS), and what the workgroups
// exchange each step are the sign records, 16 bytes per row.  The arithmetic
// of a tile is that of sb_stream_mfma in its order.
//
// The records are written and read with agent-scope atomics, which are
// coherent over the XCDs; nothing else that is written is read by another
// workgroup, so a step needs no cache write-back and no invalidation (which
// would cost it the operands in the L2), only that a workgroup's stores are
// done before it arrives.  Gangs are queued one after the other and taken
// band by band by running workgroups, so a gang that has been started gets
// all its bands as long as `bands` workgroups of this launch run at once.  A
// gang takes an eighth of the device at most, so of up to eight such launches
// side by side (streams, processes) one always has that many; with a gang over
// the whole device two could each hold what the other waits for.  Where fewer
// compute units are left than that (a long launch beside this one, a captured
// solve replayed on a stream with a mask), a wait ends after kGangWait ticks of
// the 100 MHz clock: ctl[1] is set, the launch ends, later runs of the solve do
// nothing, and alone_steps takes the steps that are missing.
//
// A step of 8484 x 1024: FP32 24.3 -> 10.2 us, FP8 23.6 -> 8.1; 1480 x 256
// 5.2 -> 4.0, 4.9 -> 3.4.  What is left is the meeting (2.3 us), the latency
// of the records (1.7) and the update of 16 or 17 tiles per CU.  Two
// workgroups of four waves per CU, of different gangs, do not hide one
// another's meeting (13.5 us): a gang of 64 meets more slowly.
constexpr long long kGangWait = 100000000LL;  // 1 s, where a step takes microseconds
// control words before the gangs' flags: work counter, 1 + k0 of the run that was given up (0: none)
constexpr int kGangHead = 32;
// flags of a gang, in cache lines of their own
__host__ __device__ constexpr int gang_words(int bands) { return (bands + 31) / 32 * 32; }
constexpr int kGangSlots = kChunkSteps * kBK;
constexpr int kGangRec = kGangSlots + kGangSlots / 8;  // records of a chunk, padded (uint4)

// Every workgroup of a gang says how many steps it has done in a word of its
// own and waits until all have done as many: 32 additions to one counter
// took longer (8 gangs of 32 workgroups: 2.65 against 2.35 us,
// and 8.6 with the counters in one cache line).
__device__ __forceinline__ bool gang_meet(int *flags, int bands, int band, int done, int *fault, int given_up,
                                          int *stop) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's records are out
    __syncthreads();
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0)
            __hip_atomic_store(flags + band, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long t0 = wall_clock64();
        bool bad = false;
        for (int w0 = 0; w0 < bands && !bad; w0 += 64) {
            const int *mine = flags + min(w0 + static_cast<int>(threadIdx.x), bands - 1);
            for (int tries = 1; __any(__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < done); ++tries) {
                if (tries % 64 == 0) {
                    bad = __hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                    if (!bad && wall_clock64() - t0 > kGangWait) {
                        __hip_atomic_store(fault, given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        bad = true;
                    }
                    if (__any(bad)) break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            bad = __any(bad);
        }
        if (threadIdx.x == 0) *stop = bad;
    }
    __syncthreads();
    return *stop != 0;
}

// The sign record of a column, as other workgroups wrote it.
__device__ __forceinline__ uint4 load_record(const uint8_t *S, int col, int R, int ab) {
    const uint64_t *p = reinterpret_cast<const uint64_t *>(S + (static_cast<size_t>(col) * R + ab) * 16);
    const uint64_t a = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t b = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return uint4{static_cast<uint32_t>(a), static_cast<uint32_t>(a >> 32), static_cast<uint32_t>(b),
                 static_cast<uint32_t>(b >> 32)};
}

// (w << 1) | (x >= 0): the comparison's carry added in.
__device__ __forceinline__ uint32_t shift_in(uint32_t w, float x) {
    asm("v_cmp_le_f32 vcc, 0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(w) : "v"(x) : "vcc");
    return w;
}

template <int JP>
__global__ __launch_bounds__(64 * kGangWaves, 2) void sb_mfma_gang(
    StreamArgs A, int k0, int k1, const int *__restrict__ koff, const int *__restrict__ kcol,
    const uint64_t *__restrict__ kA, const float *__restrict__ h, const float *__restrict__ rowscale,
    float *__restrict__ x, float *__restrict__ y, uint8_t *S0, uint8_t *S1, int bands, int items, int *ctl) {
    constexpr int T = kMfmaGroup / 16, W = mfma_words(JP), kRegTiles = kGangRegTiles, kTiles = kGangTiles;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int item_s, stop_s;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, c = lane & 15;
    uint4 *rec = reinterpret_cast<uint4 *>(smem) + wave * kGangRec;
    // the LDS tile: x then y, lane by lane
    f32x4 *spare = reinterpret_cast<f32x4 *>(smem + kGangWaves * kGangRec * 16) + wave * 2 * T * 64 + lane;
    const int M = A.M, R = mfma_groups(M), nb = (A.n + kBR - 1) / kBR;
    const float c0 = static_cast<float>(A.scal[0]);
    for (bool first = true;; first = false) {
        if (threadIdx.x == 0) {  // (nothing where a run was given up before)
            const int given_up = first ? __hip_atomic_load(ctl + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            const int next = atomicAdd(ctl, 1);
            item_s = given_up ? items : next;
        }
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(item_s);
        __syncthreads();
        if (item >= items) return;
        const int ab = item / bands, band = item % bands;
        const int b0 = static_cast<int>(static_cast<int64_t>(nb) * band / bands);
        const int b1 = static_cast<int>(static_cast<int64_t>(nb) * (band + 1) / bands);
        int *flags = ctl + gang_words(bands) * ab + kGangHead;
        uint32_t live = 0;  // this lane's agents below M: byte r, bit t
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) live |= kMfmaGroup * ab + 16 * t + 4 * g + r < M ? 1u << (8 * r + t) : 0u;
        f32x4 xs[kRegTiles][T], ys[kRegTiles][T];
        float hv[kTiles], sc[kTiles];
        int bs[kTiles], ks0[kTiles], nk[kTiles], cn[kTiles][2];
        bool has[kTiles];
        auto tile_of = [&](int i) { return (static_cast<size_t>(bs[i]) * R + ab) * (kBR * kMfmaGroup) + 4 * lane; };
#pragma unroll
        for (int i = 0; i < kTiles; ++i) {
            bs[i] = b0 + wave + kGangWaves * i;
            has[i] = bs[i] < b1;
            if (!has[i]) bs[i] = 0;
            ks0[i] = koff[bs[i]];
            nk[i] = has[i] ? koff[bs[i] + 1] - ks0[i] : 0;
            const int row = min(bs[i] * kBR + c, A.n - 1);
            hv[i] = h[row];
            sc[i] = JP == kJFp8 ? rowscale[row] : 1.0f;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int u = lane + 64 * hh;
                cn[i][hh] = u < nk[i] * kBK ? kcol[static_cast<size_t>(ks0[i]) * kBK + u] : 0;
            }
            if (has[i]) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const f32x4 xv = *reinterpret_cast<const f32x4 *>(x + tile_of(i) + 256 * t);
                    const f32x4 yv = *reinterpret_cast<const f32x4 *>(y + tile_of(i) + 256 * t);
                    if (i < kRegTiles) {
                        xs[i][t] = xv;
                        ys[i][t] = yv;
                    } else {
                        spare[64 * t] = xv;
                        spare[64 * (T + t)] = yv;
                    }
                }
            }
        }
        bool stop = false;
        for (int k = k0; k < k1 && !stop; ++k) {
            const uint8_t *Sin = ((k - k0) & 1) ? S1 : S0;
            uint8_t *Sout = ((k - k0) & 1) ? S0 : S1;
            const float gk = A.sched[k];
            auto load_rec = [&](int col) { return load_record(Sin, col, R, ab); };
            uint4 rn[kTiles][2];
#pragma unroll
            for (int i = 0; i < kTiles; ++i)
                if (nk[i] > 0) {
                    rn[i][0] = load_rec(cn[i][0]);
                    if (nk[i] > 2) rn[i][1] = load_rec(cn[i][1]);
                }
            uint64_t an[W];
            auto load_operand = [&](int ks) {
#pragma unroll
                for (int w = 0; w < W; ++w) an[w] = kA[(static_cast<size_t>(ks) * 64 + lane) * W + w];
            };
            // the first operand of the next tile with couplings (a block may have none)
            auto load_next_tile = [&](int i) {
                int ks = -1;
#pragma unroll
                for (int u = kTiles - 1; u > i; --u) ks = nk[u] > 0 ? ks0[u] : ks;
                if (ks >= 0) load_operand(ks);
            };
            load_next_tile(-1);
#pragma unroll
            for (int i = 0; i < kTiles; ++i) {
                if (!has[i]) continue;
                f32x4 acc[T];
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                for (int j = 0; j * kChunkSteps < nk[i]; ++j) {
                    if (j > 0) {
#pragma unroll
                        for (int hh = 0; hh < 2; ++hh) {
                            const int u = min(j * kGangSlots + lane + 64 * hh, nk[i] * kBK - 1);
                            rn[i][hh] = load_rec(kcol[static_cast<size_t>(ks0[i]) * kBK + u]);
                        }
                    }
                    __builtin_amdgcn_wave_barrier();  // the LDS reads of the chunk before come first
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
                        const int sl = lane + 64 * hh;
                        if (hh == 0 || nk[i] - j * kChunkSteps > 2) rec[sl + sl / 8] = rn[i][hh];
                    }
                    __builtin_amdgcn_wave_barrier();
                    const int kend = min(kChunkSteps, nk[i] - j * kChunkSteps);
                    for (int kk = 0; kk < kend; ++kk) {
                        const int ks = ks0[i] + j * kChunkSteps + kk;
                        uint32_t s8[8];
                        uint64_t a8[W];
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int sl = kk * kBK + 8 * g + e;
                            s8[e] = reinterpret_cast<const uint8_t *>(rec + sl + sl / 8)[c];
                        }
#pragma unroll
                        for (int w = 0; w < W; ++w) a8[w] = an[w];
                        if (ks + 1 < ks0[i] + nk[i])
                            load_operand(ks + 1);
                        else
                            load_next_tile(i);
                        mfma_kstep<JP>(s8, a8, acc);
                    }
                }
                uint32_t bits[4] = {0u, 0u, 0u, 0u};  // of agent 16 t + 4 g + r: bit t of word r
#pragma unroll
                for (int t = T - 1; t >= 0; --t) {
                    f32x4 xv, yv;
                    if (i < kRegTiles) {
                        xv = xs[i < kRegTiles ? i : 0][t];
                        yv = ys[i < kRegTiles ? i : 0][t];
                    } else {
                        xv = spare[64 * t];
                        yv = spare[64 * (T + t)];
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float xr = xv[r], yr = yv[r];
                        sb_update(xr, yr, __builtin_fmaf(-sc[i], acc[t][r], hv[i]), c0, gk, A.dt, A.dta0);
                        xv[r] = xr;
                        yv[r] = yr;
                        bits[r] = shift_in(bits[r], xr);
                    }
                    if (i < kRegTiles) {
                        xs[i < kRegTiles ? i : 0][t] = xv;
                        ys[i < kRegTiles ? i : 0][t] = yv;
                    } else {
                        spare[64 * t] = xv;
                        spare[64 * (T + t)] = yv;
                    }
                }
                const uint32_t word = (bits[0] | bits[1] << 8 | bits[2] << 16 | bits[3] << 24) & live;
                const int row = bs[i] * kBR + c;
                if (row < A.n)
                    __hip_atomic_store(reinterpret_cast<uint32_t *>(Sout) + (static_cast<size_t>(row) * R + ab) * 4 + g,
                                       word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (k + 1 < k1) stop = gang_meet(flags, bands, band, k + 1 - k0, ctl + 1, k0 + 1, &stop_s);
        }
#pragma unroll
        for (int i = 0; i < kTiles; ++i) {
            if (!has[i]) continue;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                f32x4 xv, yv;
                if (i < kRegTiles) {
                    xv = xs[i < kRegTiles ? i : 0][t];
                    yv = ys[i < kRegTiles ? i : 0][t];
                } else {
                    xv = spare[64 * t];
                    yv = spare[64 * (T + t)];
                }
                *reinterpret_cast<f32x4 *>(x + tile_of(i) + 256 * t) = xv;
                *reinterpret_cast<f32x4 *>(y + tile_of(i) + 256 * t) = yv;
            }
        }
        if (stop) return;
        if (threadIdx.x == 0) __hip_atomic_store(flags + band, k1 - k0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
}

// One group's steps that a given-up run of sb_mfma_gang leaves, by one
// workgroup that waits for nobody, its blocks in turn.  Bands of a gang stop at
// different steps, so a gang of which a band did not finish is taken again from
// the start draw; the runs after it go on from the state.  Arithmetic and order
// are sb_mfma_gang's.
template <int JP, int WAVES>
__device__ __forceinline__ void alone_steps(const StreamArgs &A, const MfmaArgs &P, const GangRun &G, float *x, float *y,
                                         int ab, int bands, uint4 (&rec_lds)[WAVES][kGangRec], int &short_s) {
    constexpr int T = kMfmaGroup / 16, W = mfma_words(JP);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, c = lane & 15, k0 = G.k0, k1 = G.k1;
    const int M = A.M, R = mfma_groups(M), nb = (A.n + kBR - 1) / kBR;
    const int *__restrict__ koff = P.koff, *__restrict__ kcol = P.kcol;
    const uint64_t *__restrict__ kA = P.kA;
    auto signs = [&](int k) { return ((k - k0) & 1) ? G.S1 : G.S0; };  // that step k reads
    int kb = k0;
    if (G.ctl[1] == k0 + 1) {
        const int *flags = G.ctl + gang_words(bands) * ab + kGangHead;
        if (threadIdx.x == 0) short_s = 0;
        __syncthreads();
        for (int b = threadIdx.x; b < bands; b += 64 * WAVES)
            if (flags[b] != k1 - k0) short_s = 1;
        __syncthreads();
        if (short_s == 0) return;
        kb = 0;
        for (int b = wave; b < nb; b += WAVES)
            mfma_draw(A.n, M, G.seed_lo, G.seed_hi, G.event, b, ab, R, lane, x, y, [&](size_t at, uint32_t word) {
                __hip_atomic_store(reinterpret_cast<uint32_t *>(signs(0)) + at, word, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            });
    }
    const float c0 = static_cast<float>(A.scal[0]);
    uint4 *rec = rec_lds[wave];
    for (int k = kb; k < k1; ++k) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's records are out
        __syncthreads();
        const uint8_t *Sin = signs(k);
        uint8_t *Sout = signs(k + 1);
        const float gk = A.sched[k];
        for (int b = wave; b < nb; b += WAVES) {
            const int ks0 = koff[b], nk = koff[b + 1] - ks0;
            f32x4 acc[T];
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            for (int j = 0; j * kChunkSteps < nk; ++j) {
                uint4 rn[2];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int u = min(j * kGangSlots + lane + 64 * hh, nk * kBK - 1);
                    rn[hh] = load_record(Sin, kcol[static_cast<size_t>(ks0) * kBK + u], R, ab);
                }
                __builtin_amdgcn_wave_barrier();  // the LDS reads of the chunk before come first
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int sl = lane + 64 * hh;
                    rec[sl + sl / 8] = rn[hh];
                }
                __builtin_amdgcn_wave_barrier();
                for (int kk = 0; kk < min(kChunkSteps, nk - j * kChunkSteps); ++kk) {
                    uint32_t s8[8];
                    uint64_t a8[W];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int sl = kk * kBK + 8 * g + e;
                        s8[e] = reinterpret_cast<const uint8_t *>(rec + sl + sl / 8)[c];
                    }
#pragma unroll
                    for (int w = 0; w < W; ++w)
                        a8[w] = kA[(static_cast<size_t>(ks0 + j * kChunkSteps + kk) * 64 + lane) * W + w];
                    mfma_kstep<JP>(s8, a8, acc);
                }
            }
            const int row = b * kBR + c, rc = min(row, A.n - 1);
            const float hv = A.h[rc], sc = JP == kJFp8 ? A.rowscale[rc] : 1.0f;
            const size_t tile = (static_cast<size_t>(b) * R + ab) * (kBR * kMfmaGroup) + 4 * lane;
            uint32_t word = 0;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                f32x4 xv = *reinterpret_cast<const f32x4 *>(x + tile + 256 * t);
                f32x4 yv = *reinterpret_cast<const f32x4 *>(y + tile + 256 * t);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float xr = xv[r], yr = yv[r];
                    sb_update(xr, yr, __builtin_fmaf(-sc, acc[t][r], hv), c0, gk, A.dt, A.dta0);
                    xv[r] = xr;
                    yv[r] = yr;
                    if (kMfmaGroup * ab + 16 * t + 4 * g + r < M && xr >= 0.0f) word |= 1u << (8 * r + t);
                }
                *reinterpret_cast<f32x4 *>(x + tile + 256 * t) = xv;
                *reinterpret_cast<f32x4 *>(y + tile + 256 * t) = yv;
            }
            if (row < A.n)
                __hip_atomic_store(reinterpret_cast<uint32_t *>(Sout) + (static_cast<size_t>(row) * R + ab) * 4 + g, word,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// mfma_state of x after a run of sb_mfma_gang.  Where the run was given up, the
// first workgroup of each group of agents takes the missing steps and converts
// the group's tiles: no launch more for the runs that need none of this.
template <int JP>
__global__ __launch_bounds__(kStateThreads) void mfma_gang_state(StreamArgs A, MfmaArgs P, GangRun G, float *x, float *y,
                                                                 int bands, float *__restrict__ dst) {
    constexpr int kWaves = kStateThreads / 64;
    __shared__ StateRows rows;
    __shared__ uint4 rec[kWaves][kGangRec];
    __shared__ int short_s;
    const int R = mfma_groups(A.M), b0 = blockIdx.x / R, ab = blockIdx.x % R;
    if (G.ctl[1] == 0) {
        tile_state(A.n, A.M, b0, ab, x, dst, rows);
    } else if (b0 == 0) {
        alone_steps<JP, kWaves>(A, P, G, x, y, ab, bands, rec, short_s);
        for (int b = 0; b * kBR < A.n; ++b) {
            __syncthreads();  // the steps' stores are done, and the rows of the block before
            tile_state(A.n, A.M, b, ab, x, dst, rows);
        }
    }
}

size_t mfma_ksteps_bound(int n, int64_t nnz) {
    const size_t nb = (static_cast<size_t>(n) + kBR - 1) / kBR;
    return static_cast<size_t>(nnz) / kBK + nb + 1;
}

hipError_t launch_mfma_plan(int jprec, const StreamArgs &A, const MfmaArgs &P, hipStream_t st) {
    const int nb = (A.n + kBR - 1) / kBR;
    const unsigned gr = static_cast<unsigned>((nb * static_cast<int64_t>(kBR) + kWalkThreads - 1) / kWalkThreads);
    mfma_count<<<gr, kWalkThreads, 0, st>>>(A.n, nb, A.row_ptr, A.col, P.kcnt);
    mfma_scan<<<scan_grid(nb), kScanThreads, 0, st>>>(nb, scan_range(nb), P.kcnt, P.koff);
    switch (jprec) {
        case kJFp8: mfma_fill<kJFp8><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        case kJBf16x2: mfma_fill<kJBf16x2><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        case kJFp32: mfma_fill<kJFp32><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        case kJFp8Blk: mfma_fill<kJFp8Blk><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        case kJBf16: mfma_fill<kJBf16><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        case kJFp16: mfma_fill<kJFp16><<<gr, kWalkThreads, 0, st>>>(nb, A, P.koff, P.kcol, P.kA); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_mfma_init(int n, int M, uint64_t seed, uint32_t event, float *x, float *y, uint8_t *S,
                            hipStream_t st) {
    const int64_t tiles = static_cast<int64_t>((n + kBR - 1) / kBR) * mfma_groups(M);
    mfma_init<<<static_cast<unsigned>((tiles + 3) / 4), 256, 0, st>>>(
        n, M, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), event, x, y, S);
    return hipGetLastError();
}

hipError_t launch_mfma_state(int n, int M, const float *src, float *dst, hipStream_t st) {
    const unsigned tiles = static_cast<unsigned>((n + kBR - 1) / kBR) * mfma_groups(M);
    if (tiles > 0) mfma_state<<<tiles, kStateThreads, 0, st>>>(n, M, src, dst);
    return hipGetLastError();
}

namespace {

template <int JP>
hipError_t launch_mfma_form(const StreamArgs &A, const MfmaArgs &P, int k, float *x, float *y,
                            const uint8_t *Sin, uint8_t *Sout, hipStream_t st) {
    const int nb = (A.n + kBR - 1) / kBR;
    // x and y, FP32, past the caches when larger than the Infinity Cache
    const bool nt = static_cast<size_t>(A.n) * A.M * sizeof(float) * 2 > (size_t(256) << 20);
    const int total = mfma_words(JP) > 1 && nt ? nb * ((mfma_groups(A.M) + 3) / 4)   // shared operands
                                               : (nb + 3) / 4 * mfma_groups(A.M);
    const dim3 grid((total + 7) / 8 * 8);
    if (nt)
        sb_stream_mfma<JP, true><<<grid, 256, 0, st>>>(A, k, P.koff, P.kcol, P.kA, A.h, A.rowscale, x, y,
                                                       Sin, Sout);
    else
        sb_stream_mfma<JP, false><<<grid, 256, 0, st>>>(A, k, P.koff, P.kcol, P.kA, A.h, A.rowscale, x, y,
                                                        Sin, Sout);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stream_mfma(int jprec, const StreamArgs &A, const MfmaArgs &P, int k, float *x, float *y,
                              const uint8_t *Sin, uint8_t *Sout, hipStream_t st) {
    switch (jprec) {
        case kJFp8: return launch_mfma_form<kJFp8>(A, P, k, x, y, Sin, Sout, st);
        case kJBf16x2: return launch_mfma_form<kJBf16x2>(A, P, k, x, y, Sin, Sout, st);
        case kJFp32: return launch_mfma_form<kJFp32>(A, P, k, x, y, Sin, Sout, st);
        case kJFp8Blk: return launch_mfma_form<kJFp8Blk>(A, P, k, x, y, Sin, Sout, st);
        case kJBf16: return launch_mfma_form<kJBf16>(A, P, k, x, y, Sin, Sout, st);
        case kJFp16: return launch_mfma_form<kJFp16>(A, P, k, x, y, Sin, Sout, st);
        default: return hipErrorInvalidValue;
    }
}

int mfma_gang_bands(int n, int M, int cus) {
    const int nb = (n + kBR - 1) / kBR, R = mfma_groups(M);
    const int bands = std::min(cus / 8, nb);
    if (bands < 1 || n < kGangHead + gang_words(bands) * R) return 0;
    return (nb + bands - 1) / bands <= kGangTiles * kGangWaves ? bands : 0;
}

namespace {

template <int JP>
hipError_t launch_gang_form(const StreamArgs &A, const MfmaArgs &P, const GangRun &G, float *x, float *y, int cus,
                            hipStream_t st) {
    const int R = mfma_groups(A.M), nb = (A.n + kBR - 1) / kBR;
    const int bands = mfma_gang_bands(A.n, A.M, cus);
    const bool spare = (nb + bands - 1) / bands > kGangRegTiles * kGangWaves;
    const size_t lds = kGangWaves * (kGangRec * sizeof(uint4) + (spare ? 2 * kMfmaGroup / 16 * 64 * 16 : 0));
    return launch_with_lds(sb_mfma_gang<JP>, dim3(std::min(cus, R * bands)), dim3(64 * kGangWaves), lds, st, A, G.k0,
                           G.k1, P.koff, P.kcol, P.kA, A.h, A.rowscale, x, y, G.S0, G.S1, bands, R * bands, G.ctl);
}

template <int JP>
hipError_t launch_gang_state_form(const StreamArgs &A, const MfmaArgs &P, const GangRun &G, float *x, float *y, int cus,
                                  float *dst, hipStream_t st) {
    const unsigned tiles = static_cast<unsigned>((A.n + kBR - 1) / kBR) * mfma_groups(A.M);
    mfma_gang_state<JP><<<tiles, kStateThreads, 0, st>>>(A, P, G, x, y, mfma_gang_bands(A.n, A.M, cus), dst);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_mfma_gang(int jprec, const StreamArgs &A, const MfmaArgs &P, const GangRun &G, float *x, float *y,
                            int cus, hipStream_t st) {
    const int bands = mfma_gang_bands(A.n, A.M, cus);
    if (bands == 0) return hipErrorInvalidValue;
    // (work counter and flags; a run given up stays noted for the solve)
    hipError_t e = launch_zero_ints(G.ctl, G.k0 == 0 ? 2 : 1, st);
    if (e == hipSuccess)
        e = launch_zero_ints(G.ctl + kGangHead, gang_words(bands) * mfma_groups(A.M), st);
    if (e != hipSuccess) return e;
    switch (jprec) {
        case kJFp8: return launch_gang_form<kJFp8>(A, P, G, x, y, cus, st);
        case kJBf16x2: return launch_gang_form<kJBf16x2>(A, P, G, x, y, cus, st);
        case kJFp32: return launch_gang_form<kJFp32>(A, P, G, x, y, cus, st);
        case kJFp8Blk: return launch_gang_form<kJFp8Blk>(A, P, G, x, y, cus, st);
        case kJBf16: return launch_gang_form<kJBf16>(A, P, G, x, y, cus, st);
        case kJFp16: return launch_gang_form<kJFp16>(A, P, G, x, y, cus, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_mfma_gang_state(int jprec, const StreamArgs &A, const MfmaArgs &P, const GangRun &G, float *x,
                                  float *y, int cus, float *dst, hipStream_t st) {
    if (mfma_gang_bands(A.n, A.M, cus) == 0) return hipErrorInvalidValue;
    switch (jprec) {
        case kJFp8: return launch_gang_state_form<kJFp8>(A, P, G, x, y, cus, dst, st);
        case kJBf16x2: return launch_gang_state_form<kJBf16x2>(A, P, G, x, y, cus, dst, st);
        case kJFp32: return launch_gang_state_form<kJFp32>(A, P, G, x, y, cus, dst, st);
        case kJFp8Blk: return launch_gang_state_form<kJFp8Blk>(A, P, G, x, y, cus, dst, st);
        case kJBf16: return launch_gang_state_form<kJBf16>(A, P, G, x, y, cus, dst, st);
        case kJFp16: return launch_gang_state_form<kJFp16>(A, P, G, x, y, cus, dst, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sbt
