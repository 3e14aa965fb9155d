// Batched SB over many events in one persistent kernel (gfx950).
//
// Paper section "Simulated Bifurcation" (bSB Eq. 5-8, dSB Eq. 9-12) applied
// to a batch of independent events (the paper solves one event at a time;
// batching is this library's scheduling, not a change of the method).
//
// Work items are (event, group of A agents) with A a power of two chosen so
// that the event's spins times A / 2 fill one workgroup's slots; items are
// ordered by decreasing cost and handed out by an atomic counter to a
// persistent grid.  Two workgroup shapes exist (the tuner decides which
// events use which): 1024 threads, one workgroup per CU, and 512 threads,
// two per CU (each workgroup's barrier stalls overlap the other's work);
// both hold 9 slots per thread within 128 VGPRs.  Couplings are stored in
// 16 bits (FP16 or BF16, the reduced precision form) next to a 16-bit LDS
// address; accumulation is FP32 and energies FP64.  The item's solve itself
// is rows_item (sb_rows_step.hpp).
//
// sb_batch_mode.hip instantiates the kernel for one (mode, coupling format,
// shape) per build of that file (in parallel), sb_batch.hip holds the
// per-event preparation and the best-agent selection.
#pragma once

#include "sb_rows_step.hpp"

namespace sbt {

// At least four waves per SIMD for either shape (128 VGPRs): 1024 threads
// are four waves per SIMD by themselves, 512 threads need the hint so that
// two workgroups fit a CU.
//
// LONG: one agent per word, for the items of events whose rows are too long
// for two (a launch of its own, which other batches do not need).  Events of
// more than kBatchSlotsSmall spins are told apart here, by batch_prep's count
// of their couplings past the registers: the launch of two agents leaves their
// items to this one.
template <int MODE, int JP, int TPB, bool LONG>
__global__ __launch_bounds__(TPB, 4) void sb_batch(BatchArgs B) {
    constexpr int kAgents = LONG ? 1 : kBatchAgents;
    extern __shared__ __align__(16) unsigned char smem[];
    using L = RowsLds<MODE, TPB, kBatchSPT, kAgents>;
    static_assert(TPB != kBatchTPB || LONG || L::kTailWords == kBatchListWords[MODE], "list of two agents");
    int *item_s = reinterpret_cast<int *>(smem + L::kItem);
    for (;;) {
        if (threadIdx.x == 0) *item_s = atomicAdd(B.counter, 1);
        __syncthreads();
        const int local = __builtin_amdgcn_readfirstlane(*item_s);
        __syncthreads();
        if (local >= B.n_items) return;
        // LONG: the items of two agents come first, an agent at a time
        const bool over = LONG && local < kBatchAgents * B.over_items;
        const int sub = over ? local % kBatchAgents : 0;
        const int item = B.item_begin + (over ? local / kBatchAgents : local - (LONG ? (kBatchAgents - 1) * B.over_items : 0));
        const int e = __builtin_amdgcn_readfirstlane(B.item_event[item]);
        const int agent0 = __builtin_amdgcn_readfirstlane(B.item_agent0[item]) + sub;
        const int lg = __builtin_amdgcn_readfirstlane(B.item_lg[item]);
        const int n = __builtin_amdgcn_readfirstlane(B.ev[e].n);
        if constexpr (TPB == kBatchTPB) {
            const bool rows_long = n > kBatchSlotsSmall && __builtin_amdgcn_readfirstlane(B.long_rows[e]) != 0;
            if (LONG ? over && (!rows_long || sub >> lg || agent0 >= B.M) : rows_long) continue;
        }
        auto solve = [&](auto jc) __attribute__((always_inline)) {
            constexpr int J = decltype(jc)::value;
            if constexpr (LONG) {
                rows_item<MODE, J, TPB, kBatchSPT, 1, false>(B, smem, e, agent0, over ? 0 : lg);
            } else {
                // an item of at most two slots runs without a branch in its
                // steps (an event of 64 spins x 16 agents: 0.45 -> 0.19 us a step)
                const int lg_groups = max(0, lg - (kBatchAgents - 1));
                if ((n << lg_groups) <= 2 * TPB)
                    rows_item<MODE, J, TPB, 2, kBatchAgents, false>(B, smem, e, agent0, lg_groups);
                else
                    rows_item<MODE, J, TPB, kBatchSPT, kBatchAgents, false>(B, smem, e, agent0, lg_groups);
            }
        };
        // BF16 couplings that are FP16 values too are held as FP16: the
        // multiply-add takes those as they are, where a BF16 value costs an
        // instruction to mask (couplings of track events lie in 0.23..0.25:
        // 128 events of 20-1000 particles, dSB: 94.3 -> 90.8 ms)
        if constexpr (JP == kJBf16) {
            if (__builtin_amdgcn_readfirstlane(B.halves[e]) != 0) {
                solve(std::integral_constant<int, kJBf16Half>{});
                continue;
            }
        }
        solve(std::integral_constant<int, JP>{});
    }
}

// The step kernel of one mode, coupling format and workgroup shape (the
// launch's work counter must already be zero).
template <int MODE, int JP, int TPB, bool LONG>
hipError_t launch_batch_kernel(const BatchArgs &B, hipStream_t st) {
    using L = RowsLds<MODE, TPB, kBatchSPT, LONG ? 1 : kBatchAgents>;
    BatchArgs A = B;
    A.lds = static_cast<int>(L::bytes(L::tail_words(B.tail_cap)));
    // the 16-bit LDS addresses assume the dynamic LDS starts at address 0,
    // which holds when the kernel has no static LDS
    static const bool base_zero = [] {
        hipFuncAttributes fa{};
        return hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(sb_batch<MODE, JP, TPB, LONG>)) ==
                   hipSuccess &&
               fa.sharedSizeBytes == 0;
    }();
    if (!base_zero) return hipErrorInvalidConfiguration;
    return launch_with_lds(sb_batch<MODE, JP, TPB, LONG>, dim3(A.grid), dim3(TPB), A.lds, st, A);
}

template <int MODE, int JP, int TPB>
hipError_t launch_batch_steps_tu(const BatchArgs &B, bool long_rows, hipStream_t st) {
    if constexpr (TPB == kBatchTPB)
        if (long_rows) return launch_batch_kernel<MODE, JP, TPB, true>(B, st);
    return long_rows ? hipErrorInvalidValue : launch_batch_kernel<MODE, JP, TPB, false>(B, st);
}

}  // namespace sbt
