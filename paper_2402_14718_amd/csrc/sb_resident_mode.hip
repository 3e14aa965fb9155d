// The resident single-event kernel (gfx950): all steps of one event in one
// launch, FP32 couplings, a workgroup per one or two agents.  The solve is
// rows_item (sb_rows_step.hpp), the step loop of the batched kernel.
//
// Paper section "Simulated Bifurcation" (bSB Eq. 5-8, dSB Eq. 9-12, aSB
// Eq. 1-4).  Built once per mode (SBT_RESIDENT_MODE), in parallel.
#include "sb_rows_step.hpp"

#if !defined(SBT_RESIDENT_MODE)
#error "build with -DSBT_RESIDENT_MODE=<0|1|2>"
#endif

namespace sbt {

template <int MODE, int TPB, int S, int W>
__global__ __launch_bounds__(TPB) void sb_resident_rows(BatchArgs B) {
    extern __shared__ __align__(16) unsigned char smem[];
    rows_item<MODE, kJFp32, TPB, S, W, true>(B, smem, 0, static_cast<int>(blockIdx.x) * W, 0);
}

namespace {

template <int MODE, int TPB, int S, int W>
hipError_t launch_shape(const BatchArgs &B, hipStream_t st) {
    using L = RowsLds<MODE, TPB, S, W>;
    if (B.one.n > S * TPB) return hipErrorInvalidValue;
    BatchArgs A = B;
    A.tail_cap = L::tail_words(B.tail_cap);
    // the 16-bit LDS addresses assume the dynamic LDS starts at address 0,
    // which holds when the kernel has no static LDS
    static const bool base_zero = [] {
        hipFuncAttributes fa{};
        return hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(sb_resident_rows<MODE, TPB, S, W>)) ==
                   hipSuccess &&
               fa.sharedSizeBytes == 0;
    }();
    if (!base_zero) return hipErrorInvalidConfiguration;
    return launch_with_lds(sb_resident_rows<MODE, TPB, S, W>, dim3((B.M + W - 1) / W), dim3(TPB),
                           L::bytes(A.tail_cap), st, A);
}

template <int MODE, int TPB>
hipError_t launch_threads(const BatchArgs &B, const RowsShape &R, hipStream_t st) {
    if (R.slots == 2 && R.agents == 1) return launch_shape<MODE, TPB, 2, 1>(B, st);
    if (R.slots == kBatchSPT && R.agents == 1) return launch_shape<MODE, TPB, kBatchSPT, 1>(B, st);
    if constexpr (TPB > 64)
        if (R.slots == 2 && R.agents == 2) return launch_shape<MODE, TPB, 2, 2>(B, st);
    if constexpr (TPB == 1024) {
        if (R.slots == 4)
            return R.agents == 2 ? launch_shape<MODE, TPB, 4, 2>(B, st) : launch_shape<MODE, TPB, 4, 1>(B, st);
        if (R.slots == kBatchSPT && R.agents == 2) return launch_shape<MODE, TPB, kBatchSPT, 2>(B, st);
        if (R.slots == 6)
            return R.agents == 2 ? launch_shape<MODE, TPB, 6, 2>(B, st) : launch_shape<MODE, TPB, 6, 1>(B, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

template <int MODE>
hipError_t launch_resident_rows_tu(const BatchArgs &B, const RowsShape &R, hipStream_t st) {
    switch (R.threads) {
        case 64: return launch_threads<MODE, 64>(B, R, st);
        case 256: return launch_threads<MODE, 256>(B, R, st);
        case 512: return launch_threads<MODE, 512>(B, R, st);
        case 1024: return launch_threads<MODE, 1024>(B, R, st);
        default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_resident_rows_tu<SBT_RESIDENT_MODE>(const BatchArgs &B, const RowsShape &R,
                                                               hipStream_t st);

}  // namespace sbt
