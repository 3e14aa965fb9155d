// The step loop of solves whose whole state stays on chip (gfx950): one
// workgroup holds every spin of a few agents from the start draw to the
// last step.  The batched kernel (sb_batch_step.hpp) and the resident
// single-event kernel (sb_resident_mode.hip) are this body.
//
// Paper section "Simulated Bifurcation": bSB (Eq. 5-8), dSB (Eq. 9-12), aSB
// (Eq. 1-4).
//
// Layout.  An item is one event with G groups of W agents (G a power of
// two).  Its spins are ranked by decreasing row length, and position
// j = rank * G + group is one LDS word of W shared values (x, or sgn x for
// dSB).  Thread t's slot s is position s * T + t, so a wave's stores are
// consecutive words and need no address of their own (odd slots hand their
// positions to the waves in reverse order, so that no wave holds the longest
// rows of every slot); x and y of the W
// agents, the field and the row's couplings live in VGPRs.  A coupling is
// read once from LDS for all W agents, and held once.  For dSB a word holds
// the W = 2 signs as two halves +-1.0, which the fused multiply-add takes
// as they are (v_fma_mix), so a gather moves half the bytes of FP32 values.
//
// Why W = 2 and no branches per coupling but per pair: this loop is bound
// by VALU issue and by the LDS.  Rows of 64 consecutive ranks have nearly
// the same length, so each wave keeps its longest row per slot in an SGPR
// and skips whole groups of couplings past it: gathers and multiply-adds
// come to 1.03-1.1 times the couplings on events of 100 to 1000 particles,
// where fixed counts per slot came to 1.4 times.
//
// Couplings past a slot's register capacity are packed into an LDS array
// once per item and summed from there, in CSR order after the held ones; an
// item whose tails do not fit reads them from global memory.  Absent
// couplings of a group are a zero coupling to the spin itself: they add an
// exact zero.
//
// No branch around the state is divergent: lanes without work read another
// lane's data and select, and write to a dump word.  With the registers all
// in use, the register allocator places copies at the joins of divergent
// branches, ahead of the instruction that switches the lanes back on
// (seen in the ISA of an earlier form of this loop: lanes lost an address).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cstdint>
#include <type_traits>

#include "sb_device.hpp"
#include "sb_kernels.hpp"

namespace sbt {

namespace {

// Couplings held per slot, by slot: slot 0 holds the longest rows.  On the
// 1000-particle event (n = 8484, 9 slots of 1024) the longest rows by slot
// are 19-26, 6-7, 4, 3, 2, 2, 2, 2, 1.  FEW: nine slots, whose state leaves
// room for fewer (two agents, and one of FP32 dSB).  With the larger set the
// step spilled: two agents, FP32, 8484 spins x 1024, bSB 8.4 against 5.3 us a
// step; batch of 96 events of 20-400 particles, bSB, FP16, 6.19 against
// 5.95 ms; 128 of 20-1000, dSB, FP16, 31.8 against 31.2.
template <bool FEW>
struct Held {
    static __host__ __device__ constexpr int cap(int s) { return kHeldCaps[FEW ? 1 : 0][s]; }
    static __host__ __device__ constexpr int before(int s) {
        int o = 0;
        for (int i = 0; i < s; ++i) o += cap(i);
        return o;
    }
    // gathered while the slot before is summed
    static __host__ __device__ constexpr int ahead(int s) { return cap(s) < 2 ? cap(s) : 2; }
};
constexpr int kWideSlots = 6;  // slots up to which FP32 couplings have address registers of their own
constexpr uint16_t kColUpper = 0x8000;  // colr: the column is above the row (j > i)

typedef float f32x2 __attribute__((ext_vector_type(2)));

// Hides a loop-invariant register from the optimiser (an empty asm that
// "modifies" it), so that values derived from it are recomputed where used
// instead of being hoisted out of the step loop and kept live.
__device__ __forceinline__ void launder(uint32_t &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void launder_uniform(int &v) { asm volatile("" : "+s"(v)); }

// Exchanges and the largest value of a wave, for code beside the step loop:
// `lane` comes from a fresh copy (see rows_item), where __shfl_xor's six
// lane addresses would be kept in registers through the loop.
__device__ __forceinline__ int lane_xor(int v, int lane, int off) {
    return __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, v);
}
__device__ __forceinline__ double lane_xor(double v, int lane, int off) {
    const int lo = lane_xor(__double2loint(v), lane, off), hi = lane_xor(__double2hiint(v), lane, off);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ int wave_max_at(int v, int lane) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, lane_xor(v, lane, off));
    return __builtin_amdgcn_readfirstlane(v);
}

// Calls f(integral_constant<int, I>) for I = 0 .. N-1.
template <int N, int I = 0, class F>
__device__ __forceinline__ void unrolled(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<N, I + 1>(f);
    }
}

// What one LDS word holds: the shared values of W agents.
template <int MODE, int W>
struct Shared {
    static_assert(W == 1 || W == 2, "one or two agents per word");
    static constexpr bool kSigns = MODE == kDSB && W == 2;  // two halves +-1.0
    using type = std::conditional_t<kSigns, uint32_t, std::conditional_t<W == 2, f32x2, float>>;
    static constexpr uint32_t kBytes = sizeof(type);

    static __device__ __forceinline__ type pack(const float (&x)[W]) {
        if constexpr (kSigns) {
            // upper halves of both, their sign bits onto 1.0 (0x3C00)
            const uint32_t u = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]),
                                                     0x07060302u);
            uint32_t r;  // (one bitfield insert; as C++ it becomes an and and an or)
            asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(0x7FFF7FFFu), "v"(0x3C003C00u), "v"(u));
            return r;
        } else if constexpr (W == 2) {
            return f32x2{shared_value<MODE>(x[0]), shared_value<MODE>(x[1])};
        } else {
            return shared_value<MODE>(x[0]);
        }
    }
    template <int A>
    static __device__ __forceinline__ float get(type v) {
        if constexpr (kSigns)
            return static_cast<float>(__ushort_as_half(static_cast<uint16_t>(A == 0 ? v : v >> 16)));
        else if constexpr (W == 2)
            return v[A];
        else
            return v;
    }
};

// sb_step with the position's multiply-add in a register of its own: in
// place it costs a copy, because the wall test and the clamp both read it.
template <int MODE>
__device__ __forceinline__ void rows_step(float &x, float &y, float F, float c0, float g, float dt,
                                          float dta0) {
    if constexpr (MODE == kASB) {
        sb_update_asb(x, y, F, c0, g, dt, dta0);
    } else {
        const float force = __builtin_fmaf(c0, F, -(g * x));
        const float yn = __builtin_fmaf(dt, force, y);
        float xn;
        asm("v_fma_f32 %0, %1, %2, %3" : "=v"(xn) : "s"(dta0), "v"(yn), "v"(x));
        y = __builtin_fabsf(xn) > 1.0f ? 0.0f : yn;
        x = __builtin_amdgcn_fmed3f(xn, -1.0f, 1.0f);
    }
    asm volatile("" : "+v"(y));  // the select stays here
}

__device__ __forceinline__ float uniform(float v) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

// *p = v where `mine`, into the trash words elsewhere: a store with no
// branch around it.
template <class T>
__device__ __forceinline__ void put(bool mine, T *p, T v, void *trash) {
    *(mine ? p : static_cast<T *>(trash)) = v;
}

template <class T>
__device__ __forceinline__ T lds_read(uint32_t addr) {
    typedef __attribute__((address_space(3))) T lds_t;
    return *(const lds_t *)(static_cast<uintptr_t>(addr));
}

template <class T>
__device__ __forceinline__ void lds_write(uint32_t addr, T v) {
    typedef __attribute__((address_space(3))) T lds_t;
    *(lds_t *)(static_cast<uintptr_t>(addr)) = v;
}

}  // namespace

// LDS of one workgroup: two position buffers of S * TPB words, the
// reduction area where the idle position buffer is too small for it, the
// item word, the tails.
template <int MODE, int TPB, int S, int W>
struct RowsLds {
    static constexpr uint32_t kBuf = static_cast<uint32_t>(S) * TPB * Shared<MODE, W>::kBytes;
    static constexpr uint32_t kRed = sizeof(double) * TPB * W;
    static constexpr bool kRedInBuf = kRed <= kBuf;  // energies reduce in the buffer not read
    // with nine slots the VGPRs do not hold everything: what the step can
    // read back from the LDS at one word per slot leaves them -- the
    // positions where the buffers hold them whole (bSB, aSB), the fields
    // and, of two agents, the last slots' positions for dSB (a spilled
    // register costs a memory access per step instead)
    static constexpr bool kXInLds = S == kBatchSPT && MODE != kDSB;
    static constexpr bool kHInLds = S == kBatchSPT && MODE == kDSB;
    static constexpr uint32_t kH = 2 * kBuf + (kRedInBuf ? 0 : kRed);
    static constexpr int kXFrom = kXInLds ? 0 : (kHInLds && W == 2 ? 6 : S);  // slots from here on: x in the LDS
    static constexpr uint32_t kX = kH + (kHInLds ? 4u * S * TPB : 0);
    static constexpr uint32_t kItem = kX + (kHInLds ? 4u * W * (S - kXFrom) * TPB : 0);
    static constexpr uint32_t kDump = kItem + 32;  // two words that absorb writes of no one
    static constexpr uint32_t kTails = kItem + 64;
    static constexpr uint32_t kMax = TPB <= 512 && S == kBatchSPT ? 81920 : 163840;
    static constexpr int kTailWords = static_cast<int>((kMax - kTails) / 4);
    static int tail_words(int asked) { return asked < 0 ? 0 : (asked < kTailWords ? asked : kTailWords); }
    static size_t bytes(int tails) { return kTails + sizeof(uint32_t) * static_cast<size_t>(tails); }
};

// Solves one item: agents agent0 .. of event e, 2^lg groups of W; SINGLE: the
// one event, agents b * W .. in workgroup b.  (All three wave-uniform.)
template <int MODE, int JP, int TPB, int S, int W, bool SINGLE>
__device__ __forceinline__ void rows_item(const BatchArgs &B, unsigned char *smem, int e, int agent0, int lgG) {
    constexpr bool kHalf = JP == kJFp16 || JP == kJBf16Half;  // held as FP16
    using V = Shared<MODE, W>;
    using word = typename V::type;
    using L = RowsLds<MODE, TPB, S, W>;
    constexpr bool kWide = JP == kJFp32;            // coupling and address in words of their own
    constexpr uint32_t kB = V::kBytes;
    // a held address is 16 bits: the byte address where every word of the
    // first buffer has one, else the position
    constexpr bool kBytesHeld = L::kBuf <= 65536;
    constexpr uint32_t kScale = kBytesHeld ? kB : 1;
    using H = Held<S == kBatchSPT && (W == 2 || (kWide && MODE == kDSB))>;
    constexpr int kHeld = H::before(S);
    // FP32 couplings: their addresses two to a register, or one, where the
    // registers allow it (an instruction less per coupling; with the finer
    // classes of row lengths 3329 spins x 32, bSB: 0.57 -> 0.50 us a step)
    constexpr bool kPairs = !(S <= kWideSlots && W == 1);
    static_assert(H::before(1) <= 16 && S <= kBatchSPT && (kBytesHeld || L::kBuf <= 8 * 65536), "positions fit 16 bits");

    double *red_own = reinterpret_cast<double *>(smem + 2 * L::kBuf);
    int *item_s = reinterpret_cast<int *>(smem + L::kItem);
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int T = TPB, nwaves = TPB / 64;
    auto sync = [&]() __attribute__((always_inline)) {
        if constexpr (TPB == 64) {
            // one wave: the LDS executes its accesses in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    };

    const BatchEvent E = SINGLE ? B.one : B.ev[e];
    const int n = E.n;
    const int G = 1 << lgG;
    const int g = t & (G - 1);
    const int agent = agent0 + g * W;  // the first of this thread's agents
    // this thread's position within an odd slot (a wave keeps its lanes'
    // groups as long as a group fits a wave), and the position of slot s
    const int t_odd = G <= 64 ? (nwaves - 1 - wave) * 64 + (t & 63) : t;
    struct Place {
        uint32_t even, odd;
    };
    // dSB positions kept in the LDS, by thread
    using xs_t = std::conditional_t<W == 2, f32x2, float>;
    auto x_at = [&](int s) -> uint32_t {
        return L::kX + static_cast<uint32_t>(((s - L::kXFrom) * T + t) * 4 * W);
    };
    auto to_xs = [](const float (&x)[W]) __attribute__((always_inline)) -> xs_t {
        if constexpr (W == 2)
            return f32x2{x[0], x[1]};
        else
            return x[0];
    };
    auto from_xs = [](xs_t v, float (&x)[W]) __attribute__((always_inline)) {
        if constexpr (W == 2) {
            x[0] = v[0];
            x[1] = v[1];
        } else {
            x[0] = v;
        }
    };
    // what rarely runs inside the step loop computes its addresses from
    // a fresh copy instead of keeping them in registers beside the state
    auto fresh = [&]() __attribute__((always_inline)) -> Place {
        Place P{static_cast<uint32_t>(t), static_cast<uint32_t>(t_odd)};
        launder(P.even);
        launder(P.odd);
        return P;
    };
    auto place = [&](int s, const Place &P) -> int { return s * T + static_cast<int>(s & 1 ? P.odd : P.even); };
    // the agents that thread `t` (t < G) reports energies and stamps of
    auto reports = [&](int w) -> bool { return (t < G) & (agent0 + t * W + w < B.M); };
    const bool wave_reports = wave * 64 < G;
    // when each agent's work starts and reaches each checkpoint (the
    // device's constant-rate wall clock), for time-to-target
    auto stamp = [&](int slot) {
        if (!SINGLE && B.ckpt_clock && wave_reports)
            for (int w = 0; w < W; ++w)
                put(reports(w),
                    B.ckpt_clock + (static_cast<size_t>(e) * (B.n_ckpt + 1) + slot) * B.M + agent0 + t * W + w,
                    static_cast<long long>(wall_clock64()), B.trash);
    };
    stamp(0);

    float xr[L::kXInLds ? 1 : L::kXFrom][W], yr[S][W], hr[L::kHInLds ? 1 : S];
    // held couplings: 16-bit forms are one word (address low, coupling
    // high); FP32 a word each and two addresses per word
    uint32_t cw[kHeld], ca[kWide ? (kPairs ? (kHeld + 1) / 2 : kHeld) : 1];
    int cnt[S];  // longest row of this wave per slot, up to the capacity
    // tail lengths of the slots, 8 bits each in tp_lo of up to four
    // slots, else 5: slots 0-5 in tp_lo, 6-8 in the low 15 bits of
    // tp_hi; the tails' first entry above those; the wave's longest per
    // slot likewise in tm_lo, tm_hi
    constexpr int kBits = S <= 4 ? 8 : 5, kLongest = (1 << kBits) - 1;
    uint32_t tp_lo = 0, tp_hi = 0, tm_lo = 0, tm_hi = 0;
    int tsum = 0, tbig = 0, act = 0;
    // (the workgroup's LDS starts at address 0; launchers check it)
    auto tail_of = [](uint32_t lo, uint32_t hi, auto sc) -> int {
        constexpr int s = decltype(sc)::value;
        return static_cast<int>((s < 6 ? lo >> (kBits * (s < 6 ? s : 0)) : hi >> (5 * (s < 6 ? 0 : s - 6))) &
                                kLongest);
    };
    // the spin of slot s and whether there is one (otherwise another's)
    auto spin_at = [&](int s, const Place &P, bool &there) -> int {
        const int q = place(s, P) >> lgG;
        there = q < n;
        return B.perm[E.row_off + min(q, n - 1)];
    };
    auto row_of = [&](int i, bool there, int &p0) -> int {  // length of the row, 0 without a spin
        uint32_t r0 = static_cast<uint32_t>(B.row_ptr[E.rp_off + i]);
        uint32_t r1 = static_cast<uint32_t>(B.row_ptr[E.rp_off + i + 1]);
        launder(r0);  // (or the loads move under a branch)
        launder(r1);
        p0 = static_cast<int>(r0);
        return there ? static_cast<int>(r1 - r0) : 0;
    };
    auto address = [&](uint32_t colr) -> uint32_t {
        return ((colr & (kColUpper - 1)) * G + g) * kScale;
    };
    auto coupling_of = [&](uint16_t j) -> uint32_t {
        if constexpr (JP == kJBf16Half)
            return static_cast<uint32_t>(
                       __half_as_ushort(__float2half_rn(__uint_as_float(static_cast<uint32_t>(j) << 16)))) << 16;
        else
            return static_cast<uint32_t>(j) << 16;
    };
    auto coupling = [&](int p) -> uint32_t {
        if constexpr (kWide)
            return __float_as_uint(B.J32[p]);
        else
            return coupling_of(B.J16[p]);
    };
    auto self_of = [&](int s, const Place &P) -> uint32_t { return static_cast<uint32_t>(place(s, P)) * kScale; };
    if constexpr (kWide) {
#pragma unroll
        for (int c = 0; c < (kPairs ? (kHeld + 1) / 2 : kHeld); ++c) ca[c] = 0;
    }
    unrolled<S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int CAP = H::cap(s), O = H::before(s);
        const Place P = fresh();
        bool there;
        int p0;
        const int i = spin_at(s, P, there);
        const int len = row_of(i, there, p0);
        uint32_t h = __float_as_uint(B.h[E.row_off + i]);
        // every load of the row in flight (past its end: entry 0 again)
        uint32_t al[CAP], vl[CAP];
#pragma unroll
        for (int c = 0; c < CAP; ++c) {
            const int p = c < len ? E.nz_off + p0 + c : 0;
            al[c] = B.colr[p];
            vl[c] = coupling(p);
        }
        float x[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const Philox4 r = philox4x32_10(static_cast<uint32_t>(i), static_cast<uint32_t>(agent + w),
                                            static_cast<uint32_t>(E.event_id), 0u, B.seed_lo, B.seed_hi);
            x[w] = there ? philox_word_to_unit(r.v[0]) : 0.0f;
            if constexpr (s < L::kXFrom) xr[s][w] = x[w];
            yr[s][w] = there ? philox_word_to_unit(r.v[1]) : 0.0f;
        }
        if constexpr (L::kHInLds && s >= L::kXFrom) lds_write<xs_t>(x_at(s), to_xs(x));
        launder(h);
        const float hf = there ? __uint_as_float(h) : 0.0f;
        if constexpr (L::kHInLds)
            lds_write<float>(L::kH + 4u * static_cast<uint32_t>(s * T + t), hf);
        else
            hr[s] = hf;
        cnt[s] = wave_max_int(len < CAP ? len : CAP);
        const uint32_t self = self_of(s, P);
#pragma unroll
        for (int c = 0; c < CAP; ++c) {
            launder(al[c]);
            launder(vl[c]);
            const uint32_t a = c < len ? address(al[c]) : self, v = c < len ? vl[c] : 0u;
            if constexpr (kWide) {
                cw[O + c] = v;
                if constexpr (kPairs)
                    ca[(O + c) / 2] |= a << (16 * ((O + c) & 1));
                else
                    ca[O + c] = a;
            } else {
                cw[O + c] = v | a;
            }
        }
        const int tl = max(0, len - CAP);
        tbig |= tl > kLongest ? 1 : 0;
        const uint32_t tlen = static_cast<uint32_t>(min(tl, kLongest));
        const uint32_t most = static_cast<uint32_t>(wave_max_int(min(tl, kLongest)));
        if constexpr (s < 6) {
            tp_lo |= tlen << (kBits * s);
            tm_lo |= most << (kBits * s);
        } else {
            tp_hi |= tlen << (5 * (s - 6));
            tm_hi |= most << (5 * (s - 6));
        }
        tsum += tl;
        act |= there ? 1 << s : 0;
        lds_write<word>(static_cast<uint32_t>(place(s, P)) * kB, V::pack(x));
    });
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) act |= __shfl_xor(act, off, 64);
    act = __builtin_amdgcn_readfirstlane(act);
    int n_act = act ? 32 - __builtin_clz(act) : 0;  // slots with a spin: a prefix
    const int any_tail = wave_max_int(tsum);
    // offsets of the tails by a block scan; an item whose tails do not
    // fit, or that has more than a field holds, reads them from global
    // memory.  The scan's scratch is the buffer no wave reads yet.
    int *scan = reinterpret_cast<int *>(L::kRedInBuf ? smem + L::kBuf : smem + 2 * L::kBuf);
    int t_total = 0, big_total = 0;
    const int tail_cap = SINGLE ? B.tail_cap : min(B.tail_cap, (B.lds - static_cast<int>(L::kTails)) / 4);
    const int t_base = block_exclusive_scan(tsum, scan, t_total);
    (void)block_exclusive_scan(tbig, scan, big_total);
    constexpr int kTW = kWide ? 2 : 1;  // words per tail entry
    const bool lds_tails = __builtin_amdgcn_readfirstlane(t_total) * kTW <= tail_cap &&
                           __builtin_amdgcn_readfirstlane(big_total) == 0;
    if (lds_tails && any_tail > 0) {
        int o = t_base;
        unrolled<S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            const int most = tail_of(tm_lo, tm_hi, sc), len = tail_of(tp_lo, tp_hi, sc);
            if (most > 0) {
                bool there;
                int p0;
                const int i = spin_at(s, fresh(), there);
                (void)row_of(i, there, p0);
                for (int u = 0; u < most; ++u) {
                    const bool mine = u < len;
                    const int p = mine ? E.nz_off + p0 + H::cap(s) + u : 0;
                    const uint32_t a = address(B.colr[p]), v = coupling(p);
                    const uint32_t at = mine ? L::kTails + 4u * kTW * (o + u) : L::kDump;
                    if constexpr (kWide) {
                        lds_write<uint32_t>(at, v);
                        lds_write<uint32_t>(at + 4, a);
                    } else {
                        lds_write<uint32_t>(at, v | a);
                    }
                }
                o += len;
            }
        });
    }
    // slots of this wave whose rows go on in tails, or past the couplings
    // that are always gathered
    int tailed = 0, slow = 0;
    unrolled<S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if (tail_of(tm_lo, tm_hi, sc) > 0) tailed |= 1 << s;
        if (cnt[s] > H::ahead(s)) slow |= 1 << s;
    });
    tailed = __builtin_amdgcn_readfirstlane(tailed);
    slow = __builtin_amdgcn_readfirstlane(slow | tailed);
    tp_hi |= lds_tails ? static_cast<uint32_t>(t_base) << 15 : 0u;
    __syncthreads();

    const float c0 = uniform(SINGLE ? static_cast<float>(B.scal[0]) : B.c0[e]);
    const float dt = B.dt, dta0 = B.dta0;
    // the schedule a step ahead, as a vector load: a scalar one would
    // make every wait for LDS values a wait for all of them
    float gap_next = 0.0f;
    // LDS addresses of slots 0 and 1 in the first buffer, less whole slots
    uint32_t own = static_cast<uint32_t>(t) * kB, own_odd = static_cast<uint32_t>(t_odd) * kB;
    launder(own);
    launder(own_odd);
    uint32_t own_h = L::kH + 4u * static_cast<uint32_t>(t);
    uint32_t own_x = L::kX + 4u * W * static_cast<uint32_t>(t);
    if constexpr (L::kHInLds) launder(own_h);
    if constexpr (L::kHInLds && L::kXFrom < S) launder(own_x);
    int ck = 0;

    // positions of slot s in buffer `buf`
    auto state = [&](auto sc, const Place &P, int buf, float (&x)[W]) {
        constexpr int s = decltype(sc)::value;
        if constexpr (L::kXInLds) {
            const word xw = lds_read<word>(static_cast<uint32_t>(buf) * L::kBuf + static_cast<uint32_t>(place(s, P)) * kB);
            unrolled<W>([&](auto wc) { x[decltype(wc)::value] = V::template get<decltype(wc)::value>(xw); });
        } else if constexpr (s >= L::kXFrom) {
            from_xs(lds_read<xs_t>(x_at(s)), x);
        } else {
            for (int w = 0; w < W; ++w) x[w] = xr[s][w];
        }
    };

    // FP64 energy of the current state per agent (Eq. 13): out[w] is
    // agent (agent0 + t * W + w)'s in threads t < G.  The sums run
    // through the buffer that this step does not read.
    //
    // In a batch each spin's term (its row in CSR order) is split into a
    // multiple of 2^-38 and one of 2^-77 of the largest term, whose sums over
    // at most 2^14 spins are exact.  So an agent's energy does not depend on
    // which thread holds a spin: agents with equal spins have equal energies
    // under any schedule (the best of a tie is the lowest), a checkpoint's
    // energy is the final one of that state, and a target taken from either
    // is reached.  What is dropped is below 2^-64 of the largest term.
    constexpr int kParts = SINGLE ? 1 : 2;
    auto agent_energy = [&](int buf, double (&out)[W]) {
        const Place P = fresh();
        const int lane = static_cast<int>(P.even & 63u);
        double *red = L::kRedInBuf ? reinterpret_cast<double *>(smem + (buf ^ 1) * L::kBuf) : red_own;
        double v[kParts][W] = {};
        const double at = SINGLE ? 0.0 : B.split_at[e];
        unrolled<S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if (s >= n_act) return;
            bool there;
            int p0;
            const int i = spin_at(s, P, there);
            const int len = row_of(i, there, p0);
            const int most = wave_max_at(len, lane);
            const double a = B.a[E.row_off + i];
            double er[W];
            for (int w = 0; w < W; ++w) er[w] = a;
            for (int u = 0; u < most; ++u) {
                const int p = u < len ? E.nz_off + p0 + u : 0;
                const int c = B.colr[p];
                const double b = B.b[p];
                const bool pair = (u < len) & ((c & kColUpper) != 0);
                const word x = lds_read<word>(static_cast<uint32_t>(buf) * L::kBuf +
                                              (pair ? (c & (kColUpper - 1)) * G + g : 0) * kB);
                unrolled<W>([&](auto wc) {
                    constexpr int w = decltype(wc)::value;
                    er[w] += (pair & (V::template get<w>(x) >= 0.0f)) ? b : 0.0;
                });
            }
            float x[W];
            state(sc, P, buf, x);
            for (int w = 0; w < W; ++w) {
                const double term = (there & (x[w] >= 0.0f)) ? er[w] : 0.0;
                if constexpr (SINGLE)
                    v[0][w] += term;
                else
                    add_split(term, at, v[0][w], v[kParts - 1][w]);
            }
        });
        // (both parts at once where the buffer has room for them)
        constexpr int kAtOnce = L::kRedInBuf && kParts * L::kRed <= L::kBuf ? kParts : 1;
        double tot[W] = {};
        for (int part = 0; part < kParts; part += kAtOnce) {
            for (int h = 0; h < kAtOnce; ++h)
                for (int w = 0; w < W; ++w) {
                    // lanes with equal t % G hold the same agents
                    double sum = v[part + h][w];
                    for (int off = 32; off >= G; off >>= 1) sum += lane_xor(sum, lane, off);
                    red[(h * W + w) * T + t] = sum;
                }
            __syncthreads();
            for (int h = 0; h < kAtOnce; ++h)
                for (int w = 0; w < W; ++w) {
                    // group t: lane t of every wave when G <= 64; otherwise lane
                    // t % 64 of the waves whose first group is t rounded down to 64
                    double sum = 0.0;
                    if (wave_reports)
                        for (int v2 = 0; v2 < nwaves; ++v2)
                            if (G <= 64 || ((v2 * 64) & (G - 1)) == wave * 64)
                                sum += red[(h * W + w) * T + v2 * 64 + (t & 63)];
                    tot[w] += sum;  // (of exact sums: one rounding)
                }
            __syncthreads();
        }
        for (int w = 0; w < W; ++w) out[w] = tot[w];
    };

    auto held_value = [&](auto oc) __attribute__((always_inline)) -> float {
        constexpr int o = decltype(oc)::value;
        if constexpr (kWide)
            return __uint_as_float(cw[o]);
        else if constexpr (kHalf)
            return static_cast<float>(__ushort_as_half(static_cast<uint16_t>(cw[o] >> 16)));
        else
            return __uint_as_float(cw[o] & 0xFFFF0000u);
    };

    // One step reading buffer BUF and writing the other.
    auto step = [&](auto bufc, int k) __attribute__((always_inline)) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr uint32_t XO = BUF * L::kBuf, XN = (BUF ^ 1) * L::kBuf;
        const float gap = gap_next;
        gap_next = B.sched[min(k + 1, B.K - 1)];
        // (comparisons with the counts belong in the step, not in masks kept for it)
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (H::cap(s) > 3) launder_uniform(cnt[s]);
        launder_uniform(n_act);
        launder_uniform(slow);
        auto read = [&](uint32_t a16) __attribute__((always_inline)) -> word {
            return lds_read<word>(kBytesHeld ? a16 + XO : a16);
        };
        // the 16-bit address of held coupling o as a byte address
        auto addr_of = [&](auto oc) __attribute__((always_inline)) -> uint32_t {
            constexpr int o = decltype(oc)::value;
            const uint32_t wv = kWide ? ca[kPairs ? o / 2 : o] : cw[o];
            if constexpr (kWide && !kPairs) {
                static_assert(kBytesHeld, "byte addresses");
                return wv;
            } else if constexpr (kBytesHeld) {
                return kWide && (o & 1) ? wv >> 16 : wv & 0xFFFFu;
            } else {
                // position * bytes + buffer in one instruction
                uint32_t a;
                if constexpr (kWide && (o & 1))
                    a = (wv >> 16) * kB + XO;
                else if constexpr (XO == 0)
                    asm("v_mad_u32_u16 %0, %1, %2, 0" : "=v"(a) : "v"(wv), "n"(kB));
                else
                    asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(a) : "v"(wv), "n"(kB), "s"(XO));
                return a;
            }
        };
        // couplings [C0, C1) of slot s, all gathers in flight at once
        auto load = [&](auto sc, auto c0c, auto c1c, word *v) __attribute__((always_inline)) {
            constexpr int O = H::before(decltype(sc)::value), C0 = decltype(c0c)::value;
            unrolled<decltype(c1c)::value - C0>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value, o = O + C0 + u;
                if constexpr (!kWide)
                    launder(cw[o]);
                else if constexpr (!kPairs)
                    ;
                else if constexpr ((o & 1) == 0 || u == 0)
                    launder(ca[o / 2]);
                v[u] = read(addr_of(std::integral_constant<int, O + C0 + u>{}));
            });
        };
        auto add = [&](auto sc, auto c0c, auto c1c, const word *v, float (&acc)[W])
                       __attribute__((always_inline)) {
            constexpr int O = H::before(decltype(sc)::value), C0 = decltype(c0c)::value;
            unrolled<decltype(c1c)::value - C0>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                const float jv = held_value(std::integral_constant<int, O + C0 + u>{});
                unrolled<W>([&](auto wc) __attribute__((always_inline)) {
                    constexpr int w = decltype(wc)::value;
                    acc[w] = __builtin_fmaf(jv, V::template get<w>(v[u]), acc[w]);
                });
            });
        };
        using std::integral_constant;
        // the first couplings of a slot are gathered while the slot
        // before it is summed
        word base[2][2], xw[2];
        float hw[2];
        xs_t xs[2];
        auto read_ahead = [&](auto nc) __attribute__((always_inline)) {
            constexpr int n2 = decltype(nc)::value;
            load(nc, integral_constant<int, 0>{}, integral_constant<int, H::ahead(n2)>{}, base[n2 & 1]);
            if constexpr (L::kXInLds)
                xw[n2 & 1] = lds_read<word>((n2 & 1 ? own_odd : own) + (XO + static_cast<uint32_t>(n2 * T) * kB));
            if constexpr (L::kHInLds && n2 >= L::kXFrom)
                xs[n2 & 1] = lds_read<xs_t>(own_x + 4u * W * static_cast<uint32_t>((n2 - L::kXFrom) * T));
            if constexpr (L::kHInLds) hw[n2 & 1] = lds_read<float>(own_h + 4u * static_cast<uint32_t>(n2 * T));
        };
        read_ahead(integral_constant<int, 0>{});
        unrolled<S>([&](auto sc) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
            if (s >= n_act) return;
            constexpr int CAP = H::cap(s);
            float acc[W], x[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if constexpr (L::kHInLds)
                    acc[w] = hw[s & 1];
                else
                    acc[w] = hr[s];
            }
            if constexpr (s + 1 < S) read_ahead(integral_constant<int, s + 1>{});
            if (!((slow >> s) & 1)) {
                add(sc, integral_constant<int, 0>{}, integral_constant<int, H::ahead(s)>{}, base[s & 1], acc);
#pragma unroll
                for (int w = 0; w < W; ++w) asm volatile("; slot %1 short" : "+v"(acc[w]) : "n"(s));
            } else {
                // couplings [ahead, C), at most six in flight: one
                // straight run per length class
                auto row = [&](auto cc) __attribute__((always_inline)) {
                    constexpr int C = decltype(cc)::value;
                    if constexpr (C > H::ahead(s)) {
                        word v[C - H::ahead(s)];
                        load(sc, integral_constant<int, H::ahead(s)>{}, cc, v);
                        add(sc, integral_constant<int, 0>{}, integral_constant<int, H::ahead(s)>{}, base[s & 1], acc);
                        add(sc, integral_constant<int, H::ahead(s)>{}, cc, v, acc);
                    } else {
                        add(sc, integral_constant<int, 0>{}, integral_constant<int, H::ahead(s)>{}, base[s & 1], acc);
                    }
                    // (distinct per class, or the classes' ends are
                    // merged at the price of a copy per operand)
#pragma unroll
                    for (int w = 0; w < W; ++w)
                        asm volatile("; slot %1 class %2" : "+v"(acc[w]) : "n"(s), "n"(C));
                };
                auto more = [&](auto c0c, auto c1c) __attribute__((always_inline)) {
                    word v[decltype(c1c)::value - decltype(c0c)::value];
                    load(sc, c0c, c1c, v);
                    add(sc, c0c, c1c, v, acc);
                };
                // (a class of three, five or six where a slot's rows
                // often end there: a class wider is four instructions
                // per coupling that none of the rows has)
                auto upto = [&](auto cc) __attribute__((always_inline)) -> bool {
                    if constexpr (decltype(cc)::value >= CAP)
                        return true;
                    else
                        return cnt[s] <= decltype(cc)::value;
                };
                using C3 = integral_constant<int, 3>;
                using C4 = integral_constant<int, 4>;
                using C6 = integral_constant<int, 6>;
                using C8 = integral_constant<int, 8>;
                using C10 = integral_constant<int, 10>;
                using C12 = integral_constant<int, 12>;
                using End = integral_constant<int, CAP>;
                if constexpr (CAP <= 5) {
                    if (CAP > 3 && upto(C3{}))
                        row(integral_constant<int, (CAP < 3 ? CAP : 3)>{});
                    else if (CAP > 4 && upto(C4{}))
                        row(integral_constant<int, (CAP < 4 ? CAP : 4)>{});
                    else
                        row(End{});
                } else {
                    if (upto(C4{}))
                        row(C4{});
                    else if (upto(C6{}))
                        row(C6{});
                    else
                        row(integral_constant<int, (CAP < 8 ? CAP : 8)>{});
                    if constexpr (CAP > 8)
                        if (cnt[s] > 8) {
                            if (upto(C10{})) {
                                more(C8{}, C10{});
                            } else {
                                more(C8{}, C12{});
                                if constexpr (CAP > 12)
                                    if (!upto(C12{})) more(C12{}, End{});
                            }
                        }
                }
                if (__builtin_expect((tailed >> s) & 1, 0)) {
                // CSR order within the row, after the held couplings;
                // lanes past their row's end add a zero coupling
                const Place P = fresh();
                uint32_t tl_lo = tp_lo, tl_hi = tp_hi;
                launder(tl_lo);
                launder(tl_hi);
                const uint32_t self = self_of(s, P);
                auto tail_word = [&](uint32_t a16) __attribute__((always_inline)) -> word {
                    return lds_read<word>((kBytesHeld ? a16 : a16 * kB) + XO);
                };
                auto tail_add = [&](uint32_t v, word x) __attribute__((always_inline)) {
                    float jv;
                    if constexpr (kHalf)
                        jv = static_cast<float>(__ushort_as_half(static_cast<uint16_t>(v >> 16)));
                    else
                        jv = __uint_as_float(kWide ? v : v & 0xFFFF0000u);
                    unrolled<W>([&](auto wc) {
                        constexpr int w = decltype(wc)::value;
                        acc[w] = __builtin_fmaf(jv, V::template get<w>(x), acc[w]);
                    });
                };
                if (lds_tails) {
                    int o = static_cast<int>(tl_hi >> 15);
                    unrolled<s>([&](auto bc) { o += tail_of(tl_lo, tl_hi, bc); });
                    const int len = tail_of(tl_lo, tl_hi, sc), most = tail_of(tm_lo, tm_hi, sc);
                    // four at a time, so that a wave with long rows waits
                    // twice for the LDS per four couplings
                    constexpr int U = 4;
                    for (int u0 = 0; u0 < most; u0 += U) {
                        uint32_t tw[U], a16[U];
                        word x[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t at = u0 + u < len ? L::kTails + 4u * kTW * (o + u0 + u) : L::kDump;
                            tw[u] = lds_read<uint32_t>(at);
                            if constexpr (kWide) a16[u] = lds_read<uint32_t>(at + 4);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const bool mine = u0 + u < len;
                            if constexpr (kWide) {
                                tw[u] = mine ? tw[u] : 0u;
                                a16[u] = mine ? a16[u] : self;
                            } else {
                                tw[u] = mine ? tw[u] : self;
                                a16[u] = tw[u] & 0xFFFFu;
                            }
                            x[u] = tail_word(a16[u]);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) tail_add(tw[u], x[u]);
                    }
                } else {
                    bool there;
                    int p0;
                    const int i = spin_at(s, P, there);
                    const int len = row_of(i, there, p0);
                    const int most = wave_max_at(len, static_cast<int>(P.even & 63u));
                    // eight at a time (one at a time they cost a memory
                    // latency each), as runs of memory: lanes hold rows of
                    // their own, so an access costs a cache line per lane
                    // whatever its width (entries past the row's end are
                    // read, at most seven past the last row's, and not used:
                    // the arrays lie in the workspace with others after them)
                    constexpr int U = 8;
                    for (int u0 = CAP; u0 < most; u0 += U) {
                        uint32_t v[U], a[U];
                        word x[U];
                        const int at = u0 < len ? E.nz_off + p0 + u0 : 0;
                        struct __attribute__((packed, aligned(2))) Half8 {
                            uint16_t v[U];
                        };
                        const Half8 cols = *reinterpret_cast<const Half8 *>(B.colr + at);
                        if constexpr (kWide) {
                            struct __attribute__((packed, aligned(4))) Float8 {
                                float v[U];
                            };
                            const Float8 js = *reinterpret_cast<const Float8 *>(B.J32 + at);
#pragma unroll
                            for (int u = 0; u < U; ++u) v[u] = __float_as_uint(js.v[u]);
                        } else {
                            const Half8 js = *reinterpret_cast<const Half8 *>(B.J16 + at);
#pragma unroll
                            for (int u = 0; u < U; ++u) v[u] = coupling_of(js.v[u]);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) a[u] = cols.v[u];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            launder(v[u]);
                            launder(a[u]);
                            const bool mine = u0 + u < len;
                            v[u] = mine ? v[u] : 0u;
                            x[u] = tail_word(mine ? address(a[u]) : self);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) tail_add(v[u], x[u]);
                    }
                }
            }
            }
            if constexpr (L::kHInLds && s >= L::kXFrom) from_xs(xs[s & 1], x);
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if constexpr (L::kXInLds)
                    x[w] = w == 0 ? V::template get<0>(xw[s & 1]) : V::template get<W - 1>(xw[s & 1]);
                else if constexpr (s < L::kXFrom)
                    x[w] = xr[s][w];
                rows_step<MODE>(x[w], yr[s][w], acc[w], c0, gap, dt, dta0);
                if constexpr (s < L::kXFrom) xr[s][w] = x[w];
            }
            if constexpr (L::kHInLds && s >= L::kXFrom)
                lds_write<xs_t>(own_x + 4u * W * static_cast<uint32_t>((s - L::kXFrom) * T), to_xs(x));
            lds_write<word>((s & 1 ? own_odd : own) + (XN + static_cast<uint32_t>(s * T) * kB), V::pack(x));
        });
        sync();
    };
    // Steps [k, end) of a wave of up to two slots without tails, whose
    // longest rows have at most C0 and C1 couplings: no branch, every
    // gather of the step in flight at once, and the schedule read once
    // per 64 steps.  These small events are bound by the latency of a
    // step (the waves of a CU are few), not by its instructions: against
    // the branching step, 20 spins x 32 agents take 54 instead of 122 ns
    // a step, 1444 x 256 214 instead of 315 ns.
    auto straight = [&](auto c0c, auto c1c, int &k, int end) __attribute__((always_inline)) {
        constexpr int C0 = decltype(c0c)::value, C1 = decltype(c1c)::value;
        constexpr int kSlots = C1 >= 0 ? 2 : 1, kC1 = C1 > 0 ? C1 : 0;
        const int lane = t & 63;
        auto gaps_from = [&](int k0) -> float { return B.sched[min(k0 + lane, B.K - 1)]; };
        float gaps = gaps_from(k & ~63), gaps_next = gaps_from((k & ~63) + 64);
        uint32_t at[C0 + kC1];
        unrolled<C0 + kC1>([&](auto cc) {
            constexpr int c = decltype(cc)::value, o = c < C0 ? c : H::before(1) + c - C0;
            if constexpr (kWide && !kPairs)
                at[c] = ca[o];
            else
                at[c] = (kWide ? ((o & 1) ? ca[o / 2] >> 16 : ca[o / 2] & 0xFFFFu) : cw[o] & 0xFFFFu) *
                        (kBytesHeld ? 1u : kB);
        });
        auto one = [&](auto bufc, int k) __attribute__((always_inline)) {
            constexpr uint32_t XO = decltype(bufc)::value * L::kBuf, XN = (decltype(bufc)::value ^ 1) * L::kBuf;
            const float gap = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gaps), k & 63));
            word v[C0 + kC1];
#pragma unroll
            for (int c = 0; c < C0 + kC1; ++c) v[c] = lds_read<word>(at[c] + XO);
            unrolled<kSlots>([&](auto sc) __attribute__((always_inline)) {
                constexpr int s = decltype(sc)::value, O = s == 0 ? 0 : C0;
                float acc[W];
#pragma unroll
                for (int w = 0; w < W; ++w) acc[w] = hr[s];
                unrolled<(s == 0 ? C0 : kC1)>([&](auto cc) __attribute__((always_inline)) {
                    constexpr int c = decltype(cc)::value;
                    const float jv = held_value(std::integral_constant<int, H::before(s) + c>{});
                    unrolled<W>([&](auto wc) __attribute__((always_inline)) {
                        constexpr int w = decltype(wc)::value;
                        acc[w] = __builtin_fmaf(jv, V::template get<w>(v[O + c]), acc[w]);
                    });
                });
#pragma unroll
                for (int w = 0; w < W; ++w) rows_step<MODE>(xr[s][w], yr[s][w], acc[w], c0, gap, dt, dta0);
                lds_write<word>((s & 1 ? own_odd : own) + (XN + static_cast<uint32_t>(s * T) * kB), V::pack(xr[s]));
            });
            sync();
        };
        auto turn = [&]() {
            if ((k & 63) == 0) {
                gaps = gaps_next;
                gaps_next = gaps_from(k + 64);
            }
        };
        if (k & 1) {
            one(std::integral_constant<int, 1>{}, k++);
            turn();
        }
        while (k + 1 < end) {
            const int stop = min(end - 1, (k & ~63) + 63);
            for (; k < stop; k += 2) {
                one(std::integral_constant<int, 0>{}, k);
                one(std::integral_constant<int, 1>{}, k + 1);
            }
            turn();
        }
        if (k < end) one(std::integral_constant<int, 0>{}, k++);
    };
    // the straight run for this wave's rows, or none
    auto straight_run = [&](auto &k, int end) __attribute__((always_inline)) -> bool {
        if (tailed != 0) return false;
        const int l0 = cnt[0], l1 = n_act > 1 ? cnt[1] : -1;
        using std::integral_constant;
        auto first = [&](auto c0c) __attribute__((always_inline)) {
            if (l1 < 0)
                straight(c0c, integral_constant<int, -1>{}, k, end);
            else if (l1 <= 2)
                straight(c0c, integral_constant<int, 2>{}, k, end);
            else if (l1 <= 4)
                straight(c0c, integral_constant<int, 4>{}, k, end);
            else
                straight(c0c, integral_constant<int, H::cap(1)>{}, k, end);
        };
        if (l0 <= 2)
            first(integral_constant<int, 2>{});
        else if (l0 <= 4)
            first(integral_constant<int, 4>{});
        else if (l0 <= 8)
            first(integral_constant<int, 8>{});
        else if (l0 <= 12)
            first(integral_constant<int, 12>{});
        else
            first(integral_constant<int, H::cap(0)>{});
        return true;
    };
    // steps in runs between checkpoints; the buffer read at step k is k & 1
    int k = 0;
    while (k < B.K) {
        const int kend = B.ckpt_every > 0 ? min(B.K, k - k % B.ckpt_every + B.ckpt_every) : B.K;
        bool done = false;
        if constexpr (S <= 2) done = straight_run(k, kend);
        if (!done) {
            gap_next = B.sched[k];
            if (k & 1) step(std::integral_constant<int, 1>{}, k++);
            for (; k + 1 < kend; k += 2) {
                step(std::integral_constant<int, 0>{}, k);
                step(std::integral_constant<int, 1>{}, k + 1);
            }
            if (k < kend) step(std::integral_constant<int, 0>{}, k++);
        }
        const bool checkpoint = B.ckpt_every > 0 && k % B.ckpt_every == 0;
        if (checkpoint || (!SINGLE && !B.energy_apart && k == B.K)) {
            double en[W];
            agent_energy(k & 1, en);
            if (!SINGLE && wave_reports)
                for (int w = 0; w < W; ++w)
                    put(reports(w), B.energy + static_cast<size_t>(e) * B.M + agent0 + t * W + w, en[w], B.trash);
            if (!checkpoint) break;
            if (wave_reports)
                for (int w = 0; w < W; ++w)
                    put(reports(w), B.etrace + (static_cast<size_t>(e) * B.n_ckpt + ck) * B.M + agent0 + t * W + w,
                        en[w], B.trash);
            stamp(ck + 1);
            ++ck;
            // target mode: the event's work stops at the first
            // checkpoint where one of its agents (of this item or,
            // through the event's flag, of another) reaches the target
            if (!SINGLE && B.target) {
                // (an OR over the workgroup through the item word)
                bool hit = false;
                for (int w = 0; w < W; ++w) hit |= reports(w) & (en[w] <= B.target[e]);
                if (wave == 0) *item_s = 0;
                __syncthreads();
                if (__ballot(hit)) *item_s = 1;
                __syncthreads();
                if (wave == 0) {
                    const int any = __builtin_amdgcn_readfirstlane(*item_s);
                    if (any)
                        __hip_atomic_store(B.done + e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    *item_s = any | __hip_atomic_load(B.done + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                __syncthreads();
                const bool stop = __builtin_amdgcn_readfirstlane(*item_s) != 0;
                __syncthreads();
                if (stop) break;
            }
        }
    }
    // checkpoints a target stop skipped read NaN (no state was reached)
    if (wave_reports)
        for (int c = ck; c < B.n_ckpt; ++c)
            for (int w = 0; w < W; ++w) {
                put(reports(w), B.etrace + (static_cast<size_t>(e) * B.n_ckpt + c) * B.M + agent0 + t * W + w,
                    static_cast<double>(NAN), B.trash);
                if (B.ckpt_clock)
                    put(reports(w),
                        B.ckpt_clock + (static_cast<size_t>(e) * (B.n_ckpt + 1) + c + 1) * B.M + agent0 + t * W + w,
                        0ll, B.trash);
            }
    unrolled<S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if (s >= n_act) return;
        const Place P = fresh();
        bool there;
        const int i = spin_at(s, P, there);
        const size_t o = (static_cast<size_t>(E.row_off) + i) * B.M + agent;
        float x[W];
        state(sc, P, k & 1, x);
        for (int w = 0; w < W; ++w) {
            const bool mine = there & (agent + w < B.M);
            if (!SINGLE) put(mine, B.T + o + w, static_cast<int8_t>(x[w] >= 0.0f ? 1 : 0), B.trash);
            if (SINGLE || B.x_out) put(mine, B.x_out + o + w, x[w], B.trash);
            if (SINGLE && B.y_out) put(mine, B.y_out + o + w, yr[s][w], B.trash);
        }
    });
    __syncthreads();
}

}  // namespace sbt
