// Kernel argument blocks and launchers of the SB solver (host <-> device).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sbt {

constexpr int kEnergyRows = 64;  // rows per workgroup in energy_rows

struct ResidentArgs {
    int n, nnz, M, K;
    int ckpt_every;              // > 0: FP64 energy every that many steps
    double a0;
    float dt, dta0;
    const int *row_ptr;          // [n+1]
    const int *col;              // [nnz]
    const float *J;              // [nnz] FP32 couplings
    const float *h;              // [n]   FP32 field
    const double *scal;          // [0] = c0
    const double *a;             // [n]   FP64 QUBO (checkpoint energies)
    const double *b;             // [nnz]
    float *x;                    // [n*M] in: start, out: final
    float *y;                    // [n*M]
    double *etrace;              // [n_ckpt*M]
    const float *sched;          // [K] a0 - a_k (schedule table)
};

// The LDS-row resident kernel, for events past the step loop's shapes.
constexpr int kResidentThreads = 1024;
constexpr int kResidentSlots = 16;  // spins per thread
constexpr int kResidentSpins = kResidentThreads * kResidentSlots;
struct ResidentShape {
    bool jlds;                   // J held in LDS
    size_t lds_bytes;            // 0: the event does not fit
};

// Shape of the resident kernel whose rows are held in registers
// (sb_resident_mode.hip); slots = 0: the event does not fit it.
struct RowsShape {
    int threads;                 // 64, 256, 512 or 1024
    int slots;                   // spins per thread: 2, 4, 6 or 9
    int agents;                  // per workgroup: 1 or 2
};

// ---------------------------------------------------------------- batch

constexpr int kBatchTPB = 1024;                     // threads per workgroup, large shape
constexpr int kBatchTPBSmall = 512;                 // small shape (two workgroups per CU)
constexpr int kBatchSPT = 9;                        // slots per thread (both shapes)
constexpr int kBatchAgents = 2;                     // agents per slot
constexpr int kBatchSlots = kBatchTPB * kBatchSPT;  // largest n * agents / 2 per item
constexpr int kBatchSlotsSmall = kBatchTPBSmall * kBatchSPT;
constexpr int kBatchTailCap = 8192;                 // default LDS words for couplings past the
                                                    //   slots' register capacity (32 KB)
// Couplings of a row that the step loop holds in registers, by slot (slot 0 has
// the longest rows); [1]: nine slots whose state leaves room for fewer.
constexpr int kHeldCaps[2][kBatchSPT] = {{16, 8, 5, 4, 3, 2, 2, 2, 1}, {12, 6, 4, 3, 2, 2, 2, 2, 1}};
// LDS words left for other couplings by nine slots of two agents on 1024
// threads, by mode.
constexpr int kBatchListWords[3] = {4080, 7152, 4080};
// coupling formats: 16-bit (batch), FP32, FP8 e4m3 with a per-row scale,
// FP8 e4m3 with a per-block scale (blocks of 8 padded couplings of a row),
// BF16 hi + lo pairs (streaming kernels, sb_stream_kernels.hpp)
enum : int { kJFp16 = 0, kJBf16 = 1, kJFp32 = 2, kJFp8 = 3, kJFp8Blk = 4, kJBf16x2 = 5,
              kJBf16Half = 6 };  // BF16 couplings of an event where all are FP16 values too

struct BatchEvent {
    int n, nnz;
    int row_off;                 // offset into per-spin arrays (a, h, perm, best_T, T rows)
    int rp_off;                  // offset into row_ptr (row_off + event index)
    int nz_off;                  // offset into col, b, J16
    int event_id;                // Philox counter word 2
    float c0_scale;              // c0 of the event = (fixed or auto c0) * c0_scale
    int gang;                    // solved as gangs of row bands
    int chunk0;                  // first chunk of the event
};

constexpr int kEnergyChunk = 512;  // rows per workgroup of batch_energy

struct BatchArgs {
    int E, M, K, ckpt_every, n_ckpt;
    int n_items, item_begin;     // this launch's items: [item_begin, item_begin + n_items)
    int grid, tail_cap;          // persistent workgroups; LDS words for staged couplings
    int lds;                     // batch: LDS bytes of a workgroup
    uint32_t seed_lo, seed_hi;
    float dt, dta0;
    double c0_fixed;             // > 0: fixed c0 for every event
    const BatchEvent *ev;        // [E]
    const int *item_event;       // [n_items], decreasing cost
    const int *item_agent0;      // [n_items]
    const int *item_lg;          // [n_items] log2 of the agents an item holds
    const int *row_ptr;          // [sum (n + 1)] per-event row pointers (local)
    const int *col;              // [sum nnz] per-event spin ids (local)
    const double *a;             // [sum n]
    const double *b;             // [sum nnz]
    uint16_t *J16;               // [sum nnz] 16-bit couplings (prep output)
    uint16_t *colr;              // [sum nnz] rank of each column in the spin order, bit 15:
                                 //   the column is above its row (prep output; events of
                                 //   at most kBatchSlots spins)
    float *h;                    // [sum n]
    float *c0;                   // [E]
    double *offset;              // [E] Ising offset C
    int *perm;                   // [sum n] spin order per event
    int *rank;                   // [sum n] its inverse
    const float *sched;          // [K]
    void *trash;                 // 64 bytes that absorb stores of lanes without work
    int *counter;                // this launch's work queue counter
    double *etrace;              // [E * n_ckpt * M]
    int *halves;                 // [E] BF16 couplings: all of the event are FP16 values
    int *long_rows;              // [E] events of more than kBatchSlotsSmall spins whose couplings past the
                                 //   registers of two agents are more than list_room (prep output)
    int list_room;
    int over_items;              // first items of the launch for long rows that belong to the one of two agents
    double *split_at;            // [E] where rows_item splits an event's energy terms (prep output)
    double *energy;              // [E * M] final O(T)
    // batches of many items: final energies by batch_energy instead of the step kernel
    int energy_apart, n_chunks;  // chunks of kEnergyChunk rows of all events without gangs
    const int *chunk_event;      // [n_chunks]
    double *esum;                // [E * M * 2] both parts' sums (zeroed by prep)
    double *trace;               // [E * n_ckpt] best so far, or null
    double *best_energy;         // [E]
    int *best_agent;             // [E]
    int8_t *T;                   // [sum n * M] final T per agent
    float *x_out;                // [sum n * M] final positions, or null
    int8_t *best_T;              // [sum n]
    long long *ckpt_clock;       // [E * (n_ckpt + 1) * M] device wall clock at each
                                 //   agent's item start and checkpoints, or null
    // a single event solved by the same step loop (FP32 couplings)
    const float *J32;            // [nnz]
    const double *scal;          // [0] = c0
    float *y_out;                // [n * M] final momenta, or null
    BatchEvent one;              // the event
    const double *target;        // [E] or null: stop an event's work at the first
                                 //   checkpoint where an agent reaches O(T) <= target
    int *done;                   // [E] events whose target was reached (target mode)
    // events run as gangs of row bands (sb_batch_gang.hip)
    int gang_items;              // (gang, band) items, gang-major
    const int *gitem_gang;       // [gang_items]
    const int *gitem_band;       // [gang_items]
    const struct GangDesc *gangs;
    float *xg;                   // per gang: two position buffers of n floats
    int *arrive;                 // per gang: bands arrived at its barriers
    double *gpart;               // per gang: [bands][n_ckpt + 1] partial energies
    long long *gclock;           // per gang: [bands][n_ckpt + 1] wall-clock stamps
    int *gang_fault;             // set when a bounded gang wait ran out
    int *gang_counter;           // work queue of the gang launch
};

// One gang: the `bands` row bands of one (event, agent), each of at most
// `rows` consecutive spins, run by as many workgroups at once; positions
// cross bands through the gang's global buffers, one barrier per step.
struct GangDesc {
    int e, agent, bands, rows;
    long long x_off;             // offset of the gang's two position buffers in xg
    int part_off;                // offset of its [bands][n_ckpt + 1] in gpart / gclock
};

hipError_t launch_batch_prep(int jprec, const BatchArgs &B, hipStream_t st);
// resets the launch counters (kernels, so the reset can be graph-captured)
hipError_t launch_batch_reset(int *counters, int n, hipStream_t st);
// (long_rows: the items of one agent per word, 1024 threads)
hipError_t launch_batch_steps(int mode, int jprec, int tpb, bool long_rows, const BatchArgs &B, hipStream_t st);
// the step kernel of one mode, coupling format and shape, instantiated in
// its own translation unit (sb_batch_mode.hip, built once per triple)
template <int MODE, int JP, int TPB>
hipError_t launch_batch_steps_tu(const BatchArgs &B, bool long_rows, hipStream_t st);

// final energies of every event without gangs, from its agents' T
hipError_t launch_batch_energy(const BatchArgs &B, hipStream_t st);
hipError_t launch_batch_select(const BatchArgs &B, hipStream_t st);
// the gang launch (persistent grid of `B.grid` 1024-thread workgroups) and
// the reduction of its partial energies and stamps; n_gangs gangs
hipError_t launch_batch_gang(int mode, int jprec, const BatchArgs &B, hipStream_t st);
hipError_t launch_batch_gang_reduce(const BatchArgs &B, int n_gangs, hipStream_t st);
// zeroes n ints (a kernel, so it can be graph-captured)
hipError_t launch_zero_ints(int *p, int n, hipStream_t st);

hipError_t launch_prep(int n, const double *a, const int *row_ptr, const int *col, const double *b,
                       float *J, float *h, double *part, double *scal, double c0_fixed,
                       hipStream_t st);
hipError_t launch_init(int n, int M, uint64_t seed, uint32_t event, float *x, float *y,
                       hipStream_t st);
hipError_t launch_schedule(int K, double a0, float *sched, hipStream_t st);
hipError_t launch_resident(int mode, const ResidentArgs &A, const ResidentShape &S, hipStream_t st);
hipError_t launch_resident_rows(int mode, const BatchArgs &B, const RowsShape &R, hipStream_t st);
template <int MODE>
hipError_t launch_resident_rows_tu(const BatchArgs &B, const RowsShape &R, hipStream_t st);
// spin order by decreasing row length (perm, its inverse rank) and the
// columns in it (colr), for the kernels that hold rows in registers
hipError_t launch_rank_spins(int n, const int *row_ptr, const int *col, int *perm, int *rank,
                             uint16_t *colr, hipStream_t st);
hipError_t launch_energy(int n, int M, const double *a, const int *row_ptr, const int *col,
                         const double *b, const float *x, double *part, double *out,
                         hipStream_t st);
hipError_t launch_select_best(int n, int M, const double *E, const float *x, double *best_e,
                              int *best_m, int8_t *T, hipStream_t st);
hipError_t launch_trace_reduce(int n_ckpt, int M, const double *et, double *trace, hipStream_t st);

}  // namespace sbt
