// Internal declarations shared by the kernels (esq_kernels.hip) and the
// host library (esq_api.hip).  Not part of the public C-ABI.
//
// Coordinates.  Odd numbers are addressed by their "odd index"
// i(m) = (m - 1) / 2, so m = 2i + 1.  For odd n, n - 2^k has odd index
// i(n) - 2^(k-1): the k-th candidate of Algorithm 2 (Section 3) sits
// 2^(k-1) bits below n in a bitmap over odd numbers.  The odd multiples of
// p^2 are p^2 (2t + 1), i.e. the odd indices congruent to (p^2 - 1) / 2
// modulo p^2 -- spaced p^2 apart, as Algorithm 1 steps by 2 p^2 in integers.
//
// A segment covers S = 2^log2S consecutive odd indices (its "main" part)
// plus hlo_words * 64 indices below it (the halo, so that candidates of the
// segment's n up to depth kh fall inside LDS) and hup_words * 64 above it.
// Bitmap bits are 1 for "not squarefree or not a positive odd number".
//
// Column layout (k_column).  A region is R = 32 W bits in W 32-bit words:
// bit j of word i is odd index B1 + j W + i, so n - 2^k sits at the same bit
// 2^(k-1) - 1 words lower (B1 is one odd index below the first n's halo): the
// search's windows are plain reads of other words, where the row layout needs
// two funnel shifts per step and word.  Word i - t < 0 is word W + i - t one
// bit up; the bit that comes in is below the region, and only the halo's own
// slots -- the first kColHalo positions, which are no n of the segment -- look
// there.
//
// Work is a list of intervals; each interval is cut into segments, and runs
// of consecutive segments ("items") are pulled by persistent workgroups from
// a device queue.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace esq {

constexpr uint32_t kWheelPeriod = 9u * 25u * 49u;  // 11025 words: the table stays in L2
constexpr uint32_t kWheelExtra = 16640;   // >= largest region in 64-bit words
constexpr uint32_t kWheel2Period = 121u * 169u;  // 20449 words: second table (11^2, 13^2)
constexpr size_t kWheelAlloc = 2u << 20;  // bytes holding both tables, at both origins
// Column layout (k_column): summary mode at the default depth, segment length
// and block size.
constexpr int kColLog2 = 18;              // log2 of the region's bits
constexpr uint32_t kColBlock = 512;       // threads per workgroup
constexpr uint32_t kColHalo = 4096;       // region bits below the segment's first n
constexpr uint32_t kColGuard = 32;        // 32-bit words below the region's word 0 in LDS
constexpr uint32_t kColSingle = 3;        // primes with at most so many marks per region go without tasks
// its two tables, in 32-bit words: one period and a region's words more each
constexpr size_t kColTableWords = (size_t)kWheelPeriod + kWheel2Period + 2 * ((1u << kColLog2) / 32);

constexpr uint32_t kFirstMedium = 5;      // primes[0 .. 5) = 3, 5, 7, 11, 13: the two tables
constexpr int kMaxKh = 13;                // deepest in-LDS level supported
constexpr int kMaxMedium = 1536;          // medium primes per launch (LDS offsets)
constexpr unsigned long long kNone = ~0ull;
constexpr int kMaxSegLog2 = 20;
constexpr uint32_t kFlushSegs = 4096;     // segments per run and per flush of partial totals
constexpr int kMinSegLog2 = 10;
constexpr int kShortSegLog2 = 14;         // shortest segment of a short launch at the default knobs
constexpr uint32_t kFinalizeSortCap = 16384;  // LDS sort capacity of the finalize pass
constexpr uint32_t kAccCopies = 16;       // of one interval's accumulators (a power of two)
constexpr uint32_t kOwnSegs = 256;        // segments per workgroup of k_bucket_own, at most
constexpr uint64_t kCofactorPrime = 1u << 20; // largest direct/cofactor cut-over considered
constexpr uint32_t kCofactorLanes = 16;   // lanes of a cofactor with a wide range of primes

// Per-interval accumulators in device scratch.  A launch of one interval has
// kAccCopies of them: workgroup b adds its counts and least n to copy b mod
// that, and k_finalize merges them.  Device-scope operations on one address take
// about 12 ns each, one after the other: a thousand workgroups that end
// together waited 12 us for each other's.
struct Acc {
    unsigned long long cnt[16];        // cnt[k]: #n still unresolved after step k (k <= k_lds)
    unsigned long long first[65];      // first[k]: least n-index with depth >= k
    unsigned long long deep_hist[65];  // tail pass: [0] no representation, [k] least k
    unsigned int status;               // ESQ_STATUS_* bits
    unsigned int pad;
};

// One interval of a launch.
struct Interval {
    int64_t A0;             // odd index of segment 0's first main bit (row layout: multiple of 64; column layout: I0)
    uint64_t I0, I1;        // verify: odd indices of the n examined; sieve: of the output bits
    uint32_t nseg;          // segments
    uint32_t seg_base;      // global index of segment 0 (bucket slots)
    uint32_t wheel_base0;   // row layout: floor((A0 - 64 hlo_words) / 64) mod kWheelPeriod
    uint32_t pmax_end;      // primes[0 .. pmax_end) are all the primes this interval needs
    uint32_t b_direct_end;  // bucket primes by first hit: primes[med_end .. b_direct_end)
    uint32_t n_cof;         // odd cofactors j = 1, 3, ... for primes from b_direct_end on
    Acc* acc;
    uint8_t* out_mink;      // per-n bytes (n-index - I0), or null
    uint64_t* out_bits;     // sieve output words, or null
    uint32_t out_shift;     // sieve: I0 - A0
    double sqrt_lo, sqrt_hi; // square roots of the least and the largest odd number of its regions
    uint32_t n_cof_wide;    // the first n_cof_wide cofactors (widest ranges) take kCofactorLanes lanes each
};

// Medium-prime lane-task, packed in a uint2: x = v q | (idx << 21), y = c q;
// it marks f + v q + t c q, t >= 0, of medium prime idx (0 = the prime 17),
// f its first hit in the region.  In the column layout y is the step scaled
// by 2^(32 - kColLog2), or 2^32 - 1 where the step is no shorter than the region,
// and only primes with more than kColSingle marks have any.

// Geometry and resources shared by every interval of a launch.
struct Launch {
    uint32_t S;                   // odd numbers per segment
    uint64_t s_inv;               // floor((2^64 - 1) / S)
    uint32_t hlo_words, hup_words, rw;  // rw = hlo_words + S/64 + hup_words (column layout: R/64)
    uint32_t n_iv;                // intervals
    uint32_t n_acc;               // accumulators: n_iv, or one interval's copies
    uint32_t n_items;             // work items in the queue
    uint32_t run_long, run_short; // one interval: see run_of
    uint32_t stage;               // per-n mode: depth bytes staged through LDS per wave
    uint32_t mode;                // 0 verify, 1 verify + per-n, 2 sieve, 3 verify in the column layout (k_column)
    uint32_t med_end;             // medium primes primes[kFirstMedium .. med_end)
    uint32_t n_tasks;
    uint32_t k_lds, kmax_eff;     // k_lds >= kmax_eff: every n unresolved in LDS is an exception
    uint32_t exc_list;            // 1: the call lists its exceptions (single interval)
    uint32_t bucket_cap;          // hit slots per segment
    uint32_t nprimes;
    const Interval* iv;
    Interval iv0;                 // one interval: its descriptor
    const uint4* items;           // (interval, first segment, segments, 0), or null: one interval
    const uint32_t* primes;       // odd primes ascending
    const uint32_t* pbits;        // bit i: 2 i + 1 is prime, for the odd numbers up to plimit
    uint32_t plimit;
    const uint64_t* qinv;         // qinv[i] = floor(2^64 / primes[i]^2) for i < n_qinv
    uint32_t n_qinv;              // every prime <= kCofactorPrime has one
    const uint2* medq;            // per medium prime: (q, S mod q)
    const uint2* tasks;           // medium-prime lane-tasks
    uint32_t tasks_in_lds;        // 1: the task table is copied into LDS
    uint32_t stagger;             // start delay per workgroup slot, in units of 64 clocks (0: none)
    uint32_t priority;            // 1: wave priority from the share of the run left
    unsigned long long* phase;    // non-null: per-phase clock ticks of the segment loop (init, marking, search or store, segments)
    const uint64_t* wheel;        // kWheelPeriod + kWheelExtra words (9, 25, 49)
    const uint64_t* wheel2;       // kWheel2Period + kWheelExtra words (121, 169)
    const uint32_t* col;          // column layout: its tables (9, 25, 49) and (121, 169)
    uint32_t n_multi;             // column layout: the first n_multi of them go by lane-tasks
    const uint32_t* task_min;     // column layout: marks that every task of a wave's 64 makes
    uint32_t origin;              // 1: a region's bit 0 is the odd index one below its word
                                  // boundary (search modes; wheel tables shifted to match)
    uint32_t* bucket_cnt;         // per global segment
    uint32_t* bucket_slot;        // bucket_cap per global segment
    unsigned int* queue;          // work-queue head
    unsigned long long* tail_n;   // n-indices unresolved after the LDS steps
    uint32_t* tail_iv;            // their interval
    uint8_t* tail_d;              // their depth from the tail pass
    unsigned long long* tail_count;
    uint64_t tail_cap;
};

// launchers (esq_kernels.hip); all return hipError_t of the launch
hipError_t launch_wheel_build(uint64_t* wheel, uint64_t* wheel2, uint32_t shift, hipStream_t s);
hipError_t launch_col_build(uint32_t* tab, hipStream_t s);
hipError_t launch_prepare(const Launch& L, Acc* accs, uint32_t nseg_total, hipStream_t s);
hipError_t launch_bucket(const Launch& L, Acc* accs, uint32_t n_heavy, uint32_t max_direct, uint32_t max_cof,
                         uint32_t p_cof, bool in_doubles, const uint4* ranges, uint32_t n_ranges, hipStream_t s);
hipError_t launch_verify(const Launch& L, uint32_t grid, uint32_t block, hipStream_t s);
hipError_t launch_tail(const Launch& L, hipStream_t s);
hipError_t launch_finalize(const Launch& L, const Acc* accs, void* out_summaries, void* out_records,
                           uint64_t* out_exceptions, uint64_t exc_cap, hipStream_t s);
hipError_t configure_kernels();
int verify_occupancy(int mode, uint32_t block, size_t lds_bytes);
size_t verify_lds_bytes(const Launch& L, uint32_t block);
constexpr size_t kVerifyLdsMax = 159 * 1024;  // dynamic LDS per workgroup
constexpr uint32_t kTailList = 64;              // n that a segment lists in LDS for the tail pass or as exceptions
constexpr uint32_t kVerifyCtrlWords = 28 + 1 + kTailList;       // the segment kernels' LDS control block, in 8-byte words
constexpr uint32_t kPhaseSlots = 8;             // phase-clock counters (3 used)
constexpr uint32_t kStageWordsPerWave = 528;    // per-n mode: one wave's 4096 depth bytes + 2 x 64 B guard

// k_verify's dynamic LDS, in 8-byte words: the region bitmap (rw), the
// control block, the medium primes' (q, S mod q) and first-hit offsets, the
// task table when it is held in LDS, and -- when per-n output is staged -- a
// store-staging area of kStageWordsPerWave words per wave, 16-byte aligned.
__host__ __device__ inline size_t verify_stage_word(uint32_t rw, uint32_t nmed, uint32_t n_tasks_lds)
{
    return ((size_t)rw + kVerifyCtrlWords + nmed + (nmed + 1) / 2 + n_tasks_lds + 1) & ~(size_t)1;
}
__host__ __device__ inline size_t verify_lds_size(uint32_t rw, uint32_t nmed, uint32_t n_tasks_lds,
                                                  bool stage, uint32_t block)
{
    if (stage)
        return (verify_stage_word(rw, nmed, n_tasks_lds) + (size_t)(block / 64) * kStageWordsPerWave) * 8;
    return ((size_t)rw + kVerifyCtrlWords + nmed + (nmed + 1) / 2 + n_tasks_lds) * 8;
}

}  // namespace esq
