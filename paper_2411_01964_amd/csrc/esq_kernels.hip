// HIP kernels for gfx950 (wave64).  Exact integer work only: no floating
// point on any result and no matrix cores -- the sieve and the search are bit
// operations over 64-bit words.
//
//   k_wheel_build  periodic patterns of odd multiples of 9, 25, 49 and of 121, 169 (once)
//   k_prepare      zero the per-launch accumulators, hit counts and work queue
//                  (k_bucket_own does this itself)
//   k_bucket       primes above the medium range: every odd multiple of p^2
//                  that falls in a segment region goes to that segment's hit
//                  slots (by first hit up to a cut-over chosen per launch, at
//                  most 2^20; by cofactor enumeration above it); k_bucket_own
//                  where there are segments enough to give each workgroup its
//                  own
//   k_column       k_verify's summary form in the column layout: the default
//                  for aggregates-only calls
//   k_verify       persistent workgroups pull runs of consecutive segments;
//                  per segment: Algorithm 1 in LDS, then Algorithm 2 as a
//                  bit-sliced scan of the LDS bitmap (in per-n mode also one
//                  byte per n to HBM, staged through LDS; in sieve mode the
//                  bitmap itself to HBM)
//   k_tail         exact search for the n not resolved from LDS: a launch of its
//                  own only where they may be many (depths below 12 in LDS)
//   k_finalize     per interval: the tail search where it has no launch of its
//                  own; aggregates, record-setters, exceptions
#include <type_traits>

#include "esq.h"
#include "esq_internal.h"

namespace esq {

// ------------------------------------------------------------ wheel table

// Word w holds bits for odd indices 64w .. 64w+63 (mod the period).  An odd
// index x is an odd multiple of q = p^2 iff x = (q - 1)/2 (mod q).  A word
// pattern repeats every `period` words when gcd(64, period) = 1: 9 * 25 * 49
// for the first table, 121 * 169 for the second.  Both tables carry
// kWheelExtra more words so that a region never wraps; together they take
// about 0.5 MB and stay in L2.  A second pair of tables holds the same
// patterns one position lower (word w: odd indices 64w - 1 .. 64w + 62), for
// the search's regions, whose bit 0 sits one position below a word boundary.
__global__ void k_wheel_build(uint64_t* wheel, uint64_t* wheel2, uint32_t shift)
{
    const uint32_t n1 = kWheelPeriod + kWheelExtra, n2 = kWheel2Period + kWheelExtra;
    for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < n1 + n2;
         w += gridDim.x * blockDim.x) {
        const bool second = w >= n1;
        const uint32_t ww = second ? w - n1 : w;
        const uint32_t period = second ? kWheel2Period : kWheelPeriod;
        const uint32_t base = (uint32_t)(((uint64_t)ww * 64u + period - shift) % period);
        uint64_t word = 0;
        for (uint32_t b = 0; b < 64; b++) {
            const uint32_t x = base + b;
            const bool hit = second ? (x % 121u == 60u || x % 169u == 84u)
                                    : (x % 9u == 4u || x % 25u == 12u || x % 49u == 24u);
            if (hit)
                word |= 1ull << b;
        }
        if (second)
            wheel2[ww] = word;
        else
            wheel[ww] = word;
    }
}

hipError_t launch_wheel_build(uint64_t* wheel, uint64_t* wheel2, uint32_t shift, hipStream_t s)
{
    hipLaunchKernelGGL(k_wheel_build, dim3(1024), dim3(256), 0, s, wheel, wheel2, shift);
    return hipGetLastError();
}

// Column layout: word x of a table marks, in bit j, odd index x + j W (W =
// 2^kColLog2 / 32) modulo the table's period; W more words follow one period so
// that a region's words are consecutive.  The tables lie one after the other.
__global__ void k_col_build(uint32_t* tab)
{
    constexpr uint32_t W = (1u << kColLog2) / 32, n1 = kWheelPeriod + W, n2 = n1 + kWheel2Period + W;
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < n2; t += gridDim.x * blockDim.x) {
        uint32_t word = 0;
        for (uint32_t j = 0; j < 32; j++) {
            const uint32_t x = (t < n1 ? t : t - n1) + j * W;
            const bool hit = t < n1 ? (x % 9u == 4u || x % 25u == 12u || x % 49u == 24u)
                                    : (x % 121u == 60u || x % 169u == 84u);
            if (hit)
                word |= 1u << j;
        }
        tab[t] = word;
    }
}

hipError_t launch_col_build(uint32_t* tab, hipStream_t s)
{
    hipLaunchKernelGGL(k_col_build, dim3(512), dim3(256), 0, s, tab);
    return hipGetLastError();
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Output pointers read from an Interval in memory are generic: stores through
// them become flat stores, which also count on the LDS wait counter, so every
// later wait for an LDS read would wait for the stores to reach memory too.
// Stores to the output buffers go through these global-space views instead.
typedef __attribute__((address_space(1))) uint8_t g_u8;
typedef __attribute__((address_space(1))) uint32_t g_u32;
typedef __attribute__((address_space(1))) uint64_t g_u64;
typedef __attribute__((address_space(1))) u32x4 g_u32x4;
typedef __attribute__((address_space(1))) u64x2 g_u64x2;
typedef __attribute__((address_space(1))) unsigned long long g_ull;
typedef __attribute__((address_space(1))) unsigned int g_uint;
__device__ __forceinline__ void g_add(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_fetch_add((g_ull*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void g_min(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_fetch_min((g_ull*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void g_or(unsigned int* p, unsigned int v)
{
    __hip_atomic_fetch_or((g_uint*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t rfl(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// popcount(x) + acc in one v_bcnt_u32_b32
__device__ __forceinline__ uint32_t bcnt_acc(uint32_t x, uint32_t acc)
{
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// --------------------------------------------------------------- prepare

typedef const __attribute__((address_space(4))) Launch CLaunch;
typedef const __attribute__((address_space(4))) Interval CInterval;

// The kernel's Launch argument (the first of each kernel) and an interval's
// descriptor as constant memory, for scalar loads: one interval's lies among
// the arguments themselves, a load that is in flight from the start.
__device__ __forceinline__ CLaunch* launch_args() { return (CLaunch*)__builtin_amdgcn_kernarg_segment_ptr(); }
__device__ __forceinline__ CInterval* interval_at(const Interval* iv, uint32_t n_iv, uint32_t ivi)
{
    return n_iv == 1 ? &launch_args()->iv0 : (CInterval*)(uintptr_t)(iv + ivi);
}

// What a launch needs cleared, by thread t of n: the accumulators, the queue
// and the list's length; for one interval its descriptor's copy in memory.
__device__ __forceinline__ void prepare(const Launch& L, Acc* accs, uint32_t t, uint32_t n)
{
    if (L.n_iv == 1 && t == 0)
        *const_cast<Interval*>(L.iv) = L.iv0;
    for (uint32_t i = t; i < L.n_acc * 65u; i += n) {
        Acc* a = accs + i / 65u;
        const uint32_t k = i % 65u;
        if (k < 16)
            a->cnt[k] = 0;
        a->first[k] = kNone;
        a->deep_hist[k] = 0;
        if (k == 0) {
            a->status = 0;
            a->pad = 0;
        }
    }
    if (t == 0) {
        *L.queue = 0;
        *L.tail_count = 0;
    }
}

__global__ void k_prepare(Launch L, Acc* accs, uint32_t nseg_total)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t stride = gridDim.x * blockDim.x;
    prepare(L, accs, t, stride);
    if (L.bucket_cnt)
        for (uint32_t i = t; i < nseg_total; i += stride)
            L.bucket_cnt[i] = 0;
}

hipError_t launch_prepare(const Launch& L, Acc* accs, uint32_t nseg_total, hipStream_t s)
{
    // a thread per counter or accumulator level, at most 256 workgroups
    const uint64_t work = L.n_acc * 65ull > nseg_total ? L.n_acc * 65ull : nseg_total;
    const uint32_t grid = work >= 65536 ? 256u : (uint32_t)(work / 256) + 1;
    hipLaunchKernelGGL(k_prepare, dim3(grid), dim3(256), 0, s, L, accs, nseg_total);
    return hipGetLastError();
}

// ------------------------------------------------------- large primes

// least y >= 0 with B0 + y an odd multiple of q, in odd-index terms
__device__ __forceinline__ uint64_t first_hit(int64_t B0, uint64_t q)
{
    const int64_t d = (int64_t)((q - 1) >> 1) - B0;
    int64_t f = d % (int64_t)q;
    if (f < 0)
        f += (int64_t)q;
    return (uint64_t)f;
}

// x mod q for any x < 2^64 by Barrett reduction (Barrett, CRYPTO '86): with
// m = floor(2^64 / q), t = floor(x m / 2^64) is floor(x / q) or one less, so
// x - t q lies in [0, 2q) and one conditional subtraction finishes it
__device__ __forceinline__ uint64_t mod_barrett(uint64_t x, uint64_t q, uint64_t m)
{
    const uint64_t r = x - __umul64hi(x, m) * q;
    return r >= q ? r - q : r;
}

// first_hit with the prime's Barrett reciprocal m = floor(2^64 / q)
__device__ __forceinline__ uint64_t first_hit_b(int64_t B0, uint64_t q, uint64_t m)
{
    const int64_t h = (int64_t)((q - 1) >> 1);
    if (B0 <= h)
        return mod_barrett((uint64_t)(h - B0), q, m);
    const uint64_t r = mod_barrett((uint64_t)(B0 - h), q, m);
    return r ? q - r : 0;
}

__device__ __forceinline__ uint64_t isqrt_floor(uint64_t x)
{
    uint64_t r = (uint64_t)sqrt((double)x);
    while (r > 0 && r * r > x)
        r--;
    while ((r + 1) * (r + 1) <= x)
        r++;
    return r;
}

// first_hit in doubles, for |B0| < 2^52, 17^2 <= q < 2^41 and inv = recip_d(q): the
// quotient is below 2^44, so its error below 2^44 2^-46 = 1/4 and its floor off
// by at most one; the remainder's fma is exact, and two corrections finish it.
// A tenth of the issue time of the 64-bit integer reduction, whose multiplies
// run at a quarter of the rate or less.
__device__ __forceinline__ double first_hit_d(double B0, double q, double inv)
{
    const double d = (q - 1.0) * 0.5 - B0;
    double r = __builtin_fma(-__builtin_floor(d * inv), q, d);
    r = r < 0.0 ? r + q : r;
    return r >= q ? r - q : r;
}

// 1 / q to within a relative 2^-46: the hardware's estimate is good to 2^-23 (2^29
// units in the last place), and a Newton step squares that.
__device__ __forceinline__ double recip_d(double q)
{
    const double y = __builtin_amdgcn_rcp(q);
    return __builtin_fma(__builtin_fma(-q, y, 1.0), y, y);
}

// Segment s of an interval covers region offsets y in [s S, s S + R): a hit
// belongs to segment floor(y / S) and to each earlier segment still reaching it.
// A hit's slot number comes back from a device-scope atomic, microseconds
// later: where there are many, the hits go out kEmit at a time (y[0 .. n)).
constexpr uint32_t kEmit = 4;
template <uint32_t N>
__device__ __forceinline__ void bucket_put(const Launch& L, uint32_t seg_base, uint32_t nseg,
                                           const uint64_t (&y)[N], uint32_t n)
{
    const uint64_t S = L.S;
    const uint32_t R = L.rw * 64;
    uint64_t seg[N];
    uint32_t off[N], pos[N];
    bool again = false;
#pragma unroll
    for (uint32_t u = 0; u < N; u++) {
        // y div S through the reciprocal: at most one too small (y < 2^56)
        seg[u] = __umul64hi(y[u], L.s_inv);
        off[u] = (uint32_t)(y[u] - seg[u] * S);
        if (off[u] >= S) {
            seg[u]++;
            off[u] -= (uint32_t)S;
        }
        const bool in = u < n;
        again = again || (in && off[u] + S < R);
        pos[u] = ~0u;
        if (in && seg[u] < nseg)
            pos[u] = atomicAdd(&L.bucket_cnt[seg_base + seg[u]], 1u);
        else if (!in)
            seg[u] = 0;
    }
#pragma unroll
    for (uint32_t u = 0; u < N; u++)
        if (pos[u] < L.bucket_cap)
            L.bucket_slot[(seg_base + seg[u]) * L.bucket_cap + pos[u]] = off[u];
    if (again)  // hits in the overlap with earlier segments
        for (uint32_t u = 0; u < N; u++) {
            uint64_t g = seg[u];
            uint64_t o = off[u] + S;
            while (u < n && o < R && g > 0) {
                g--;
                const uint32_t at = atomicAdd(&L.bucket_cnt[seg_base + g], 1u);
                if (at < L.bucket_cap)
                    L.bucket_slot[(seg_base + g) * L.bucket_cap + at] = (uint32_t)o;
                o += S;
            }
        }
}

// the hits y, y + step, ... < E
__device__ __forceinline__ void bucket_emit(const Launch& L, uint32_t seg_base, uint32_t nseg, uint64_t y0,
                                            uint64_t step, uint64_t E)
{
    while (y0 < E) {
        uint64_t y[kEmit];
        uint32_t n = 0;
#pragma unroll
        for (uint32_t u = 0; u < kEmit; u++) {
            y[u] = y0 + u * step;
            n += y[u] < E ? 1u : 0u;
        }
        bucket_put(L, seg_base, nseg, y, n);
        y0 += kEmit * step;
    }
}

// The odd cofactor j's odd multiples j p^2 in the regions whose least and
// largest odd number have the square roots sqrt_lo and sqrt_hi: the p form one
// range, empty for most j when the regions are short.  Its ends, and whether an
// integer no smaller than p_cof lies in it.  The estimate of 1 / sqrt(j) is good
// to 2^-23, after a Newton step to 1.5 2^-46, so the ends (below 2^28) to 6e-6: the
// 1e-4 that they are moved outwards by covers it.
__device__ __forceinline__ bool cofactor_range(uint64_t j, double sqrt_lo, double sqrt_hi, uint32_t p_cof,
                                               double* lo_d, double* hi_d)
{
    const double jd = (double)j;
    double y = __builtin_amdgcn_rsq(jd);
    y = __builtin_fma(__builtin_fma(-jd * y, y, 1.0), 0.5 * y, y);
    *lo_d = sqrt_lo * y - 1e-4;
    *hi_d = __builtin_floor(sqrt_hi * y + 1e-4);
    return *hi_d >= *lo_d && *hi_d >= (double)p_cof;
}

// hit(y) for the region offset y of each of j's multiples of a prime p >= p_cof
// in that range; the regions' bit 0 is odd index B0 and they hold E bits.  The
// range's ends come from the estimates by exact corrections.  Its primes come
// from the bitmap of odd primes, of which lane g takes words g, g + lanes, ... of
// the range's: one load for 32 odd numbers.  What bounds a wide range is the chain
// of a lane's loads and of the hits' atomics.  2^30 odd n from 2^40, where j = 1
// has a range of 1024 numbers: k_bucket 46 us a number a load over 8 lanes, 16 a
// word a load, 9 over 16 lanes (and over 32 and 64, or with four hits in flight).
template <typename Hit>
__device__ __forceinline__ void cofactor_hits(const Launch& L, uint64_t j, double lo_d, double hi_d, int64_t B0,
                                              uint64_t E, uint32_t p_cof, uint32_t g, uint32_t lanes, Hit hit)
{
    const uint64_t m_lo = B0 > 0 ? 2 * (uint64_t)B0 + 1 : 1;
    const uint64_t m_hi = 2 * (uint64_t)(B0 + (int64_t)E - 1) + 1;
    uint64_t pa = lo_d > 0.0 ? (uint64_t)lo_d : 0;
    while (pa > 0 && j * pa * pa >= m_lo)
        pa--;
    while (j * pa * pa < m_lo)
        pa++;
    uint64_t pb = (uint64_t)hi_d + 1;
    while (j * pb * pb > m_hi)
        pb--;
    pb = min(pb, (uint64_t)L.plimit);
    const uint64_t a = max(pa, (uint64_t)p_cof) | 1, w_end = pb >> 6;
    if (a > pb)  // no odd number
        return;
    for (uint64_t w = (a >> 6) + g; w <= w_end; w += lanes) {
        // bit b: 64 w + 2 b + 1; those from a on, and up to pb
        uint32_t bits = L.pbits[w];
        if (w == a >> 6)
            bits &= ~0u << ((a >> 1) & 31u);
        if (w == w_end)
            bits &= (uint32_t)((1ull << (((pb & 63u) + 1) >> 1)) - 1);
        for (; bits; bits &= bits - 1) {
            const uint64_t p = 64 * w + 2 * (uint64_t)(__ffs((int)bits) - 1) + 1;
            hit((j * p * p - 1) / 2 - (uint64_t)B0);
        }
    }
}

// Few segments: grid.y = interval.  Work units, in order: kHeavyLanes-wide
// groups of lanes for each of the first n_heavy bucket primes (many hits: the
// group strides over them), then one thread per remaining prime of the direct
// range primes[med_end, b_direct_end), then, for the primes above it
// (p_cof and up), kCofactorLanes lanes for each of the first n_cof_wide odd
// cofactors j (wide ranges) and one thread for each remaining j.
constexpr uint32_t kHeavyLanes = 64;

__global__ __launch_bounds__(256) void k_bucket(Launch L, uint32_t n_heavy, uint32_t max_direct, uint32_t p_cof,
                                                int in_doubles)
{
    CInterval* iv = interval_at(L.iv, L.n_iv, blockIdx.y);
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t heavy_units = (uint64_t)n_heavy * kHeavyLanes;
    if (iv->nseg == 0)
        return;
    const int64_t B0 = iv->A0 - (int64_t)L.hlo_words * 64 - (int64_t)L.origin;  // region bit 0
    const uint64_t E = (uint64_t)(iv->nseg - 1) * L.S + (uint64_t)L.rw * 64;
    if (t < heavy_units + max_direct) {
        const bool heavy = t < heavy_units;
        const uint64_t pi = L.med_end + (heavy ? t / kHeavyLanes : n_heavy + (t - heavy_units));
        if (pi >= iv->b_direct_end)
            return;
        const uint64_t p = L.primes[pi];
        const uint64_t q = p * p;
        uint64_t f;
        if (in_doubles)
            f = (uint64_t)first_hit_d((double)B0, (double)q, recip_d((double)q));
        else
            f = pi < L.n_qinv ? first_hit_b(B0, q, L.qinv[pi]) : first_hit(B0, q);
        const uint64_t g = heavy ? t % kHeavyLanes : 0, stride = heavy ? kHeavyLanes : 1;
        bucket_emit(L, iv->seg_base, iv->nseg, f + g * q, stride * q, E);
        return;
    }
    const uint64_t tc = t - heavy_units - max_direct;
    const uint64_t wide_threads = (uint64_t)iv->n_cof_wide * kCofactorLanes;
    const bool wide = tc < wide_threads;
    const uint64_t c = wide ? tc / kCofactorLanes : iv->n_cof_wide + (tc - wide_threads);
    if (c >= iv->n_cof)
        return;
    double lo_d, hi_d;
    if (cofactor_range(2 * c + 1, iv->sqrt_lo, iv->sqrt_hi, p_cof, &lo_d, &hi_d))
        cofactor_hits(L, 2 * c + 1, lo_d, hi_d, B0, E, p_cof, wide ? (uint32_t)(tc % kCofactorLanes) : 0u,
                      wide ? kCofactorLanes : 1u, [&](uint64_t y) {
                          const uint64_t one[1] = {y};
                          bucket_put(L, iv->seg_base, iv->nseg, one, 1);
                      });
}

// Many segments: a workgroup owns up to kOwnSegs consecutive segments of one
// interval, takes every bucket prime and every cofactor over them, and counts
// their hits in LDS, so no counter is shared between workgroups, nor cleared
// beforehand: the launch's other clearing is done here too and k_prepare left
// out.  Counters in memory bound the other form here: the dies' atomic
// operations on them pass the L2 caches, about ten in a nanosecond.  What is
// left to bound it is finding out that a prime or cofactor has no hit in the
// range, about a dozen double-precision operations each, 3e4 of them per
// workgroup near 2^50.  1024 intervals of 2^16 .. 2^28 odd n: 156 us with
// 64-bit integer reductions, exact square roots for all and counters in memory,
// 110 with the arithmetic in doubles, 57 here; 2^33 odd n: 20 and 16 us.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_bucket_own(Launch L, Acc* accs, const uint4* ranges, uint32_t p_cof, int in_doubles)
{
    __shared__ uint32_t s_cnt[kOwnSegs];
    // The cofactors with an integer in their range and the primes with a hit,
    // about one in a hundred and one in twenty: listed, then a lane each for
    // the rest of their work, which every wave would go through for the sake
    // of a lane or two otherwise.
    constexpr uint32_t kListed = 2048;
    __shared__ uint32_t s_cof[kListed], s_prime[kListed], s_hit[kListed];
    __shared__ uint32_t s_n_cof, s_n_prime;
    uint32_t ivi = 0, s0, n;
    if (ranges) {
        const uint4 r = ranges[blockIdx.x];
        ivi = rfl(r.x);
        s0 = rfl(r.y);
        n = rfl(r.z);
    } else {
        const uint64_t ns = L.iv0.nseg;
        s0 = (uint32_t)(blockIdx.x * ns / gridDim.x);
        n = (uint32_t)((blockIdx.x + 1) * ns / gridDim.x) - s0;
    }
    CInterval* iv = interval_at(L.iv, L.n_iv, ivi);
    prepare(L, accs, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x)
        s_cnt[i] = 0;
    if (threadIdx.x == 0)
        s_n_cof = s_n_prime = 0;
    __syncthreads();
    const uint32_t S = L.S, R = L.rw * 64, cap = L.bucket_cap;
    const uint32_t gs = iv->seg_base + s0;
    // the range's regions: E bits from odd index B0 (E < 2^32)
    const int64_t B0 = iv->A0 - (int64_t)L.hlo_words * 64 - (int64_t)L.origin + (int64_t)s0 * (int64_t)S;
    const uint64_t E = (uint64_t)(n - 1) * S + R;
    uint32_t* slots = L.bucket_slot + (uint64_t)gs * cap;
    auto emit = [&](uint64_t y) {  // y < E: to its segment and each earlier one that still reaches it
        uint32_t seg = (uint32_t)__umul64hi(y, L.s_inv);
        uint32_t off = (uint32_t)y - seg * S;
        if (off >= S) {
            seg++;
            off -= S;
        }
        for (; off < R; off += S) {
            if (seg < n) {
                const uint32_t pos = atomicAdd(&s_cnt[seg], 1u);
                if (pos < cap)
                    slots[(uint64_t)seg * cap + pos] = off;
            }
            if (seg == 0)
                break;
            seg--;
        }
    };
    const uint32_t n_direct = iv->b_direct_end - L.med_end, n_cof = iv->n_cof;
    const double Ed = (double)E, B0d = (double)B0;
    const double sqrt_lo = sqrt(B0 > 0 ? 2.0 * B0d + 1.0 : 1.0), sqrt_hi = sqrt(2.0 * (B0d + Ed) - 1.0);
    auto cofactor = [&](uint32_t c, uint32_t g, uint32_t lanes) {
        double lo_d, hi_d;
        if (cofactor_range(2 * (uint64_t)c + 1, sqrt_lo, sqrt_hi, p_cof, &lo_d, &hi_d))
            cofactor_hits(L, 2 * (uint64_t)c + 1, lo_d, hi_d, B0, E, p_cof, g, lanes, emit);
    };
    for (uint32_t c = threadIdx.x; c < n_cof; c += blockDim.x) {
        double lo_d, hi_d;
        if (cofactor_range(2 * (uint64_t)c + 1, sqrt_lo, sqrt_hi, p_cof, &lo_d, &hi_d)) {
            const uint32_t at = atomicAdd(&s_n_cof, 1u);
            if (at < kListed)
                s_cof[at] = c;
            else
                cofactor(c, 0, 1);
        }
    }
    constexpr int kAhead = 4;  // primes per thread in flight
    for (uint32_t t0 = threadIdx.x; t0 < n_direct; t0 += kAhead * blockDim.x) {
        uint32_t pr[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; u++)
            pr[u] = L.primes[min(L.med_end + t0 + u * blockDim.x, L.nprimes - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
            const uint32_t t = t0 + u * blockDim.x;
            const uint64_t q = (uint64_t)pr[u] * pr[u];
            uint64_t f = E;
            if (t < n_direct) {
                if (in_doubles) {
                    const double fd = first_hit_d(B0d, (double)q, recip_d((double)q));
                    if (fd < Ed)
                        f = (uint64_t)fd;
                } else {
                    const uint32_t pi = L.med_end + t;
                    f = pi < L.n_qinv ? first_hit_b(B0, q, L.qinv[pi]) : first_hit(B0, q);
                }
            }
            if (f < E) {
                const uint32_t at = atomicAdd(&s_n_prime, 1u);
                if (at < kListed) {
                    s_prime[at] = pr[u];
                    s_hit[at] = (uint32_t)f;
                } else {
                    for (; f < E; f += q)
                        emit(f);
                }
            }
        }
    }
    __syncthreads();
    // the two lists from opposite ends of the workgroup
    const uint32_t n_listed = min(s_n_prime, kListed), c_listed = min(s_n_cof, kListed);
    for (uint32_t i = threadIdx.x; i < n_listed; i += blockDim.x)
        for (uint64_t f = s_hit[i], q = (uint64_t)s_prime[i] * s_prime[i]; f < E; f += q)
            emit(f);
    // Few cofactors have all the hits at low positions, in ranges (the widest:
    // that of j = 1) of several words of the bitmap: a lane for each word, as far
    // as there are.  2^33 odd n near 2^36: 22.6 us with a lane for each range,
    // 13.6 so; from 3 on, where the first workgroup has a range of 8192 numbers,
    // 360 and 14.8.
    uint32_t shift = 0;
    if (sqrt_hi - sqrt_lo >= 64.0)
        shift = 32u - __clz((int)((sqrt_hi - sqrt_lo) * (1.0 / 64.0)) + 1);
    while (shift && c_listed << shift > blockDim.x)
        shift--;
    for (uint32_t i = blockDim.x - 1 - threadIdx.x; i < c_listed << shift; i += blockDim.x)
        cofactor(s_cof[i >> shift], i & ((1u << shift) - 1), 1u << shift);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x)
        L.bucket_cnt[gs + i] = s_cnt[i];
}

hipError_t launch_bucket(const Launch& L, Acc* accs, uint32_t n_heavy, uint32_t max_direct, uint32_t max_cof, uint32_t p_cof,
                         bool in_doubles, const uint4* ranges, uint32_t n_ranges, hipStream_t s)
{
    if (n_ranges) {
        hipLaunchKernelGGL(k_bucket_own, dim3(n_ranges), dim3(1024), 0, s, L, accs, ranges, p_cof, in_doubles ? 1 : 0);
        return hipGetLastError();
    }
    const uint64_t threads = (uint64_t)n_heavy * kHeavyLanes + max_direct + (uint64_t)max_cof;
    if (threads == 0 || L.n_iv == 0)
        return hipSuccess;
    const uint32_t bx = (uint32_t)((threads + 255) / 256);
    hipLaunchKernelGGL(k_bucket, dim3(bx, L.n_iv), dim3(256), 0, s, L, n_heavy, max_direct, p_cof,
                       in_doubles ? 1 : 0);
    return hipGetLastError();
}

// ------------------------------------------------------- segment kernel

// 4 bits -> 4 bytes holding 0 or 1
__device__ __forceinline__ uint32_t spread4(uint32_t nib) { return (nib * 0x00204081u) & 0x01010101u; }

// bits of the 64 n-indices j0 .. j0+63 that lie in [I0, I1)
__device__ __forceinline__ uint64_t valid_mask(uint64_t j0, uint64_t I0, uint64_t I1)
{
    if (j0 + 64 <= I0 || j0 >= I1)
        return 0;
    uint64_t m = ~0ull;
    if (I0 > j0)
        m &= ~0ull << (I0 - j0);
    if (I1 < j0 + 64)
        m &= ~0ull >> (j0 + 64 - I1);
    return m;
}

// Store the 64 depth bytes D (4 per dword) of one word at out[0..63], only
// where V has a bit.  Interior dwords that are wholly ours and valid go out
// as aligned 32-bit stores; the rest byte by byte.
__device__ __forceinline__ void store_depths(g_u8* out, const uint32_t (&D)[16], uint64_t V)
{
    // whole word, 16-byte aligned (every word of an interval whose first
    // n-index is a multiple of 16): four 16-byte stores
    if (V == ~0ull && ((uintptr_t)out & 15u) == 0) {
        g_u32x4* o = (g_u32x4*)out;
#pragma unroll
        for (int q = 0; q < 4; q++)
            o[q] = u32x4{D[4 * q], D[4 * q + 1], D[4 * q + 2], D[4 * q + 3]};
        return;
    }
    const uint32_t mis = (uint32_t)((uintptr_t)out & 3u);
    g_u8* al = out - mis;
#pragma unroll
    for (int t = 0; t <= 16; t++) {
        // the aligned dword at al + 4t holds stream bytes 4t - mis .. 4t - mis + 3
        const uint32_t lo = t > 0 ? D[t - 1] : 0u;
        const uint32_t hi = t < 16 ? D[t] : 0u;
        const uint32_t val = mis ? ((hi << (8 * mis)) | (lo >> (32 - 8 * mis))) : hi;
        const int b0 = 4 * t - (int)mis;
        bool all = true;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int b = b0 + i;
            all = all && b >= 0 && b < 64 && ((V >> (b & 63)) & 1ull);
        }
        if (all) {
            *(g_u32*)(al + 4 * t) = val;
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int b = b0 + i;
                if (b >= 0 && b < 64 && ((V >> (b & 63)) & 1ull))
                    al[4 * t + i] = (uint8_t)(val >> (8 * i));
            }
        }
    }
}

__device__ __forceinline__ void mark(uint32_t* bm32, uint32_t pos)
{
    // the byte address of the word as (pos >> 3) & ~3: one shift (a half-rate
    // operation on this chip, like the mask's) and one full-rate AND, where
    // (pos >> 5) << 2 would take two shifts
    // The bitmap starts at LDS address 0 (the kernel has no static LDS), so
    // the byte offset is the LDS address itself.
    (void)bm32;
    uint32_t a;
    asm("v_lshrrev_b32 %0, 3, %1" : "=v"(a) : "v"(pos));
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    lds_u32* w = (lds_u32*)(uintptr_t)(a & ~3u);
    __hip_atomic_fetch_or(w, 1u << (pos & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Column layout: set the bit of the position whose log2R bits are the top of
// P (the bits below are ignored): the top five are the bit, the rest the word.
template <int LR>
__device__ __forceinline__ void mark_col(uint32_t P)
{
    const uint32_t a = (P >> (30 - LR)) & (((1u << (LR - 5)) - 1) << 2);
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    __hip_atomic_fetch_or((lds_u32*)(uintptr_t)a + kColGuard, 1u << (P >> 27), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Store bytes [b0, b1) of the 16 bytes v at the 16-byte aligned p (b0, b1
// wave-uniform): whole dwords as dwords, the rest byte by byte.
__device__ __forceinline__ void store_part16(g_u8* p, const u32x4 v, uint32_t b0, uint32_t b1)
{
#pragma unroll
    for (uint32_t t = 0; t < 4; t++) {
        if (4 * t >= b0 && 4 * t + 4 <= b1) {
            *(g_u32*)(p + 4 * t) = v[t];
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; j++)
                if (4 * t + j >= b0 && 4 * t + j < b1)
                    p[4 * t + j] = (uint8_t)(v[t] >> (8 * j));
        }
    }
}

// Position of 16-byte slot s (-4 <= s < 260) in a staging area: the 4 slots
// of word w = s/4 are rotated by (w/2 xor w/8) mod 4, so that any 8 (or 16)
// consecutive lanes writing one slot of their words, or reading consecutive
// slots, touch distinct groups of LDS banks, with 32 or with 64 banks.
__device__ __forceinline__ int stage_pos(int s)
{
    const int w = s >> 2;
    return 4 * w + (((s & 3) + ((w >> 1) ^ (w >> 3))) & 3);
}

// The 16 output bytes of aligned chunk c, which begins delta bytes before
// staged slot c, from the slots A = c - 1 and B = c: x holds the five dwords
// that start KQ = ceil(delta / 4) dwords before slot c, and each output dword
// is the window of two neighbours that starts sh = (-delta) mod 4 bytes in.
template <int KQ>
__device__ __forceinline__ u32x4 stage_shift(const u32x4 A, const u32x4 B, uint32_t sh)
{
    uint32_t x[5];
#pragma unroll
    for (int i = 0; i < 5; i++)
        x[i] = i < KQ ? A[4 + i - KQ] : B[(i - KQ) & 3];
    return u32x4{__builtin_amdgcn_alignbyte(x[1], x[0], sh), __builtin_amdgcn_alignbyte(x[2], x[1], sh),
                 __builtin_amdgcn_alignbyte(x[3], x[2], sh), __builtin_amdgcn_alignbyte(x[4], x[3], sh)};
}

// Per-n mode: write a wave's 4096 depth bytes (lane l holds bytes 64l ..
// 64l+63 of the run in D) to out .. out+4095 through the wave's staging area
// st (slot 0; 4 guard slots on either side), so that each global store
// writes 1 KB of consecutive bytes.  The run starts delta = out mod 16 bytes
// past an aligned chunk; the first and last chunks, shared with the
// neighbouring runs, are written in part.
template <int KQ>
__device__ __forceinline__ void stage_store_run(u32x4* st, g_u8* out, const uint32_t (&D)[16],
                                                uint32_t lane, uint32_t delta)
{
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; q++)
        st[stage_pos(4 * (int)lane + q)] = u32x4{D[4 * q], D[4 * q + 1], D[4 * q + 2], D[4 * q + 3]};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    g_u8* g = out - delta;  // 16-byte aligned
    g_u32x4* go = (g_u32x4*)g;
    const uint32_t sh = (0u - delta) & 3u;
    u32x4 last;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int c = 64 * r + (int)lane;
        const u32x4 B = st[stage_pos(c)];
        if (KQ == 0) {
            go[c] = B;
            continue;
        }
        const u32x4 v = stage_shift<KQ>(st[stage_pos(c - 1)], B, sh);
        if (r == 0 && lane == 0)
            store_part16(g, v, delta, 16);
        else
            go[c] = v;
        last = B;
    }
    if (KQ != 0 && lane == 63)
        store_part16(g + 4096, stage_shift<KQ>(last, last, sh), 0, delta);
}

// Run `it` of a launch over one interval of ns segments: the first `grid` runs
// are run_long segments each, the rest of the segments is cut into runs of
// run_short; or, with run_long = 0, n_items equal runs.
__device__ __forceinline__ void run_of(uint32_t it, uint32_t ns, uint32_t n_items, uint32_t run_long,
                                       uint32_t run_short, uint32_t grid, uint32_t* first, uint32_t* n)
{
    if (run_long == 0) {
        *first = (uint32_t)((uint64_t)it * ns / n_items);
        *n = (uint32_t)((uint64_t)(it + 1) * ns / n_items) - *first;
    } else if (it < grid) {
        *first = it * run_long;
        *n = run_long;
    } else {
        *first = grid * run_long + (it - grid) * run_short;
        *n = min(run_short, ns - *first);
    }
}

// LDS layout of k_verify: the region bitmap (rw words), a control block of
// kVerifyCtrlWords words (per-item first-n slots, level counts, the item,
// phase-clock sums), then the medium primes' (q, S mod q), their current
// first-hit offsets, the lane-task table when it fits, and in per-n mode
// (when it fits) one store-staging area per wave, 16-byte aligned.
// MODE 0: verify, aggregates only; MODE 1: verify + per-n bytes;
// MODE 2: Algorithm 1 alone, bitmap to HBM.  PH: the phase-clock instance
// (measurement only).
template <int MODE, bool PH = false>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(MODE == 0 ? 8 : 4))) void k_verify(Launch L)
{
    // No static LDS: the bitmap sits at LDS address 0, so a bit position
    // turns into a word address without a base offset.
    extern __shared__ uint64_t lds[];

    const uint32_t tid = threadIdx.x, T = blockDim.x, lane = tid & 63u;
    const uint32_t S = L.S, SW = S >> 6;
    const uint32_t R = L.rw * 64;
    const uint32_t HW = L.hlo_words;
    const uint32_t nmed = L.med_end - kFirstMedium;
    const uint32_t klds = L.k_lds;
    const uint32_t wstep = SW % kWheelPeriod;
    uint64_t* bm = lds;
    uint32_t* bm32 = reinterpret_cast<uint32_t*>(bm);
    constexpr uint32_t kCntAt = kMaxKh + 2, kItemAt = kCntAt + (kMaxKh + 2) / 2, kPhAt = kItemAt + 2;
    constexpr uint32_t kNTailAt = kPhAt + 3, kTailAt = kNTailAt + 1;
    static_assert(kTailAt + kTailList <= kVerifyCtrlWords, "k_verify control block");
    unsigned long long* s_first = reinterpret_cast<unsigned long long*>(lds + L.rw);  // kMaxKh + 2
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(lds + L.rw + kCntAt);               // kMaxKh + 1
    uint32_t* s_item = reinterpret_cast<uint32_t*>(lds + L.rw + kItemAt);             // 4
    unsigned long long* s_ph = reinterpret_cast<unsigned long long*>(lds + L.rw + kPhAt);  // 3 (phase clock)
    // the segment's n that go to the tail pass or the list of exceptions
    uint32_t* s_ntail = reinterpret_cast<uint32_t*>(lds + L.rw + kNTailAt);
    unsigned long long* s_tail = reinterpret_cast<unsigned long long*>(lds + L.rw + kTailAt);  // kTailList
    if (tid == 0) {
        s_ntail[0] = 0;
        s_ntail[1] = kTailList;
    }
    uint2* s_medq = reinterpret_cast<uint2*>(lds + L.rw + kVerifyCtrlWords);
    uint32_t* s_f = reinterpret_cast<uint32_t*>(s_medq + nmed);
    uint2* s_task = reinterpret_cast<uint2*>(lds + L.rw + kVerifyCtrlWords + nmed + (nmed + 1) / 2);
    // per-n mode: this wave's 4 KB staging area for the depth bytes
    u32x4* s_stage = reinterpret_cast<u32x4*>(lds + verify_stage_word(L.rw, nmed, L.tasks_in_lds ? L.n_tasks : 0u)) +
                     (tid >> 6) * (kStageWordsPerWave / 2) + 4;

    // per-launch tables into LDS (the bitmap region is rewritten per segment)
    for (uint32_t i = tid; i < nmed; i += T)
        s_medq[i] = L.medq[i];
    if (L.tasks_in_lds)
        for (uint32_t i = tid; i < L.n_tasks; i += T)
            s_task[i] = L.tasks[i];

    // per-lane counts of levels 1 .. kRegLevels; deeper levels, reached by few
    // words, count straight into s_cnt
    constexpr int kRegLevels = 5;
    uint32_t cnt[kRegLevels + 1];
    uint32_t found = 0;       // levels whose least n this wave has already offered
    uint32_t cur_iv = ~0u;    // interval of the partial totals (~0: none)
    uint32_t acc_segs = 0;    // segments in the partial totals
    auto flush = [&](uint32_t iv) {
        if (MODE != 2) {
            Acc* acc = L.items ? L.iv[iv].acc : L.iv0.acc + (blockIdx.x & (L.n_acc - 1));
#pragma unroll
            for (int k = 1; k <= kRegLevels; k++) {
                if (k > (int)klds)
                    break;
                uint32_t v = cnt[k];
                for (int o = 32; o > 0; o >>= 1)
                    v += __shfl_xor(v, o);
                if (lane == 0 && v)
                    atomicAdd(&s_cnt[k], v);
            }
            __syncthreads();
            if (tid >= 1 && tid <= klds && s_cnt[tid])
                g_add(&acc->cnt[tid], (unsigned long long)s_cnt[tid]);
            if (tid >= 2 && tid <= klds + 1 && s_first[tid] != kNone)
                g_min(&acc->first[tid], s_first[tid]);
        }
        __syncthreads();
    };

    // phase clock (the PH instance only, for measurement): workgroup time per
    // phase of the segment loop from the constant-rate counter, summed in LDS
    // and added to L.phase once per workgroup at exit
    uint64_t t_ph = 0;
    if (PH && tid < 3)
        s_ph[tid] = 0;
    auto phase_tick = [&](int ph) {
        if (PH) {
            const uint64_t t = __builtin_amdgcn_s_memrealtime();
            if (ph >= 0 && tid == 0)
                atomicAdd(&s_ph[ph], (unsigned long long)(t - t_ph));
            t_ph = t;
        }
    };

    // optional start delay by launch-order slot (the workgroups sharing a CU
    // come from different quarters of the grid), so that their phases --
    // L2-bound init, LDS-bound marking, VALU-bound search -- do not line up
    if (L.stagger) {
        const uint32_t slot = (uint32_t)(((uint64_t)blockIdx.x * 4u) / gridDim.x);
        for (uint32_t i = 0; i < slot * L.stagger; i++)
            __builtin_amdgcn_s_sleep(1);
    }

    // Work items.  The first is the workgroup's own number, the others come
    // from the queue (a device-scope operation of a microsecond, and of ten
    // when all workgroups start with one), if there are more than workgroups.
    bool first_item = true;
    for (;;) {
        if (tid == 0) {
            uint32_t ok = 0, ivi = 0, b = 0, cnt = 0, it = blockIdx.x;
            if (!first_item)
                it = L.n_items > gridDim.x ? gridDim.x + atomicAdd(L.queue, 1u) : ~0u;
            if (it < L.n_items) {
                ok = 1;
                if (L.items) {
                    const uint4 x = L.items[it];
                    ivi = x.x;
                    b = x.y;
                    cnt = x.z;
                } else {
                    run_of(it, L.iv0.nseg, L.n_items, L.run_long, L.run_short, gridDim.x, &b, &cnt);
                }
            }
            s_item[0] = ivi;
            s_item[1] = b;
            s_item[2] = cnt;
            s_item[3] = ok;
        }
        first_item = false;
        __syncthreads();
        const uint32_t item_ok = rfl(s_item[3]);
        const uint32_t ivi = rfl(s_item[0]), seg0 = rfl(s_item[1]), nsegs = rfl(s_item[2]);
        // the partial totals of cur_iv go to its accumulators when the next
        // run belongs to another interval, when they would exceed kFlushSegs
        // segments (32-bit counters), and at exit: one round of global
        // atomics per flush instead of one per run
        if (cur_iv != ~0u && (!item_ok || ivi != cur_iv || acc_segs + nsegs > kFlushSegs)) {
            flush(cur_iv);
            cur_iv = ~0u;
        }
        if (!item_ok) {
            if (PH && tid < 3)
                atomicAdd(&L.phase[tid], s_ph[tid]);
            break;
        }
        if (cur_iv == ~0u) {
            if (tid < kMaxKh + 2)
                s_first[tid] = kNone;
            if (tid <= kMaxKh)
                s_cnt[tid] = 0;
#pragma unroll
            for (int k = 0; k <= kRegLevels; k++)
                cnt[k] = 0;
            found = 0;
            acc_segs = 0;
            cur_iv = ivi;
            __syncthreads();
        }
        acc_segs += nsegs;
        CInterval& IV = *interval_at(L.iv, L.n_iv, ivi);
        const uint32_t cap = L.bucket_cap;
        // The issue arbiter favours older waves, so of the workgroups sharing
        // a CU the first-launched would finish far ahead of the last.  Raising
        // the priority of a workgroup with more of its run left keeps them
        // level, and the CU busy until the end.
        // Step 1 of a segment: the words of the two tables (9, 25, 49 and
        // 121, 169) ORed into the region whose first word is gw0 (table 1 at
        // offset wb), by the nl lanes lid < nl, from pair `first` on (the
        // caller wrote the pairs below first * nl); words below odd index 0
        // are all marked.  16-byte loads (two words per lane; the tables need
        // only 8-byte alignment for global loads), 16-byte LDS stores; byte
        // offsets are 32-bit so that a load is a scalar base plus one lane
        // offset.
        auto init_region = [&](int64_t gw0, uint32_t wb, uint32_t lid, uint32_t nl, uint32_t first) {
            int64_t g2 = gw0 % (int64_t)kWheel2Period;
            if (g2 < 0)
                g2 += kWheel2Period;
            const char* src = reinterpret_cast<const char*>(L.wheel + wb);
            const char* src2 = reinterpret_cast<const char*>(L.wheel2 + g2);
            char* dst = reinterpret_cast<char*>(bm);
            if (gw0 >= 0) {
                const uint32_t st = 16 * nl;
                const uint32_t pairs = L.rw / 2;
                constexpr int kInitPairs = 2;  // pairs per lane in flight (VGPR budget)
                const uint32_t passes = (pairs - first * nl) / (kInitPairs * nl);
                uint32_t off = 16 * lid + first * st;
                for (uint32_t ps = 0; ps < passes; ps++, off += kInitPairs * st) {
                    u64x2 v[kInitPairs], x[kInitPairs];
                    uint32_t o[kInitPairs];
#pragma unroll
                    for (int u = 0; u < kInitPairs; u++) {
                        // each pair's offset as its own 32-bit value, so that
                        // its loads keep the scalar-base form
                        o[u] = off + u * st;
                        if (u > 0)
                            asm volatile("" : "+v"(o[u]));
                        v[u] = *reinterpret_cast<const u64x2*>(src + o[u]);
                        x[u] = *reinterpret_cast<const u64x2*>(src2 + o[u]);
                    }
#pragma unroll
                    for (int u = 0; u < kInitPairs; u++)
                        *reinterpret_cast<u64x2*>(dst + o[u]) = v[u] | x[u];
                }
                for (; off < 16 * pairs; off += st)
                    *reinterpret_cast<u64x2*>(dst + off) =
                        *reinterpret_cast<const u64x2*>(src + off) |
                        *reinterpret_cast<const u64x2*>(src2 + off);
                if ((L.rw & 1u) && lid == 0) {
                    const uint32_t o = 8 * (L.rw - 1);
                    *reinterpret_cast<uint64_t*>(dst + o) =
                        *reinterpret_cast<const uint64_t*>(src + o) |
                        *reinterpret_cast<const uint64_t*>(src2 + o);
                }
                // at origin 1 a region whose first word starts at odd index 0
                // has bit 0 at odd index -1, not positive: marked (lane 0
                // wrote word 0 itself)
                if (gw0 == 0 && L.origin && lid == 0)
                    bm[0] |= 1ull;
            } else {
                // words below odd index 0 are all marked; at origin 1 the word
                // at index 0 starts with odd index -1, marked too
                for (uint32_t w = lid; w < L.rw; w += nl)
                    bm[w] = (gw0 + (int64_t)w < 0)
                                ? ~0ull
                                : (reinterpret_cast<const uint64_t*>(src)[w] |
                                   reinterpret_cast<const uint64_t*>(src2)[w] |
                                   (gw0 + (int64_t)w == 0 ? (uint64_t)L.origin : 0ull));
            }
        };
        // each medium prime's first hit in the region whose bit 0 is odd index
        // B1, by the nl lanes lid < nl: from scratch for a run's first segment,
        // else one segment on from the last
        auto first_hits = [&](int64_t B1, bool restart, uint32_t lid, uint32_t nl) {
            if (restart) {
                for (uint32_t i = lid; i < nmed; i += nl) {
                    s_f[i] = (uint32_t)first_hit_b(B1, s_medq[i].x, L.qinv[kFirstMedium + i]);
                }
            } else {
                for (uint32_t i = lid; i < nmed; i += nl) {
                    const uint2 qs = s_medq[i];
                    const uint32_t f = s_f[i];
                    s_f[i] = f >= qs.y ? f - qs.y : f + qs.x - qs.y;
                }
            }
        };
        auto set_priority = [&](uint32_t seg) {
            if (L.priority) {
                const uint32_t q = min(((seg0 + nsegs - seg) * 4u) / nsegs, 3u);
                if (q == 0)
                    __builtin_amdgcn_s_setprio(0);
                else if (q == 1)
                    __builtin_amdgcn_s_setprio(1);
                else if (q == 2)
                    __builtin_amdgcn_s_setprio(2);
                else
                    __builtin_amdgcn_s_setprio(3);
            }
        };

        // Algorithm 1 alone, with the waves in two roles.  A wave's vector
        // loads and stores complete on one counter, so a wave that has stores
        // in flight and then needs a load's result waits for the stores too;
        // the compiler, not knowing which lanes take which branch, places
        // such waits on every path it cannot rule out.  So the storers (upper
        // half of the waves) run a loop of their own with no global load in
        // it: they take the medium primes' first hits, mark, and write the
        // bitmap out, and their stores drain while the loaders (lower half)
        // load the next segment's tables and hit slots.  Both loops meet at
        // the same three barriers per segment.  Needs the task table in LDS
        // and an even number of waves.
        const bool split = MODE == 2 && L.tasks_in_lds && T % 128 == 0;
        if (split) {
            const uint32_t TL = T / 2, TS = T - TL;
            // wave-uniform (TL is a multiple of 64), and known to be so: each
            // wave runs exactly one of the two loops
            const bool loader = rfl(tid) < TL;
            const uint64_t n_bits = IV.I1 - IV.I0;
            const uint32_t sh = IV.out_shift;
            auto mark_medium = [&]() {
                for (uint32_t e = tid; e < L.n_tasks; e += T) {
                    const uint2 tk = s_task[e];
                    const uint32_t idx = tk.x >> 21, step = tk.y;
                    for (uint32_t pos = s_f[idx] + (tk.x & 0x1fffffu); pos < R; pos += step)
                        mark(bm32, pos);
                }
            };
            if (loader) {
                constexpr int kPre = 4;  // pairs per lane fetched a segment ahead
                u64x2 pre_v[kPre], pre_x[kPre];
                bool have_pre = false;
                const uint32_t pairs = L.rw / 2;
                for (uint32_t seg = seg0; seg < seg0 + nsegs; seg++) {
                    phase_tick(-1);
                    set_priority(seg);
                    const int64_t Bs = IV.A0 - (int64_t)HW * 64 + (int64_t)seg * (int64_t)S;
                    const int64_t B1 = Bs - (int64_t)L.origin;
                    const int64_t gw0 = Bs / 64;
                    const uint32_t wb = (uint32_t)(((uint64_t)IV.wheel_base0 + (uint64_t)seg * wstep) % kWheelPeriod);
                    const uint32_t gs = IV.seg_base + seg;
                    // the hit-slot count and first slot, then the tables (as
                    // in the single-role loop, over the loader lanes)
                    uint32_t nb = 0, slot_pos = R;
                    if (L.bucket_cnt) {
                        nb = *(const __attribute__((address_space(4))) uint32_t*)(uintptr_t)(L.bucket_cnt + gs);
                        if (nb <= cap && tid < nb)
                            slot_pos = L.bucket_slot[(uint64_t)gs * cap + tid];
                    }
                    uint32_t first = 0;  // pairs per lane fetched a segment ahead
                    if (have_pre && gw0 >= 0) {
#pragma unroll
                        for (int u = 0; u < kPre; u++)
                            *reinterpret_cast<u64x2*>(reinterpret_cast<char*>(bm) + 16 * (tid + u * TL)) =
                                pre_v[u] | pre_x[u];
                        first = kPre;
                    }
                    init_region(gw0, wb, tid, TL, first);
                    __syncthreads();
                    phase_tick(0);

                    // medium primes (both roles), the hit slots (loaders)
                    mark_medium();
                    if (L.bucket_cnt) {
                        if (nb <= cap) {
                            if (slot_pos < R)
                                mark(bm32, slot_pos);
                            const uint32_t* sl = L.bucket_slot + (uint64_t)gs * cap;
                            for (uint32_t e = tid + TL; e < nb; e += TL) {
                                const uint32_t pos = sl[e];
                                if (pos < R)
                                    mark(bm32, pos);
                            }
                        } else {
                            for (uint32_t pi = L.med_end + tid; pi < IV.pmax_end; pi += TL) {
                                const uint64_t p = L.primes[pi];
                                const uint64_t q = p * p;
                                for (uint64_t pos = first_hit(B1, q); pos < R; pos += q)
                                    mark(bm32, (uint32_t)pos);
                            }
                        }
                    }
                    __syncthreads();
                    phase_tick(1);

                    // the next segment's first kPre pairs per lane, at the
                    // addresses its init uses
                    have_pre = seg + 1 < seg0 + nsegs && gw0 + (int64_t)SW >= 0 && pairs / TL >= (uint32_t)kPre;
                    if (have_pre) {
                        const int64_t gwn = gw0 + (int64_t)SW;
                        const uint32_t wbn = wb + wstep >= kWheelPeriod ? wb + wstep - kWheelPeriod : wb + wstep;
                        const char* sn = reinterpret_cast<const char*>(L.wheel + wbn);
                        const char* sn2 = reinterpret_cast<const char*>(L.wheel2 + gwn % (int64_t)kWheel2Period);
#pragma unroll
                        for (int u = 0; u < kPre; u++) {
                            uint32_t o = 16 * tid + u * 16 * TL;
                            if (u > 0)
                                asm volatile("" : "+v"(o));
                            pre_v[u] = *reinterpret_cast<const u64x2*>(sn + o);
                            pre_x[u] = *reinterpret_cast<const u64x2*>(sn2 + o);
                        }
                    }
                    __syncthreads();
                    phase_tick(2);
                }
            } else {
                const uint32_t sid = tid - TL;
                for (uint32_t seg = seg0; seg < seg0 + nsegs; seg++) {
                    phase_tick(-1);
                    set_priority(seg);
                    const int64_t B1 = IV.A0 - (int64_t)HW * 64 + (int64_t)seg * (int64_t)S - (int64_t)L.origin;
                    first_hits(B1, seg == seg0, sid, TS);
                    __syncthreads();
                    phase_tick(0);

                    mark_medium();
                    __syncthreads();
                    phase_tick(1);

                    // the segment's output words (as in the single-role loop)
                    const uint64_t wo0 = (uint64_t)seg * SW;
                    if (wo0 * 64 + (uint64_t)SW * 64 <= n_bits && (((uintptr_t)IV.out_bits) & 15u) == 0) {
                        for (uint32_t lw = 2 * sid; lw < SW; lw += 2 * TS) {
                            const uint64_t w0 = bm[lw], w1 = bm[lw + 1], w2 = bm[lw + 2];
                            u64x2 o;
                            o.x = ~(sh ? ((w0 >> sh) | (w1 << (64 - sh))) : w0);
                            o.y = ~(sh ? ((w1 >> sh) | (w2 << (64 - sh))) : w1);
                            *(g_u64x2*)((g_u64*)IV.out_bits + wo0 + lw) = o;
                        }
                    } else {
                        for (uint32_t lw = sid; lw < SW; lw += TS) {
                            const uint64_t wo = wo0 + lw;
                            if (wo * 64 >= n_bits)
                                break;
                            const uint64_t lo = bm[lw], hi = bm[lw + 1];
                            uint64_t out = ~(sh ? ((lo >> sh) | (hi << (64 - sh))) : lo);
                            const uint64_t rem = n_bits - wo * 64;
                            if (rem < 64)
                                out &= (1ull << rem) - 1;
                            ((g_u64*)IV.out_bits)[wo] = out;
                        }
                    }
                    __syncthreads();
                    phase_tick(2);
                }
            }
        }

        for (uint32_t seg = seg0; seg < seg0 + nsegs && !split; seg++) {
            phase_tick(-1);
            set_priority(seg);
            // the region's words start at odd index Bs (a multiple of 64) for
            // the wheel tables (at the launch's origin); its bit 0 is odd index
            // B1 = Bs - origin
            const int64_t Bs = IV.A0 - (int64_t)HW * 64 + (int64_t)seg * (int64_t)S;
            const int64_t B1 = Bs - (int64_t)L.origin;
            const int64_t gw0 = Bs / 64;  // exact: Bs is a multiple of 64
            const uint32_t wb = (uint32_t)(((uint64_t)IV.wheel_base0 + (uint64_t)seg * wstep) % kWheelPeriod);

            // 0. the segment's hit-slot count and this lane's first slot, fetched
            //    now so that their latency overlaps the wheel loads
            const uint32_t gs = IV.seg_base + seg;
            uint32_t nb = 0, slot_pos = R;
            if (L.bucket_cnt) {
                // read-only here: a scalar (constant address space) load
                nb = *(const __attribute__((address_space(4))) uint32_t*)(uintptr_t)(L.bucket_cnt + gs);
                if (nb <= cap && tid < nb)
                    slot_pos = L.bucket_slot[(uint64_t)gs * cap + tid];
            }

            // 1. the wheel: odd multiples of 9, 25, 49 and of 121, 169 from the
            //    two tables; each medium prime's first hit in the region
            init_region(gw0, wb, tid, T, 0);
            first_hits(B1, seg == seg0, tid, T);
            __syncthreads();
            phase_tick(0);

            // 2. odd multiples of p^2: medium primes by lane-tasks, larger ones
            //    from the segment's hit slots (directly if the slots overflowed)
            // A prime with h = ceil(R / q) hits per region has c <= h tasks, so
            // c q <= R + q and f + v q < R + q: 32-bit positions suffice.
            // a task carries its start past the prime's first hit (v q, 21
            // bits), the prime's index (11 bits) and its step c q: one LDS read
            // of the prime's offset, no multiply
            auto mark_tasks = [&](const uint2* tk_table) {
                for (uint32_t e = tid; e < L.n_tasks; e += T) {
                    const uint2 tk = tk_table[e];
                    const uint32_t idx = tk.x >> 21, step = tk.y;
                    for (uint32_t pos = s_f[idx] + (tk.x & 0x1fffffu); pos < R; pos += step)
                        mark(bm32, pos);
                }
            };
            if (L.tasks_in_lds)
                mark_tasks(s_task);
            else
                mark_tasks(L.tasks);
            if (L.bucket_cnt) {
                if (nb <= cap) {
                    if (slot_pos < R)
                        mark(bm32, slot_pos);
                    const uint32_t* sl = L.bucket_slot + (uint64_t)gs * cap;
                    for (uint32_t e = tid + T; e < nb; e += T) {
                        const uint32_t pos = sl[e];
                        if (pos < R)
                            mark(bm32, pos);
                    }
                } else {
                    // slots overflowed: every prime above the medium range, directly
                    for (uint32_t pi = L.med_end + tid; pi < IV.pmax_end; pi += T) {
                        const uint64_t p = L.primes[pi];
                        const uint64_t q = p * p;
                        for (uint64_t pos = first_hit(B1, q); pos < R; pos += q)
                            mark(bm32, (uint32_t)pos);
                    }
                }
            }
            __syncthreads();
            phase_tick(1);

            if (MODE == 2) {
                // output word wo = seg * SW + lw covers odd indices I0 + 64 wo ...:
                // region bits out_shift + 64 lw ... (words lw and lw + 1)
                const uint32_t sh = IV.out_shift;
                const uint64_t n_bits = IV.I1 - IV.I0;
                const uint64_t wo0 = (uint64_t)seg * SW;
                auto store_pair = [&](uint32_t lw) {
                    const uint64_t w0 = bm[lw], w1 = bm[lw + 1], w2 = bm[lw + 2];
                    u64x2 o;
                    o.x = ~(sh ? ((w0 >> sh) | (w1 << (64 - sh))) : w0);
                    o.y = ~(sh ? ((w1 >> sh) | (w2 << (64 - sh))) : w1);
                    *(g_u64x2*)((g_u64*)IV.out_bits + wo0 + lw) = o;
                };
                if (wo0 * 64 + (uint64_t)SW * 64 <= n_bits && (((uintptr_t)IV.out_bits) & 15u) == 0) {
                    // a whole segment of output: two words per lane, 16-byte stores
                    for (uint32_t lw = 2 * tid; lw < SW; lw += 2 * T)
                        store_pair(lw);
                } else {
                    for (uint32_t lw = tid; lw < SW; lw += T) {
                        const uint64_t wo = wo0 + lw;
                        if (wo * 64 >= n_bits)
                            break;
                        const uint64_t lo = bm[lw], hi = bm[lw + 1];
                        const uint64_t v = sh ? ((lo >> sh) | (hi << (64 - sh))) : lo;
                        uint64_t out = ~v;
                        const uint64_t rem = n_bits - wo * 64;
                        if (rem < 64)
                            out &= (1ull << rem) - 1;
                        ((g_u64*)IV.out_bits)[wo] = out;
                    }
                }
                __syncthreads();
                phase_tick(2);
                continue;
            }

            // 3. Algorithm 2, bit-sliced: (uhi:ulo) holds the n of one word
            //    still without a representation; step k keeps the n whose
            //    n - 2^k (2^(k-1) bits lower) is marked.  cnt[k] counts them
            //    after step k; s_first[k+1] collects the least such n.
            const uint64_t As = (uint64_t)(IV.A0 + (int64_t)seg * (int64_t)S);
            // main words wholly inside [I0, I1)
            uint32_t lo_w = 0, hi_w = SW;
            if (IV.I0 > As)
                lo_w = (uint32_t)min((IV.I0 - As + 63) / 64, (uint64_t)SW);
            if (IV.I1 < As + S)
                hi_w = IV.I1 > As ? (uint32_t)((IV.I1 - As) / 64) : 0u;
            // A segment whose main words all lie inside [I0, I1) and split
            // evenly over the workgroup, searched to the deepest in-LDS level,
            // takes the fast form: every lane active, every n valid, no
            // per-word index arithmetic, no level bound.
            const bool fast = lo_w == 0 && hi_w == SW && SW % T == 0 && klds == (uint32_t)kMaxKh;
            // per-n mode, FAST segments: a wave's 64 words are 4096 consecutive
            // output bytes, staged through LDS; every run of the segment starts
            // the same delta bytes past a 16-byte boundary
            const bool stage_ok = MODE == 1 && L.stage && IV.out_mink;
            const uint32_t delta = rfl((uint32_t)(((uintptr_t)IV.out_mink + (uintptr_t)(As - IV.I0)) & 15u));
            const uint32_t iters = (SW + T - 1) / T;
            // STEADY: the least n of depth 2 .. 5 have been offered already, so
            // steps 1 .. 4 run without any branch.
            const bool no_tail = klds >= L.kmax_eff;
            auto push_tail = [&](uint64_t j, unsigned long long idx) {
                if (idx < L.tail_cap) {
                    L.tail_n[idx] = j;
                    L.tail_iv[idx] = ivi;
                } else {
                    g_or(&IV.acc->status, no_tail ? (unsigned)ESQ_STATUS_EXCEPTIONS_INCOMPLETE
                                                  : (unsigned)ESQ_STATUS_TAIL_OVERFLOW);
                }
            };
            const uint64_t* pbase = bm + HW + tid - 1;  // FAST: word before pass 0's word
            auto word_pass = [&](auto fast_c, auto steady_c, uint32_t itw) {
                constexpr bool FAST = decltype(fast_c)::value;
                constexpr bool STEADY = decltype(steady_c)::value;
                // the word's first n-index, for the rare paths only (formed from
                // an opaque copy of tid, so that no index arithmetic is hoisted
                // into the common path)
                auto j0_of = [&]() {
                    uint32_t t = tid;
                    asm volatile("" : "+v"(t));
                    return As + (uint64_t)(t + itw * T) * 64;
                };
                const uint32_t mw = tid + itw * T;
                const bool act = FAST || mw < SW;
                // pw points at the word before this lane's word (FAST: from the
                // loop-invariant base, one add per pass)
                const uint64_t* pw = FAST ? pbase + itw * T : bm + HW + (act ? mw : 0u) - 1;
                uint64_t V;
                if (FAST)
                    V = ~0ull;
                else if (!act)
                    V = 0;
                else if (mw >= lo_w && mw < hi_w)
                    V = ~0ull;
                else
                    V = valid_mask(As + (uint64_t)mw * 64, IV.I0, IV.I1);
                const uint64_t cur = pw[1], prv = pw[0];
                const uint32_t clo = (uint32_t)cur, chi = (uint32_t)(cur >> 32);
                const uint32_t plo = (uint32_t)prv, phi = (uint32_t)(prv >> 32);
                uint32_t ulo = (uint32_t)V, uhi = (uint32_t)(V >> 32);
                // per-n depths as bit planes: the step sets U_0 = V, U_1, U_2, ...
                // are nested, so the least k of an n, the number of sets that
                // hold it, has bit b equal to the parity of its membership in
                // the U_j with j = 2^b - 1 (mod 2^b)
                uint32_t pl[4][2] = {{(uint32_t)V, (uint32_t)(V >> 32)}, {0u, 0u}, {0u, 0u}, {0u, 0u}};
                found = rfl(found);
                bool alive = true;  // wave-uniform: some lane still has an n left
#pragma unroll
                for (int k = 1; k <= kMaxKh; k++) {
                    if (!FAST && k > (int)klds)
                        break;
                    // The region's bit 0 is one odd index below its first word
                    // boundary, so bit b of a word holds the odd index one below
                    // the word's n-bit b: n - 2^k, 2^(k-1) positions below n, is
                    // t = 2^(k-1) - 1 bits below in the bitmap.  k = 1 reads the
                    // word itself; k <= 7 funnel-shifts it with the word below
                    // by t; from k = 8 on the two words d = 2^(k-7) and d - 1
                    // below, shifted by 63.
                    uint32_t wlo, whi;
                    if (k == 1) {
                        wlo = clo;
                        whi = chi;
                    } else if (k <= 6) {
                        const uint32_t sh = 33u - (1u << (k - 1));
                        wlo = __builtin_amdgcn_alignbit(clo, phi, sh);
                        whi = __builtin_amdgcn_alignbit(chi, clo, sh);
                    } else if (k == 7) {
                        wlo = __builtin_amdgcn_alignbit(phi, plo, 1);
                        whi = __builtin_amdgcn_alignbit(clo, phi, 1);
                    } else {
                        const bool any = (ulo | uhi) != 0;
                        const uint64_t y = any ? pw[1 - (1 << (k - 7))] : 0ull;
                        const uint64_t x = any ? pw[2 - (1 << (k - 7))] : 0ull;
                        wlo = __builtin_amdgcn_alignbit((uint32_t)(y >> 32), (uint32_t)y, 1);
                        whi = __builtin_amdgcn_alignbit((uint32_t)x, (uint32_t)(y >> 32), 1);
                    }
                    ulo &= wlo;
                    uhi &= whi;
                    // levels below 4 are counted here; from level 4 on, where
                    // the empty-wave test runs first, after that test (a wave
                    // that stops there has nothing to count)
                    if (k < 4)
                        cnt[k] = bcnt_acc(uhi, bcnt_acc(ulo, cnt[k]));
                    if (MODE == 1) {
#pragma unroll
                        for (int b = 0; b < 4; b++) {
                            if ((k & ((1 << b) - 1)) == (1 << b) - 1) {
                                pl[b][0] ^= ulo;
                                pl[b][1] ^= uhi;
                            }
                        }
                    }
                    // a wave of 4096 n almost never empties before step 4, so
                    // the test for an empty wave starts there
                    const bool track = !(STEADY && k <= 4) && !(found & (1u << (k + 1)));
                    if (k >= 4 || track) {
                        const uint64_t bal = __ballot((ulo | uhi) != 0);
                        if (bal == 0) {
                            alive = false;
                            break;
                        }
                        if (k >= 4) {
                            if (k <= kRegLevels)
                                cnt[k] = bcnt_acc(uhi, bcnt_acc(ulo, cnt[k]));
                            else if (ulo | uhi)
                                atomicAdd(&s_cnt[k], (uint32_t)(__popc(ulo) + __popc(uhi)));
                        }
                        if (track) {
                            const uint32_t l = rfl((uint32_t)(__ffsll((unsigned long long)bal) - 1));
                            if (lane == l) {
                                const uint64_t U = ((uint64_t)uhi << 32) | ulo;
                                const uint64_t n_first = j0_of() +
                                                         (uint64_t)(__ffsll((unsigned long long)U) - 1);
                                atomicMin(&s_first[k + 1], (unsigned long long)n_first);
                            }
                            found |= 1u << (k + 1);
                        }
                    }
                }
                // the loop ends early (alive false) for all but the rarest words
                const uint64_t U = ((uint64_t)uhi << 32) | ulo;
                // still unresolved after the in-LDS steps: to the exact tail
                // pass -- unless the search limit is the in-LDS depth, so that
                // these n are exceptions already counted in cnt[k_lds]; then
                // they are listed only when the call lists exceptions
                if (__builtin_expect(alive, 0) && U && (!no_tail || L.exc_list)) {
                    // one reservation of popcount(U) entries per word, in the
                    // list's memory once the segment's is full
                    const uint64_t j0 = j0_of();
                    const uint32_t c = (uint32_t)__popcll(U);
                    uint32_t at = atomicAdd(&s_ntail[0], c);
                    const bool here = at + c <= kTailList;
                    unsigned long long idx = 0;
                    if (!here) {
                        atomicMin(&s_ntail[1], at);  // the segment's entries end here
                        idx = atomicAdd(L.tail_count, (unsigned long long)c);
                    }
                    for (uint64_t x = U; x; x &= x - 1, at++, idx++) {
                        const uint64_t j = j0 + (uint64_t)(__ffsll((unsigned long long)x) - 1);
                        if (here)
                            s_tail[at] = j;
                        else
                            push_tail(j, idx);
                    }
                }
                if (MODE == 1 && IV.out_mink) {
                    // n without a representation yet (the tail pass decides
                    // them) get 0
#pragma unroll
                    for (int b = 0; b < 4; b++) {
                        pl[b][0] &= ~ulo;
                        pl[b][1] &= ~uhi;
                    }
                    // planes -> one byte per n: nibble t of plane b spread to
                    // bit b of 4 bytes.  Plane 2 (least k in 4 .. 7) holds
                    // 1.4e-4 of the n, so a wave of 4096 n has none more often
                    // than not, and plane 3 (k >= 8) is almost never set: both
                    // are spread only when some lane of the wave has a bit
                    uint32_t D[16];
#pragma unroll
                    for (int t = 0; t < 16; t++) {
                        const int h = t >> 3, sh = 4 * (t & 7);
                        D[t] = (((pl[0][h] >> sh) & 15u) * 0x00204081u & 0x01010101u) |
                               (((pl[1][h] >> sh) & 15u) * 0x00408102u & 0x02020202u);
                    }
                    if (__ballot((pl[2][0] | pl[2][1]) != 0)) {
#pragma unroll
                        for (int t = 0; t < 16; t++)
                            D[t] |= spread4((pl[2][t >> 3] >> (4 * (t & 7))) & 15u) << 2;
                    }
                    if (__ballot((pl[3][0] | pl[3][1]) != 0)) {
#pragma unroll
                        for (int t = 0; t < 16; t++)
                            D[t] |= spread4((pl[3][t >> 3] >> (4 * (t & 7))) & 15u) << 3;
                    }
                    if (FAST && stage_ok) {
                        g_u8* o = (g_u8*)IV.out_mink + (As - IV.I0) + (uint64_t)(itw * T + (tid & ~63u)) * 64;
                        switch ((delta + 3) >> 2) {
                        case 0: stage_store_run<0>(s_stage, o, D, lane, delta); break;
                        case 1: stage_store_run<1>(s_stage, o, D, lane, delta); break;
                        case 2: stage_store_run<2>(s_stage, o, D, lane, delta); break;
                        case 3: stage_store_run<3>(s_stage, o, D, lane, delta); break;
                        default: stage_store_run<4>(s_stage, o, D, lane, delta); break;
                        }
                    } else if (V) {
                        const uint64_t j0 = As + (uint64_t)mw * 64;
                        store_depths((g_u8*)IV.out_mink + ((int64_t)j0 - (int64_t)IV.I0), D, V);
                    }
                }
            };
            constexpr uint32_t kSteadyBits = 0x3Cu;  // levels 2 .. 5
            uint32_t itw = 0;
            if (fast) {
                for (; itw < iters && (rfl(found) & kSteadyBits) != kSteadyBits; itw++)
                    word_pass(std::true_type{}, std::false_type{}, itw);
                for (; itw < iters; itw++)
                    word_pass(std::true_type{}, std::true_type{}, itw);
            } else {
                for (; itw < iters; itw++)
                    word_pass(std::false_type{}, std::false_type{}, itw);
            }
            __syncthreads();
            // the segment's listed n, with one reservation (a device-scope
            // operation each bounded a search that lists 2400 exceptions);
            // reset two barriers before the next search
            if (tid < 64) {
                const uint32_t m = rfl(min(s_ntail[0], s_ntail[1]));
                if (m) {
                    unsigned long long base = 0;
                    if (lane == 0) {
                        base = atomicAdd(L.tail_count, (unsigned long long)m);
                        s_ntail[0] = 0;
                        s_ntail[1] = kTailList;
                    }
                    base = __shfl(base, 0);
                    if (lane < m)
                        push_tail(s_tail[lane], base + lane);
                }
            }
            phase_tick(2);
        }

        // the item's s_item slots are reused by the next fetch
        __syncthreads();
    }
}

// Summary mode in the column layout (see esq_internal.h): regions of 2^kColLog2
// bits by workgroups of kColBlock threads, four of them on a CU.
//
// What bounds it: the issue of vector instructions and the waits between them.
// Per 64-n word the row layout's summary form issues 52 vector instructions
// (30 in the search, a third of them half-rate funnel shifts) and 31 scalar
// ones; here it is 39 and 18, of which the search has 23 (8 popcounts, 8
// ANDs).  The vector units are busy for about 0.7 of the time, the LDS for
// 0.5; the rest are barriers and latencies of eight waves a SIMD, which is
// why block size, region length and trip counts are constants and the rare
// paths (first segments, deep n) have loops of their own: with runtime trip
// counts and the offers in the common path the same method took 204 us.
// On the 2^33 odd n below 2^50: 221 us in the row layout, 160 to 167 us here
// (5.2e13 n/s); a third table for 17 and 19 took 184, regions of 2^19 211, of 2^17
// 203.
template <bool PH>
__global__ __launch_bounds__(kColBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_column(Launch Larg)
{
    constexpr int LR = kColLog2;
    constexpr uint32_t T = kColBlock;
    extern __shared__ uint64_t lds[];  // at LDS address 0
    constexpr uint32_t R = 1u << LR, W = R / 32, H = kColHalo, S = R - H;
    static_assert(H <= W && H % 256 == 0, "the halo lies in the lowest bit of the region's words");
    constexpr uint32_t kS1 = S % kWheelPeriod, kS2 = S % kWheel2Period;
    // The launch's and the interval's fields are read from memory (scalar
    // loads) where they are used, through pointers that the compiler takes to
    // change from segment to segment: kept in registers they do not fit, and
    // spilled scalars cost a vector instruction each.
    CLaunch* lp = launch_args();
    (void)Larg;

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = rfl(tid >> 6);
    // kColGuard words, then the region's W; the words below word 0 wrap (the
    // whole-segment search's reads of them are the guard's)
    uint32_t* bm = reinterpret_cast<uint32_t*>(lds) + kColGuard;
    constexpr uint32_t kRw = (W + kColGuard) / 2;
    constexpr uint32_t kCntAt = kMaxKh + 2, kItemAt = kCntAt + (kMaxKh + 2) / 2, kPhAt = kItemAt + 2;
    static_assert(kPhAt + 3 <= kVerifyCtrlWords, "control block");
    unsigned long long* s_first = reinterpret_cast<unsigned long long*>(lds + kRw);  // kMaxKh + 2
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(lds + kRw + kCntAt);               // kMaxKh + 1
    uint32_t* s_item = reinterpret_cast<uint32_t*>(lds + kRw + kItemAt);             // 4
    unsigned long long* s_ph = reinterpret_cast<unsigned long long*>(lds + kRw + kPhAt);
    uint2* s_medq = reinterpret_cast<uint2*>(lds + kRw + kVerifyCtrlWords);
    const uint32_t nmed = lp->med_end - kFirstMedium, n_multi = lp->n_multi;
    uint32_t* s_f = reinterpret_cast<uint32_t*>(s_medq + nmed);
    for (uint32_t i = tid; i < nmed; i += T)
        s_medq[i] = lp->medq[i];
    // a lane's first task is its own for the whole launch
    uint2 task = {0u, 0u};
    uint32_t task_min = 0;
    if (tid < lp->n_tasks) {
        task = lp->tasks[tid];
        task_min = lp->task_min[wave];
    }
    task_min = rfl(task_min);
    const uint32_t n_tasks = lp->n_tasks, cap = lp->bucket_cap;
    const uint32_t* const bcnt = lp->bucket_cnt;
    const uint32_t* const bslot = lp->bucket_slot;
    const uint32_t* const col = lp->col;

    constexpr int kRegLevels = 5;
    uint32_t cnt[kRegLevels + 1];
    uint32_t found = 0;       // levels whose least n this run has already offered
    uint32_t cur_iv = ~0u, acc_segs = 0;
    auto flush = [&](uint32_t iv) {
        asm volatile("" : "+s"(lp));
        Acc* acc = lp->items ? lp->iv[iv].acc : lp->iv0.acc + (blockIdx.x & (lp->n_acc - 1));
        const uint32_t klds = lp->k_lds;
#pragma unroll
        for (int k = 1; k <= kRegLevels; k++) {
            uint32_t v = cnt[k];
            for (int o = 32; o > 0; o >>= 1)
                v += __shfl_xor(v, o);
            if (lane == 0 && v)
                atomicAdd(&s_cnt[k], v);
        }
        __syncthreads();
        if (tid >= 1 && tid <= klds && s_cnt[tid])
            g_add(&acc->cnt[tid], (unsigned long long)s_cnt[tid]);
        if (tid >= 2 && tid <= klds + 1 && s_first[tid] != kNone)
            g_min(&acc->first[tid], s_first[tid]);
        __syncthreads();
    };
    uint64_t t_ph = 0;
    if (PH && tid < 3)
        s_ph[tid] = 0;
    auto phase_tick = [&](int ph) {
        if (PH) {
            const uint64_t t = __builtin_amdgcn_s_memrealtime();
            if (ph >= 0 && tid == 0)
                atomicAdd(&s_ph[ph], (unsigned long long)(t - t_ph));
            t_ph = t;
        }
    };
    // Work items.  The first is the workgroup's own number; the others come
    // from the queue, fetched before the last segment's search (thread 0).  A
    // thousand workgroups taking their first item from one counter waited up
    // to 14 us for it.
    uint32_t item = blockIdx.x;
    for (;;) {
        asm volatile("" : "+s"(lp));
        if (tid == 0) {
            uint32_t ok = 0, ivi = 0, b = 0, n = 0;
            const uint32_t it = item;
            if (it < lp->n_items) {
                ok = 1;
                if (lp->items) {
                    const uint4 x = lp->items[it];
                    ivi = x.x;
                    b = x.y;
                    n = x.z;
                } else {
                    run_of(it, lp->iv0.nseg, lp->n_items, lp->run_long, lp->run_short, gridDim.x, &b, &n);
                }
            }
            s_item[0] = ivi;
            s_item[1] = b;
            s_item[2] = n;
            s_item[3] = ok;
        }
        __syncthreads();
        const uint32_t item_ok = rfl(s_item[3]);
        const uint32_t ivi = rfl(s_item[0]), seg0 = rfl(s_item[1]), nsegs = rfl(s_item[2]);
        // partial totals go out as in k_verify
        if (cur_iv != ~0u && (!item_ok || ivi != cur_iv || acc_segs + nsegs > kFlushSegs)) {
            flush(cur_iv);
            cur_iv = ~0u;
        }
        if (!item_ok) {
            if (PH && tid < 3)
                atomicAdd(&lp->phase[tid], s_ph[tid]);
            break;
        }
        if (cur_iv == ~0u) {
            if (tid < kMaxKh + 2)
                s_first[tid] = kNone;
            if (tid <= kMaxKh)
                s_cnt[tid] = 0;
#pragma unroll
            for (int k = 0; k <= kRegLevels; k++)
                cnt[k] = 0;
            // Segment 0 holds the interval's least n of depths 2 .. 5, so runs
            // that start later need not look for theirs: the n whose first
            // four candidates are multiples of 9, 25, 49 and 121 in any order
            // recur within 169400 odd numbers (a period of 9 25 49 121).  Every
            // run's first segment took the slow form for these offers: 2^31
            // odd n 66 us with it, 56 without.
            static_assert(S >= 169400, "a whole segment holds an n of depth 5 or more");
            found = seg0 ? 0x3cu : 0u;
            acc_segs = 0;
            cur_iv = ivi;
            __syncthreads();
        }
        acc_segs += nsegs;
        CInterval* ivp = lp->items ? (CInterval*)(uintptr_t)(lp->iv + ivi) : &lp->iv0;
        // n-index of region position 0's slot: slot y is n-index nh + y, its
        // k-th candidate position y - (2^(k-1) - 1), position 0 odd index nh - 1
        int64_t nh = ivp->A0 + (int64_t)seg0 * (int64_t)S - (int64_t)H;
        const uint64_t I1 = ivp->I1;
        // the region's first word in each table, carried along
        uint32_t x1, x2;
        {
            auto fmod = [](int64_t x, int64_t m) {
                const int64_t r = x % m;
                return rfl((uint32_t)(r < 0 ? r + m : r));
            };
            x1 = fmod(nh - 1, kWheelPeriod);
            x2 = fmod(nh - 1, kWheel2Period);
        }
        // Hit slots.  Lane l holds the counts of the run's segments l, l + 64,
        // ... in turn: a scalar load of each segment's own count would be
        // waited for by the next LDS read.  This lane's first slot is fetched
        // a segment ahead, after the marks: vector loads complete in order,
        // and the next one that is waited for is then a whole search away.
        uint32_t gs = ivp->seg_base + seg0, n_seg = 0;  // n_seg: segments of the run done
        auto slot_counts = [&](uint32_t done) {
            return bcnt && done + lane < nsegs ? bcnt[gs + lane] : 0u;
        };
        auto slot_of = [&](uint32_t g, uint32_t n) {
            return tid < min(n, cap) ? bslot[(uint64_t)g * cap + tid] : R;
        };
        uint32_t counts = slot_counts(0);
        uint32_t nb = rfl(counts);
        uint32_t slot_pos = slot_of(gs, nb);
        for (uint32_t left = nsegs; left > 0; left--, nh += S) {
            asm volatile("" : "+s"(lp), "+s"(ivp));
            phase_tick(-1);
            // 1. the two tables, four words per lane and load
            {
                const char* src1 = reinterpret_cast<const char*>(col + x1);
                const char* src2 = reinterpret_cast<const char*>(col + (kWheelPeriod + W) + x2);
                char* dst = reinterpret_cast<char*>(bm);
                uint32_t off = 16 * tid;
                asm volatile("" : "+v"(off));
                constexpr int kQuads = W / (4 * T), kU = 2;  // kU quads in flight (VGPR budget)
                static_assert(W % (4 * T * kU) == 0, "whole rounds of quads");
#pragma unroll
                for (int r = 0; r < kQuads; r += kU) {
                    u32x4 v[kU], x[kU];
#pragma unroll
                    for (int u = 0; u < kU; u++) {
                        v[u] = *reinterpret_cast<const u32x4u*>(src1 + off + (r + u) * (16 * T));
                        x[u] = *reinterpret_cast<const u32x4u*>(src2 + off + (r + u) * (16 * T));
                    }
#pragma unroll
                    for (int u = 0; u < kU; u++)
                        *reinterpret_cast<u32x4*>(dst + off + (r + u) * (16 * T)) = v[u] | x[u];
                }
                x1 = x1 + kS1 >= kWheelPeriod ? x1 + kS1 - kWheelPeriod : x1 + kS1;
                x2 = x2 + kS2 >= kWheel2Period ? x2 + kS2 - kWheel2Period : x2 + kS2;
            }
            // the medium primes' first hits in a run's first segment (carried
            // from segment to segment after that, see below)
            if (left == nsegs) {
                for (uint32_t i = tid; i < nmed; i += T)
                    s_f[i] = (uint32_t)first_hit_b(nh - 1, s_medq[i].x, lp->qinv[kFirstMedium + i]);
            }
            __syncthreads();
            phase_tick(0);

            // 2. odd multiples of p^2.  A position is carried with its LR bits
            //    at the top of a word: stepping past the region is the add's
            //    carry, and the mark's bit is the top five.  The bit set below
            //    the position makes the step 2^32 - 1 (no shorter than the
            //    region) carry from position 0 too.
            if (nh < 1)  // odd indices below 0 are not positive
                for (uint32_t i = tid; i < (uint32_t)(1 - nh); i += T)
                    mark_col<LR>(i << (32 - LR));
            {
                // tasks: the marks that every task of the wave makes in a
                // loop without a test, the rest one by one
                auto run_task = [&](const uint2 tk, uint32_t n) {
                    const uint32_t pos = s_f[tk.x >> 21] + (tk.x & 0x1fffffu), step = tk.y;
                    uint32_t P = (pos << (32 - LR)) | 1u;
                    bool out = pos >= R;
                    if (n) {
#pragma unroll 4
                        for (uint32_t t = 1; t < n; t++) {
                            mark_col<LR>(P);
                            P += step;
                        }
                        mark_col<LR>(P);
                        P += step;
                        out = P < step;
                    }
                    while (!out) {
                        mark_col<LR>(P);
                        P += step;
                        out = P < step;
                    }
                };
                if (tid < n_tasks)
                    run_task(task, task_min);
                for (uint32_t e = tid + T; e < n_tasks; e += T)
                    run_task(lp->tasks[e], rfl(lp->task_min[e >> 6]));
                // the other medium primes, at most kColSingle marks each, by
                // the lanes in reverse, away from the longest tasks
                for (uint32_t i = n_multi + (T - 1 - tid); i < nmed; i += T) {
                    const uint2 qs = s_medq[i];
                    const uint32_t f = s_f[i];
                    s_f[i] = f >= qs.y ? f - qs.y : f + qs.x - qs.y;  // in the next segment
                    if (f < R) {
                        uint32_t P = (f << (32 - LR)) | 1u;
                        const uint32_t step = qs.x >= R ? ~0u : qs.x << (32 - LR);
                        do {
                            mark_col<LR>(P);
                            P += step;
                        } while (P >= step);
                    }
                }
            }
            if (nb <= cap) {
                if (slot_pos < R)
                    mark_col<LR>(slot_pos << (32 - LR));
                for (uint32_t e = tid + T; e < nb; e += T) {
                    const uint32_t pos = bslot[(uint64_t)gs * cap + e];
                    if (pos < R)
                        mark_col<LR>(pos << (32 - LR));
                }
            } else {
                // slots overflowed: every prime above the medium range, directly
                for (uint32_t pi = lp->med_end + tid; pi < ivp->pmax_end; pi += T) {
                    const uint64_t p = lp->primes[pi];
                    const uint64_t q = p * p;
                    for (uint64_t pos = first_hit(nh - 1, q); pos < R; pos += q)
                        mark_col<LR>((uint32_t)pos << (32 - LR));
                }
            }
            __syncthreads();
            phase_tick(1);
            gs++;
            n_seg++;
            if ((n_seg & 63u) == 0)
                counts = slot_counts(n_seg);
            nb = n_seg < nsegs ? (uint32_t)__builtin_amdgcn_readlane((int)counts, (int)(n_seg & 63u)) : 0u;
            slot_pos = slot_of(gs, nb);
            // the next first hits of the primes with tasks, by a wave that has
            // less to do in the search than others
            if (wave == 1)
                for (uint32_t i = lane; i < n_multi; i += 64) {
                    const uint2 qs = s_medq[i];
                    const uint32_t f = s_f[i];
                    s_f[i] = f >= qs.y ? f - qs.y : f + qs.x - qs.y;
                }
            if (left == 1 && tid == 0)
                item = lp->n_items > gridDim.x ? gridDim.x + atomicAdd(lp->queue, 1u) : ~0u;

            // 3. Algorithm 2.  The n of the segment are the slots [H, yhi).
            const uint32_t yhi = (uint32_t)min((uint64_t)R, I1 - (uint64_t)nh);
            found = rfl(found);
            // least n of depth 2, 3, 4: the slots in order, one wave per level;
            // a level found in an earlier segment of the run has its least n there
            if ((found & 0x1cu) != 0x1cu) {
                for (uint32_t k = 1; k <= 3; k++) {
                    if ((found & (2u << k)) || k - 1 != wave)
                        continue;
                    constexpr int kAhead = 4;  // words of 64 slots in flight
                    for (uint32_t y0 = H; y0 < yhi; y0 += 64 * kAhead) {
                        auto bit = [&](uint32_t p) { return bm[p & (W - 1)] >> ((p >> (LR - 5)) & 31u); };
                        uint32_t u[kAhead];
#pragma unroll
                        for (int j = 0; j < kAhead; j++) {
                            const uint32_t y = y0 + 64 * j + lane;
                            u[j] = y < yhi ? bit(y) : 0u;
                            if (k > 1)
                                u[j] &= bit(y - 1);
                            if (k > 2)
                                u[j] &= bit(y - 3);
                        }
                        uint32_t at = ~0u;
#pragma unroll
                        for (int j = kAhead - 1; j >= 0; j--) {
                            const uint64_t bal = __ballot((u[j] & 1u) != 0);
                            if (bal)
                                at = y0 + 64 * j + (uint32_t)(__ffsll((unsigned long long)bal) - 1);
                        }
                        if (at != ~0u) {
                            if (lane == 0)
                                atomicMin(&s_first[k + 1], (unsigned long long)nh + at);
                            break;
                        }
                    }
                }
            }
            // word i of the region for any i > -W: below 0, word W + i one bit up
            auto word_at = [&](int32_t i) { return bm[(uint32_t)i & (W - 1)] << (i < 0 ? 1 : 0); };
            auto n_of = [&](uint32_t i, uint32_t u) {  // n-index of the least slot in u of word i
                return (unsigned long long)nh + (((uint32_t)__ffs((int)u) - 1u) << (LR - 5)) + i;
            };
            // offer the least n in the four words from i0 as least n of depth d;
            // few lanes have any, so each does its own LDS operation (the
            // address is kept from looking uniform, which would make it a
            // reduction over the wave first)
            auto offer = [&](uint32_t d, uint32_t i0, const uint32_t (&u)[4]) {
                unsigned long long at = kNone;
#pragma unroll
                for (uint32_t c = 0; c < 4; c++)
                    if (u[c])
                        at = min(at, n_of(i0 + c, u[c]));
                asm volatile("" : "+v"(d));
                if (at != kNone)
                    atomicMin(&s_first[d], at);
            };
            // Four words per lane.  KIND 0: every slot of the wave's 256 words
            // is an n of the segment; 1: all but those in bit 0 (words below 0
            // from the guard); 2: the general form, which also wraps below
            // word 0 and offers level 5.
            auto quad_pass = [&](auto kind_c, uint32_t i0) {
                constexpr int KIND = decltype(kind_c)::value;
                auto quad = [&](int32_t i) {
                    if (KIND == 2)
                        return *reinterpret_cast<const u32x4*>(bm + ((uint32_t)i & (W - 1))) << (i < 0 ? 1u : 0u);
                    return *reinterpret_cast<const u32x4*>(bm + i);
                };
                const u32x4 wc = quad((int32_t)i0), wb = quad((int32_t)i0 - 4), wa = quad((int32_t)i0 - 8);
                // words i0 - 15 .. i0 - 12 (one unaligned read of them costs
                // four times the LDS cycles)
                const u32x4 za = quad((int32_t)i0 - 16), zb = quad((int32_t)i0 - 12);
                const uint32_t wz[4] = {za[1], za[2], za[3], zb[0]};
                const uint32_t w[12] = {wa[0], wa[1], wa[2], wa[3], wb[0], wb[1], wb[2], wb[3],
                                        wc[0], wc[1], wc[2], wc[3]};
                uint32_t u[4];
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    uint32_t U = w[8 + c];
                    if (KIND == 1)
                        U &= ~1u;
                    if (KIND == 2) {
                        // bits j with H <= j W + i < yhi
                        const uint32_t i = i0 + (uint32_t)c;
                        const uint32_t jh = (yhi + W - 1 - i) >> (LR - 5);
                        U &= (jh >= 32 ? ~0u : (1u << jh) - 1u) & (i < H ? ~1u : ~0u);
                    }
                    cnt[1] = bcnt_acc(U, cnt[1]);
                    U &= w[7 + c];
                    cnt[2] = bcnt_acc(U, cnt[2]);
                    U &= w[5 + c];
                    cnt[3] = bcnt_acc(U, cnt[3]);
                    U &= w[1 + c];
                    cnt[4] = bcnt_acc(U, cnt[4]);
                    u[c] = U;
                }
                if (KIND == 2 && !(found & (1u << 5)))
                    offer(5, i0, u);
#pragma unroll
                for (int c = 0; c < 4; c++)
                    u[c] &= wz[c];
                // of 8192 n 1.2 are left after step 4 and 0.08 after step 5:
                // the first test for an empty wave pays here (at step 4 it
                // saves three tenths of the waves six instructions)
                if (__builtin_expect(__ballot((u[0] | u[1] | u[2] | u[3]) != 0) == 0, 1))
                    return;
#pragma unroll
                for (int c = 0; c < 4; c++)
                    cnt[5] = bcnt_acc(u[c], cnt[5]);
                if (!(found & (1u << 6)))
                    offer(6, i0, u);
                const uint32_t klds = lp->k_lds;
                uint32_t k = 5;
                if (klds > 5) {
                    // step 6, which leaves next to none, for the four words at once
                    const u32x4 ya = quad((int32_t)i0 - 32), yb = quad((int32_t)i0 - 28);
                    u[0] &= ya[1];
                    u[1] &= ya[2];
                    u[2] &= ya[3];
                    u[3] &= yb[0];
                    k = 6;
                    if (__ballot((u[0] | u[1] | u[2] | u[3]) != 0) == 0)
                        return;
                    const uint32_t c6 = (uint32_t)(__popc(u[0]) + __popc(u[1]) + __popc(u[2]) + __popc(u[3]));
                    if (c6)
                        atomicAdd(&s_cnt[6], c6);
                    offer(7, i0, u);
                }
#pragma nounroll
                for (uint32_t c = 0; c < 4; c++) {
                    uint32_t U = c == 0 ? u[0] : c == 1 ? u[1] : c == 2 ? u[2] : u[3];
                    for (uint32_t kk = k; U && kk < klds;) {
                        kk++;
                        U &= word_at((int32_t)(i0 + c) - (int32_t)((1u << (kk - 1)) - 1u));
                        if (U) {
                            // U: the slots of depth > kk
                            atomicAdd(&s_cnt[kk], (uint32_t)__popc(U));
                            atomicMin(&s_first[kk + 1], n_of(i0 + c, U));
                        }
                    }
                    // still unresolved: to the tail pass or the exceptions, as in k_verify
                    if (__builtin_expect(U != 0, 0) && (klds < lp->kmax_eff || lp->exc_list)) {
                        const unsigned long long cu = (unsigned long long)__popc(U);
                        unsigned long long idx = atomicAdd(lp->tail_count, cu);
                        for (uint32_t x = U; x; x &= x - 1, idx++) {
                            if (idx < lp->tail_cap) {
                                lp->tail_n[idx] = n_of(i0 + c, x);
                                lp->tail_iv[idx] = ivi;
                            } else {
                                g_or(&ivp->acc->status, klds >= lp->kmax_eff
                                                            ? (unsigned)ESQ_STATUS_EXCEPTIONS_INCOMPLETE
                                                            : (unsigned)ESQ_STATUS_TAIL_OVERFLOW);
                            }
                        }
                    }
                }
            };
            constexpr uint32_t kStep = 4 * T;  // words per round of quads
            // opaque, so that no addresses are kept from segment to segment
            uint32_t t4 = 4 * tid;
            asm volatile("" : "+v"(t4));
            if (yhi == R && (found & (1u << 5))) {
                // a whole segment, the levels up to 5 offered
                if (wave == 0 && lane < kColGuard)  // only this wave reads the guard
                    bm[(int32_t)lane - (int32_t)kColGuard] = bm[W - kColGuard + lane] << 1;
#pragma unroll
                for (uint32_t a = 0; a < W; a += kStep) {
                    const uint32_t i0 = a + t4;
                    if (a < H)
                        quad_pass(std::integral_constant<int, 1>{}, i0);
                    else
                        quad_pass(std::integral_constant<int, 0>{}, i0);
                }
                static_assert(H % kStep == 0 || H == W, "a round's words lie on one side of H");
            } else {
#pragma nounroll
                for (uint32_t i0 = t4; i0 < W; i0 += kStep)
                    quad_pass(std::integral_constant<int, 2>{}, i0);
            }
            __syncthreads();
            // the levels found by now need no offers in later segments
            if ((found & 0x7cu) != 0x7cu) {
                uint32_t fnd = found;
#pragma unroll
                for (int k = 2; k <= 6; k++)
                    fnd |= s_first[k] != kNone ? 1u << k : 0u;
                found = rfl(fnd);
            }
            phase_tick(2);
        }
        // the item's s_item slots are reused by the next fetch
        __syncthreads();
    }
}


size_t verify_lds_bytes(const Launch& L, uint32_t block)
{
    return verify_lds_size(L.rw + (L.mode == 3 ? kColGuard / 2 : 0u), L.med_end - kFirstMedium, L.tasks_in_lds ? L.n_tasks : 0u, L.stage != 0,
                           block);
}

// The instance of a mode; the phase-clock ones only when the clock is on.
using VerifyKernel = void (*)(Launch);
static VerifyKernel verify_kernel(int mode, bool phase)
{
    switch (mode) {
    case 0:
        return phase ? k_verify<0, true> : k_verify<0, false>;
    case 1:
        return phase ? k_verify<1, true> : k_verify<1, false>;
    case 2:
        return phase ? k_verify<2, true> : k_verify<2, false>;
    default:
        return phase ? k_column<true> : k_column<false>;
    }
}

hipError_t launch_verify(const Launch& L, uint32_t grid, uint32_t block, hipStream_t s)
{
    const size_t lds = verify_lds_bytes(L, block);
    if (grid == 0 || L.n_items == 0)
        return hipSuccess;
    hipLaunchKernelGGL(verify_kernel((int)L.mode, L.phase != nullptr), dim3(grid), dim3(block), lds, s, L);
    return hipGetLastError();
}

int verify_occupancy(int mode, uint32_t block, size_t lds_bytes)
{
    int occ = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &occ, reinterpret_cast<const void*>(verify_kernel(mode, false)), (int)block, lds_bytes);
    return e == hipSuccess && occ > 0 ? occ : 1;
}

// --------------------------------------------------------------- tail

// Exact search, by trial division over the resident prime squares, for an n
// (odd index j) whose first k_lds candidates were all marked (Algorithm 2
// continued), by the whole workgroup: its least k, 0 if none.
__device__ __forceinline__ uint32_t tail_search(const Launch& L, uint64_t j, int* s_hit)
{
    const uint64_t n = 2 * j + 1;
    volatile int* hitp = s_hit;
    for (uint32_t k = L.k_lds + 1; k <= 63 && k <= L.kmax_eff; k++) {
        const uint64_t pk = 1ull << k;
        if (pk >= n)
            break;
        const uint64_t m = n - pk;
        if (threadIdx.x == 0)
            *hitp = 0;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < L.nprimes; i += blockDim.x) {
            const uint64_t pr = L.primes[i];
            const uint64_t q = pr * pr;
            if (q > m || *hitp)
                break;
            if (m % q == 0) {
                *hitp = 1;
                break;
            }
        }
        __syncthreads();
        const int hit = *hitp;
        __syncthreads();
        if (!hit)
            return k;
    }
    return 0;
}

// The tail pass as a kernel of its own, where many n are expected to need it
// (see tail_in_finalize).
__global__ __launch_bounds__(256) void k_tail(Launch L)
{
    __shared__ int s_hit;
    const unsigned long long total = *L.tail_count;
    const uint64_t count = total < L.tail_cap ? total : L.tail_cap;
    for (uint64_t idx = blockIdx.x; idx < count; idx += gridDim.x) {
        const uint64_t j = L.tail_n[idx];
        const uint32_t d = tail_search(L, j, &s_hit);
        if (threadIdx.x == 0) {
            const Interval IV = L.iv[L.tail_iv[idx]];
            L.tail_d[idx] = (uint8_t)d;
            g_add(&IV.acc->deep_hist[d], 1ull);
            const uint32_t top = d ? d : 64u;
            for (uint32_t kk = L.k_lds + 2; kk <= top; kk++)
                g_min(&IV.acc->first[kk], (unsigned long long)j);
            if (IV.out_mink)
                ((g_u8*)IV.out_mink)[j - IV.I0] = (uint8_t)d;
        }
    }
}

// Whether k_finalize takes the tail pass along.  With the search limit at the
// in-LDS depth there is none (what is listed are exceptions); at 12 in-LDS
// steps and more, an n is left with probability 9e-16, so the launch of an
// empty k_tail (4 us, a fifth of a short call's kernels) is saved.
static bool tail_in_finalize(const Launch& L) { return L.k_lds >= L.kmax_eff || L.k_lds >= 12; }

hipError_t launch_tail(const Launch& L, hipStream_t s)
{
    if (tail_in_finalize(L))
        return hipSuccess;
    hipLaunchKernelGGL(k_tail, dim3(512), dim3(256), 0, s, L);
    return hipGetLastError();
}

// ------------------------------------------------------------ finalize

__device__ unsigned long long block_sum(unsigned long long v, unsigned long long* s_acc)
{
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    if (threadIdx.x == 0)
        *s_acc = 0;
    __syncthreads();
    if ((threadIdx.x & 63u) == 0)
        atomicAdd(s_acc, v);
    __syncthreads();
    const unsigned long long r = *s_acc;
    __syncthreads();
    return r;
}

// Sort the `got` distinct numbers in s_sort, by a workgroup of kSortThreads: each
// goes to the bucket of its leading bits (s_bkt: kSortBuckets + 1 words) and
// takes its rank among the bucket's, at most eight on average: exceptions lie
// about evenly over their range, being set by residues (crowded ones would
// take longer, a pass over the bucket each).  What bounds it is the latency of
// its steps: k_finalize with 2400 exceptions takes 10.5 us, with a bitonic sort
// (78 steps for 4096 entries) 31.
constexpr uint32_t kSortThreads = 1024, kSortBuckets = 4 * kSortThreads;
constexpr size_t kFinalizeLds = (size_t)kFinalizeSortCap * 8 + (kSortBuckets + 2) * 4;
__device__ __forceinline__ void bucket_sort(unsigned long long* s_sort, uint32_t* s_bkt, uint32_t got)
{
    constexpr int kEach = (int)(kFinalizeSortCap / kSortThreads);
    __shared__ unsigned long long s_lo, s_hi;
    __shared__ uint32_t s_wave[kSortThreads / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    if (tid == 0) {
        s_lo = kNone;
        s_hi = 0;
    }
    for (uint32_t i = tid; i < kSortBuckets; i += kSortThreads)
        s_bkt[i] = 0;
    unsigned long long x[kEach], lo = kNone, hi = 0;
#pragma unroll
    for (int u = 0; u < kEach; u++) {
        const uint32_t i = tid + u * kSortThreads;
        x[u] = kNone;
        if (i < got) {
            x[u] = s_sort[i];
            lo = min(lo, x[u]);
            hi = max(hi, x[u]);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (unsigned long long)__shfl_xor(lo, o));
        hi = max(hi, (unsigned long long)__shfl_xor(hi, o));
    }
    __syncthreads();
    if (lane == 0) {
        atomicMin(&s_lo, lo);
        atomicMax(&s_hi, hi);
    }
    __syncthreads();
    lo = s_lo;
    const int bits = 64 - __clzll((long long)(s_hi - lo));
    const int shift = bits > 12 ? bits - 12 : 0;
    static_assert(kSortBuckets == 1u << 12, "the leading bits");
    uint32_t at[kEach];  // place in the bucket, later in s_sort
#pragma unroll
    for (int u = 0; u < kEach; u++)
        if (tid + u * kSortThreads < got)
            at[u] = atomicAdd(&s_bkt[(uint32_t)((x[u] - lo) >> shift)], 1u);
    __syncthreads();
    // the buckets' starts: four buckets a thread
    uint32_t n[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        n[j] = s_bkt[4 * tid + j];
        sum += n[j];
    }
    uint32_t up = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(up, o);
        up += lane >= (uint32_t)o ? v : 0u;
    }
    if (lane == 63)
        s_wave[wave] = up;
    __syncthreads();
    uint32_t start = up - sum;
    for (uint32_t w = 0; w < wave; w++)
        start += s_wave[w];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        s_bkt[4 * tid + j] = start;
        start += n[j];
    }
    if (tid == kSortThreads - 1)
        s_bkt[kSortBuckets] = start;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEach; u++)
        if (tid + u * kSortThreads < got)
            s_sort[s_bkt[(uint32_t)((x[u] - lo) >> shift)] + at[u]] = x[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEach; u++)
        if (tid + u * kSortThreads < got) {
            const uint32_t b = (uint32_t)((x[u] - lo) >> shift), end = s_bkt[b + 1];
            at[u] = s_bkt[b];
            for (uint32_t i = s_bkt[b]; i < end; i++)
                at[u] += s_sort[i] < x[u] ? 1u : 0u;
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEach; u++)
        if (tid + u * kSortThreads < got)
            s_sort[at[u]] = x[u];
    __syncthreads();
}

// One workgroup per interval; the aggregates by its first wave, a level per
// lane (one thread taking the 65 levels in turn took 4 of the kernel's 6 us).
__global__ __launch_bounds__(1024) void k_finalize(Launch L, const Acc* accs, void* out_summaries, void* out_records,
                                                   uint64_t* out_exceptions, uint64_t exc_cap, int tail)
{
    extern __shared__ unsigned long long s_sort[];
    __shared__ unsigned long long s_acc;
    __shared__ unsigned int s_fill;
    __shared__ int s_hit;
    __shared__ unsigned long long s_first[66], s_h[65], s_cnt[16];
    const uint32_t ivi = blockIdx.x;
    CInterval* IV = interval_at(L.iv, L.n_iv, ivi);
    const Acc* A = accs + ivi;
    const uint32_t tid = threadIdx.x, T = blockDim.x;
    const unsigned long long tail_total = *L.tail_count;
    const uint64_t nlist = tail_total < L.tail_cap ? tail_total : L.tail_cap;
    const uint64_t I0 = IV->I0, n_odd = IV->I1 - I0;
    const uint32_t status = A->status;
    // with the search limit at the in-LDS depth there is no tail pass: the n
    // still unresolved after step k_lds are the exceptions, and they are
    // deeper than every level, so first[k] for k > k_lds + 1 is first[k_lds + 1]
    const bool no_tail = L.k_lds >= L.kmax_eff;
    // one interval's copies: a thread per copy and level (256 of them)
    static_assert(kAccCopies * 16 <= 256 && kMaxKh + 1 < 16, "the copies' levels");
    const uint32_t copy = tid >> 4, lev = tid & 15u;
    const bool merge = L.n_iv == 1 && copy > 0 && copy < L.n_acc;
    const unsigned long long c_cnt = merge ? A[copy].cnt[lev] : 0ull;
    const unsigned long long c_first = merge ? A[copy].first[lev] : kNone;
    for (uint32_t i = tid; i < 65; i += T) {
        s_first[i] = A->first[i];
        s_h[i] = no_tail ? 0ull : A->deep_hist[i];
        if (i < 16)
            s_cnt[i] = A->cnt[i];
    }
    __syncthreads();
    if (c_cnt)
        atomicAdd(&s_cnt[lev], c_cnt);
    if (c_first != kNone)
        atomicMin(&s_first[lev], c_first);
    __syncthreads();
    if (no_tail) {
        for (uint32_t i = tid; i < 65; i += T)
            if (i > L.k_lds + 1)
                s_first[i] = s_first[L.k_lds + 1];
        __syncthreads();
    }
    if (tail && !no_tail)
        for (uint64_t idx = 0; idx < nlist; idx++) {
            if (L.tail_iv[idx] != ivi)
                continue;
            const uint64_t j = L.tail_n[idx];
            const uint32_t d = tail_search(L, j, &s_hit);
            if (tid == 0) {
                L.tail_d[idx] = (uint8_t)d;
                s_h[d]++;
                for (uint32_t kk = L.k_lds + 2; kk <= (d ? d : 64u); kk++)
                    s_first[kk] = min(s_first[kk], (unsigned long long)j);
                if (IV->out_mink)
                    ((g_u8*)IV->out_mink)[j - I0] = (uint8_t)d;
            }
            __threadfence_block();
            __syncthreads();
        }
    const uint64_t n_exc = no_tail ? s_cnt[L.k_lds] : s_h[0];
    const uint64_t want = n_exc < exc_cap ? n_exc : exc_cap;
    auto listed = [&](uint64_t i) { return L.tail_iv[i] == ivi && (no_tail || L.tail_d[i] == 0); };

    if (out_exceptions && want > 0) {
        // the want-th smallest exception of this interval (binary search on
        // its odd index), then an LDS sort of those up to it
        uint64_t thr = kNone;
        if (want < n_exc) {
            uint64_t lo = I0, hi = I0 + n_odd;
            while (lo < hi) {
                const uint64_t mid = lo + (hi - lo) / 2;
                unsigned long long c = 0;
                for (uint64_t i = tid; i < nlist; i += T)
                    c += (listed(i) && L.tail_n[i] <= mid) ? 1ull : 0ull;
                c = block_sum(c, &s_acc);
                if (c >= want)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            thr = lo;
        }
        if (tid == 0)
            s_fill = 0;
        __syncthreads();
        for (uint64_t i0 = tid; i0 < nlist; i0 += 4 * T) {
            unsigned long long x[4];
            bool take[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const uint64_t i = min(i0 + u * T, nlist - 1);
                x[u] = L.tail_n[i];
                take[u] = listed(i) && i0 + u * T < nlist;
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (take[u] && x[u] <= thr) {
                    const unsigned int slot = atomicAdd(&s_fill, 1u);
                    if (slot < kFinalizeSortCap)
                        s_sort[slot] = x[u];
                }
        }
        __syncthreads();
        const uint32_t got = min(s_fill, kFinalizeSortCap);
        bucket_sort(s_sort, (uint32_t*)(s_sort + kFinalizeSortCap), got);
        for (uint32_t i = tid; i < want && i < got; i += T)
            out_exceptions[i] = 2 * s_sort[i] + 1;
    }
    if (tid >= 64)
        return;
    // lane l: level k = l + 1.  The LDS steps' counts give the levels up to
    // k_lds, the tail pass the deeper ones.
    const uint32_t k = tid + 1;
    unsigned long long h;
    if (k <= L.k_lds)
        h = (k == 1 ? n_odd : s_cnt[k - 1]) - s_cnt[k];
    else
        h = s_h[k];
    unsigned long long ksum = (unsigned long long)k * h;
    for (int o = 32; o > 0; o >>= 1)
        ksum += __shfl_xor(ksum, o);
    const uint64_t seen = __ballot(h != 0);
    // record-setters: first[k] = least n-index with depth >= k; each distinct
    // value is a record, labelled with the deepest level sharing it
    const unsigned long long v = k == 1 ? I0 : s_first[k];
    const bool last = k == 64 || s_first[k + 1] != v;
    const bool is_rec = n_odd && v != kNone && last;
    const uint64_t recs = __ballot(is_rec);
    const uint32_t nrec = (uint32_t)__popcll(recs);
    if (out_records && is_rec) {
        esq_record* rec = reinterpret_cast<esq_record*>(out_records) + (uint64_t)ivi * ESQ_RECORDS_CAP +
                          __popcll(recs & ((1ull << tid) - 1));
        const uint64_t n = 2 * v + 1;
        rec->n = n;
        rec->k = k == 64 ? 0u : k;
        // an exception found by the search limit, with a larger k still
        // positive, vs one for which every k with 2^k < n failed
        rec->flags = (k == 64 && L.kmax_eff < 63 && (1ull << (L.kmax_eff + 1)) < n) ? (uint32_t)ESQ_RECORD_KMAX_LIMIT
                                                                                   : 0u;
    }
    esq_summary* out = reinterpret_cast<esq_summary*>(out_summaries) + ivi;
    out->hist[k] = h;
    if (tid == 0) {
        out->n0 = n_odd ? 2 * I0 + 1 : 0;
        out->n_odd = n_odd;
        out->hist[0] = n_exc;
        out->ksum = ksum;
        out->kmax_seen = seen ? 64u - (uint32_t)__clzll((long long)seen) : 0u;
        out->n_records = nrec;
        out->n_exceptions = n_exc;
        out->status = status;
        out->reserved = 0;
    }
}

hipError_t launch_finalize(const Launch& L, const Acc* accs, void* out_summaries, void* out_records,
                           uint64_t* out_exceptions, uint64_t exc_cap, hipStream_t s)
{
    if (L.n_iv == 0)
        return hipSuccess;
    const size_t lds = out_exceptions ? kFinalizeLds : 0;
    hipLaunchKernelGGL(k_finalize, dim3(L.n_iv), dim3(out_exceptions ? kSortThreads : 256), lds, s, L, accs,
                       out_summaries, out_records, out_exceptions, exc_cap, tail_in_finalize(L) ? 1 : 0);
    return hipGetLastError();
}

hipError_t configure_kernels()
{
    hipError_t e;
    const int lds_max = (int)kVerifyLdsMax;
    for (int mode = 0; mode < 4; mode++)
        for (int phase = 0; phase < 2; phase++) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(verify_kernel(mode, phase != 0)),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
            if (e != hipSuccess) return e;
        }
    e = hipFuncSetAttribute((const void*)k_finalize, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kFinalizeLds);
    return e;
}

}  // namespace esq
