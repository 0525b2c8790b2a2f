// Layer-wise percentile threshold and pruning mask (Section 3.2, paragraph before Eq. (2), and
// Eq. (2)).
//
// tau is the order statistic of rank floor(p * N) among the N participating entries of the mean
// maps of all heads of a layer.  It is found exactly, with one sweep over the maps in which the
// mask is written too:
//
//   sample   clusters of 16 entries, every stride-th of the map (two million entries, more for large maps; all of
//            them if the map is small), are counted into a histogram of their leading 12 key bits, then
//            the bins around the wanted rank once more into 1024 sub-bins.  That gives a narrow value
//            interval [lo, hi] that is meant to hold tau: the sample's own rank, five standard
//            deviations of a clustered sample to either side (typically 0.2 to 0.6 % of the map).
//   sweep    every entry above the interval is kept, every entry below it pruned; the entries
//            inside it (the candidates) are copied out, and the entries above it counted.
//   select   the count says whether the interval holds the wanted rank.  If so, tau is found among
//            the candidates by two histograms over their key bits, and their mask bytes are written.
//
// If the sample says that the candidates will not fit the workspace (ties, values close together), the sweep only
// counts, in 16384 bins of the interval, and the bin that holds the rank becomes the interval: it is a
// single key (ties: tau is known), or its entries fit and are collected by a sweep in the place of the first
// selection level, or two levels of 65536 bins go on from there, as they do from the whole range of keys if the interval
// misses the rank.  A last sweep then writes what is left of the mask.  For maps so large that only a sample of an
// eighth of them or more would do, such a counting sweep comes first.  Which path runs is decided on the device (the
// launches of the others return at once), so the call never synchronises with the host; the result is the
// same element of the map either way.
//
// What bounds it: reading the map and writing the mask once (805 MB for 16 x 4096 x 4096 causal maps).
// A full first sweep for an exact histogram costs a read of the map more and, worse, one LDS atomic per
// entry on a few hot bins.  Measured there: 451 us with the histogram sweep (126 us), one-workgroup
// selections (26 + 52 us) and a mask sweep of 214 us; now 260 us, of which the sweep is 162 (5.0 TB/s),
// the sample 35 and the candidates 31.  At 12 x 512 x 512 (launches
// only) 63 -> 50 us; rows that start anywhere (Lk = 4095) 644 -> 252 us.
// Other maps, with the two radix sweeps of 15 bits before: 16 x 4096 x 4096 causal, all equal 1640 -> 437 us, 60 %
// zeros 1116 -> 451 to 460 us (440 where the rank lies next to their mass, 524 before), normal within 1 % 636 -> 428 us;
// 16 x 16384 x 16384 causal 6.0 -> 4.1 ms, 60 % zeros 15.6 -> 4.7 ms; 12 x 512 x 512, all equal 91 -> 88 us.
//
// Float bit patterns are mapped to unsigned keys whose integer order is the numeric order
// (sign bit flipped for non-negative values, all bits flipped for negative ones; -0 counts as +0).
#include <hip/hip_runtime.h>
#include <algorithm>
#include <stdint.h>

#include "ap_internal.h"

namespace ap {

namespace {

constexpr int kCoarse = 4096;                // first look at the sample: leading 12 key bits
constexpr int kCoarseShift = 20;
constexpr int kSubBits = 10, kSub = 1 << kSubBits;   // second look: sub-bins of the bins around the rank
constexpr int kCandBits = 10, kCandBins = 1 << kCandBits;   // first histogram over the candidates
constexpr int kLastBits = 13, kLastBins = 1 << kLastBits;   // second one
constexpr int kNarrowBits = 14, kNarrowBins = 1 << kNarrowBits;   // a narrowing sweep
constexpr int kMaxBracketBits = kCandBits + kLastBits;   // widest interval the selection resolves
constexpr int kExactBins = 65536;            // a level of the exact way: 16 key bits
constexpr uint32_t kCap = 978240;            // candidates the workspace can hold
constexpr double kAim = 650000.0;            // candidates aimed at where the map is large
constexpr unsigned long long kSample = 1ull << 21;   // entries looked at, at least (all, if there are fewer)
constexpr double kRefineShare = 8.0;         // a sample larger than this part of the map gives way to an exact pass
constexpr double kDesign = 6.0;              // variance of the clustered sample over an independent one's
constexpr double kSigmas = 5.0;              // half width of the interval in standard deviations of the sample
constexpr int kThreads = 1024;
constexpr int kSweepThreads = 512;

// way: the sweep collects candidates (0: the state is cleared before use); it narrows the interval instead; what it
// left is collected in place of the first level of the selection; it is narrowed further, as [in_lo, in_hi]; tau is
// known.
enum { COLLECT = 0, NARROW = 1, LATE = 2, EXACT = 3, KNOWN = 4 };

struct SelectState {
    unsigned long long rank;                 // wanted rank among the participating entries
    unsigned long long n;                    // number of participating entries
    unsigned long long above;                // sweep: entries above the interval
    unsigned long long ncand;                // sweep: entries inside it (the candidates)
    unsigned long long in_rank;              // exact way: wanted rank among the entries of [in_lo, in_hi]
    uint32_t s_lo, s_hi;                     // ranks of the sample that the interval runs between
    uint32_t s_total;
    uint32_t range_lo, range_shift, range_below;   // second look: first key, sub-bin width, sample entries before it
    uint32_t lo, hi;                         // the interval, as keys, inclusive
    uint32_t way;                            // what comes next
    uint32_t cand_lo, cand_shift, cand_rank; // chosen bin of the candidates
    uint32_t in_lo, in_hi;
    uint32_t tau_key;
    uint32_t done[8];                        // finished workgroups of each kernel that ends with a selection
};

struct Workspace {
    SelectState* st;
    uint32_t* coarse;                        // [kCoarse]
    uint32_t* sub;                           // [kSub]
    uint32_t* cand;                          // [kCandBins]
    uint32_t* last;                          // [kLastBins]
    unsigned long long* exact;               // [2][kExactBins]
    uint32_t* cand_key;                      // [kCap]
    unsigned long long* cand_idx;            // [kCap] linear index into the maps
};
constexpr size_t kStateBytes = 256;
static_assert(sizeof(SelectState) <= kStateBytes, "the state has a block of its own");
// everything up to the candidate lists is cleared before use
constexpr size_t kClearBytes = kStateBytes + (size_t)(kCoarse + kSub + kCandBins + kLastBins) * 4 +
                               (size_t)2 * kExactBins * 8;

__host__ __device__ inline Workspace carve(void* p)
{
    Workspace w;
    char* c = reinterpret_cast<char*>(p);
    w.st = reinterpret_cast<SelectState*>(c);
    w.coarse = reinterpret_cast<uint32_t*>(c + kStateBytes);
    w.sub = w.coarse + kCoarse;
    w.cand = w.sub + kSub;
    w.last = w.cand + kCandBins;
    w.exact = reinterpret_cast<unsigned long long*>(w.last + kLastBins);
    w.cand_idx = reinterpret_cast<unsigned long long*>(c + kClearBytes);
    w.cand_key = reinterpret_cast<uint32_t*>(w.cand_idx + kCap);
    return w;
}
// The size that callers of the C ABI have always been told; kCap is what is left of it.
constexpr size_t kWorkspaceBytes = 64 + (size_t)32768 * 8 + (size_t)(1 << 20) * 12;
static_assert(kClearBytes + (size_t)kCap * 12 <= kWorkspaceBytes, "the candidate lists fit");
static_assert(kClearBytes % 16 == 0, "cleared in 16-byte pieces");

constexpr uint32_t kKeyMinusInf = 0x007fffffu, kKeyPlusInf = 0xff800000u, kKeyZero = 0x80000000u;

__device__ __forceinline__ uint32_t key_of(float v)
{
    uint32_t b = __float_as_uint(v);
    if ((b << 1) == 0) b = 0;                                // -0 -> +0
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float value_of(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

__device__ __forceinline__ int bits_for(unsigned long long width)   // smallest b with width <= 2^b
{
    return width <= 1 ? 0 : 64 - __clzll((long long)(width - 1));
}

__global__ __launch_bounds__(256) void select_init_kernel(void* ws, unsigned long long rank, unsigned long long n,
                                                          float* tau_out, int none)
{
    uint4* p = reinterpret_cast<uint4*>(ws);                 // the state is the first block
    for (int i = blockIdx.x * 256 + threadIdx.x; i < (int)(kClearBytes / 16); i += gridDim.x * 256) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (i == 0) v = make_uint4((uint32_t)rank, (uint32_t)(rank >> 32), (uint32_t)n, (uint32_t)(n >> 32));
        p[i] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && none && tau_out) *tau_out = INFINITY;   // rank N: everything is pruned
}

// The last of a launch's `count` workgroups that get here returns true, and then sees what all of them wrote.
__device__ __forceinline__ bool last_workgroup(uint32_t* done, uint32_t count)
{
    __shared__ uint32_t s_last;
    // What is handed over are counts in memory that only atomics of agent scope touch, and they are read
    // back with loads of that scope: it is enough that this thread's have been performed (a full fence
    // would write back the L2, once per wavefront).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(done, 1u) == count - 1 ? 1u : 0u;
    __syncthreads();
    return s_last != 0;
}

template <typename T>
__device__ __forceinline__ T load_agent(const T* p)          // past this XCD's caches: another one's atomics wrote it
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// For a workgroup of NT threads: the bins of a histogram that hold the given ranks, R of them.  `base`:
// entries before the first bin.  The lane whose bin holds a rank reports it: found(r, bin, entries
// before the bin).  Returns the number of entries counted.  A wavefront owns consecutive rows of 64 bins and reads
// a row with consecutive lanes: the loads go past the caches, so a line would be fetched once per bin otherwise
// (65536 bins of 64 bit: 50 us with consecutive bins per thread).
template <int NB, int NT, int R, typename T, typename F>
__device__ __forceinline__ unsigned long long find_ranks(const T* hist, unsigned long long base,
                                                         const unsigned long long (&ranks)[R], F&& found)
{
    constexpr int ROWS = NB / NT;                            // rows of a wavefront
    constexpr int CH = ROWS < 16 ? ROWS : 16;                // of them, in flight
    static_assert(ROWS * NT == NB && ROWS % CH == 0, "whole rows");
    __shared__ unsigned long long s_wave[NT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bin0 = wave * ROWS * 64 + lane;
    auto load = [&](int r0, T* c) {
#pragma unroll
        for (int i = 0; i < CH; ++i) c[i] = load_agent(hist + bin0 + (r0 + i) * 64);
    };
    T sum = 0;                                               // 32-bit bins count a sample or candidates: below 2^32 in all
    for (int r0 = 0; r0 < ROWS; r0 += CH) {
        T c[CH];
        load(r0, c);
#pragma unroll
        for (int i = 0; i < CH; ++i) sum += c[i];
    }
    sum = wave_sum(sum);
    if (lane == 0) s_wave[wave] = sum;
    __syncthreads();
    unsigned long long before = base, all = 0;
    for (int w = 0; w < NT / 64; ++w) {
        if (w < wave) before += s_wave[w];
        all += s_wave[w];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (ranks[r] < before || ranks[r] >= before + sum) continue;   // uniform over the wavefront
        unsigned long long b = before;
        for (int r0 = 0; r0 < ROWS && b <= ranks[r]; r0 += CH) {
            T c[CH];
            load(r0, c);
            T chunk = 0;
#pragma unroll
            for (int i = 0; i < CH; ++i) chunk += c[i];
            chunk = wave_sum(chunk);
            if (ranks[r] >= b + chunk) {
                b += chunk;
                continue;
            }
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                T incl = c[i];
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const T up = __shfl_up(incl, o, 64);
                    if (lane >= o) incl += up;
                }
                const unsigned long long first = b + incl - c[i];
                if (ranks[r] >= first && ranks[r] < b + incl) found(r, bin0 + (r0 + i) * 64, first);
                b += __shfl(incl, 63, 64);
            }
            break;
        }
    }
    __syncthreads();
    return all;
}

// The maps are walked in units, one wavefront per unit, all of (nearly) the same size so that
// any dealing of units to wavefronts is balanced: a unit is one row, or, for a causal map, the
// pair of rows i and Lq-1-i of a head, whose visible prefixes together hold Lk + (Lk - Lq) + 1
// entries whatever i is.  Inside a unit the two prefixes are laid end to end (the first padded
// to a multiple of 4 positions, so that no quad of positions spans both rows and 128-bit loads
// stay aligned) and lane l takes the 4 entries at position 256 * step + 4 * l.  All row
// arithmetic is wave-uniform.
struct Walk {
    const float* abar;
    int units;                   // below 2^31: the entry point checks H * Lq
    int H, Lq, Lk;
    int causal;
    int per_head;                // units per head
};

__host__ __device__ inline Walk walk_of(const float* abar, int H, int Lq, int Lk, int causal)
{
    Walk w;
    w.abar = abar;
    w.H = H;
    w.Lq = Lq;
    w.Lk = Lk;
    w.causal = causal;
    w.per_head = causal ? (Lq + 1) / 2 : Lq;
    w.units = H * w.per_head;
    return w;
}

// Kernels take the maps' description and the workspace as these scalars and not as structures: arguments arrive in
// registers when a wavefront starts (kernel-argument preloading), structures by a round trip to memory first.
#define AP_WALK_PARAMS const float *p_abar, void *p_ws, int p_H, int p_Lq, int p_Lk, int p_causal
#define AP_WALK_LOCALS                                             \
    const Walk w = walk_of(p_abar, p_H, p_Lq, p_Lk, p_causal);     \
    const Workspace ws = carve(p_ws);

struct Unit {                    // wave-uniform
    const float* row[2];
    long long base[2];           // linear index of the first entry of each row
    int n[2];                    // visible entries of each row (n[1] = 0: single row)
    int p0;                      // n[0] padded
    int total;                   // p0 + n[1]
};

__device__ __forceinline__ Unit decode_unit(const Walk& w, int unit)
{
    Unit u;
    const int h = (int)((uint32_t)unit / (uint32_t)w.per_head);
    const int t = unit - h * w.per_head;
    const long long off = (long long)w.Lk - w.Lq;
    const int i0 = t;
    const int i1 = w.causal ? w.Lq - 1 - t : t;
    u.n[0] = w.causal ? (int)min((long long)w.Lk, i0 + off + 1) : w.Lk;
    u.n[1] = (w.causal && i1 != i0) ? (int)min((long long)w.Lk, i1 + off + 1) : 0;
    u.base[0] = ((long long)h * w.Lq + i0) * w.Lk;
    u.base[1] = ((long long)h * w.Lq + i1) * w.Lk;
    u.row[0] = w.abar + u.base[0];
    u.row[1] = w.abar + u.base[1];
    u.p0 = (u.n[0] + 3) & ~3;                                // positions come in quads
    u.total = u.p0 + u.n[1];
    return u;
}

// rows of a map whose Lk is no multiple of 4 start anywhere: the same loads and stores, 4- and 1-byte aligned
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_a4;
typedef __attribute__((aligned(1))) uint32_t u32_a1;

// Entries col .. col + 3 of a row of which n are visible: one 128-bit load, also where the visible prefix
// ends inside the four; entry by entry only where the row itself ends inside them.
__device__ __forceinline__ f32x4 load_quad(const float* row, int col, int n, int Lk)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (col < n) {
        if (col + 4 <= Lk) {
            v = *reinterpret_cast<const f32x4_a4*>(row + col);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < n) v[e] = row[col + e];
        }
    }
    return v;
}

// ---- sample

// Entry clusters of the sample: 16 positions (four lanes, a quad each), every stride-th cluster of a
// unit, starting at a place that depends on the unit.
struct Sample {
    unsigned long long slots;    // clusters, some of them beyond their unit's end
    uint32_t per_unit, stride;
};

template <typename F>
__device__ __forceinline__ void for_sample(const Walk& w, const Sample& s, F&& body)
{
    constexpr int U = 4;                                     // quads of a lane in flight
    const unsigned long long lanes = s.slots * 4, step = (unsigned long long)gridDim.x * kThreads;
    for (unsigned long long i0 = (unsigned long long)blockIdx.x * kThreads + threadIdx.x; i0 < lanes; i0 += U * step) {
        f32x4 v[U];
        int cnt[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const unsigned long long i = i0 + k * step;
            const unsigned long long slot = i >> 2;
            const uint32_t unit = slot >> 32 ? (uint32_t)(slot / s.per_unit) : (uint32_t)slot / s.per_unit;
            const uint32_t j = (uint32_t)(slot - (unsigned long long)unit * s.per_unit);
            const uint32_t phase = ((unit * 2654435761u) >> 8) % s.stride;
            const unsigned long long pos = ((unsigned long long)j * s.stride + phase) * 16 + 4 * (i & 3);
            cnt[k] = 0;
            v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (i >= lanes) continue;
            const Unit u = decode_unit(w, (int)unit);
            if (pos >= (unsigned long long)u.total) continue;
            const bool second = (int)pos >= u.p0;
            const int col = second ? (int)pos - u.p0 : (int)pos, n = second ? u.n[1] : u.n[0];
            v[k] = load_quad(second ? u.row[1] : u.row[0], col, n, w.Lk);
            cnt[k] = n - col;
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < cnt[k]) body(key_of(v[k][e]));
    }
}

__global__ __launch_bounds__(kThreads) void sample_coarse_kernel(AP_WALK_PARAMS, unsigned long long p_slots,
                                                             uint32_t p_per_unit, uint32_t p_stride)
{
    AP_WALK_LOCALS
    const Sample s = {p_slots, p_per_unit, p_stride};
    __shared__ uint32_t h[kCoarse];
    const int t = threadIdx.x;
    for (int i = t; i < kCoarse; i += kThreads) h[i] = 0;
    __syncthreads();
    for_sample(w, s, [&](uint32_t key) { atomicAdd(&h[key >> kCoarseShift], 1u); });
    __syncthreads();
    for (int i = t; i < kCoarse; i += kThreads)
        if (h[i]) atomicAdd(&ws.coarse[i], h[i]);
    if (!last_workgroup(&ws.st->done[0], gridDim.x)) return;

    __shared__ int s_bin[2];
    __shared__ unsigned long long s_below, s_total;
    if (t == 0) {
        s_bin[0] = 0;
        s_bin[1] = kCoarse - 1;
        s_below = s_total = 0;
    }
    unsigned long long mine = 0;
    for (int i = t; i < kCoarse; i += kThreads) mine += load_agent(ws.coarse + i);
    __syncthreads();
    atomicAdd(&s_total, mine);
    __syncthreads();
    const unsigned long long rank = ws.st->rank, n = ws.st->n, total = s_total;
    // the sample's own rank, and how far the map's may be from it: binomial with the variance of
    // clusters whose entries resemble each other
    unsigned long long s_mid = rank, margin = 0;
    if (s.stride > 1) {
        const double f = (double)rank / (double)n;
        s_mid = (unsigned long long)(f * (double)total);
        margin = (unsigned long long)(kSigmas * sqrt((double)total * f * (1.0 - f) * kDesign)) + 16;
    }
    const unsigned long long top = total > 0 ? total - 1 : 0;
    const unsigned long long s_lo = s_mid > margin ? min(s_mid - margin, top) : 0;
    const unsigned long long s_hi = min(s_mid + margin, top);
    const unsigned long long want[2] = {s_lo, s_hi};
    find_ranks<kCoarse, kThreads>(ws.coarse, 0ull, want, [&](int r, int bin, unsigned long long below) {
        s_bin[r] = bin;
        if (r == 0) s_below = below;
    });
    if (t == 0) {
        const int bits = bits_for((unsigned long long)(s_bin[1] - s_bin[0] + 1) << kCoarseShift);
        ws.st->s_lo = (uint32_t)s_lo;
        ws.st->s_hi = (uint32_t)s_hi;
        ws.st->s_total = (uint32_t)total;
        ws.st->range_lo = (uint32_t)s_bin[0] << kCoarseShift;
        ws.st->range_shift = (uint32_t)(bits > kSubBits ? bits - kSubBits : 0);
        ws.st->range_below = (uint32_t)s_below;
    }
}

// `refine`: the first of two sweeps narrows the interval, whatever it holds.
__global__ __launch_bounds__(kThreads) void sample_fine_kernel(AP_WALK_PARAMS, unsigned long long p_slots,
                                                           uint32_t p_per_unit, uint32_t p_stride, int refine)
{
    AP_WALK_LOCALS
    const Sample s = {p_slots, p_per_unit, p_stride};
    __shared__ uint32_t h[kSub];
    const int t = threadIdx.x;
    for (int i = t; i < kSub; i += kThreads) h[i] = 0;
    __syncthreads();
    const uint32_t range_lo = ws.st->range_lo, shift = ws.st->range_shift;
    for_sample(w, s, [&](uint32_t key) {
        const uint32_t bin = (key - range_lo) >> shift;
        if (key >= range_lo && bin < kSub) atomicAdd(&h[bin], 1u);
    });
    __syncthreads();
    for (int i = t; i < kSub; i += kThreads)
        if (h[i]) atomicAdd(&ws.sub[i], h[i]);
    if (!last_workgroup(&ws.st->done[1], gridDim.x)) return;

    __shared__ int s_bin[2];
    __shared__ uint32_t s_inside;
    if (t == 0) {
        s_bin[0] = 0;
        s_bin[1] = kSub - 1;
        s_inside = 0;
    }
    __syncthreads();
    const uint32_t s_lo = ws.st->s_lo, s_hi = ws.st->s_hi;
    const unsigned long long want[2] = {s_lo, s_hi};
    find_ranks<kSub, kThreads>(ws.sub, (unsigned long long)ws.st->range_below, want,
                     [&](int r, int bin, unsigned long long) { s_bin[r] = bin; });
    // What the sample says about the number of candidates.  If they are more than the list can hold (ties, or values
    // so close together that the bins do not tell them apart) the sweep counts instead of collecting: staging
    // them all, one atomic on one address per few hundred, took 7 ms instead of 0.25 on a map of 16 x 4096 x 4096.
    for (int i = t; i < kSub; i += kThreads)
        if (i >= s_bin[0] && i <= s_bin[1]) atomicAdd(&s_inside, load_agent(ws.sub + i));
    __syncthreads();
    if (t == 0) {
        const bool many = (unsigned long long)s_inside * s.stride > kCap;
        // a sample that ends inside the margin says nothing about the values beyond it
        const bool open = s.stride > 1;
        unsigned long long lo = (unsigned long long)range_lo + ((unsigned long long)s_bin[0] << shift);
        unsigned long long hi = (unsigned long long)range_lo + ((unsigned long long)(s_bin[1] + 1) << shift) - 1;
        if (open && s_lo == 0) lo = 0;
        if (open && s_hi + 1 >= ws.st->s_total) hi = 0xffffffffull;
        // the sweep compares values: keep to keys that are values, and to +0 for zero
        if (lo < kKeyMinusInf) lo = kKeyMinusInf;
        if (hi > kKeyPlusInf) hi = kKeyPlusInf;
        if (hi == kKeyZero - 1) hi = kKeyZero;
        ws.st->lo = (uint32_t)lo;
        ws.st->hi = (uint32_t)hi;
        const bool narrow = refine || many || bits_for(hi - lo + 1) > kMaxBracketBits;
        ws.st->way = hi < lo ? EXACT : (narrow ? NARROW : COLLECT);
        ws.st->in_hi = 0xffffffffu;                          // in_lo = 0 and in_rank = rank complete the whole range
        ws.st->in_rank = ws.st->rank;
    }
}

// Did the sweep collect, and did its interval hold the wanted rank, with all its candidates in the list?
__device__ __forceinline__ bool interval_ok(const SelectState* st, unsigned long long* rank_inside)
{
    const unsigned long long below = st->n - st->above - st->ncand;
    *rank_inside = st->rank - below;
    return (st->way == COLLECT || st->way == LATE) && st->ncand <= kCap && st->rank >= below && st->rank - below < st->ncand;
}

// ---- sweep: the mask of every entry that the interval decides, and the list of those it does not

// Candidates are staged per wavefront in LDS and moved to the global list in blocks, so that the global
// counter sees one atomic per few hundred candidates.  Their places come from ballots.
constexpr int kStage = 384;                  // staged candidates per wavefront
constexpr int kStageFlush = kStage - 256;    // a step adds at most 64 lanes x 4 entries

// Zeros for dst[0 .. n): whole wavefront, any alignment.
__device__ __forceinline__ void zero_bytes(uint8_t* dst, int n, int lane)
{
    const int head = min(n, (int)(-(uintptr_t)dst & 15u));
    if (lane < head) dst[lane] = 0;
    const int body = (n - head) >> 4;
    uint4* q = reinterpret_cast<uint4*>(dst + head);
    for (int i = lane; i < body; i += 64) q[i] = make_uint4(0, 0, 0, 0);
    const int tail = head + 16 * body + lane;
    if (lane < 16 && tail < n) dst[tail] = 0;
}

// COLLECT: the interval decides or makes candidates.
// NARROW: the entries inside the interval are counted in kNarrowBins bins of it, and the bin that holds the wanted rank
//   becomes the interval.  `again`: another sweep follows, which collects if that bin's entries fit the list (this is
//   the way of maps so large that the interval of any reasonable sample holds too much); otherwise the exact
//   way goes on from there.
// KNOWN: every entry is decided by tau.
// For a workgroup of NT threads; `lds`: room for the staged candidates of NT / 64 wavefronts, or for the bins.
template <int MODE, int NT>
__device__ __forceinline__ void sweep(const Walk& w, const Workspace& ws, uint8_t* mask, float* tau_out, int again,
                                      unsigned long long* lds)
{
    constexpr int U = 8;                                     // quads of a lane in flight
    constexpr int WAVES = NT / 64;
    __shared__ unsigned long long s_above;
    uint32_t* s_bins = reinterpret_cast<uint32_t*>(lds);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = (int)gridDim.x * WAVES;
    unsigned long long* s_idx = lds + wave * kStage;         // of this wavefront
    uint32_t* s_key = reinterpret_cast<uint32_t*>(lds + WAVES * kStage) + wave * kStage;
    const float lo = MODE == KNOWN ? 0.f : value_of(ws.st->lo);
    const float hi = MODE == KNOWN ? 0.f : value_of(ws.st->hi);
    const float tau = MODE == KNOWN ? value_of(ws.st->tau_key) : 0.f;
    uint32_t lo_key = 0;
    int shift = 0;                                           // NARROW: width of a bin
    if (MODE == NARROW) {
        lo_key = ws.st->lo;
        shift = max(0, bits_for((unsigned long long)ws.st->hi - lo_key + 1) - kNarrowBits);
        for (int i = threadIdx.x; i < kNarrowBins; i += NT) s_bins[i] = 0;
    }
    if (threadIdx.x == 0) s_above = 0;
    if (MODE == NARROW) __syncthreads();
    int fill = 0;                                            // staged candidates (wave-uniform)
    // NARROW: entries of one bin, the first that the wavefront meets in a unit, are counted in a register: in a map
    // full of ties the lanes would take turns on one address otherwise
    uint32_t hot = ~0u, hot_n = 0;
    unsigned long long above = 0;                            // of this lane

    auto flush = [&]() {                                     // wave-uniform
        if (fill == 0) return;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // staged entries written by other lanes
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&ws.st->ncand, (unsigned long long)fill);
        base = __shfl(base, 0, 64);
        for (int i = lane; i < fill; i += 64) {
            const unsigned long long slot = base + i;
            if (slot < kCap) {                               // the count runs on: it tells that they did not fit
                ws.cand_key[slot] = s_key[i];
                ws.cand_idx[slot] = s_idx[i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        fill = 0;
    };

    // Entries [lin, lin + 4) of the maps, of which the first cnt count: decide, collect, write.
    auto one = [&](const f32x4& v, long long lin, int cnt, bool whole, bool room) {
        bool a[4], c[4];
        uint32_t out = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool vis = whole || e < cnt;               // whole is a compile-time constant
            a[e] = MODE == KNOWN ? !(v[e] < tau) : !(v[e] <= hi);
            c[e] = MODE != KNOWN && v[e] >= lo && !a[e];
            if (!whole) {
                a[e] = a[e] && vis;
                c[e] = c[e] && vis;
            }
            out |= a[e] ? 1u << (8 * e) : 0u;
        }
        if (MODE != KNOWN) {
            above += (uint32_t)__popc(out);
            if (MODE == NARROW) {
                if (hot == ~0u) {
                    const unsigned long long m = __ballot(c[0]);
                    if (m) hot = __builtin_amdgcn_readlane((key_of(v[0]) - lo_key) >> shift, __ffsll((long long)m) - 1);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c[e]) {
                        const uint32_t bin = (key_of(v[e]) - lo_key) >> shift;
                        if (bin == hot) ++hot_n;
                        else atomicAdd(&s_bins[bin], 1u);
                    }
                return;
            }
            if (__ballot(c[0] || c[1] || c[2] || c[3]) != 0) {
                if (fill > kStageFlush) flush();
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned long long m = __ballot(c[e]);
                    if (m == 0) continue;
                    if (c[e]) {
                        const int pos = fill + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                        s_key[pos] = key_of(v[e]);
                        s_idx[pos] = (unsigned long long)(lin + e);
                    }
                    fill += __popcll(m);
                }
            }
        }
        // candidates get 0 here, their byte comes later; four entries cut by the visible prefix also
        // write the zeros of the hidden ones (inside the row)
        if (mask && (whole || cnt > 0)) {
            if (whole || room) {
                *reinterpret_cast<u32_a1*>(mask + lin) = out;
            } else {
                for (int e = 0; e < cnt; ++e) mask[lin + e] = (uint8_t)((out >> (8 * e)) & 1u);
            }
        }
    };

    for (long long unit = (long long)blockIdx.x * WAVES + wave; unit < w.units; unit += nwaves) {
        const Unit u = decode_unit(w, (int)unit);
        // what is left of each row behind its last 256 visible entries: requested first
        f32x4 rest[2];
        int rest_col[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            rest_col[r] = (u.n[r] & ~255) + 4 * lane;
            rest[r] = load_quad(u.row[r], rest_col[r], u.n[r], w.Lk);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int steps = u.n[r] >> 8;                   // 256 entries of the row each, all visible
            const float* row = u.row[r] + 4 * lane;
            const long long lin = u.base[r] + 4 * lane;
            for (int s0 = 0; s0 < steps; s0 += U) {
                f32x4 v[U];
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (s0 + k < steps) v[k] = *reinterpret_cast<const f32x4_a4*>(row + (s0 + k) * 256);
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (s0 + k < steps) one(v[k], lin + (s0 + k) * 256, 4, true, true);
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (u.n[r] == 0) continue;                       // a unit of one row
            one(rest[r], u.base[r] + rest_col[r], u.n[r] - rest_col[r], false, rest_col[r] + 4 <= w.Lk);
            if (mask) {                                      // the hidden tail of the row
                const int up = (u.n[r] + 3) & ~3;            // written with the last four, if they fitted the row
                const int start = up <= w.Lk ? up : u.n[r];
                if (start < w.Lk) zero_bytes(mask + u.base[r] + start, w.Lk - start, lane);
            }
        }
        if (MODE == NARROW && hot != ~0u) {
            const uint32_t n = wave_sum(hot_n);
            if (lane == 0) atomicAdd(&s_bins[hot], n);
            hot = ~0u;
            hot_n = 0;
        }
    }
    if (MODE != KNOWN) {
        flush();
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) above += __shfl_xor(above, o, 64);
        __syncthreads();
        if (lane == 0 && above) atomicAdd(&s_above, above);
        __syncthreads();
        if (threadIdx.x == 0 && s_above) atomicAdd(&ws.st->above, s_above);
    }
    if (MODE == NARROW) {
        unsigned long long* hist = ws.exact;                 // borrowed from the exact way, given back cleared
        for (int i = threadIdx.x; i < kNarrowBins; i += NT)
            if (s_bins[i]) atomicAdd(&hist[i], (unsigned long long)s_bins[i]);
        if (!last_workgroup(&ws.st->done[again ? 6 : 7], gridDim.x)) return;
        __shared__ unsigned long long s_inside, s_count, s_rank;
        __shared__ int s_found;
        if (threadIdx.x == 0) {
            s_inside = 0;
            s_found = -1;
        }
        __syncthreads();
        unsigned long long mine = 0;
        for (int i = threadIdx.x; i < kNarrowBins; i += NT) mine += load_agent(hist + i);
        atomicAdd(&s_inside, mine);
        __syncthreads();
        const unsigned long long rank = ws.st->rank, below = ws.st->n - load_agent(&ws.st->above) - s_inside;
        const unsigned long long want[1] = {rank};
        find_ranks<kNarrowBins, NT>(hist, below, want, [&](int, int bin, unsigned long long first) {
            s_found = bin;
            s_rank = rank - first;
            s_count = load_agent(hist + bin);
        });
        for (int i = threadIdx.x; i < kNarrowBins; i += NT) hist[i] = 0;
        if (threadIdx.x == 0) {
            ws.st->above = 0;                                // the next sweep counts again
            if (s_found < 0) {
                ws.st->way = EXACT;                          // the interval misses the rank: from the whole range
            } else {
                const uint32_t lo2 = lo_key + ((uint32_t)s_found << shift);
                uint32_t hi2 = min(ws.st->hi, lo2 + ((1u << shift) - 1u));
                if (hi2 == kKeyZero - 1) --hi2;              // as a value it is -0, which counts as +0 (the next key)
                if (hi2 == lo2) {
                    ws.st->way = KNOWN;
                    ws.st->tau_key = lo2;
                    if (tau_out) *tau_out = value_of(lo2);
                } else if (again) {
                    const bool fits = s_count <= kCap && bits_for((unsigned long long)hi2 - lo2 + 1) <= kMaxBracketBits;
                    ws.st->way = fits ? COLLECT : NARROW;
                    ws.st->lo = lo2;
                    ws.st->hi = hi2;
                } else if (s_count <= kCap && hi2 - lo2 < kExactBins) {
                    ws.st->way = LATE;
                    ws.st->lo = lo2;
                    ws.st->hi = hi2;
                } else {
                    ws.st->way = EXACT;
                    ws.st->in_lo = lo2;
                    ws.st->in_hi = hi2;
                    ws.st->in_rank = s_rank;
                }
            }
        }
    }
}

__global__ __launch_bounds__(kSweepThreads) void mask_sweep_kernel(AP_WALK_PARAMS, uint8_t* mask, float* tau_out, int again)
{
    AP_WALK_LOCALS
    __shared__ unsigned long long lds[kNarrowBins / 2];
    static_assert(sizeof lds >= kSweepThreads / 64 * kStage * 12, "the staged candidates fit");
    const uint32_t way = ws.st->way;
    if (way == COLLECT) sweep<COLLECT, kSweepThreads>(w, ws, mask, tau_out, again, lds);
    else if (way == NARROW) sweep<NARROW, kSweepThreads>(w, ws, nullptr, tau_out, again, lds);
}

// The mask where the sweep did not write all of it: the candidates' bytes, or, after the exact way, every entry.
__global__ __launch_bounds__(kSweepThreads) void mask_finish_kernel(AP_WALK_PARAMS, uint8_t* mask)
{
    AP_WALK_LOCALS
    unsigned long long dummy;
    if (!interval_ok(ws.st, &dummy)) return sweep<KNOWN, kSweepThreads>(w, ws, mask, nullptr, 0, nullptr);
    const uint32_t n = (uint32_t)ws.st->ncand, tau_key = ws.st->tau_key;
    for (uint32_t i = blockIdx.x * kSweepThreads + threadIdx.x; i < n; i += gridDim.x * kSweepThreads)
        if (ws.cand_key[i] >= tau_key) mask[ws.cand_idx[i]] = 1;
}

// ---- select: tau among the candidates, in two histograms over their key bits.  `h` is LDS, `parts` the
// workgroups of the launch that take part.
__device__ __forceinline__ void candidate_bins(const Workspace& ws, uint32_t* h, unsigned long long rank, uint32_t parts)
{
    const int t = threadIdx.x;
    const uint32_t n = (uint32_t)ws.st->ncand, lo = ws.st->lo;
    const int bits = bits_for((unsigned long long)ws.st->hi - lo + 1);
    const int shift = bits > kCandBits ? bits - kCandBits : 0;
    for (int i = t; i < kCandBins; i += kThreads) h[i] = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x * kThreads + t; i < n; i += parts * kThreads)
        atomicAdd(&h[(ws.cand_key[i] - lo) >> shift], 1u);
    __syncthreads();
    for (int i = t; i < kCandBins; i += kThreads)
        if (h[i]) atomicAdd(&ws.cand[i], h[i]);
    if (!last_workgroup(&ws.st->done[2], parts)) return;
    const unsigned long long want[1] = {rank};
    find_ranks<kCandBins, kThreads>(ws.cand, 0ull, want, [&](int, int bin, unsigned long long below) {
        ws.st->cand_lo = lo + ((uint32_t)bin << shift);
        ws.st->cand_shift = (uint32_t)shift;
        ws.st->cand_rank = (uint32_t)(rank - below);
    });
}

__device__ __forceinline__ void candidate_last(const Workspace& ws, uint32_t* h, float* tau_out, uint32_t parts)
{
    const int t = threadIdx.x;
    const uint32_t n = (uint32_t)ws.st->ncand, lo = ws.st->cand_lo, width = 1u << ws.st->cand_shift;   // <= kLastBins
    for (int i = t; i < kLastBins; i += kThreads) h[i] = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x * kThreads + t; i < n; i += parts * kThreads) {
        const uint32_t d = ws.cand_key[i] - lo;
        if (d < width) atomicAdd(&h[d], 1u);
    }
    __syncthreads();
    for (int i = t; i < kLastBins; i += kThreads)
        if (h[i]) atomicAdd(&ws.last[i], h[i]);
    if (!last_workgroup(&ws.st->done[3], parts)) return;
    const unsigned long long want[1] = {ws.st->cand_rank};
    find_ranks<kLastBins, kThreads>(ws.last, 0ull, want, [&](int, int bin, unsigned long long) {
        ws.st->tau_key = lo + (uint32_t)bin;
        if (tau_out) *tau_out = value_of(lo + (uint32_t)bin);
    });
}

// LATE: the whole selection in one level, the interval has at most kExactBins keys.  16-bit halves of LDS words: a
// workgroup has at most kCap / 64 + kThreads candidates.
__device__ __forceinline__ void candidate_only(const Workspace& ws, uint32_t* h, unsigned long long rank, float* tau_out,
                                               uint32_t parts)
{
    const int t = threadIdx.x;
    const uint32_t n = (uint32_t)ws.st->ncand, lo = ws.st->lo;
    unsigned long long* hist = ws.exact + kExactBins;
    for (int i = t; i < kExactBins / 2; i += kThreads) h[i] = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x * kThreads + t; i < n; i += parts * kThreads) {
        const uint32_t d = ws.cand_key[i] - lo;
        atomicAdd(&h[d >> 1], 1u << (16 * (d & 1)));
    }
    __syncthreads();
    for (int i = t; i < kExactBins / 2; i += kThreads) {
        const uint32_t v = h[i];
        if (v & 0xffffu) atomicAdd(&hist[2 * i], (unsigned long long)(v & 0xffffu));
        if (v >> 16) atomicAdd(&hist[2 * i + 1], (unsigned long long)(v >> 16));
    }
    if (!last_workgroup(&ws.st->done[3], parts)) return;
    const unsigned long long want[1] = {rank};
    find_ranks<kExactBins, kThreads>(hist, 0ull, want, [&](int, int bin, unsigned long long) {
        ws.st->tau_key = lo + (uint32_t)bin;
        if (tau_out) *tau_out = value_of(lo + (uint32_t)bin);
    });
}

// One of the two levels of the selection: a histogram over the candidates or, only if the interval failed,
// the exact way: the entries of [in_lo, in_hi] (at first the whole range of keys, or what a narrowing sweep left)
// in 65536 bins per level over all entries, the counts of a workgroup kept as 16-bit halves of
// LDS words and moved out before one of them can overflow.  Both in one launch: a launch that returns at once
// costs 4.6 us between its neighbours, as does the mask sweep of the exact way, which shares the launch that
// writes the candidates' mask bytes (16 x 4096 x 4096 causal: 9 us of a call).
template <int LEVEL>
__global__ __launch_bounds__(kThreads) void select_level_kernel(AP_WALK_PARAMS, uint8_t* mask, float* tau_out, uint32_t parts)
{
    AP_WALK_LOCALS
    constexpr int STEP = 256;                                // entries of a wavefront's step
    constexpr int STEPS = 65535 / (STEP * (kThreads / 64));  // steps of all wavefronts between two moves: 15
    __shared__ __attribute__((aligned(8))) uint32_t h[kExactBins / 2];
    static_assert(sizeof h >= kThreads / 64 * kStage * 12, "the staged candidates fit");
    unsigned long long rank_inside;
    if (LEVEL == 0 && ws.st->way == LATE)
        return sweep<COLLECT, kThreads>(w, ws, mask, tau_out, 0, reinterpret_cast<unsigned long long*>(h));
    if (interval_ok(ws.st, &rank_inside)) {
        if (blockIdx.x >= parts) return;
        if (LEVEL == 0) candidate_bins(ws, h, rank_inside, parts);
        else if (ws.st->way == LATE) candidate_only(ws, h, rank_inside, tau_out, parts);
        else candidate_last(ws, h, tau_out, parts);
        return;
    }
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const long long nwaves = (long long)gridDim.x * (kThreads / 64);
    if (ws.st->way == KNOWN) return;
    const uint32_t in_lo = ws.st->in_lo, in_hi = ws.st->in_hi, in_width = in_hi - in_lo;
    const unsigned long long in_rank = ws.st->in_rank;
    const int in_bits = bits_for((unsigned long long)in_width + 1), in_shift = in_bits > 16 ? in_bits - 16 : 0;
    unsigned long long* hist = ws.exact + (size_t)LEVEL * kExactBins;
    for (int i = t; i < kExactBins / 2; i += kThreads) h[i] = 0;
    __syncthreads();
    long long unit = (long long)wave * gridDim.x + blockIdx.x;   // runs past w.units
    int pos0 = 0;
    // every wavefront takes the same number of rounds, those that have run out with nothing to do
    const long long units_per_wave = ((long long)w.units + nwaves - 1) / nwaves;
    const int steps_per_unit = (int)(((long long)w.Lk + (w.causal ? (long long)w.Lk - w.Lq + 5 : 0) + STEP - 1) / STEP) + 1;
    const long long rounds = (units_per_wave * steps_per_unit + STEPS - 1) / STEPS;
    constexpr int U = 8;                                     // quads of a lane in flight
    Unit u = {};
    for (long long round = 0; round < rounds; ++round) {
        for (int k0 = 0; k0 < STEPS && unit < w.units; k0 += U) {
            f32x4 v[U];
            int cnt[U];                                      // visible entries of the lane's quad
#pragma unroll
            for (int k = 0; k < U; ++k) {
                cnt[k] = 0;
                v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (k0 + k >= STEPS || unit >= w.units) continue;   // uniform
                if (pos0 == 0) u = decode_unit(w, (int)unit);
                const int pos = pos0 + lane * 4;
                const bool second = pos >= u.p0;
                const int col = second ? pos - u.p0 : pos, n = second ? u.n[1] : u.n[0];
                v[k] = load_quad(second ? u.row[1] : u.row[0], col, n, w.Lk);
                cnt[k] = n - col;
                pos0 += STEP;
                if (pos0 >= u.total) {
                    pos0 = 0;
                    unit += nwaves;
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t key = key_of(v[k][e]);
                    const bool part = e < cnt[k] && key - in_lo <= in_width;
                    const uint32_t bin = (key - in_lo) >> in_shift;
                    // the lanes that share the first lane's bin add once: ties (zeros, equal values)
                    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
                    const unsigned long long same = __ballot(part && bin == first);
                    if (same != 0 && lane == 0) atomicAdd(&h[first >> 1], (uint32_t)__popcll(same) << (16 * (first & 1)));
                    if (part && bin != first) atomicAdd(&h[bin >> 1], 1u << (16 * (bin & 1)));
                }
        }
        __syncthreads();
        for (int i = t; i < kExactBins / 2; i += kThreads) {
            const uint32_t v = h[i];
            if (v == 0) continue;
            h[i] = 0;
            if (v & 0xffffu) atomicAdd(&hist[2 * i], (unsigned long long)(v & 0xffffu));
            if (v >> 16) atomicAdd(&hist[2 * i + 1], (unsigned long long)(v >> 16));
        }
        __syncthreads();
    }
    if (!last_workgroup(&ws.st->done[4 + LEVEL], gridDim.x)) return;
    const unsigned long long want[1] = {in_rank};
    find_ranks<kExactBins, kThreads>(hist, 0ull, want, [&](int, int bin, unsigned long long below) {
        const uint32_t lo = in_lo + ((uint32_t)bin << in_shift);
        if (in_shift == 0) {
            ws.st->way = KNOWN;
            ws.st->tau_key = lo;
            if (tau_out) *tau_out = value_of(lo);
        } else {
            ws.st->way = EXACT;
            ws.st->in_lo = lo;
            ws.st->in_hi = min(in_hi, lo + ((1u << in_shift) - 1u));
            ws.st->in_rank = in_rank - below;
        }
    });
}

__global__ __launch_bounds__(256) void zero_mask_kernel(uint8_t* mask, unsigned long long n)   // everything is pruned
{
    const unsigned long long words = n / 4, step = (unsigned long long)gridDim.x * 256;
    const unsigned long long i0 = (unsigned long long)blockIdx.x * 256 + threadIdx.x;
    for (unsigned long long i = i0; i < words; i += step) reinterpret_cast<uint32_t*>(mask)[i] = 0u;
    if (i0 < (n & 3)) mask[words * 4 + i0] = 0;
}

}  // namespace

size_t prune_mask_workspace_bytes() { return kWorkspaceBytes; }

hipError_t launch_prune_mask(const float* abar, int H, int Lq, int Lk, int causal,
                             unsigned long long rank, unsigned long long n, bool none, uint8_t* mask,
                             float* tau_out, void* workspace, hipStream_t stream)
{
    const Walk w = walk_of(abar, H, Lq, Lk, causal);

    hipLaunchKernelGGL(select_init_kernel, dim3(64), dim3(256), 0, stream, workspace, rank, n, tau_out, none ? 1 : 0);
    if (none) {
        if (mask)
            hipLaunchKernelGGL(zero_mask_kernel, dim3(2048), dim3(256), 0, stream, mask,
                               (unsigned long long)H * Lq * Lk);
        return hipGetLastError();
    }
    // positions of the longest unit: a row, or a pair of rows with the first padded to a quad
    const long long unit_len = causal ? (long long)Lk + (Lk - Lq) + 1 + 3 : Lk;
    Sample s;
    // A sample for which the interval holds about kAim candidates: 2 kSigmas standard deviations of the
    // sample, as a share of the n entries.  It grows with the square of n: 2.3 million entries at 16 x 4096 x 4096,
    // every third cluster at 16 x 16384 x 16384.  There a small sample and one exact pass over the map come cheaper.
    const double f = (double)rank / (double)n, share = (double)n / kAim;
    const double want = 4.0 * kSigmas * kSigmas * kDesign * f * (1.0 - f) * share * share;
    const int sweep_wgs = (w.units + kSweepThreads / 64 - 1) / (kSweepThreads / 64);
    // Two wavefronts per SIMD with 8 KB in flight each.  More wavefronts mean more places of the map and
    // the mask that are read and written at a time, and that costs more than it hides: whole call at
    // 16 x 4096 x 4096 causal 245 us with 256 workgroups, 258 with 384, 271 with 512, 288 with 768.
    const unsigned grid = (unsigned)min(256, sweep_wgs);
    // entries that one workgroup of the exact pass may meet: it counts them in 32 bits
    const double per_wg = (double)((sweep_wgs + grid - 1) / grid) * (kSweepThreads / 64) * (double)unit_len;
    const bool refine = want > (double)n / kRefineShare && n > 2 * kSample && per_wg < 4294967296.0;
    // (std::min: the min of host code takes ints, and of a double beyond them anything may come)
    const unsigned long long size =
        want > (double)kSample && !refine ? (unsigned long long)std::min({want, (double)n, 2147483648.0}) : kSample;
    s.stride = (uint32_t)std::min(std::max(n / size, 1ull), 1ull << 30);
    s.per_unit = (uint32_t)(((unit_len + 15) / 16 + s.stride - 1) / s.stride);
    s.slots = (unsigned long long)w.units * s.per_unit;
    const unsigned sgrid = (unsigned)std::min(128ull, (s.slots * 4 + kThreads - 1) / kThreads);
    // the exact levels take 128 KB of LDS: one workgroup of 16 wavefronts per compute unit
    const unsigned egrid = (unsigned)min(256, (w.units + kThreads / 64 - 1) / (kThreads / 64));
    const unsigned cgrid = (unsigned)std::min(64ull, (n + kThreads - 1) / kThreads);

    hipLaunchKernelGGL(sample_coarse_kernel, dim3(sgrid), dim3(kThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                       s.slots, s.per_unit, s.stride);
    hipLaunchKernelGGL(sample_fine_kernel, dim3(sgrid), dim3(kThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                       s.slots, s.per_unit, s.stride, refine ? 1 : 0);
    if (refine)
        hipLaunchKernelGGL(mask_sweep_kernel, dim3(grid), dim3(kSweepThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                           mask, tau_out, 1);
    hipLaunchKernelGGL(mask_sweep_kernel, dim3(grid), dim3(kSweepThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                       mask, tau_out, 0);
    const unsigned lgrid = max(egrid, cgrid);
    hipLaunchKernelGGL(select_level_kernel<0>, dim3(lgrid), dim3(kThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                       mask, tau_out, cgrid);
    hipLaunchKernelGGL(select_level_kernel<1>, dim3(lgrid), dim3(kThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                       mask, tau_out, cgrid);
    if (mask)
        hipLaunchKernelGGL(mask_finish_kernel, dim3(256), dim3(kSweepThreads), 0, stream, abar, workspace, H, Lq, Lk, causal,
                           mask);
    return hipGetLastError();
}

}  // namespace ap
