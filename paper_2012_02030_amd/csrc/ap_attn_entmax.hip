// Masked attention forward with the 1.5-entmax normaliser (Section 6: the experiments are
// repeated with 1.5-entmax in place of softmax, together with the pruning mask).
//
// With x_j = scale * <q, k_j> / 2 over the kept, visible keys of a query, 1.5-entmax is
//     p_j = [x_j - tau]_+^2,   tau such that sum_j p_j = 1
// (the optimality conditions of its defining problem).  Unlike softmax this needs a per-row
// threshold before any probability is known:
//
//   maximum     row maximum m of the kept visible keys' scores
//   steps       with y = x - m <= 0, d = [y - tau]_+: the norm |d| and the sum g of d, and a Newton
//               step on h(tau) = |d| - 1:  tau += (|d| - 1) |d| / g.  h is convex and decreasing
//               with its root in [-1, 0); started at -1 (where h >= 0 because the maximum
//               contributes 1) the steps increase monotonically to the root and never pass it.
//               The norm is much closer to linear than its square, which saves about half of
//               the steps.  A row is done when | |d|^2 - 1 | <= 1e-5 at its tau, or after the
//               step taken from a tau with | |d|^2 - 1 | <= 1e-2: the steps converge quadratically,
//               so that step usually leaves a few 1e-5 and the one that would only confirm it is
//               saved.  The block row goes on until all its rows are done.
//   output      P = [y - tau]_+^2, O^T += V^T P^T, O / sum P.  The sum of P is what an unconfirmed step
//               leaves: where it is more than 1e-4 above 1 (many scores just above tau that leave the
//               support: 2.4e-3 with 3400 of them within 0.002), the block row starts again from its
//               tau, every step confirmed.
//
// A workgroup of four wavefronts takes a block row, a wavefront a 32 x 32 quarter of every entry.  The scores of up to
// E (2 to 8) entries stay in registers, 16 per entry and lane: K is read once, a Newton step is three vector
// instructions per score and an exchange of the key halves through LDS, and V travels under the steps.  Of longer
// block rows the first HL entries are held and the others' scores are formed again in every sweep, as all were before.
// B4 H16 L2048 (3.9 entries a block row) D128 112 -> 64 us, D64 78 -> 42; B32 H8 117 x 141 D64 25 -> 11.4; 32 entries
// a block row (nothing pruned) D128 735 -> 680, D64 541 -> 444; without schedules (up to 32 tiles, every tenth key) D128
// 487 -> 361.
//
// Same operand layouts and LDS-direct loads as the softmax kernel; walks the layout's 64x64 tiles or, if given, the
// entries of its visit schedule.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"
#include "ap_mfma_common.h"

namespace ap {

namespace {

using namespace mfma;

constexpr float kEntmaxTol = 1e-5f;          // on sum p - 1
constexpr float kEntmaxEarly = 1e-2f;        // residual from which one more step is taken unconfirmed
constexpr float kEntmaxLeft = 1e-4f;         // largest residual that such a step may leave
constexpr int kEntmaxMaxIter = 60;

// s[32 x 32] = T * B^T for 32 rows of a tile in LDS (SWZ_BOTH; `row` is this lane's row) and an operand in registers.
template <int D>
__device__ __forceinline__ void product_32(const uint16_t* T, int row, int k_swz, const bf16x8* b, f32x16& s)
{
    constexpr int KSTEPS = D / 16;
    constexpr int AHEAD = KSTEPS < 4 ? KSTEPS : 4;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    bf16x8 x[KSTEPS];
    int at = row * D + k_swz * 8;                            // chunk 2 kk: this ^ (16 kk)
    asm volatile("" : "+v"(at));
    auto read = [&](int kk) { x[kk] = *reinterpret_cast<const bf16x8*>(T + (at ^ (16 * kk))); };
#pragma unroll
    for (int kk = 0; kk < AHEAD; ++kk) read(kk);
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        if (kk + AHEAD < KSTEPS) read(kk + AHEAD);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[kk], b[kk], s, 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);   // pin that order
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        if (kk + AHEAD < KSTEPS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
}

// [y - tau]_+ for y <= 0 and tau in [-1, 0): at most 1, so that the subtraction's own clamp does it (NaN and -inf: 0)
__device__ __forceinline__ float above(float y, float tau) { return __builtin_amdgcn_fmed3f(y - tau, 0.f, 1.f); }

template <bool V> struct Flag {
    static constexpr bool value = V;
};

__device__ __forceinline__ float both_halves_max(float v)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
}
__device__ __forceinline__ float both_halves_sum(float v)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}

// LDS of a workgroup: four tiles (a ring of three and the Q rows), gather keys of the held entries, and what the key
// halves of a query exchange, by parity.
template <int D, int E>
struct EntmaxLds {
    uint16_t tiles[4 * kBN * D];
    int32_t cols[E][64];
    float2 pair[2][2][64];
    uint32_t pend[2][4];
};

// One wavefront's view of its workgroup's block row.  Four wavefronts: `qh` and `kh` say which 32 x 32 quarter of
// every entry this one forms.  Entries are those of the visit schedule (runs of 64 consecutive keys or 64 gathered
// keys, causal limit already folded into their bitmaps), or the layout's tiles.
template <int D, int E>
struct EntmaxRow {
    static constexpr int TILE = kBN * D, KSTEPS = D / 16, DBLK = D / 32;
    static constexpr int RPI = 64 / (D / 8);                 // tile rows per load instruction
    static constexpr int NLOAD = (D / 8) / 4;                // load instructions per wavefront and tile
    const FwdArgs& a;
    EntmaxLds<D, E>& m;
    lds_u16* lds;
    int wave, lane, n, hh, qh, kh, brow, k_swz;
    int t0, ne;
    bool use_sched;
    long long diag;                                          // last visible key of this lane's query if causal
    float c;                                                 // x = c * <q, k>
    int sk_bytes, sv_bytes;
    rsrc_t k_rsrc, v_rsrc;
    const int32_t* starts;                                   // start of an entry, or block column of a tile
    const int32_t* cols;                                     // gather keys, or null
    const uint32_t* words;
    TrReadU<D> tr;
    // state of the row
    int par = 0;
    float tau = -1.f, mc = 0.f, psum = 0.f;
    bool empty = true;

    __device__ __forceinline__ EntmaxRow(const FwdArgs& args, EntmaxLds<D, E>& mem, int tid_, int b, int h, int qb, int t0_,
                                         int ne_, const int32_t* starts_, const int32_t* cols_, const uint32_t* words_)
        : a(args), m(mem), lds((lds_u16*)mem.tiles), t0(t0_), ne(ne_), starts(starts_), cols(cols_), words(words_)
    {
        wave = __builtin_amdgcn_readfirstlane(tid_ >> 6);
        lane = tid_ & 63;
        n = lane & 31;
        hh = lane >> 5;
        qh = wave & 1;
        kh = wave >> 1;
        brow = qh * 32 + n;
        k_swz = hh ^ swz_u<D>(n);
        use_sched = cols != nullptr;
        diag = (long long)qb * 64 + brow + a.Lk - a.Lq;
        c = 0.5f * a.scale;
        sk_bytes = (int)a.sk[2] * 2;
        sv_bytes = (int)a.sv[2] * 2;
        k_rsrc = make_rsrc((const uint16_t*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1],
                           (unsigned)((a.Lk - 1) * sk_bytes + D * 2));
        v_rsrc = make_rsrc((const uint16_t*)a.V + (size_t)b * a.sv[0] + (size_t)h * a.sv[1],
                           (unsigned)((a.Lk - 1) * sv_bytes + D * 2));
        tr = make_tr_read_u<D>(lane);
    }
    // first key of an entry, -1: gathered
    __device__ __forceinline__ int first_key(int t) const { return use_sched ? starts[t] : starts[t] * kBN; }
    // this lane's half of its bitmap word; without a schedule the causal limit is still to be applied
    __device__ __forceinline__ uint32_t raw_word(int t) const { return words[((size_t)t * 64 + brow) * 2 + kh]; }
    __device__ __forceinline__ uint32_t visible(uint32_t w, int k0) const
    {
        if (a.causal && !use_sched) {
            const long long lim = diag - k0 - 32 * kh;
            if (lim < 0) w = 0;
            else if (lim < 31) w &= (2u << lim) - 1u;
        }
        return w;
    }
    // K or V rows of an entry.  ANEW: addresses are formed for this tile alone; held over many, they would cost
    // registers that the scores need.
    template <bool ANEW>
    __device__ __forceinline__ void issue(bool v, int place, int k0, const int* gk) const
    {
        int l = lane;
        if (ANEW) asm volatile("" : "+v"(l));
        const rsrc_t rs = v ? v_rsrc : k_rsrc;
        const int stride = v ? sv_bytes : sk_bytes;
        if (k0 >= 0) issue_tile_loads<D, 4, SWZ_BOTH>(rs, lds + place * TILE, k0, stride, wave, l);
        else issue_gather_loads<D, 4, SWZ_BOTH>(rs, lds + place * TILE, gk, stride, wave, l);
    }
    // slot of this lane's row in load instruction u
    __device__ __forceinline__ int load_row(int u) const { return (wave + 4 * u) * RPI + lane / (D / 8); }

    // scores of pruned and hidden entries become -inf
    __device__ __forceinline__ void mask_scores(uint32_t word, f32x16& x) const
    {
        const int wbits = (int)(word >> (4 * hh));
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(wbits, 8 * (i / 4) + (i % 4), 1);
            x[i] = __uint_as_float((__float_as_uint(x[i]) & keep) | (0xff800000u & ~keep));
        }
    }
    // (x, y) of the two key halves of this lane's query
    __device__ __forceinline__ float4 exchange(float x, float y)
    {
        if (hh == 0) m.pair[par][kh][brow] = make_float2(x, y);
        __syncthreads();
        const float2 u = m.pair[par][0][brow], v = m.pair[par][1][brow];
        par ^= 1;
        return make_float4(u.x, u.y, v.x, v.y);
    }
    __device__ __forceinline__ void set_max(float mx)
    {
        const float4 x = exchange(both_halves_max(mx), 0.f);
        mx = fmaxf(x.x, x.z);
        empty = mx == -INFINITY;
        mc = empty ? 0.f : mx * c;
    }
    __device__ __forceinline__ void set_psum()
    {
        const float4 x = exchange(both_halves_sum(psum), 0.f);
        psum = x.x + x.z;
    }
    __device__ __forceinline__ bool left_too_much() const { return __syncthreads_or(psum - 1.0f > kEntmaxLeft ? 1 : 0) != 0; }
    // One Newton step from the sums over all of a query's keys of d = [y - tau]_+ and d^2.
    __device__ __forceinline__ void newton_step(float g1, float g2, bool confirm, bool& done)
    {
        if (done) return;
        const float f = g2 - 1.0f;
        if (fabsf(f) <= kEntmaxTol || g1 <= 0.f) {
            done = true;
        } else {
            const float nd = sqrtf(g2);
            tau = fminf(fmaxf(tau + (nd - 1.0f) * nd / g1, -1.0f), 0.f);
            done = !confirm && fabsf(f) <= kEntmaxEarly;     // this step is the last one
        }
    }
    // O^T += V^T P^T for x = y - tau, cut at 0, of a quarter and the V rows in a place
    __device__ __forceinline__ void add_tile(f32x16& x, int place, f32x16* oacc)
    {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            x[i] = x[i] * x[i];
            psum += x[i];
        }
        bf16x8 pb[2];
        to_operands(x, pb);
        tr_mm_32<D, false>(lds + place * TILE + kh * 32 * D, pb, oacc, tr);
    }
};

// A block row of at most E entries: every score stays in registers.  False: an unconfirmed step left too much.
template <int D, int E>
__device__ __forceinline__ bool entmax_short_row(EntmaxRow<D, E>& w, f32x16* oacc)
{
    constexpr int NS = 3, TILE = kBN * D, NLOAD = EntmaxRow<D, E>::NLOAD;
    const uint16_t* tiles = w.m.tiles;
    const int ne = w.ne;
    const int start_l = w.lane < ne ? w.first_key(w.t0 + w.lane) : 0;   // lane e: first key of entry e
    uint32_t word[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        word[e] = 0;
        if (e < ne) word[e] = w.visible(w.raw_word(w.t0 + e), __builtin_amdgcn_readlane(start_l, e));
    }
    if (w.use_sched)
        for (int e = w.wave; e < ne; e += 4) w.m.cols[e][w.lane] = w.cols[(size_t)(w.t0 + e) * 64 + w.lane];
    __syncthreads();
    uint32_t live = 0;                                       // bit e: this quarter of entry e keeps something
#pragma unroll
    for (int e = 0; e < E; ++e) live |= __ballot(word[e] != 0) != 0 ? 1u << e : 0u;

    // The tiles arrive through a ring: K of entry 0, 1, .., then V of entry 0, 1, ..
    const int items = 2 * ne;
    auto issue_item = [&](int item, int place) {
        if (item >= items) return;
        const bool is_v = item >= ne;
        const int e = is_v ? item - ne : item;
        const int k0 = __builtin_amdgcn_readlane(start_l, e);
        int gk[NLOAD];
        if (k0 < 0)
#pragma unroll
            for (int u = 0; u < NLOAD; ++u) gk[u] = w.m.cols[e][w.load_row(u)];
        if (is_v) w.template issue<true>(true, place, k0, gk);
        else w.template issue<true>(false, place, k0, gk);
    };
    int item = 0, place = 0;
    // item `item` is there for everybody; the place before its own is free and takes item + 2
    auto next_item = [&]() {
        if (item + 1 < items) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NLOAD) : "memory");
        else wait_vmem();
        __syncthreads();
        issue_item(item + 2, place >= 1 ? place - 1 : NS - 1);
    };
    auto advance = [&]() {
        ++item;
        place = place + 1 == NS ? 0 : place + 1;
    };
    issue_item(0, 0);
    issue_item(1, 1);

    f32x16 y[E];
    float m = -INFINITY;
    {
        bf16x8 qreg[EntmaxRow<D, E>::KSTEPS];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e >= ne) continue;
            next_item();
            if (e == 0) read_operand<D>(tiles + NS * TILE, w.brow, w.k_swz, qreg);
            if ((live >> e) & 1u) {
                product_32<D>(tiles + place * TILE, w.kh * 32 + w.n, w.k_swz, qreg, y[e]);
                w.mask_scores(word[e], y[e]);
#pragma unroll
                for (int i = 0; i < 16; ++i) m = fmaxf(m, y[e][i]);
            }
            advance();
        }
    }
    w.set_max(m);
#pragma unroll
    for (int e = 0; e < E; ++e)
        if ((live >> e) & 1u)
#pragma unroll
            for (int i = 0; i < 16; ++i) y[e][i] = fmaf(y[e][i], w.c, -w.mc);

    // Newton steps (relative to the row maximum the root lies in [-1, 0)) until every row has its tau
    bool done = w.empty;
    for (int iter = 0; iter < kEntmaxMaxIter; ++iter) {
        const bool pend = __ballot(!done) != 0;
        const int now = w.par;
        if (w.lane == 0) w.m.pend[now][w.wave] = pend ? 1u : 0u;
        float g1 = 0.f, g2 = 0.f;
        if (pend)
#pragma unroll
            for (int e = 0; e < E; ++e)
                if ((live >> e) & 1u)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float d = above(y[e][i], w.tau);
                        g1 += d;
                        g2 = fmaf(d, d, g2);
                    }
        const float4 x = w.exchange(both_halves_sum(g1), both_halves_sum(g2));
        const uint4 p = *reinterpret_cast<const uint4*>(w.m.pend[now]);
        if ((p.x | p.y | p.z | p.w) == 0) break;
        w.newton_step(x.x + x.z, x.y + x.w, false, done);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e >= ne) continue;
        next_item();
        if ((live >> e) & 1u) {
#pragma unroll
            for (int i = 0; i < 16; ++i) y[e][i] = above(y[e][i], w.tau);
            w.add_tile(y[e], place, oacc);
        }
        advance();
    }
    w.set_psum();
    return !w.left_too_much();
}

// Any number of entries: the scores of the first HL stay in registers, those of the others are formed again in every
// sweep.  `confirm`: no Newton step is the last one before its result has been looked at.
template <int D, int HL, int E>
__device__ __forceinline__ void entmax_long_row(EntmaxRow<D, E>& w, f32x16* oacc, bool confirm)
{
    constexpr int TILE = kBN * D, NLOAD = EntmaxRow<D, E>::NLOAD;
    uint16_t* tiles = w.m.tiles;
    const int t_end = w.t0 + w.ne, t_begin = w.t0 + HL;
    // First keys of entries: 64 at a time are kept in a register, one per lane, so that nothing but words and tiles is
    // loaded for an entry that is not gathered.  (Loaded in every sweep together with gather keys: rows of 24 entries
    // D64 263 us, 248 so; 1000 keys in 16 entries D32 111, 104.)
    int start_l = 0, window = -1;
    auto first_keys = [&](int e, int* k0) {                  // of entries e, e + 1 of the block row (e even)
        if (__builtin_expect(e >> 6 != window, 0)) {
            window = e >> 6;
            start_l = w.first_key(w.t0 + min(64 * window + w.lane, w.ne - 1));
            asm volatile("" : "+v"(start_l));                // waited for here and not where the branch ends
        }
        k0[0] = __builtin_amdgcn_readlane(start_l, e & 63);
        k0[1] = __builtin_amdgcn_readlane(start_l, (e & 63) + 1);
    };
    bf16x8 qreg[EntmaxRow<D, E>::KSTEPS];
    wait_vmem();
    __syncthreads();                                         // Q rows have landed
    read_operand<D>(tiles + 3 * TILE, w.brow, w.k_swz, qreg);

    // Two entries per step, so that a wavefront has two chains of matrix instructions and a barrier serves both;
    // body(scores, which).  Without V: two pairs of places (that of the Q rows is free now), the next K tiles travel
    // while the current ones are used.  With V (last sweep): K in the first pair, V in the second.
    auto sweep = [&](auto with_v_, auto&& body) {
        constexpr bool with_v = decltype(with_v_)::value;
        // gather keys and words of the entries after those on their way, one step ahead
        int start[2] = {0, 0}, key[2] = {0, 0};
        uint32_t fetched[2] = {0, 0}, ahead[2] = {0, 0};
        auto fetch = [&](int t) {
            first_keys(t - w.t0, start);                     // (of the last entry again if there is one left)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int tt = min(t + j, t_end - 1);
                if (start[j] < 0) key[j] = w.cols[(size_t)tt * 64 + w.lane];
                fetched[j] = w.raw_word(tt);
            }
        };
        auto issue = [&](int t, int to) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k0 = start[j];
                ahead[j] = t + j < t_end ? w.visible(fetched[j], k0) : 0;
                if (t + j >= t_end) continue;
                int gk[NLOAD];
                if (k0 < 0)
#pragma unroll
                    for (int u = 0; u < NLOAD; ++u) gk[u] = __shfl(key[j], w.load_row(u), 64);
                w.template issue<with_v>(false, 2 * to + j, k0, gk);
                if (with_v) w.template issue<true>(true, 2 + j, k0, gk);
            }
        };
        if (t_begin >= t_end) return;
        fetch(t_begin);
        __syncthreads();                                     // what was there is consumed
        if (!with_v) {
            issue(t_begin, 0);
            if (t_begin + 2 < t_end) fetch(t_begin + 2);
        }
        int to = 0;
        for (int t = t_begin; t < t_end; t += 2) {
            if (with_v) {
                __syncthreads();                             // the previous tiles are consumed
                issue(t, 0);
                if (t + 2 < t_end) fetch(t + 2);
            }
            wait_vmem();
#pragma unroll
            for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(key[j]), "+v"(fetched[j]));
            const uint32_t word[2] = {ahead[0], ahead[1]};
            __syncthreads();
            if (!with_v && t + 2 < t_end) {
                issue(t + 2, to ^ 1);
                if (t + 4 < t_end) fetch(t + 4);
            }
            const bool some0 = __ballot(word[0] != 0) != 0, some1 = __ballot(word[1] != 0) != 0;
            const uint16_t* base = tiles + 2 * to * TILE;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (j ? some1 : some0) {
                    f32x16 x;
                    product_32<D>(base + j * TILE, w.kh * 32 + w.n, w.k_swz, qreg, x);
                    w.mask_scores(word[j], x);
                    body(x, j);
                }
            if (!with_v) to ^= 1;
        }
    };
    // tiles of held entries e, e + 1 into the first two places
    auto bring = [&](int e, bool v) {
        __syncthreads();                                     // what was there is consumed
        int start[2];
        first_keys(e, start);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = w.t0 + e + j, k0 = start[j];
            int gk[NLOAD];
            if (k0 < 0)
#pragma unroll
                for (int u = 0; u < NLOAD; ++u) gk[u] = w.cols[(size_t)t * 64 + w.load_row(u)];
            w.template issue<true>(v, j, k0, gk);
        }
        wait_vmem();
        __syncthreads();
    };
    f32x16 y[HL > 0 ? HL : 1];
    uint32_t live = 0;                                       // bit e: this quarter of held entry e keeps something
    float m = -INFINITY;
#pragma unroll
    for (int e = 0; e < HL; ++e) {
        if (e % 2 == 0) bring(e, false);
        const uint32_t word = w.visible(w.raw_word(w.t0 + e), __builtin_amdgcn_readlane(start_l, e));
        if (__ballot(word != 0) == 0) continue;
        live |= 1u << e;
        product_32<D>(tiles + e % 2 * TILE, w.kh * 32 + w.n, w.k_swz, qreg, y[e]);
        w.mask_scores(word, y[e]);
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, y[e][i]);
    }
    sweep(Flag<false>{}, [&](const f32x16& x, int) {
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, x[i]);
    });
    w.set_max(m);
#pragma unroll
    for (int e = 0; e < HL; ++e)
        if ((live >> e) & 1u)
#pragma unroll
            for (int i = 0; i < 16; ++i) y[e][i] = fmaf(y[e][i], w.c, -w.mc);
    bool done = w.empty;
    for (int iter = 0; iter < kEntmaxMaxIter; ++iter) {
        if (__syncthreads_or(done ? 0 : 1) == 0) break;
        float g1 = 0.f, g2 = 0.f;
        auto add = [&](float d) {
            g1 += d;
            g2 = fmaf(d, d, g2);
        };
        sweep(Flag<false>{}, [&](const f32x16& x, int) {
#pragma unroll
            for (int i = 0; i < 16; ++i) add(above(fmaf(x[i], w.c, -w.mc), w.tau));
        });
#pragma unroll
        for (int e = 0; e < HL; ++e)
            if ((live >> e) & 1u)
#pragma unroll
                for (int i = 0; i < 16; ++i) add(above(y[e][i], w.tau));
        const float4 x = w.exchange(both_halves_sum(g1), both_halves_sum(g2));
        w.newton_step(x.x + x.z, x.y + x.w, confirm, done);
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    w.psum = 0.f;
#pragma unroll
    for (int e = 0; e < HL; ++e) {
        if (e % 2 == 0) bring(e, true);
        if ((live >> e) & 1u) {
#pragma unroll
            for (int i = 0; i < 16; ++i) y[e][i] = above(y[e][i], w.tau);
            w.add_tile(y[e], e % 2, oacc);
        }
    }
    sweep(Flag<true>{}, [&](f32x16& x, int which) {
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = above(fmaf(x[i], w.c, -w.mc), w.tau);
        w.add_tile(x, 2 + which, oacc);
    });
    w.set_psum();
}

// E entries of a short row, the first HL of a longer one are held; W wavefronts per SIMD.  The leading arguments repeat
// fields of `a` (p_cnt and p_cols null: the layout's tiles); they arrive in registers when a wavefront starts.
template <int D, int E, int HL, int W>
__global__ __launch_bounds__(256, W) void entmax15_fwd_kernel(
    const int32_t* __restrict__ p_row_ptr, const int32_t* __restrict__ p_cnt, const int32_t* __restrict__ p_starts,
    const int32_t* __restrict__ p_cols, const uint32_t* __restrict__ p_words, int nQB, int total, int p_H, FwdArgs a,
    float* tau_out)
{
    static_assert(HL <= E && HL % 2 == 0, "a longer row has the entries that are held, two of them per step");
    __shared__ __attribute__((aligned(1024))) EntmaxLds<D, E> mem;
    const int blk = block_index();
    if (blk >= total) return;
    const int bid = xcd_contiguous(blk, total);
    const int qb = nQB - 1 - (bid % nQB);                    // long causal rows first
    const int h = (bid / nQB) % p_H;
    const int b = bid / (nQB * p_H);
    const int r = h * nQB + qb;
    const int t0 = p_row_ptr[r];
    int ne = p_cnt ? p_cnt[r] : p_row_ptr[r + 1] - t0;
    const int tid = threadIdx.x;
    auto load_q = [&]() {                                    // (the last row again beyond Lq)
        constexpr int RPI = EntmaxRow<D, E>::RPI;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        const uint16_t* Qp = (const uint16_t*)a.Q + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
        lds_u16* dst = (lds_u16*)mem.tiles + 3 * kBN * D;
#pragma unroll
        for (int u = 0; u < EntmaxRow<D, E>::NLOAD; ++u) {
            const int r = (wave + 4 * u) * RPI + lane / (D / 8);
            load16_to_lds(lds_addr_of(dst + (wave + 4 * u) * 512),
                          Qp + (long long)min(qb * 64 + r, a.Lq - 1) * a.sq[2] + ((lane % (D / 8)) ^ swz_u<D>(r)) * 8);
        }
    };
    load_q();
    if (!p_cnt && a.causal) {                                // columns ascend: hidden tiles are at the end
        const long long block_diag = (long long)qb * 64 + 63 + a.Lk - a.Lq;
        while (ne > 0 && (long long)p_starts[t0 + ne - 1] * kBN > block_diag) --ne;
    }
    f32x16 oacc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    EntmaxRow<D, E> w(a, mem, tid, b, h, qb, t0, ne, p_starts, p_cols, p_words);
    // What the other ways need they form anew from an index that the compiler takes for another one, so that
    // nothing of theirs stays in registers on the first one.
    auto other_view = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        EntmaxRow<D, E> v(a, mem, t, b, h, qb, t0, ne, p_starts, p_cols, p_words);
        v.par = w.par;
        v.tau = w.tau;
        return v;
    };
    auto take_over = [&](const EntmaxRow<D, E>& v) {
        w.tau = v.tau;
        w.mc = v.mc;
        w.psum = v.psum;
        w.empty = v.empty;
        w.par = v.par;
    };
    bool fine;
    if (ne <= E) {
        fine = entmax_short_row<D, E>(w, oacc);
    } else {
        EntmaxRow<D, E> v = other_view();
        entmax_long_row<D, HL>(v, oacc, false);
        take_over(v);
        fine = !v.left_too_much();
    }
    // An unconfirmed step that left too much: once more, every step confirmed.
    if (__builtin_expect(!fine, 0)) {
        EntmaxRow<D, E> v = other_view();
        load_q();                                            // their place may have been used
        entmax_long_row<D, 0>(v, oacc, true);
        take_over(v);
    }
    const float inv = (!w.empty && w.psum > 0.f) ? 1.0f / w.psum : 0.f;
    wait_vmem();                                             // without entries nobody has waited for the Q rows
    __syncthreads();                                         // all wavefronts are done with the tiles
    const int row0 = qb * 64 + w.qh * 32;
    uint16_t* Op = (uint16_t*)a.O + (size_t)b * a.so[0] + (size_t)h * a.so[1];
    store_key_halves<D>(mem.tiles, oacc, w.wave, w.lane, inv, Op + (size_t)row0 * a.so[2], a.so[2], a.Lq - row0);
    if (tau_out && w.hh == 0 && w.kh == 0 && row0 + w.n < a.Lq)
        tau_out[((size_t)b * a.H + h) * a.Lq + row0 + w.n] = w.empty ? INFINITY : w.mc + w.tau;
}

template <int D, int E, int HL, int W>
hipError_t launch(const FwdArgs& a, float* tau_out, hipStream_t stream)
{
    const int nQB = (a.Lq + 63) / 64, total = a.B * a.H * nQB;
    const bool sched = a.sched.cnt != nullptr;
    hipLaunchKernelGGL((entmax15_fwd_kernel<D, E, HL, W>), grid_of(total, 256), dim3(256), 0, stream, a.row_ptr, a.sched.cnt,
                       sched ? a.sched.start : a.col_idx, sched ? a.sched.cols : nullptr,
                       (const uint32_t*)(sched ? a.sched.bitmaps : a.bitmaps), nQB, total, a.H, a, tau_out);
    return hipGetLastError();
}

// No block row has more entries than there are key tiles.  Registers go into entries held or into a third wavefront per
// SIMD.  With up to two tiles two entries are all there is, and a fourth wavefront fits (the same at D = 32: B256 H8 40 x 40
// 20.7 us with room for six entries, 16.5 with two).  At D = 64 with up to six tiles every row fits either way (16 x 12 x
// 330, all tiles full: 42 us with two wavefronts, 32 with three); with seven or eight only two wavefronts hold them all
// (500: 60 against 92).  Beyond that it is
// the rows that decide, and they are not known here.  Two wavefronts (512 workgroups at a time) against three (768), 8 heads of
// 1024 keys with block rows of 3, of 6 to 8 and of 16 entries, us:
//   512 workgroups    11.7 / 11.3    17.1 / 27.2    58 / 67        one round of either
//   640               19.5 / 13.0    28.1 / 31.5    98 / 83        two rounds against one
//   1024              22.0 / 20.5    32.1 / 45.8   118 / 124       two of either
//   2048              42.4 / 32.8    60 / 74       231 / 217       four against three
// So the entries are held up to 1024 workgroups, at a price between 513 and 768.
hipError_t launch_64(const FwdArgs& a, float* tau_out, hipStream_t stream)
{
    const int tiles = (a.Lk + 63) / 64;
    const long long workgroups = (long long)a.B * a.H * ((a.Lq + 63) / 64);
    if (tiles <= 2) return launch<64, 2, 0, 4>(a, tau_out, stream);
    if (tiles <= 6) return launch<64, 6, 0, 3>(a, tau_out, stream);
    if (tiles <= 8 || workgroups <= 1024) return launch<64, 8, 6, 2>(a, tau_out, stream);
    return launch<64, 5, 2, 3>(a, tau_out, stream);
}

}  // namespace

hipError_t launch_entmax15_fwd(const FwdArgs& a, float* tau_out, hipStream_t stream)
{
    switch (a.D) {
        case 32:
            if (a.Lk <= 128) return launch<32, 2, 0, 4>(a, tau_out, stream);   // as in launch_64
            return launch<32, 6, 4, 3>(a, tau_out, stream);
        case 64: return launch_64(a, tau_out, stream);
        case 128: return launch<128, 8, 4, 2>(a, tau_out, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ap
