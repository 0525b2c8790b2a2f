// Backward pass over visit schedules: the same arithmetic as ap_attn_bwd.hip, but dQ walks the
// entries of the row schedule (runs of 64 consecutive keys or 64 gathered keys per block row) and
// dK, dV walk the entries of the column schedule (runs of 64 consecutive queries or 64 gathered
// queries per block column), so the backward pass skips what the forward pass skips.  Causal
// limits are folded into the entry bitmaps by the schedule builders.
//
// One workgroup of four wavefronts per block row (dQ) or block column (dK, dV); a wavefront forms the
// scores of one 32 x 32 quarter of every entry.  Every tile is stored once in LDS, with a swizzle that
// suits both the row-wise reads (scores) and the transposing reads (gradient products).  Two LDS
// stages: the next entry's tiles travel while the current entry is computed; the metadata of the entry
// after that (start, gather indices, bitmap words, per-query statistics) is fetched into registers in
// the same step.
//
// What bounds these kernels is the issue of instructions around the matrix work, so what counts is a
// second wavefront on every SIMD, i.e. at most 256 registers at D = 128.  Two wavefronts per workgroup
// that each formed a 32 x 64 half and, for dK and dV, kept both accumulators needed 314 (dQ) and 393 of
// them: one wavefront per SIMD, every wait exposed.  A quarter per wavefront and
//   dQ      partial sums over the two key halves, added at the end,
//   dK, dV  accumulators divided by what they hold (one wavefront of a pair sums dV over both query
//           halves, the other dK) with the probabilities or score gradients that the partner needs
//           handed over through LDS in bf16, the precision the products use anyway,
// fit.  B4 H16 L4096 D128, 10 % kept: dQ 229 -> 175 us (29 of the 229 a pass of its own for delta), dK and dV
// 269 -> 230 us; B4 H16 L2048 218 -> 156 us in all.  Of a dQ workgroup's 20 us there, 7 pass before its first
// entry (a chain of cold loads), 1.5 per entry, 2 in the sum over key halves and the store; of a dK, dV
// workgroup's 27 us 5.4, 2.4 per entry and 1.5.  Inside an entry the LDS pipe is busy about 70 % of the time.
// Timed in parts there (dQ / dK, dV, of 174 / 216 us): loads and barriers alone 131 / 138, no entry at all 85 / 74
// (402 MB read and written once are 80 at the rate of a large copy), no score products 149 / 185, no gradient
// products 155 / 171.  With the next entry's tiles waited for behind the products of this one dQ takes 154 (beside 213 for
// dK, dV), a call 337 us instead of 349.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"
#include "ap_mfma_common.h"

namespace ap {

namespace {

using namespace mfma;

// What the kernels compute per entry.  SOFTMAX: P = exp(s - lse), dS = P (dP - delta) with the
// per-query statistics lse and delta = <dO, O>.  ENTMAX15 (the 1.5-entmax normaliser of Section 6):
// u = [s / 2 - tau]_+, P = u^2, dS = u (dP - gbar) with the per-query statistics tau (from the
// forward pass) and gbar = sum_j u_j dP_j / sum_j u_j: the dQ kernel walks a block row's entries twice, first for
// gbar (two products of three), then for dQ.  There BwdArgs::lse holds tau and BwdArgs::delta gets gbar.  (The
// first walk as a launch of its own: B4 H16 L2048 D128 40 us + 52 for dQ, 72 in one; 3 heads of 5000 x 9000 D64 89 + 143 us, both
// still waiting for their tiles before the products, 165 in one.)
enum { SOFTMAX = 0, ENTMAX15 = 1 };

template <int N> struct Int {
    static constexpr int value = N;
};

__device__ __forceinline__ float lse2_of(float lse) { return lse == -INFINITY ? INFINITY : lse * kLog2e; }

// The leading arguments repeat fields of `a`: they arrive in registers when a wavefront starts
// (kernel-argument preloading), so the chain row pointer -> entry -> tiles starts at once.
template <int D, int MODE>
__global__ __launch_bounds__(256, 2) void bwd_dq_sched_kernel(
    const int32_t* __restrict__ p_row_ptr, const int32_t* __restrict__ p_cnt, const int32_t* __restrict__ p_start,
    const int32_t* __restrict__ p_cols, const uint32_t* __restrict__ p_words, int nQB, int p_B, int n_blocks, BwdArgs a)
{
    constexpr int TILE = kBN * D;
    constexpr int KSTEPS = D / 16;
    constexpr int DBLK = D / 32;
    constexpr int RPI = 64 / (D / 8);
    constexpr int NLOAD = (D / 8) / 4;
    constexpr int STAGE = 2 * TILE;                          // K rows, V rows
    __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * STAGE];
    __shared__ float s_pair[2][2][64];                       // sums that the two key halves of a query add up
    lds_u16* lds = (lds_u16*)smem;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = lane & 31, hh = lane >> 5;
    const int qh = wave & 1, kh = wave >> 1;                 // this wavefront's quarter of every entry
    const int g_row = lane / (D / 8);
    // A zero the compiler cannot see through.  Indexing with it turns the per-entry load of a
    // start into a vector load: a scalar load inside the loop would make every later wait for an
    // LDS read (same counter, scalar loads return out of order) wait for memory as well.
    int vzero = 0;
    asm volatile("" : "+v"(vzero));

    const int blk = block_index();
    if (blk >= n_blocks) return;
    const int bid = xcd_contiguous(blk, n_blocks);
    const int qb = nQB - 1 - (bid % nQB);
    const int b = (bid / nQB) % p_B;                         // the examples of a head one after another: they share its schedule
    const int h = bid / (nQB * p_B);
    const int r = h * nQB + qb;
    const int t0 = p_row_ptr[r];
    const int t1 = t0 + p_cnt[r];

    const uint16_t* Qp = (const uint16_t*)a.Q + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    const uint16_t* Gp = (const uint16_t*)a.dO + (size_t)b * a.so[0] + (size_t)h * a.so[1];
    const uint16_t* Kp = (const uint16_t*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1];
    const uint16_t* Vp = (const uint16_t*)a.V + (size_t)b * a.sv[0] + (size_t)h * a.sv[1];
    const int sq_bytes = (int)a.sq[2] * 2, so_bytes = (int)a.so[2] * 2;
    const rsrc_t q_rsrc = make_rsrc(Qp, (unsigned)((a.Lq - 1) * sq_bytes + D * 2));
    const rsrc_t g_rsrc = make_rsrc(Gp, (unsigned)((a.Lq - 1) * so_bytes + D * 2));
    uint16_t* dQp = (uint16_t*)a.dQ + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    const int sk_bytes = (int)a.sk[2] * 2, sv_bytes = (int)a.sv[2] * 2;
    const rsrc_t k_rsrc = make_rsrc(Kp, (unsigned)((a.Lk - 1) * sk_bytes + D * 2));
    const rsrc_t v_rsrc = make_rsrc(Vp, (unsigned)((a.Lk - 1) * sv_bytes + D * 2));

    const int brow = qh * 32 + n;
    const int qrow = qb * 64 + brow;
    const bool row_ok = qrow < a.Lq;

    // metadata of an entry: where it starts (or -1), gather key `lane` (read for every entry,
    // used by gathered ones only) and this lane's half of its bitmap word: three loads per entry
    struct Meta {
        int start;
        int key;
        uint32_t word;
    };
    auto fetch = [&](int t, Meta& m) {
        m.start = p_start[t + vzero];                        // a vector load: see vzero
        m.key = p_cols[(size_t)t * 64 + lane];
        m.word = p_words[((size_t)t * 64 + brow) * 2 + kh];
    };
    auto issue = [&](const Meta& m, int stage) {
        lds_u16* base = lds + stage * STAGE;
        const int start = __builtin_amdgcn_readfirstlane(m.start);
        if (start >= 0) {
            issue_tile_loads<D, 4, SWZ_BOTH>(k_rsrc, base, start, sk_bytes, wave, lane);
            issue_tile_loads<D, 4, SWZ_BOTH>(v_rsrc, base + TILE, start, sv_bytes, wave, lane);
        } else {
            int gk[NLOAD];                                   // keys of the rows this lane loads
#pragma unroll
            for (int u = 0; u < NLOAD; ++u) gk[u] = __shfl(m.key, (wave + 4 * u) * RPI + g_row, 64);
            issue_gather_loads<D, 4, SWZ_BOTH>(k_rsrc, base, gk, sk_bytes, wave, lane);
            issue_gather_loads<D, 4, SWZ_BOTH>(v_rsrc, base + TILE, gk, sv_bytes, wave, lane);
        }
    };

    // A first entry of 64 consecutive keys is requested before anything else: its start is a scalar load, so this waits for
    // no vector load.
    const int start0 = t0 < t1 ? p_start[t0] : -1;
    // step i of the walks is entry i % (t1 - t0)
    constexpr int WALKS = MODE == ENTMAX15 ? 2 : 1;
    const int n_entries = t1 - t0, steps = WALKS * n_entries;
    auto entry_of = [&](int i) { return t0 + (WALKS > 1 && i >= n_entries ? i - n_entries : i); };
    Meta cur, nxt;
    cur.start = start0;
    cur.key = 0;
    cur.word = 0;
    if (start0 >= 0) issue(cur, 0);
    if (t0 < t1) fetch(t0, cur);
    // Q and dO rows of the block row (rows >= Lq read as zeros) into the second stage
    issue_tile_loads<D, 4, SWZ_BOTH>(q_rsrc, lds + STAGE, qb * 64, sq_bytes, wave, lane);
    issue_tile_loads<D, 4, SWZ_BOTH>(g_rsrc, lds + STAGE + TILE, qb * 64, so_bytes, wave, lane);
    const size_t stat_base = ((size_t)b * a.H + h) * a.Lq;
    // SOFTMAX: log-sum-exp; ENTMAX15: tau (+inf for a query without keys).  Loaded for every
    // lane and looked at later: a branch on the row would wait here, before the first tile is requested.
    float lse2 = a.lse[stat_base + (row_ok ? qrow : a.Lq - 1)];
    float delta = 0.f;                                       // ENTMAX15: gbar, from the second walk on
    // delta = <dO, O> is formed here, where dO is at hand (a pass of its own reads dO once more).  The dK, dV
    // kernel reads it from memory.
    constexpr int CPR = D / 8, NO = 64 * CPR / 256;          // 16-byte pieces of a row; pieces of O per thread
    uint4 o[NO];
    if (MODE == SOFTMAX) {
        const uint16_t* Op = (const uint16_t*)a.O + (size_t)b * a.so[0] + (size_t)h * a.so[1];
#pragma unroll
        for (int u = 0; u < NO; ++u) {
            const int idx = u * 256 + tid, row = min(qb * 64 + idx / CPR, a.Lq - 1);
            o[u] = *reinterpret_cast<const uint4*>(Op + (size_t)row * a.so[2] + idx % CPR * 8);
        }
    }
    nxt = cur;
    if (t0 < t1) {
        if (start0 < 0) issue(cur, 0);
        if (WALKS > 1 || t0 + 1 < t1) fetch(entry_of(1), nxt);
    }
    const float sc = MODE == SOFTMAX ? a.scale * kLog2e : a.scale * 0.5f;
    float num = 0.f, den = 0.f;                              // first walk: this lane's share of sum u dP and sum u
    const int k_row = kh * 32 + n;
    const int k_swz = hh ^ swz_u<D>(n);
    const TrReadU<D> tr = make_tr_read_u<D>(lane);

    f32x16 dqacc[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dqacc[db][i] = 0.f;

    // everything has landed here, so that no wait for loaded registers lands inside the loop
    wait_vmem();
    asm volatile("" : "+v"(lse2), "+v"(delta));
    __syncthreads();
    bf16x8 qreg[KSTEPS], greg[KSTEPS];                       // Q^T and dO^T operands
    read_operand<D>(smem + STAGE, brow, k_swz, qreg);
    read_operand<D>(smem + STAGE + TILE, brow, k_swz, greg);
    lse2 = row_ok ? (MODE == SOFTMAX ? lse2_of(lse2) : lse2) : INFINITY;
    if (MODE == SOFTMAX) {
#pragma unroll
        for (int u = 0; u < NO; ++u) {
            const int idx = u * 256 + tid, row = idx / CPR, c = idx % CPR;
            const uint4 g4 = *reinterpret_cast<const uint4*>(smem + STAGE + TILE + row * D + (c ^ swz_u<D>(row)) * 8);
            const uint32_t ow[4] = {o[u].x, o[u].y, o[u].z, o[u].w}, gw[4] = {g4.x, g4.y, g4.z, g4.w};
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                d = fmaf(__uint_as_float(ow[k] << 16), __uint_as_float(gw[k] << 16), d);
                d = fmaf(__uint_as_float(ow[k] & 0xffff0000u), __uint_as_float(gw[k] & 0xffff0000u), d);
            }
            d = group_sum<CPR>(d);
            if (c == 0) {
                s_pair[0][0][row] = d;
                if (qb * 64 + row < a.Lq) a.delta[stat_base + qb * 64 + row] = d;
            }
        }
        __syncthreads();
        delta = s_pair[0][0][brow];
    }

    auto set_gbar = [&]() {                                  // half-wavefronts and key halves hold different keys
        num += __shfl_xor(num, 32, 64);
        den += __shfl_xor(den, 32, 64);
        if (hh == 0) {
            s_pair[kh][0][brow] = num;
            s_pair[kh][1][brow] = den;
        }
        __syncthreads();
        num = s_pair[0][0][brow] + s_pair[1][0][brow];
        den = s_pair[0][1][brow] + s_pair[1][1][brow];
        delta = den > 0.f ? num / den : 0.f;
        if (row_ok && hh == 0 && kh == 0) a.delta[stat_base + qrow] = delta;
    };
    int stage = 0;
    // steps first .. last - 1: the gradient (GRAD), the first walk (SUMS), or both, the second after the first (ALL)
    enum { GRAD, SUMS, ALL };
    auto walk = [&](int first, int last, auto what_) {
        constexpr int WHAT = decltype(what_)::value;
        for (int i = first; i < last; ++i) {
            __syncthreads();                                 // this entry has landed for everybody; the other stage is free
            const uint32_t word = cur.word;
            if (i + 1 < steps) issue(nxt, stage ^ 1);
            // (of the last entry again at the end: behind a branch the compiler copies what is fetched, and so waits for it and
            // for the tiles before the products: 1.5-entmax, 3 heads of 5000 x 9000 D64, 165 us for both walks, 260 so)
            Meta after;
            fetch(entry_of(min(i + 2, steps - 1)), after);
            int sums = WHAT == SUMS;
            if (WHAT == ALL) {
                sums = i < n_entries;
                asm volatile("" : "+v"(sums));               // one loop (D = 128: addresses for two do not fit)
                if (i == n_entries) set_gbar();
                sums = __builtin_amdgcn_readfirstlane(sums);
            }
            if (__ballot(word != 0) != 0) {
                uint16_t* base = smem + stage * STAGE;
                f32x16 s, p;
                two_products_32<D>(base, base + TILE, k_row, k_swz, qreg, greg, s, p);   // S^T = K Q^T, dP^T = V dO^T
                const int wbits = (int)(word >> (4 * hh));
                if (MODE == ENTMAX15) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) {           // u, pruned: 0
                        const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(wbits, 8 * (k / 4) + (k % 4), 1);
                        s[k] = fmaxf(__uint_as_float(__float_as_uint(fmaf(s[k], sc, -lse2)) & keep), 0.f);
                    }
                }
                if (sums) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        num = fmaf(s[k], p[k], num);
                        den += s[k];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        if (MODE == SOFTMAX) {
                            const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(wbits, 8 * (k / 4) + (k % 4), 1);
                            s[k] = __builtin_amdgcn_exp2f(or_minus_inf(fmaf(s[k], sc, -lse2), keep));
                        }
                        s[k] *= p[k] - delta;                // dS^T
                    }
                    bf16x8 pb[2];
                    to_operands(s, pb);
                    tr_mm_32<D>(lds + stage * STAGE + kh * 32 * D, pb, dqacc, tr);   // dQ^T += K^T dS^T
                }
            }
            stage ^= 1;
            wait_vmem();                                     // the next entry and the metadata of the one after it
            asm volatile("" : "+v"(after.start), "+v"(after.key), "+v"(after.word));
            cur = nxt;
            nxt = after;
        }
    };
    if constexpr (MODE == SOFTMAX) {
        walk(0, steps, Int<GRAD>{});
    } else if constexpr (D <= 64) {
        walk(0, n_entries, Int<SUMS>{});
        set_gbar();
        walk(n_entries, steps, Int<GRAD>{});
    } else {
        walk(0, steps, Int<ALL>{});
        if (n_entries == 0) set_gbar();                      // (0, which the dK, dV kernel does not look at)
    }
    __syncthreads();                                         // all wavefronts are done with the tiles
    const int row0 = qb * 64 + qh * 32;
    store_key_halves<D>(smem, dqacc, wave, lane, a.scale, dQp + (size_t)row0 * a.sq[2], a.sq[2], a.Lq - row0);
}

// A pair of wavefronts per 32 keys.  Wavefront `role` of it forms the scores of query half `role` of every
// entry; role 0 sums dV over both query halves, role 1 sums dK, and each hands the other what it needs of
// its own half: role 0 the score gradients, role 1 the probabilities.
template <int D, int NORM>
__global__ __launch_bounds__(256, 2) void bwd_dkv_sched_kernel(
    const int32_t* __restrict__ p_col_ptr, const int32_t* __restrict__ p_cnt, const int32_t* __restrict__ p_start,
    const int32_t* __restrict__ p_cols, const uint32_t* __restrict__ p_words, int nKB, int p_H, int p_B, int NP, BwdArgs a)
{
    constexpr int TILE = kBN * D;
    constexpr int KSTEPS = D / 16;
    constexpr int DBLK = D / 32;
    constexpr int RPI = 64 / (D / 8);
    constexpr int NLOAD = (D / 8) / 4;
    constexpr int STAGE = 2 * TILE;                          // Q rows, dO rows
    __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * STAGE];
    __shared__ __attribute__((aligned(16))) bf16x8 s_hand[4][2][64];     // what a wavefront hands its partner
    __shared__ __attribute__((aligned(16))) float s_stat[4][64];         // of its 32 queries: lse (or tau), delta (or gbar)
    __shared__ __attribute__((aligned(16))) uint32_t s_word[4][32];      // ... and words of kept keys, its half
    __shared__ uint32_t s_live[2][4];                        // does a wavefront's quarter hold anything?  by parity of the entry
    lds_u16* lds = (lds_u16*)smem;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = lane & 31, hh = lane >> 5;
    const int kh = wave & 1, role = wave >> 1;
    const int g_row = lane / (D / 8);
    // A zero the compiler cannot see through.  Indexing with it turns the per-entry load of a
    // start into a vector load: a scalar load inside the loop would make every later wait for an
    // LDS read (same counter, scalar loads return out of order) wait for memory as well.
    int vzero = 0;
    asm volatile("" : "+v"(vzero));

    // Which (example, head) pair and which position of the head's visiting order this workgroup
    // takes.  Every XCD gets a contiguous range of pairs (they share Q and dO rows in its L2); when
    // the pairs divide evenly over the 8 XCDs, the heavy columns of all pairs of the range come
    // first, so that the longest workgroups start at once, then the other columns pair by pair.
    const int blk = block_index();
    if (blk >= NP * nKB) return;
    const int32_t* order = p_cnt + (size_t)p_H * nKB;
    const int32_t* n_heavy = order + (size_t)p_H * nKB;
    int pair, idx;
    if (NP % 8 == 0 && NP / 8 <= 64) {
        // lane p looks at pair P0 + p: one load and two wave-wide prefix sums instead of a chain of
        // dependent scalar loads
        const int PP = NP / 8, P0 = (blk & 7) * PP;
        const int l = blk >> 3;
        const int hv = lane < PP ? n_heavy[(P0 + lane) / p_B] : 0;
        const int lt = lane < PP ? nKB - hv : 0;
        int hv_incl = hv, lt_incl = lt;                      // inclusive prefix sums over the lanes
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(hv_incl, o, 64), y = __shfl_up(lt_incl, o, 64);
            if (lane >= o) {
                hv_incl += x;
                lt_incl += y;
            }
        }
        const int hv_total = __shfl(hv_incl, 63, 64);
        const bool in_heavy = l < hv_total;
        const int ll = in_heavy ? l : l - hv_total;
        const int incl = in_heavy ? hv_incl : lt_incl, mine = in_heavy ? hv : lt;
        // the lane whose range [incl - mine, incl) holds ll
        const unsigned long long hit = __ballot(lane < PP && ll >= incl - mine && ll < incl);
        if (hit == 0) return;                                // cannot happen for grid = pairs x columns
        const int p = __ffsll((long long)hit) - 1;           // exactly one lane
        pair = P0 + p;
        idx = ll - (__shfl(incl, p, 64) - __shfl(mine, p, 64)) + (in_heavy ? 0 : __shfl(hv, p, 64));
        pair = __builtin_amdgcn_readfirstlane(pair);
        idx = __builtin_amdgcn_readfirstlane(idx);
    } else {
        const int bid = xcd_contiguous(blk, NP * nKB);
        pair = bid / nKB;
        idx = bid % nKB;
    }
    const int h = pair / p_B;                                // the examples of a head share its schedule
    const int b = pair % p_B;
    const int kb = order[(size_t)h * nKB + idx];
    const int c = h * nKB + kb;
    const int t0 = p_col_ptr[c];
    const int t1 = t0 + p_cnt[c];

    const uint16_t* Qp = (const uint16_t*)a.Q + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    const uint16_t* Gp = (const uint16_t*)a.dO + (size_t)b * a.so[0] + (size_t)h * a.so[1];
    const uint16_t* Kp = (const uint16_t*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1];
    const uint16_t* Vp = (const uint16_t*)a.V + (size_t)b * a.sv[0] + (size_t)h * a.sv[1];
    const int sq_bytes = (int)a.sq[2] * 2, so_bytes = (int)a.so[2] * 2;
    const rsrc_t q_rsrc = make_rsrc(Qp, (unsigned)((a.Lq - 1) * sq_bytes + D * 2));
    const rsrc_t g_rsrc = make_rsrc(Gp, (unsigned)((a.Lq - 1) * so_bytes + D * 2));
    const size_t stat_base = ((size_t)b * a.H + h) * a.Lq;

    // metadata of an entry: where it starts (or -1) and gathered query `lane` (read for every
    // entry, used by gathered ones only)
    struct Meta {
        int start;
        int row;
    };
    // statistics of this wavefront's 32 query slots of an entry, fetched one step ahead: lower lanes lse (or
    // tau) and the word of kept keys, upper lanes delta (or gbar)
    struct Stat {
        float v;
        uint32_t word;
    };
    const float* stat_src = (hh ? a.delta : a.lse) + stat_base;
    auto fetch = [&](int t, Meta& m) {
        m.start = p_start[t + vzero];                        // a vector load: see vzero
        m.row = p_cols[(size_t)t * 64 + lane];
    };
    auto fetch_stat = [&](int t, const Meta& m, Stat& s) {
        const int gathered = __shfl(m.row, role * 32 + n, 64);
        const int q = m.start >= 0 ? m.start + role * 32 + n : gathered;   // (all lanes hold the same start)
        const float v = stat_src[q < a.Lq ? q : a.Lq - 1];
        s.v = q < a.Lq ? v : (hh ? 0.f : (NORM == SOFTMAX ? -INFINITY : INFINITY));
        s.word = p_words[((size_t)t * 64 + role * 32 + n) * 2 + kh];
    };
    auto issue = [&](const Meta& m, int stage) {
        lds_u16* base = lds + stage * STAGE;
        const int start = __builtin_amdgcn_readfirstlane(m.start);
        if (start >= 0) {
            issue_tile_loads<D, 4, SWZ_BOTH>(q_rsrc, base, start, sq_bytes, wave, lane);
            issue_tile_loads<D, 4, SWZ_BOTH>(g_rsrc, base + TILE, start, so_bytes, wave, lane);
        } else {
            int gq[NLOAD];                                   // queries of the rows this lane loads
#pragma unroll
            for (int u = 0; u < NLOAD; ++u) gq[u] = __shfl(m.row, (wave + 4 * u) * RPI + g_row, 64);
            issue_gather_loads<D, 4, SWZ_BOTH>(q_rsrc, base, gq, sq_bytes, wave, lane);
            issue_gather_loads<D, 4, SWZ_BOTH>(g_rsrc, base + TILE, gq, so_bytes, wave, lane);
        }
    };

    // as in the dQ kernel
    const int start0 = t0 < t1 ? p_start[t0] : -1;
    Meta cur, nxt;
    cur.start = start0;
    cur.row = 0;
    Stat st;
    st.v = 0.f;
    st.word = 0;
    if (start0 >= 0) {
        issue(cur, 0);
        fetch_stat(t0, cur, st);
    } else if (t0 < t1) {
        fetch(t0, cur);
    }
    {   // K and V rows of the block column (rows >= Lk read as zeros) into the second stage
        const int sk_bytes = (int)a.sk[2] * 2, sv_bytes = (int)a.sv[2] * 2;
        issue_tile_loads<D, 4, SWZ_BOTH>(make_rsrc(Kp, (unsigned)((a.Lk - 1) * sk_bytes + D * 2)), lds + STAGE, kb * 64,
                                         sk_bytes, wave, lane);
        issue_tile_loads<D, 4, SWZ_BOTH>(make_rsrc(Vp, (unsigned)((a.Lk - 1) * sv_bytes + D * 2)), lds + STAGE + TILE,
                                         kb * 64, sv_bytes, wave, lane);
    }
    const float sc = NORM == SOFTMAX ? a.scale * kLog2e : a.scale * 0.5f;
    const int q_tile_row = role * 32 + n;
    const int k_swz = hh ^ swz_u<D>(n);
    const TrReadU<D> tr = make_tr_read_u<D>(lane);

    f32x16 acc[DBLK];                                        // role 0: dV^T, role 1: dK^T
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;

    nxt = cur;
    if (t0 < t1) {
        if (start0 < 0) {
            issue(cur, 0);
            fetch_stat(t0, cur, st);
        }
        if (t0 + 1 < t1) fetch(t0 + 1, nxt);
    }
    wait_vmem();
    __syncthreads();
    bf16x8 kreg[KSTEPS], vreg[KSTEPS];                       // K^T and V^T operands
    read_operand<D>(smem + STAGE, kh * 32 + n, k_swz, kreg);
    read_operand<D>(smem + STAGE + TILE, kh * 32 + n, k_swz, vreg);

    int stage = 0;
    for (int t = t0; t < t1; ++t) {
        wait_vmem();                                         // entry t, its statistics and the metadata of t + 1
        // read and written by this wavefront only: LDS order is all they need
        s_stat[wave][lane] = NORM == SOFTMAX && hh == 0 ? lse2_of(st.v) : st.v;
        if (hh == 0) s_word[wave][n] = st.word;
        const bool live = __ballot(st.word != 0) != 0;
        if (lane == 0) s_live[stage][wave] = live ? 1u : 0u;
        __syncthreads();                                     // entry t is there for everybody; the other stage is free
        if (t + 1 < t1) {
            issue(nxt, stage ^ 1);
            fetch_stat(t + 1, nxt, st);
            if (t + 2 < t1) fetch(t + 2, nxt);
        }
        uint16_t* base = smem + stage * STAGE;
        // the tile that this wavefront's gradient is a product of: dO for dV, Q for dK
        lds_u16* grad_tile = lds + stage * STAGE + (role ? 0 : TILE);
        if (live) {
            f32x16 s, p;
            two_products_32<D>(base, base + TILE, q_tile_row, k_swz, kreg, vreg, s, p);   // S = Q K^T, dP = dO V^T
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r0 = 8 * g + 4 * hh;               // 4 consecutive query slots
                const float4 l4 = *reinterpret_cast<const float4*>(&s_stat[wave][r0]);
                const float4 d4 = *reinterpret_cast<const float4*>(&s_stat[wave][32 + r0]);
                const uint4 w4 = *reinterpret_cast<const uint4*>(&s_word[wave][r0]);
                const float le[4] = {l4.x, l4.y, l4.z, l4.w}, de[4] = {d4.x, d4.y, d4.z, d4.w};
                const uint32_t we[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * g + e;
                    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)we[e], n, 1);
                    const float x = fmaf(s[i], sc, -le[e]);
                    if (NORM == SOFTMAX) {
                        s[i] = __builtin_amdgcn_exp2f(or_minus_inf(x, keep));   // P
                        p[i] = s[i] * (p[i] - de[e]);        // dS
                    } else {
                        const float u = fmaxf(__uint_as_float(__float_as_uint(x) & keep), 0.f);   // pruned: 0
                        s[i] = u * u;                        // P
                        p[i] = u * (p[i] - de[e]);           // dS
                    }
                }
            }
            bf16x8 own[2], hand[2];
            {
                bf16x8 pp[2], dd[2];
                to_operands(s, pp);
                to_operands(p, dd);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    own[ks] = role ? dd[ks] : pp[ks];
                    hand[ks] = role ? pp[ks] : dd[ks];
                }
            }
            s_hand[wave][0][lane] = hand[0];
            s_hand[wave][1][lane] = hand[1];
            tr_mm_32<D>(grad_tile + role * 32 * D, own, acc, tr);
        }
        __syncthreads();                                     // what the partner hands over is there
        if (s_live[stage][wave ^ 2]) {
            bf16x8 got[2];
            got[0] = s_hand[wave ^ 2][0][lane];
            got[1] = s_hand[wave ^ 2][1][lane];
            tr_mm_32<D>(grad_tile + (1 - role) * 32 * D, got, acc, tr);
        }
        stage ^= 1;
    }
    __syncthreads();                                         // all wavefronts are done with the tiles
    const int krow0 = kb * 64 + kh * 32;
    uint16_t* stg = smem + wave * 32 * D;
    if (role) {
        uint16_t* dKp = (uint16_t*)a.dK + (size_t)b * a.sk[0] + (size_t)h * a.sk[1];
        store_rows_bf16<D>(stg, acc, a.scale, lane, dKp + (size_t)krow0 * a.sk[2], a.sk[2], a.Lk - krow0);
    } else {
        uint16_t* dVp = (uint16_t*)a.dV + (size_t)b * a.sv[0] + (size_t)h * a.sv[1];
        store_rows_bf16<D>(stg, acc, 1.0f, lane, dVp + (size_t)krow0 * a.sv[2], a.sv[2], a.Lk - krow0);
    }
}

template <int D>
hipError_t launch_d(const BwdArgs& a, bool dq, bool dkv, hipStream_t stream)
{
    const int nQB = (a.Lq + 63) / 64, nKB = (a.Lk + 63) / 64, NP = a.B * a.H;
    const dim3 qgrid = grid_of((long long)NP * nQB, 256), kgrid = grid_of((long long)NP * nKB, 256), block(256);
    const Schedule &rs = a.sched, &cs = a.csched;
    auto run_dq = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, qgrid, block, 0, stream, a.row_ptr, rs.cnt, rs.start, rs.cols,
                           (const uint32_t*)rs.bitmaps, nQB, a.B, NP * nQB, a);
        return hipGetLastError();
    };
    auto run_dkv = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, kgrid, block, 0, stream, a.col_ptr, cs.cnt, cs.start, cs.cols,
                           (const uint32_t*)cs.bitmaps, nKB, a.H, a.B, NP, a);
        return hipGetLastError();
    };
    hipError_t e = hipSuccess;
    if (a.entmax) {                                          // the dQ kernel leaves gbar for the other
        e = run_dq(bwd_dq_sched_kernel<D, ENTMAX15>);
        return e == hipSuccess ? run_dkv(bwd_dkv_sched_kernel<D, ENTMAX15>) : e;
    }
    if (dq) e = run_dq(bwd_dq_sched_kernel<D, SOFTMAX>);
    if (e == hipSuccess && dkv) e = run_dkv(bwd_dkv_sched_kernel<D, SOFTMAX>);
    return e;
}

}  // namespace

hipError_t launch_bwd_sched(const BwdArgs& a, bool dq, bool dkv, hipStream_t stream)
{
    switch (a.D) {
        case 32: return launch_d<32>(a, dq, dkv, stream);
        case 64: return launch_d<64>(a, dq, dkv, stream);
        case 128: return launch_d<128>(a, dq, dkv, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ap
