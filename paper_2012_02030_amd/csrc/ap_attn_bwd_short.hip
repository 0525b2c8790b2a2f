// Backward pass of short sequences (at most 256 queries and 256 keys, D <= 64): one workgroup per (example, head)
// forms dQ, dK and dV in one go.  The arithmetic is that of ap_attn_bwd.hip, over the layout's own bitmaps.
//
// Wavefront w owns keys 32 w .. 32 w + 31: K^T and V^T operands and the dK, dV accumulators stay in its registers, and
// Q, dO and K rows in LDS.  For every 64 queries it forms S = Q K^T and dP = dO V^T of its keys (lane = key), sums
// dV += P^T dO and dK += dS^T Q straight from registers, and leaves dS in LDS; then the 32 x 32 pieces of those
// queries' dQ are dealt to the wavefronts, each a sum over all keys.
//
// Short sequences are bound by the chain of cold loads of a launch and not by arithmetic, so what counts is one launch
// instead of two (dQ, then dK and dV, which recompute the scores and load everything again): five products per tile
// instead of seven and every row read once.  B32 H8 117 x 141 D64 (backward pass) 19.4 -> 14.0 us, of which loading and
// storing are 8; B64 H16 128 x 128 53 -> 37; B64 H16 64 x 64 25.5 -> 17.7.  32 queries a round were 16 us at the first.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"
#include "ap_mfma_common.h"

namespace ap {

namespace {

using namespace mfma;

// N: most 32-row blocks of queries and of keys.  The leading arguments repeat fields of `a`: they arrive in registers
// when a wavefront starts (kernel-argument preloading).
template <int D, int N>
__global__ __launch_bounds__(64 * N, 2) void bwd_short_kernel(
    const int32_t* __restrict__ p_row_ptr, const int32_t* __restrict__ p_col_idx, const uint64_t* __restrict__ p_bitmaps,
    int nq, int nk, int total, int p_B, int p_Lq, BwdArgs a)
{
    constexpr int KSTEPS = D / 16, DBLK = D / 32;
    constexpr int CPR = D / 8, RPI = 64 / CPR;               // 16-byte pieces of a row; rows per load instruction
    constexpr int BLOCK = 32 * D;                            // elements of 32 rows
    // K rows, Q rows, dO rows; V rows, whose place dS takes afterwards (two times 32 x 32 per 32 keys); staging of dQ
    constexpr int DS = 32 * 32;
    constexpr int LAST = BLOCK > 2 * DS ? BLOCK : 2 * DS;
    __shared__ __attribute__((aligned(1024))) uint16_t smem[N * (3 * BLOCK + LAST) + N * DS];
    __shared__ __attribute__((aligned(16))) uint32_t s_word[N][32 * N];       // kept keys of a query, by 32 keys
    __shared__ __attribute__((aligned(16))) float s_lse[32 * N], s_delta[32 * N];
    uint16_t* const Ks = smem;
    uint16_t* const Qs = smem + N * BLOCK;
    uint16_t* const Gs = smem + 2 * N * BLOCK;
    uint16_t* const Vs = smem + 3 * N * BLOCK;
    uint16_t* const dSs = Vs;

    const int blk = block_index();
    if (blk >= total) return;
    const int bid = xcd_contiguous(blk, total);
    const int b = bid % p_B;                                 // the examples of a head share its layout
    const int h = bid / p_B;
    const int nQB = (p_Lq + 63) / 64;
    const int first_tile = p_row_ptr[h * nQB];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = lane & 31, hh = lane >> 5;

    // ---- everything that does not depend on the layout is requested at once (rows that do not exist read as zeros)
    auto load_rows = [&](const void* base, const long long* stride, int rows, int blocks, uint16_t* dst) {
        const int bytes = (int)stride[2] * 2;
        const rsrc_t rs = make_rsrc((const uint16_t*)base + (size_t)b * stride[0] + (size_t)h * stride[1],
                                    (unsigned)((rows - 1) * bytes + D * 2));
        for (int j = wave; j < blocks * (32 / RPI); j += nk) {
            const int r = j * RPI + lane / CPR;
            load16_to_lds(lds_addr_of((lds_u16*)dst + j * 512), (lane / CPR) * bytes + ((lane % CPR) ^ swz_u<D>(r)) * 16, rs,
                          j * RPI * bytes);
        }
    };
    int row_end = 0;                                         // lane r: end of block row r's tiles
    if (lane < nQB) row_end = p_row_ptr[h * nQB + lane + 1];
    load_rows(a.K, a.sk, a.Lk, nk, Ks);
    load_rows(a.V, a.sv, a.Lk, nk, Vs);
    load_rows(a.Q, a.sq, a.Lq, nq, Qs);
    load_rows(a.dO, a.so, a.Lq, nq, Gs);
    const size_t stat_base = ((size_t)b * a.H + h) * a.Lq;
    const int nt = 64 * nk;                                  // threads
    // pieces of O (for delta) of this thread, the first NO of them ahead of time
    constexpr int NO = 4;
    const uint16_t* Op = (const uint16_t*)a.O + (size_t)b * a.so[0] + (size_t)h * a.so[1];
    auto o_piece = [&](int idx) {
        return *reinterpret_cast<const uint4*>(Op + (long long)min(idx / CPR, a.Lq - 1) * a.so[2] + idx % CPR * 8);
    };
    uint4 o[NO];
#pragma unroll
    for (int u = 0; u < NO; ++u) o[u] = o_piece(tid + u * nt);
    const float lse = tid < a.Lq ? a.lse[stat_base + tid] : -INFINITY;

    // ---- kept keys of every query, causal limit included: tile after tile of the head, one per wavefront, the
    // first two of them ahead of time
    const int last_tile = __builtin_amdgcn_readlane(row_end, nQB - 1);
    struct Tile {
        int kb;
        uint64_t word;                                       // of query row `lane` of the tile
    };
    auto fetch_tile = [&](int t) {
        Tile x = {0, 0};
        if (t < last_tile) {
            x.kb = p_col_idx[t];
            x.word = p_bitmaps[(size_t)t * 64 + lane];
        }
        return x;
    };
    auto put_tile = [&](int t, const Tile& x) {
        if (t >= last_tile) return;
        const int r = __popcll(__ballot(lane < nQB && row_end <= t));   // the block row it belongs to
        const int q = r * 64 + lane;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t w = (uint32_t)(x.word >> (32 * half));
            if (a.causal) {
                const int lim = q + (a.Lk - a.Lq) - (x.kb * 64 + 32 * half);   // last visible bit
                w = lim < 0 ? 0u : (lim < 31 ? w & ((2u << lim) - 1u) : w);
            }
            if (2 * x.kb + half < nk && q < 32 * nq) s_word[2 * x.kb + half][q] = w;
        }
    };
    const Tile tile0 = fetch_tile(first_tile + wave), tile1 = fetch_tile(first_tile + wave + nk);

    for (int i = tid; i < nk * 32 * N; i += nt) s_word[0][i] = 0;
    if (tid < 32 * nq) s_lse[tid] = lse == -INFINITY ? INFINITY : lse * kLog2e;   // 32 nq <= 64 nk threads (bwd_short_fits)
    __syncthreads();
    put_tile(first_tile + wave, tile0);
    put_tile(first_tile + wave + nk, tile1);
    for (int t = first_tile + wave + 2 * nk; t < last_tile; t += nk) put_tile(t, fetch_tile(t));
    wait_vmem();                                             // the rows have landed
    __syncthreads();                                         // ... for everybody

    // bit 8 i + k: some query of block i (32 queries) keeps one of key block k.  A lane looks at one such pair, starting
    // at a word of its own, so that the lanes share no LDS bank.
    uint32_t kept_some = 0;
    if (lane % 8 < nk && lane / 8 < nq)
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const uint4 w = *reinterpret_cast<const uint4*>(&s_word[lane % 8][lane / 8 * 32 + (g + lane) % 8 * 4]);
            kept_some |= w.x | w.y | w.z | w.w;
        }
    const uint64_t live_blocks = __ballot(kept_some != 0);
    // keys of this wavefront's block that some query keeps: the OR over i
    uint32_t used_keys = kept_some | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)kept_some, 0x128, 0xf, 0xf, false);   // row_ror:8
    if constexpr (N > 2) {
        const auto r = __builtin_amdgcn_permlane16_swap(used_keys, used_keys, false, false);
        used_keys = r[0] | r[1];
    }
    if constexpr (N > 4) {
        const auto r = __builtin_amdgcn_permlane32_swap(used_keys, used_keys, false, false);
        used_keys = r[0] | r[1];
    }
    used_keys = (uint32_t)__builtin_amdgcn_readlane((int)used_keys, wave);

    // ---- delta_i = <dO_i, O_i>
    auto add_delta = [&](int idx, const uint4& x) {
        const int row = idx / CPR, c = idx % CPR;
        const uint4 g = *reinterpret_cast<const uint4*>(Gs + row * D + (c ^ swz_u<D>(row)) * 8);
        const float row_lse = s_lse[row];
        const uint32_t ow[4] = {x.x, x.y, x.z, x.w}, gw[4] = {g.x, g.y, g.z, g.w};
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d = fmaf(__uint_as_float(ow[k] << 16), __uint_as_float(gw[k] << 16), d);
            d = fmaf(__uint_as_float(ow[k] & 0xffff0000u), __uint_as_float(gw[k] & 0xffff0000u), d);
        }
        d = group_sum<CPR>(d);
        if (c == 0) s_delta[row] = row_lse != INFINITY ? d : 0.f;
    };
    const int pieces = 32 * nq * CPR;                        // a multiple of 64: a wavefront has all or none of a step
#pragma unroll
    for (int u = 0; u < NO; ++u)
        if (tid + u * nt < pieces) add_delta(tid + u * nt, o[u]);
    for (int idx = tid + NO * nt; idx < pieces; idx += nt) add_delta(idx, o_piece(idx));
    const int k_swz = hh ^ swz_u<D>(n);
    // Rows of keys that nobody keeps and of queries that keep nothing become zeros: a tile brings them too, nobody need have
    // written them, and they would be multiplied by exact zeros (entries of a schedule do not hold them).
    const uint4 zero = make_uint4(0, 0, 0, 0);
    if (!((used_keys >> n) & 1))                             // the pieces that this lane reads below
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            const int at = wave * BLOCK + n * D + ((2 * kk) ^ k_swz) * 8;
            *reinterpret_cast<uint4*>(Ks + at) = zero;
            *reinterpret_cast<uint4*>(Vs + at) = zero;
        }
    if (tid < a.Lq && lse == -INFINITY)                      // (their delta is zero whatever is read of them meanwhile)
#pragma unroll
        for (int c = 0; c < CPR; ++c) {
            *reinterpret_cast<uint4*>(Qs + tid * D + c * 8) = zero;
            *reinterpret_cast<uint4*>(Gs + tid * D + c * 8) = zero;
        }
    bf16x8 kreg[KSTEPS], vreg[KSTEPS];                       // K^T and V^T operands
    read_operand<D>(Ks + wave * BLOCK, n, k_swz, kreg);
    read_operand<D>(Vs + wave * BLOCK, n, k_swz, vreg);
    __syncthreads();                                         // delta is there; the place of V is free

    const float sc = a.scale * kLog2e;
    const TrReadU<D> tr = make_tr_read_u<D>(lane);
    const TrReadU<32> tr32 = make_tr_read_u<32>(lane);
    f32x16 dk[DBLK], dv[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dk[db][i] = dv[db][i] = 0.f;
    uint16_t* const dQp = (uint16_t*)a.dQ + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    uint16_t* const stage_q = smem + N * (3 * BLOCK + LAST) + wave * DS;

    // 64 queries a round: two independent chains of latencies
    for (int qi = 0; qi < nq; qi += 2) {
        const int q0 = qi * 32;
        bf16x8 dd[2][2];
        const uint32_t live_keys = (uint32_t)(live_blocks >> (8 * qi));   // of both query blocks of the round
        const bool live = (live_keys & (0x0101u << wave)) != 0;
        if (live) {
            f32x16 s[2], p[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                two_products_32<D>(Qs + (qi + j) * BLOCK, Gs + (qi + j) * BLOCK, n, k_swz, kreg, vreg, s[j], p[j]);
            bf16x8 pp[2][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int r0 = q0 + 32 * j + 8 * g + 4 * hh;            // 4 consecutive queries
                    const float4 l4 = *reinterpret_cast<const float4*>(s_lse + r0);
                    const float4 d4 = *reinterpret_cast<const float4*>(s_delta + r0);
                    const uint4 w4 = *reinterpret_cast<const uint4*>(&s_word[wave][r0]);
                    const float le[4] = {l4.x, l4.y, l4.z, l4.w}, de[4] = {d4.x, d4.y, d4.z, d4.w};
                    const uint32_t we[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = 4 * g + e;
                        const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)we[e], n, 1);
                        s[j][i] = __builtin_amdgcn_exp2f(or_minus_inf(fmaf(s[j][i], sc, -le[e]), keep));   // P
                        p[j][i] = s[j][i] * (p[j][i] - de[e]);              // dS
                    }
                }
                to_operands(s[j], pp[j]);
                to_operands(p[j], dd[j]);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                tr_mm_32<D>((lds_u16*)Gs + (qi + j) * BLOCK, pp[j], dv, tr);   // dV^T += dO^T P
                tr_mm_32<D>((lds_u16*)Qs + (qi + j) * BLOCK, dd[j], dk, tr);   // dK^T += Q^T dS
            }
        }
        if (qi > 0) __syncthreads();                         // dS of the round before is consumed
        // queries 8 g + 4 hh .. + 3 of this lane's key: half a 16-byte piece
        if (live) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const bf16x8 x = dd[j][g >> 1];
                    const bf16x4 v = (g & 1) ? __builtin_shufflevector(x, x, 4, 5, 6, 7)
                                             : __builtin_shufflevector(x, x, 0, 1, 2, 3);
                    *reinterpret_cast<bf16x4*>(dSs + (j * N + wave) * DS + n * 32 + (g ^ swz_u<32>(n)) * 8 + 4 * hh) = v;
                }
        }
        __syncthreads();                                     // dS of these queries is complete
        // dQ^T[32 columns of D][32 queries] += K^T dS^T over the key blocks that these queries keep something of: K rows of
        // the others need not be finite.  2 DBLK pieces a round, dealt to the wavefronts.
#pragma unroll
        for (int piece = 0; piece < 2 * DBLK; ++piece) {
            const int j = piece / DBLK, db = piece % DBLK;
            if ((DBLK * qi + piece) % nk != wave) continue;
            f32x16 dq[1], odd;
#pragma unroll
            for (int i = 0; i < 16; ++i) dq[0][i] = odd[i] = 0.f;
            bf16x8 ka[2], sb[2], ka_next[2], sb_next[2];
            auto read = [&](int kb, bf16x8* x, bf16x8* y) {
                lds_u16* kt = (lds_u16*)Ks + kb * BLOCK;
                lds_u16* st = (lds_u16*)dSs + (j * N + kb) * DS;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const bf16x4 a0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(kt + 16 * ks * D + tr.off[0][db]));
                    const bf16x4 a1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(kt + 16 * ks * D + tr.off[1][db]));
                    const bf16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(st + 16 * ks * 32 + tr32.off[0][0]));
                    const bf16x4 b1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(st + 16 * ks * 32 + tr32.off[1][0]));
                    x[ks] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
                    y[ks] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            };
            const uint32_t used = (live_keys >> (8 * j)) & 0xffu;
            auto multiply = [&]() {
                dq[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[0], sb[0], dq[0], 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[1], sb[1], odd, 0, 0, 0);
            };
            // Where all blocks are used, operands of the next one are requested under the matrix instructions of this one (two
            // chains).  Walked like that from bit to bit, a call of the usual case takes 2 to 5 % longer (16 x 12 x 200 x 200
            // 20.4 -> 21.5 us, 20.7 with this branch; 64 x 16 x 256 x 256 causal, which skips half, 91.4 -> 88.7).
            if (used == (1u << nk) - 1u) {
                read(0, ka, sb);
                for (int kb = 0; kb < nk; ++kb) {
                    read(min(kb + 1, nk - 1), ka_next, sb_next);
                    multiply();
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        ka[ks] = ka_next[ks];
                        sb[ks] = sb_next[ks];
                    }
                }
            } else {
                for (uint32_t rest = used; rest; rest &= rest - 1) {
                    read(__ffs(rest) - 1, ka, sb);
                    multiply();
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) dq[0][i] += odd[i];
            store_rows_bf16<32>(stage_q, dq, a.scale, lane, dQp + (size_t)(q0 + 32 * j) * a.sq[2] + 32 * db, a.sq[2],
                                a.Lq - q0 - 32 * j);
        }
    }
    __syncthreads();                                         // K rows are consumed: their place becomes the stores' staging
    const int k0 = wave * 32;
    uint16_t* const stage_k = Ks + wave * BLOCK;
    uint16_t* const dKp = (uint16_t*)a.dK + (size_t)b * a.sk[0] + (size_t)h * a.sk[1];
    uint16_t* const dVp = (uint16_t*)a.dV + (size_t)b * a.sv[0] + (size_t)h * a.sv[1];
    store_rows_bf16<D>(stage_k, dk, a.scale, lane, dKp + (size_t)k0 * a.sk[2], a.sk[2], a.Lk - k0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read before it is written again
    store_rows_bf16<D>(stage_k, dv, 1.0f, lane, dVp + (size_t)k0 * a.sv[2], a.sv[2], a.Lk - k0);
}

template <int D>
hipError_t launch_d(const BwdArgs& a, hipStream_t stream)
{
    const int nq = (a.Lq + 63) / 64 * 2, nk = (a.Lk + 31) / 32, total = a.B * a.H;
    const dim3 grid = grid_of(total, 64 * nk), block(64 * nk);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, a.row_ptr, a.col_idx, a.bitmaps, nq, nk, total, a.B, a.Lq, a);
    };
    if (nq <= 2 && nk <= 2) run(bwd_short_kernel<D, 2>);
    else if (nq <= 4 && nk <= 4) run(bwd_short_kernel<D, 4>);
    else run(bwd_short_kernel<D, 8>);
    return hipGetLastError();
}

}  // namespace

// Where the general kernels are the better ones: few keys per query (a wavefront per 32 keys walks all queries: 16 x 8
// x 160 x 30 21.9 us against 13.4), and long sequences of few pairs, where rounds of queries are a chain that the
// general kernels spread over workgroups (more than 128 queries: 4 x 4 x 200 x 200 18 against 15, 8 x 16 20 against 19, 16 x 12
// 21 against 24), or of D = 32 that fill the chip more than once (64 x 16 x 256 x 256 64 against 61).
bool bwd_short_fits(const BwdArgs& a)
{
    if (a.entmax || (a.D != 32 && a.D != 64) || a.Lq > 256 || a.Lk > 256) return false;
    if ((a.Lk + 31) / 32 < (a.Lq + 63) / 64) return false;
    const long long pairs = (long long)a.B * a.H;
    return a.Lq <= 128 || (pairs >= 192 && (a.D == 64 || pairs <= 256));
}

hipError_t launch_bwd_short(const BwdArgs& a, hipStream_t stream)
{
    return a.D == 32 ? launch_d<32>(a, stream) : launch_d<64>(a, stream);
}

}  // namespace ap
