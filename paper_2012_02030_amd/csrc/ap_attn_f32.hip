// Masked attention forward in fp32 on the matrix cores (Section 3.2, masked-attention equation).
//
// One workgroup of four wavefronts (two up to 64 keys) per 32 queries.  For up to 32 stored tiles at a time the
// workgroup brings the bitmap words of its queries into LDS and lists the keys that any of them keeps
// (the used columns of a tile are the OR of its 32 words), packed without gaps over the tiles, together
// with where the keep bits of each are found.  The wavefronts then take the chunks of 32 listed keys in
// turn, each with an online softmax of its own:
//   1. S^T = K Q^T with v_mfma_f32_32x32x2_f32, so that a lane holds scores of ONE query (lane % 32)
//      for 16 of the 32 keys.  Both operands come straight from global memory, 16 bytes per lane: the
//      contraction runs over the head dimension in the order those loads deliver it.
//   2. pruned scores become -inf, online softmax in fp32 in the log2 domain;
//   3. O^T += V^T P^T: the score registers already are the second operand, and the first is one
//      dword of a V row per lane, 32 lanes to a row.
// No tile goes through LDS; it holds the lists and, at the end, the four partial results for the merge.
//
// What bounds it: each wavefront's chain (words, lists, K rows, products at 64 cycles per instruction or 4 096
// per chunk at D = 64, V rows), with no unit full.  B8 H8 L500 D64, 10 % kept, 16.7 us: the matrix pipe is busy for a third
// of the kernel's cycles and the vector units for a quarter, and wavefronts wait for memory or barriers during 46 %
// of their time.  Hence the packing, which leaves far tiles their few used columns, and four wavefronts per
// 32 queries rather than one, because a long causal row is one chain.
// With one query per lane and K, V broadcast from LDS in vector arithmetic the same call was bound
// by LDS reads: B8 H8 L500 D64, 5 % kept, 69 us, now 18 us; B4 H8 L1024 D128 437 us, now 47 us; B1 H2 L64
// D32 (launch and chain of loads) 9.7 us, now 5.1 us.
//
// Matrix-core layouts (32x32x2, l = lane): A[m][k] and B[k][n]: m = n = l % 32, k = l / 32;
// C[m][n]: n = l % 32, m = 8*(i/4) + 4*(l/32) + i%4, i = 0..15.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"
#include "ap_mfma_common.h"

namespace ap {

namespace {

using namespace mfma;


// OR over the 32 lanes of each half of the wavefront
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_or(uint32_t v)
{
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t or_over_32(uint32_t v)
{
    v = dpp_or<0xB1>(v);                               // quad_perm [1,0,3,2]
    v = dpp_or<0x4E>(v);                               // quad_perm [2,3,0,1]
    v = dpp_or<0x141>(v);                              // row_half_mirror
    v = dpp_or<0x140>(v);                              // row_mirror
    return v | (uint32_t)__shfl_xor((int)v, 16, 64);
}

// The leading arguments arrive in registers when a wavefront starts (kernel-argument preloading).
// Off: byte offsets inside a (batch, head) slice of K and V, 32 bits wide where the slices allow it (one
// register per row address instead of two, and a wavefront more per SIMD).
// kNW wavefronts per 32 queries: two where there are at most 64 keys, i.e. two chunks, and four otherwise.
template <int D, int kNW, typename Off>
__global__ __launch_bounds__(64 * kNW, sizeof(Off) == 8 ? 2 : (D == 128 ? 3 : 4)) void fwd_f32_kernel(
    const int32_t* __restrict__ p_row_ptr, const int32_t* __restrict__ p_col_idx,
    const uint64_t* __restrict__ p_bitmaps, int nQG, int p_H, int n_blocks, FwdArgs a)
{
    constexpr int kSeg = kNW == 2 ? 2 : 32;            // tiles listed at a time (64 keys: one tile)
    constexpr int kPer = kSeg / kNW;                   // of them, per wavefront
    constexpr int DBLK = D / 32;
    constexpr int NJ = D / 8;                          // 16-byte pieces of a lane's half of a row
    constexpr int DM = D < 64 ? D : 64;                // columns of the output that are merged at a time
    constexpr int OLD = DM + 4;                        // floats per row of a partial result
    // listed keys; where their bits are; bitmap words of kSeg tiles and 32 queries, then a row of zeros
    constexpr int LISTS = 2 * kSeg * 64 + kSeg * 64 + 64;
    constexpr int QUERIES = 32 * D;                    // Q^T operand: [16-byte piece of a half row][half][query]
    constexpr int MERGE = kNW * 32 * OLD;
    __shared__ __attribute__((aligned(16))) uint32_t smem[LISTS + QUERIES > MERGE ? LISTS + QUERIES : MERGE];
    __shared__ uint64_t s_or[kSeg];                    // used columns of every listed tile
    __shared__ float s_m[kNW][32], s_l[kNW][32];
    int* list = (int*)smem;
    int* where = list + kSeg * 64;                     // byte offset of the 32-bit word half << 5 | bit
    uint32_t* words = (uint32_t*)where + kSeg * 64;    // [tile][query][half]
    float4* s_q = reinterpret_cast<float4*>(smem + LISTS);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5;

    const int blk = block_index();
    if (blk >= n_blocks) return;
    const int bid = xcd_contiguous(blk, n_blocks);     // the query groups of a head share an L2
    const int qg = nQG - 1 - bid % nQG;                // long causal rows first
    const int h = (bid / nQG) % p_H;
    const int b = bid / (nQG * p_H);
    const int nQB = (nQG + 1) >> 1;
    const int r = h * nQB + (qg >> 1);
    const int t0 = p_row_ptr[r], t1 = p_row_ptr[r + 1];
    const int brow = (qg & 1) * 32 + n;                // row inside the layout's 64-query block row
    const int i = qg * 32 + n;                         // this lane's query

    const float* Qp = (const float*)a.Q + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    const char* Kp = (const char*)((const float*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1]);
    const char* Vp = (const char*)((const float*)a.V + (size_t)b * a.sv[0] + (size_t)h * a.sv[1]);
    const Off sk_bytes = (Off)a.sk[2] * 4, sv_bytes = (Off)a.sv[2] * 4;
    const int diag = i + (a.Lk - a.Lq);                // last visible key if causal

    // query rows, pre-multiplied by scale*log2(e): scores live in the log2 domain.  Shared by the four
    // wavefronts through LDS, which leaves registers for a fourth wavefront per SIMD (a third at D = 128)
    {
        const float qs = a.scale * kLog2e;
        const float* qr = Qp + (size_t)(i < a.Lq ? i : a.Lq - 1) * a.sq[2] + 4 * hh;
#pragma unroll
        for (int u = 0; u < NJ / kNW; ++u) {
            const int j = u * kNW + wave;
            float4 x = *reinterpret_cast<const float4*>(qr + 8 * j);
            x.x *= qs; x.y *= qs; x.z *= qs; x.w *= qs;
            s_q[j * 64 + lane] = x;
        }
    }

    f32x16 oacc[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
    float m = -INFINITY;                               // running max (log2 domain)
    float l = 0.f;                                     // this lane's share of the running sum of 2^(s - m)

    for (int seg = t0; seg < t1; seg += kSeg) {
        const int nt = min(kSeg, t1 - seg);
        // ---- the listed keys of tiles seg .. seg + nt - 1.  Wavefront w looks after tiles w, w + 4, ...
        int k0_lane = 0;                               // lane t: first key of tile t
        if (lane < nt) k0_lane = p_col_idx[seg + lane] * kBN;
        // what depends on the lane only is formed again in every round: kept in registers over the loop, the
        // addresses of eight tiles would cost a wavefront per SIMD
        int word_off = brow, row_off = n * 2 + hh;
        asm volatile("" : "+v"(word_off), "+v"(row_off));
        uint64_t word[kPer];                           // both halves of the wavefront hold the 32 queries' words
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kNW + wave;
            word[u] = t < nt ? p_bitmaps[(size_t)(seg + t) * 64 + word_off] : 0ull;
        }
        __syncthreads();                               // the previous segment's lists are no longer read
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kNW + wave;
            if (t >= nt) break;                        // uniform
            if (a.causal) {
                const int lim = diag - __builtin_amdgcn_readlane(k0_lane, t);
                word[u] = lim < 0 ? 0ull : word[u] & (~0ull >> (63 - min(lim, 63)));
            }
            const uint32_t lo = (uint32_t)word[u], hi = (uint32_t)(word[u] >> 32);
            words[t * 64 + row_off] = hh ? hi : lo;
            const uint32_t any = or_over_32(hh ? hi : lo);   // lower lanes: columns 0..31, upper lanes: 32..63
            if ((row_off >> 1) == 0) reinterpret_cast<uint32_t*>(s_or)[2 * t + row_off] = any;
        }
        if (wave == kNW - 1) words[kSeg * 64 + lane] = 0;
        __syncthreads();
        const uint64_t or_lane = lane < nt ? s_or[lane] : 0ull;   // lane t: used columns of tile t
        const int cnt = __popcll(or_lane);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < kSeg; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        const int total = __builtin_amdgcn_readlane(incl, kSeg - 1);
        if (total == 0) continue;                      // nothing visible (the same in all wavefronts)
        for (int t = wave; t < nt; t += kNW) {         // lane c: column c of tile t
            const int pos = __builtin_amdgcn_readlane(incl - cnt, t);
            const int k0 = __builtin_amdgcn_readlane(k0_lane, t);
            const uint64_t used = s_or[t];
            if ((used >> lane) & 1ull) {
                const int p = pos + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(used >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)used, 0));
                list[p] = k0 + lane;
                where[p] = (t * 256 + 4 * (lane >> 5)) << 5 | (lane & 31);
            }
        }
        if (wave == 0 && total & 31) {                 // fill up the last chunk: a key that is listed, kept by nobody
            const unsigned long long some = __ballot(cnt > 0);
            const int t = __ffsll((long long)some) - 1;
            const int key = __shfl(k0_lane + __ffsll((long long)or_lane) - 1, t, 64);
            if (lane >= (total & 31) && lane < 32) {
                list[(total & ~31) + lane] = key;
                where[(total & ~31) + lane] = (kSeg * 256) << 5;
            }
        }
        __syncthreads();

        // ---- chunks of 32 listed keys
        for (int ch = wave; ch * 32 < total; ch += kNW) {
            const Off k_off = (Off)list[ch * 32 + n] * sk_bytes + (Off)(16 * hh);
            constexpr int KH = D == 128 ? 2 : 1;       // K arrives in two halves where registers are short
            float4 k[NJ / KH];
            auto load_k = [&](int half) {
#pragma unroll
                for (int j = 0; j < NJ / KH; ++j)
                    k[j] = *reinterpret_cast<const float4*>(Kp + k_off + (Off)(32 * (half * (NJ / KH) + j)));
            };
            load_k(0);
            // V rows 8*g + 4*hh + e of the chunk, one dword per lane and 32-wide block of the head dimension
            float v[16][DBLK];
            auto load_v = [&](int g) {
                const int4 key = *reinterpret_cast<const int4*>(list + ch * 32 + 8 * g + 4 * hh);
                const int ke[4] = {key.x, key.y, key.z, key.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const Off v_off = (Off)ke[e] * sv_bytes + (Off)(4 * n);
#pragma unroll
                    for (int db = 0; db < DBLK; ++db)
                        v[4 * g + e][db] = *reinterpret_cast<const float*>(Vp + v_off + (Off)(128 * db));
                }
            };
            // Quarters of V that travel under the first product and before the second one, the others under
            // the second: as many as there are registers for.  At D = 64 this keeps four wavefronts per SIMD
            // (18 us at the size above; 24 with half of V early and three, 20 with none of it early)
            constexpr int EARLY = D == 128 ? 0 : (D == 64 ? 1 : 4), LATE = D >= 64 ? 2 : 4;
#pragma unroll
            for (int g = 0; g < EARLY; ++g) load_v(g);
            // Q^T pieces are read again for every chunk: an offset the compiler cannot see through keeps
            // them from being hoisted into registers, and the barriers below keep V loads in their places
            int q_off = lane;
            asm volatile("" : "+v"(q_off));
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int half = 0; half < KH; ++half) {
                if (half > 0) load_k(half);
#pragma unroll
                for (int j = 0; j < NJ / KH; ++j) {
                    const float4 q = s_q[(half * (NJ / KH) + j) * 64 + q_off];
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[j].x, q.x, s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[j].y, q.y, s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[j].z, q.z, s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[j].w, q.w, s, 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = EARLY; g < LATE; ++g) load_v(g);
            float tmax = -INFINITY;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int4 at = *reinterpret_cast<const int4*>(where + ch * 32 + 8 * g + 4 * hh);
                const int we[4] = {at.x, at.y, at.z, at.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int w = *reinterpret_cast<const int*>((const char*)words + 8 * n + (we[e] >> 5));
                    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(w, we[e] & 31, 1);   // all ones where kept
                    const float x = __uint_as_float((__float_as_uint(s[4 * g + e]) & keep) | (0xff800000u & ~keep));
                    s[4 * g + e] = x;
                    tmax = fmaxf(tmax, x);
                }
            }
            {
                const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
                tmax = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
            }
            const float m_new = fmaxf(m, tmax);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            if (__ballot(m_new > m) != 0) {
                const float alpha = __builtin_amdgcn_exp2f(m - m_use);   // m = -inf -> 0
                l *= alpha;
#pragma unroll
                for (int db = 0; db < DBLK; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
                m = m_new;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                s[e] = __builtin_amdgcn_exp2f(s[e] - m_use);   // -inf -> 0
                l += s[e];
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (LATE == 2 && g < 2) {              // quarters 2 and 3 take the place of 0 and 1
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int db = 0; db < DBLK; ++db)
                        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[4 * g + e][db], s[4 * g + e], oacc[db], 0, 0, 0);
                if (LATE == 2 && g < 2) load_v(g + 2);
            }
        }
    }

    // ---- merge the four partial states: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w
    {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        l = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    }
    if (hh == 0) {
        s_m[wave][n] = m;
        s_l[wave][n] = l;
    }
    __syncthreads();                                   // also: the lists are no longer read
    float* part = (float*)smem;                        // [wave][query][OLD]
    float f;                                           // this wavefront's weight
    {
        float M = m;
#pragma unroll
        for (int w = 0; w < kNW; ++w) M = fmaxf(M, s_m[w][n]);
        f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
    }
    constexpr int TPR = DM / 4;                        // threads per row
    float* Op = (float*)a.O + (size_t)b * a.so[0] + (size_t)h * a.so[1];
#pragma unroll
    for (int c0 = 0; c0 < D; c0 += DM) {
        if (c0 > 0) __syncthreads();
        float* p = part + (wave * 32 + n) * OLD + 4 * hh;
#pragma unroll
        for (int db = 0; db < DM / 32; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x16& o = oacc[c0 / 32 + db];
                *reinterpret_cast<float4*>(p + 32 * db + 8 * g) =
                    make_float4(o[4 * g] * f, o[4 * g + 1] * f, o[4 * g + 2] * f, o[4 * g + 3] * f);
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 32 * TPR / (64 * kNW); ++u) {
            const int idx = u * 64 * kNW + tid;
            const int row = idx / TPR, c = (idx % TPR) * 4;
            if (qg * 32 + row >= a.Lq) continue;
            float M = -INFINITY, L = 0.f;
#pragma unroll
            for (int w = 0; w < kNW; ++w) M = fmaxf(M, s_m[w][row]);
            float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int w = 0; w < kNW; ++w) {
                const float mw = s_m[w][row];
                if (mw != -INFINITY) L = fmaf(s_l[w][row], __builtin_amdgcn_exp2f(mw - M), L);
                const float4 x = *reinterpret_cast<const float4*>(part + (w * 32 + row) * OLD + c);
                o.x += x.x; o.y += x.y; o.z += x.z; o.w += x.w;
            }
            const float inv = L > 0.f ? 1.f / L : 0.f;
            *reinterpret_cast<float4*>(Op + (size_t)(qg * 32 + row) * a.so[2] + c0 + c) =
                make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
            if (c0 == 0 && a.lse && c == 0)
                a.lse[((size_t)b * a.H + h) * a.Lq + qg * 32 + row] =
                    L > 0.f ? (M + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
        }
    }
}

template <int D>
hipError_t launch_d(const FwdArgs& a, hipStream_t stream)
{
    const int nQG = (a.Lq + 31) / 32;                  // two groups per block row of the layout
    const long long blocks = (long long)nQG * a.H * a.B;
    if (blocks > 2147483647LL) return hipErrorInvalidValue;
    const auto run = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, grid_of(blocks, 64 * waves), dim3(64 * waves), 0, stream, a.row_ptr, a.col_idx,
                           a.bitmaps, nQG, a.H, (int)blocks, a);
    };
    const bool narrow = (long long)a.Lk * a.sk[2] < (1ll << 29) && (long long)a.Lk * a.sv[2] < (1ll << 29);   // 2 GB a slice
    // 64 keys are two chunks: two more wavefronts per 32 queries would hold the places of other workgroups and do
    // nothing but set up and merge.  B256 H8 40 x 40, D = 32: 28.8 us with four, 20.2 with two; 64 x 64, D = 64: 46.9, 36.5.
    if (narrow && a.Lk <= 64) run(fwd_f32_kernel<D, 2, uint32_t>, 2);
    else if (narrow) run(fwd_f32_kernel<D, 4, uint32_t>, 4);
    else run(fwd_f32_kernel<D, 4, uint64_t>, 4);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t stream)
{
    switch (a.D) {
    case 32: return launch_d<32>(a, stream);
    case 64: return launch_d<64>(a, stream);
    case 128: return launch_d<128>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ap
