// Accumulation of attention matrices into the mean attention map (Section 3.2, Eq. (1)).
//
// The attention matrix of one example, A_b = softmax(Q_b K_b^T / sqrt(d_k)), is never stored:
// it would be B*H*Lq*Lk probabilities.  Two kernels instead:
//
//   row_lse_kernel         one workgroup per (example, head, 128 queries): walks all key tiles,
//                          S^T = K Q^T on the matrix cores, keeps the online row maximum and row
//                          sum, and writes the row's log-sum-exp (base 2) to the workspace.
//   map_accumulate_kernel  one workgroup per (head, 128 queries, 128 keys): loops over the
//                          examples, recomputes the scores tile by tile, P = exp2(s - lse), and
//                          sums P in registers; the running map in memory is read and written
//                          once per call, whatever the batch size.
//
// What bounds them (B4 H16 L2048 D128, causal): the row statistics the issue of vector instructions, three per score
// (49 us; 55 with a maximum over every tile).  The accumulation: 47 us of map traffic at 5.8 TB/s, and 66 of
// arithmetic and operand traffic to LDS (570 MB at about 18 TB/s), which overlap only in part, since the workgroups
// of a round start together (90 us; 112 with query rows loaded straight into registers and two wavefronts per SIMD).
// The first batch writes the map without reading it.
//
// Both use the score layout of the attention kernel: a wavefront owns 32 queries, lane l holds
// query l % 32 and, of each 32-key block, the keys 8*(i/4) + 4*(l/32) + i%4 (i = 0..15).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"
#include "ap_mfma_common.h"

namespace ap {

namespace {

using namespace mfma;

constexpr float kRaise = 32.f;

__device__ __forceinline__ float sum_exp(const f32x16* sacc, float sc, float msc)
{
    float s[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) s[kb] += __builtin_amdgcn_exp2f(fmaf(sacc[kb][i], sc, -msc));
    return s[0] + s[1];
}

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 4) void row_lse_kernel(MapArgs a, int nQB)
{
    constexpr int BM = 32 * NW;
    constexpr int TILE = kBN * D;
    constexpr int KSTEPS = D / 16;
    __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * TILE];
    lds_u16* lds = (lds_u16*)smem;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = lane & 31, hh = lane >> 5;

    // All workgroups of a call of ordinary size are resident at once and a compute unit gets every 32nd of an
    // XCD's, so long rows first would give some of them long rows only (B4 H16 L2048 D128: 75 us, 68 in this
    // order; 55 with four wavefronts per SIMD, which 128 registers allow): the rows' order is reversed in every other
    // round of 32.
    const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int per_xcd = (gridDim.x + 7) / 8;
    const int group = bid / nQB, j = bid % nQB;
    const int round = (nQB < 32 ? ((group * nQB) % per_xcd) / 32 : group) & 1;
    const int qb = a.causal && round ? j : nQB - 1 - j;
    const int h = group % a.H;
    const int b = group / a.H;

    const uint16_t* Qp = (const uint16_t*)a.Q + (size_t)b * a.sq[0] + (size_t)h * a.sq[1];
    const uint16_t* Kp = (const uint16_t*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1];
    const int sk_bytes = (int)a.sk[2] * 2;
    const rsrc_t k_rsrc = make_rsrc(Kp, (unsigned)((a.Lk - 1) * sk_bytes + D * 2));

    const int qrow = qb * BM + wave * 32 + n;
    const bool row_ok = qrow < a.Lq;
    bf16x8 qreg[KSTEPS];
    {
        const uint16_t* qr = Qp + (size_t)(row_ok ? qrow : a.Lq - 1) * a.sq[2] + 8 * hh;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
            qreg[kk] = *reinterpret_cast<const bf16x8*>(qr + 16 * kk);
    }
    const long long off = (long long)a.Lk - a.Lq;
    const long long diag = (long long)qrow + off;            // last visible key if causal
    int nkt = (a.Lk + 63) / 64;
    if (a.causal) {
        const long long block_diag = (long long)qb * BM + (BM - 1) + off;
        nkt = (int)min((long long)nkt, block_diag / 64 + 1);
    }
    const int k_swz = hh ^ swz_k<D>(n);
    const float sc = a.scale * kLog2e;
    // reference of the exponentials: a maximum of scores seen, raised only where the sum of a lane's 32
    // exponentials exceeds kRaise, so an ordinary tile needs no maximum (16 instructions and a lane exchange of 130).
    // While every score seen is -inf (finite rows whose products overflow) it stays -inf, and so the next tile's
    // sum is +inf or NaN and raises it.
    float m = -INFINITY, msc = -INFINITY, lsum = 0.f;
    // last key that any query of this wavefront sees
    const long long wave_last = a.causal ? (long long)qb * BM + wave * 32 + 31 + off : (long long)a.Lk - 1;

    // tiles before n_whole are visible as a whole to the whole wavefront
    long long whole_keys = a.Lk;
    if (a.causal) whole_keys = min(whole_keys, (long long)qb * BM + wave * 32 + off + 1);
    const int n_whole = (int)(whole_keys / 64);

    wait_vmem();
    settle<KSTEPS>(qreg);
    issue_tile_loads<D, NW, false>(k_rsrc, lds, 0, sk_bytes, wave, lane);
    for (int kt = 0; kt < nkt; ++kt) {
        wait_vmem();                                         // tile kt has landed
        __syncthreads();                                     // ... for everybody; tile kt-1 is consumed
        if (kt + 1 < nkt)
            issue_tile_loads<D, NW, false>(k_rsrc, lds + ((kt + 1) & 1) * TILE, (kt + 1) * 64,
                                           sk_bytes, wave, lane);
        const uint16_t* Ks = smem + (kt & 1) * TILE;
        if ((long long)kt * 64 > wave_last) continue;        // uniform over the wavefront
        f32x16 sacc[2];
        qk_64<D>(Ks, qreg, n, k_swz, sacc);

        // keys of this tile that exist and that this query may see: a prefix of the tile
        if (kt >= n_whole) {                                 // uniform over the wavefront: some lane sees a part only
            const long long k0 = (long long)kt * 64;
            long long lim = (long long)a.Lk - k0;
            if (a.causal) lim = min(lim, diag - k0 + 1);
            const uint64_t word = lim >= 64 ? ~0ull : (lim <= 0 ? 0ull : (1ull << lim) - 1ull);
            const uint64_t wsh = word >> (4 * hh);
            const uint32_t wbits[2] = {(uint32_t)wsh, (uint32_t)(wsh >> 32)};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int pos = 8 * (i / 4) + (i % 4);
                    sacc[kb][i] = ((wbits[kb] >> pos) & 1u) ? sacc[kb][i] : -INFINITY;
                }
            asm volatile("");                                // a branch, not selects in every tile's way
        }
        float psum = sum_exp(sacc, sc, msc);
        if (__ballot(!(psum <= kRaise)) != 0) {              // no finite score so far (the reference is -inf), or larger ones
            float tmax = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, sacc[kb][i]);
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
            const float m_new = fmaxf(m, fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
            msc = m_new * sc;
            lsum *= (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m * sc - msc);
            m = m_new;
            psum = sum_exp(sacc, sc, m == -INFINITY ? 0.f : msc);
        }
        lsum += psum;
    }
    {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lsum), __float_as_uint(lsum), false, false);
        lsum = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if (row_ok && hh == 0)
        a.lse2[((size_t)b * a.H + h) * a.Lq + qrow] =
            (m == -INFINITY) ? -INFINITY : fmaf(m, sc, __log2f(lsum));
}

// One workgroup: 128 queries x 128 keys of one head, eight wavefronts of 32 queries x 64 keys.  The
// partial map stays in registers over the examples; 128 registers leave room for four wavefronts per SIMD, i.e. two
// workgroups per compute unit.  Query rows come through LDS like the key rows: as operands fetched straight from
// memory (16-byte pieces of 32 rows per instruction) they took as long as the arithmetic (eight wavefronts: 120 us
// instead of 77 with everything in cache).  Two stages of half rows measured the same as one buffer of whole rows.
//
// INIT: the map is written whatever it held, hidden entries 0.
template <int D, bool INIT>
__global__ __launch_bounds__(512, 4) void map_accumulate_kernel(MapArgs a, int nQB, int nKG, int total)
{
    constexpr int BM = 128, BK = 128, TILE = kBN * D;
    constexpr int KSTEPS = D / 16;
    constexpr int OUT_LD = BK + 4;                           // floats per staged output row (16-byte rows)
    constexpr int OUT_ELEMS = BM * OUT_LD * 2;               // in 2-byte units
    constexpr int STAGES = D <= 64 ? 2 : 1;                  // what fits where the output is staged
    constexpr int STAGE = 4 * TILE;
    constexpr int SMEM = STAGES * STAGE > OUT_ELEMS ? STAGES * STAGE : OUT_ELEMS;
    __shared__ __attribute__((aligned(1024))) uint16_t smem[SMEM];
    lds_u16* lds = (lds_u16*)smem;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave & 3, wk = wave >> 2;
    const int lane = tid & 63;
    const int n = lane & 31, hh = lane >> 5;

    const int linear = block_index();
    if (linear >= total) return;
    const int bid = xcd_contiguous(linear, total);
    const int kg = bid % nKG;
    const int qb = (bid / nKG) % nQB;
    const int h = bid / (nKG * nQB);
    const long long off = (long long)a.Lk - a.Lq;
    const int key0 = kg * BK;                                // first key of this workgroup
    const int q0 = qb * BM;
    // last keys that any query of the workgroup, of this wavefront sees
    const long long block_last = a.causal ? (long long)q0 + (BM - 1) + off : (long long)a.Lk - 1;
    const long long wave_last = a.causal ? (long long)q0 + wq * 32 + 31 + off : (long long)a.Lk - 1;

    // memory side of the tile: 32 threads per row, 16 rows per pass
    const int c4 = (tid & 31) * 4, r0 = tid >> 5;
    const bool vec_ok = (a.Lk & 3) == 0;                     // then every row of the map starts 16-byte aligned
    float* const map0 = a.abar + ((size_t)h * a.Lq + q0 + r0) * a.Lk + key0;
    const long long map_step = (long long)16 * a.Lk;
    auto write_zeros = [&](int z0, long long zk) {           // of the tile of rows z0.. and keys zk * BK..
        float* const z = a.abar + ((size_t)h * a.Lq + z0 + r0) * a.Lk + zk * BK;
        const int cols = (int)min((long long)BK, a.Lk - zk * BK);
#pragma unroll
        for (int pass = 0; pass < 8; ++pass) {
            if (z0 + r0 + 16 * pass >= a.Lq) continue;
            if (vec_ok) {
                if (c4 < cols) *reinterpret_cast<float4*>(z + c4 + pass * map_step) = make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((tid & 31) + 32 * e < cols) z[(tid & 31) + 32 * e + pass * map_step] = 0.f;
            }
        }
    };
    // A tile that is hidden as a whole gets its zeros from its own workgroup before anything else, or (DEAL) from one with
    // a visible tile, before its last scores.  First batches (us, own / dealt): B2 H4 8192 x 8192 D32 273 / 300, B16 H12
    // 1024 x 1024 D64 76 / 78, B1 H16 4096 x 4096 D64 225 / 234; at D = 128 B4 H16 2048 x 2048 123 / 124, B4 H12 2000 x 2000
    // 98 / 103, but B2 H8 4096 x 4096 177 / 170.
    constexpr bool DEAL = D == 128;
    if (block_last < key0) {
        if (INIT && !DEAL) write_zeros(q0, kg);
        return;
    }

    const int qrow = q0 + wq * 32 + n;
    const int sk_bytes = (int)a.sk[2] * 2;
    const unsigned k_bytes = (unsigned)((a.Lk - 1) * sk_bytes + D * 2);
    const float sc = a.scale * kLog2e;
    // some query of the wavefront sees some key of it (uniform over the wavefront)
    const bool seen = (long long)key0 + wk * 64 <= wave_last && key0 + wk * 64 < a.Lk && q0 + wq * 32 < a.Lq;
    const float* lp = a.lse2 + (size_t)h * a.Lq + min(qrow, a.Lq - 1);

    // The 128 query rows and 128 key rows of an example travel to LDS (query rows fetched straight into registers
    // are 16-byte pieces of 32 rows per instruction); a wavefront brings 16 rows of either, key rows only if any of them
    // exists.  The first ones are brought by the wavefronts of the second 64 keys, which in a small map have no scores
    // (B256 H8 40 x 40 D32 142 -> 134 us, B128 H16 40 x 40 D128 160 -> 146, B64 H16 64 x 64 D64 54.7 -> 47.7; not
    // bringing query rows that do not exist either gives 120, 132 and 42, but costs 1 % where all rows exist).
    constexpr int CPR = D / 8, RPI = 64 / CPR, NL = 16 / RPI;
    const int cp = lane % CPR;
    const int part = 16 * (wave ^ 4);
    const uint16_t* const q_head = (const uint16_t*)a.Q + (size_t)h * a.sq[1] + (long long)q0 * a.sq[2];
    const int q_last = a.Lq - 1 - q0;
    auto issue = [&](int b) {
        lds_u16* const to = lds + (b % STAGES) * STAGE;
        const rsrc_t rs = make_rsrc((const uint16_t*)a.K + (size_t)b * a.sk[0] + (size_t)h * a.sk[1], k_bytes);
        int rl = lane / CPR;                                 // addresses are formed anew: held over the loop they
        asm volatile("" : "+v"(rl));                         // would cost registers that there are not
        int k_voff[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u)
            k_voff[u] = rl * sk_bytes + (cp ^ swz_k<D>(part + u * RPI + rl)) * 16;
        if (key0 + part < a.Lk)
            load16_chain<NL, 1024>(lds_addr_of(to + part * D), (key0 + part) * sk_bytes, RPI * sk_bytes, k_voff, rs);
        const uint16_t* const base = q_head + (size_t)b * a.sq[0];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int r = part + u * RPI + rl;
            load16_to_lds(lds_addr_of(to + 2 * TILE + part * D + u * 512),
                          base + min(r, q_last) * a.sq[2] + (cp ^ swz_k<D>(r)) * 8);
        }
    };

    f32x16 acc[2], s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[kb][i] = 0.f;
    // S^T of the wavefront's 64 keys and 32 queries: three LDS reads per two matrix instructions
    const int row_chunk = n * D + (hh ^ swz_k<D>(n)) * 8;    // chunk 2 kk of the row: this ^ (16 kk)
    auto scores = [&](int b) {
        bf16x8 kr[KSTEPS][2], qr[KSTEPS];
        int rc = row_chunk;
        asm volatile("" : "+v"(rc));
        constexpr int AHEAD = 2;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
        auto read_step = [&](int kk) {
            const uint16_t* p = smem + (b % STAGES) * STAGE + (rc ^ (16 * kk));
            qr[kk] = *reinterpret_cast<const bf16x8*>(p + 2 * TILE + wq * 32 * D);
            kr[kk][0] = *reinterpret_cast<const bf16x8*>(p + wk * TILE);
            kr[kk][1] = *reinterpret_cast<const bf16x8*>(p + wk * TILE + 32 * D);
        };
#pragma unroll
        for (int kk = 0; kk < AHEAD; ++kk) read_step(kk);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            if (kk + AHEAD < KSTEPS) read_step(kk + AHEAD);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[kk][kb], qr[kk], s[kb], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 3 * AHEAD, 0);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            if (kk + AHEAD < KSTEPS) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        }
    };
    // entries outside the map or hidden by causality are computed too (from whatever is in LDS) and dropped when the tile
    // is written
    float l;
    auto add_exp = [&]() {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[kb][i] += __builtin_amdgcn_exp2f(fmaf(s[kb][i], sc, -l));
    };
    // One buffer: the next example's rows are requested once every wavefront has its scores and travel under the
    // exponentials, and under the arithmetic of the other workgroup of the compute unit.  Two (D <= 64): they travel
    // under the scores too, with one barrier less (B64 H16 D64 128 x 128 77.9 -> 75.2 us, 256 x 256 87.2 -> 83.8, against
    // 99.7 and 112 with four wavefronts and query rows in registers).
    issue(0);
    l = lp[0];
    for (int b = 0; b + 1 < a.B; ++b) {
        wait_vmem();                                         // the rows of example b have landed
        asm volatile("" : "+v"(l));
        __syncthreads();                                     // ... for everybody
        float lnext;
        auto next = [&]() {
            issue(b + 1);
            lnext = lp[(long long)(b + 1) * a.H * a.Lq];
        };
        if (STAGES == 2) next();
        if (seen) scores(b);
        if (STAGES == 1) {
            __syncthreads();                                 // everybody has read them
            next();
        }
        if (seen) add_exp();
        l = lnext;
    }
    wait_vmem();
    asm volatile("" : "+v"(l));
    __syncthreads();
    if (INIT && DEAL && a.causal) {
        // the zeros of block row nQB - 1 - qb are dealt to the workgroups of block row qb, which has at least as many visible
        // tiles
        const int zb = nQB - 1 - qb, z0 = zb * BM;
        const long long z_vis = min((long long)nKG, ((long long)z0 + (BM - 1) + off) / BK + 1);
        const long long my_vis = min((long long)nKG, block_last / BK + 1);
        for (long long zk = z_vis + kg; zk < nKG; zk += my_vis) write_zeros(z0, zk);
    }
    if (seen) scores(a.B - 1);
    // All 8 loads of a thread are in flight under the last exponentials.  A tile that lies inside the map and below the
    // causal limit for all its rows takes a branch-free path.  Where rows start 16-byte aligned the others take pieces
    // of four entries too, which are in the map or not as a whole (B3 H3 2000 x 500 D64, a quarter of the tiles: adding
    // 20.0 us with single entries that are read when the sums are there, 16.4).
    bool interior = vec_ok && q0 + BM <= a.Lq && (long long)key0 + BK <= a.Lk;
    if (a.causal) interior = interior && (long long)key0 + (BK - 1) <= (long long)q0 + off;
    float4 o[8];
    if (!INIT && interior) {
#pragma unroll
        for (int pass = 0; pass < 8; ++pass) o[pass] = *reinterpret_cast<const float4*>(map0 + c4 + pass * map_step);
    } else if (!INIT && vec_ok) {
        const float* const from = a.abar + ((size_t)h * a.Lq + q0) * a.Lk + key0 + min(c4, a.Lk - 4 - key0);
#pragma unroll
        for (int pass = 0; pass < 8; ++pass)
            o[pass] = *reinterpret_cast<const float4*>(from + (long long)min(r0 + 16 * pass, q_last) * a.Lk);
    }
    if (seen) add_exp();

    // transpose through LDS: lanes hold columns of keys per query, memory wants rows of keys
    float* outs = reinterpret_cast<float*>(smem);
    __syncthreads();                                         // K stages are consumed
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 v = make_float4(acc[kb][4 * g], acc[kb][4 * g + 1], acc[kb][4 * g + 2], acc[kb][4 * g + 3]);
            *reinterpret_cast<float4*>(outs + (wq * 32 + n) * OUT_LD + wk * 64 + 32 * kb + 8 * g + 4 * hh) = v;
        }
    __syncthreads();
    if (interior) {
        const float* src = outs + r0 * OUT_LD + c4;
#pragma unroll
        for (int pass = 0; pass < 8; ++pass) {
            if (INIT) o[pass] = make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 v = *reinterpret_cast<const float4*>(src + pass * 16 * OUT_LD);
            o[pass].x = fmaf(a.weight, v.x, o[pass].x);
            o[pass].y = fmaf(a.weight, v.y, o[pass].y);
            o[pass].z = fmaf(a.weight, v.z, o[pass].z);
            o[pass].w = fmaf(a.weight, v.w, o[pass].w);
            *reinterpret_cast<float4*>(map0 + c4 + pass * map_step) = o[pass];
        }
    } else if (vec_ok) {
        const float* src = outs + r0 * OUT_LD + c4;
#pragma unroll
        for (int pass = 0; pass < 8; ++pass) {
            const float4 v = *reinterpret_cast<const float4*>(src + pass * 16 * OUT_LD);
            // entries of this piece that the query sees; the others keep what they hold
            const long long sees = a.causal ? (long long)q0 + r0 + 16 * pass + off - key0 - c4 : 3;
            if (INIT) o[pass] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (sees >= 0) o[pass].x = fmaf(a.weight, v.x, o[pass].x);
            if (sees >= 1) o[pass].y = fmaf(a.weight, v.y, o[pass].y);
            if (sees >= 2) o[pass].z = fmaf(a.weight, v.z, o[pass].z);
            if (sees >= 3) o[pass].w = fmaf(a.weight, v.w, o[pass].w);
            if (r0 + 16 * pass <= q_last && key0 + c4 < a.Lk)
                *reinterpret_cast<float4*>(map0 + c4 + pass * map_step) = o[pass];
        }
    } else {                                                 // a row's 128 entries as four 32-entry pieces
        const int c1 = tid & 31;
        const float* src = outs + r0 * OUT_LD + c1;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float old[4][4];
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = q0 + r0 + 16 * (4 * half + p);
                    const long long key = (long long)key0 + c1 + 32 * e;
                    const bool kept = q < a.Lq && key < a.Lk && (!a.causal || key <= q + off);
                    old[p][e] = !INIT && kept ? map0[c1 + 32 * e + (4 * half + p) * map_step] : 0.f;
                }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = q0 + r0 + 16 * (4 * half + p);
                    const long long key = (long long)key0 + c1 + 32 * e;
                    const bool here = q < a.Lq && key < a.Lk, kept = here && (!a.causal || key <= q + off);
                    const float v = fmaf(a.weight, src[(4 * half + p) * 16 * OUT_LD + 32 * e], old[p][e]);
                    if (INIT ? here : kept) map0[c1 + 32 * e + (4 * half + p) * map_step] = kept ? v : 0.f;
                }
        }
    }
}

// lse2 = lse * log2(e): the row statistics as the attention forward call returns them (natural
// logarithm), in the form the accumulation kernel reads.
__global__ __launch_bounds__(256) void lse_to_base2_kernel(const float* __restrict__ lse, float* __restrict__ lse2,
                                                            long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) lse2[i] = lse[i] * kLog2e;                    // -inf (a query without keys) stays -inf
}

template <int D>
hipError_t launch_d(const MapArgs& a, const float* lse, hipStream_t stream)
{
    constexpr int NW = 4;
    const int nQB = (a.Lq + 32 * NW - 1) / (32 * NW), nKG = (a.Lk + 127) / 128;
    if (lse) {
        const long long n = (long long)a.B * a.H * a.Lq;
        hipLaunchKernelGGL(lse_to_base2_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, lse,
                           a.lse2, n);
    } else {
        hipLaunchKernelGGL((row_lse_kernel<D, NW>), dim3((unsigned)(a.B * a.H * nQB)), dim3(64 * NW), 0,
                           stream, a, nQB);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int total = a.H * nQB * nKG;
    const dim3 grid = grid_of(total, 512);
    if (a.init)
        hipLaunchKernelGGL((map_accumulate_kernel<D, true>), grid, dim3(512), 0, stream, a, nQB, nKG, total);
    else
        hipLaunchKernelGGL((map_accumulate_kernel<D, false>), grid, dim3(512), 0, stream, a, nQB, nKG, total);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_maps(const MapArgs& a, const float* lse, hipStream_t stream)
{
    switch (a.D) {
        case 32: return launch_d<32>(a, lse, stream);
        case 64: return launch_d<64>(a, lse, stream);
        case 128: return launch_d<128>(a, lse, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ap
