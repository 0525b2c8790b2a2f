// Transpose of a block-sparse layout: for every (head, block column) the stored tiles of that
// column in ascending block-row order.  The backward pass accumulates dK and dV per block
// column and walks this list.
//
// One workgroup per (head, 64 block columns), one launch.  The workgroup sweeps the tiles of its
// head (a wavefront per block row, a lane per tile), sets one bit per stored tile in an LDS table
// [column][block row], and counts the tiles of earlier columns, which makes its part of col_ptr
// independent of the other workgroups: the tiles of a head occupy the same range of positions in
// both orders.  A tile's place in its column is then the number of bits below its own.  Bits and
// integer counts are order-free, so the result is fixed without ordered atomics.
//
// The work is a chain of dependent loads, not bandwidth: a column per thread that binary-searched
// one block row after another took 67 + 9 + 61 us in three launches for 16 heads of 64 x 64 tiles
// (2080 stored per head); this form takes 7 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"

namespace ap {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kCols = 64;                                    // block columns per workgroup
constexpr int kSegRows = 4096;                               // block rows whose bits are in LDS at a time (33 KB)

__global__ __launch_bounds__(kThreads) void transpose_kernel(const int32_t* __restrict__ row_ptr,
                                                             const int32_t* __restrict__ col_idx, int H, int nQB,
                                                             int nKB, int n_chunks, long long cap,
                                                             int32_t* __restrict__ col_ptr,
                                                             int32_t* __restrict__ row_idx,
                                                             int32_t* __restrict__ tile_idx)
{
    extern __shared__ uint32_t bits[];                       // [kCols][pitch]
    __shared__ int s_cnt[kCols], s_base[kCols], s_before;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = block_index();
    if (blk >= H * n_chunks) return;
    const int h = blk / n_chunks;
    const int kb0 = (blk % n_chunks) * kCols;
    const int seg_rows = min(nQB, kSegRows);
    const int pitch = ((seg_rows + 31) >> 5) | 1;            // odd: the columns of a row fall into different banks

    // every tile (block row qb, column kb, position t) of block rows [q0, q1)
    auto sweep = [&](int q0, int q1, auto&& body) {
        constexpr int U = 4;                                 // block rows in flight per wavefront
        for (int qw = q0 + wave; qw < q1; qw += U * kWaves) {
            int lo[U], hi[U], c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int qb = qw + u * kWaves;
                const int r = h * nQB + min(qb, nQB - 1);
                lo[u] = row_ptr[r];
                hi[u] = qb < q1 ? (int)min((long long)row_ptr[r + 1], cap) : lo[u];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = lo[u] + lane < hi[u] ? col_idx[lo[u] + lane] : -1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int qb = qw + u * kWaves;
                if (c[u] >= 0) body(qb, c[u], lo[u] + lane);
                for (int t = lo[u] + 64 + lane; t < hi[u]; t += 64) body(qb, col_idx[t], t);
            }
        }
    };
    auto clear_bits = [&]() {
        for (int i = tid; i < kCols * pitch; i += kThreads) bits[i] = 0;
    };
    auto set_bit = [&](int q0, int qb, int kb) {
        atomicOr(&bits[(kb - kb0) * pitch + ((qb - q0) >> 5)], 1u << ((qb - q0) & 31));
    };

    clear_bits();
    if (tid < kCols) s_cnt[tid] = 0;
    if (tid == 0) s_before = 0;
    __syncthreads();
    int before = 0;
    sweep(0, nQB, [&](int qb, int kb, int) {
        if (kb < kb0) ++before;
        else if (kb < kb0 + kCols) {
            atomicAdd(&s_cnt[kb - kb0], 1);
            if (qb < seg_rows) set_bit(0, qb, kb);
        }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    if (lane == 0 && before) atomicAdd(&s_before, before);
    __syncthreads();
    if (wave == 0) {
        const int cnt = s_cnt[lane];
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        const int base = (int)min((long long)row_ptr[(size_t)h * nQB], cap) + s_before + incl - cnt;
        s_base[lane] = base;
        if (kb0 + lane < nKB) col_ptr[(size_t)h * nKB + kb0 + lane] = base;
        if (h == H - 1 && kb0 + lane == nKB - 1) col_ptr[(size_t)H * nKB] = base + cnt;
    }
    __syncthreads();
    for (int q0 = 0; q0 < nQB; q0 += seg_rows) {
        const int q1 = min(nQB, q0 + seg_rows);
        if (q0 > 0) {                                        // more block rows than the table holds
            clear_bits();
            __syncthreads();
            sweep(q0, q1, [&](int qb, int kb, int) {
                if (kb >= kb0 && kb < kb0 + kCols) set_bit(q0, qb, kb);
            });
            __syncthreads();
        }
        sweep(q0, q1, [&](int qb, int kb, int t) {
            if (kb < kb0 || kb >= kb0 + kCols) return;
            const uint32_t* col = bits + (kb - kb0) * pitch;
            const int w = (qb - q0) >> 5;
            int pos = s_base[kb - kb0] + __popc(col[w] & ((1u << ((qb - q0) & 31)) - 1u));
            for (int i = 0; i < w; ++i) pos += __popc(col[i]);
            row_idx[pos] = qb;
            tile_idx[pos] = t;
        });
        if (q1 < nQB) {                                      // the next block rows follow these in every column
            __syncthreads();
            if (tid < kCols) {
                int n = 0;
                for (int i = 0; i < pitch; ++i) n += __popc(bits[tid * pitch + i]);
                s_base[tid] += n;
            }
            __syncthreads();
        }
    }
}

}  // namespace

hipError_t launch_layout_transpose(const int32_t* row_ptr, const int32_t* col_idx, int H, int nQB,
                                   int nKB, long long cap, int32_t* col_ptr, int32_t* row_idx,
                                   int32_t* tile_idx, hipStream_t stream)
{
    const int n_chunks = (nKB + kCols - 1) / kCols;
    const int seg_rows = nQB < kSegRows ? nQB : kSegRows;
    const size_t lds = (size_t)kCols * (((seg_rows + 31) / 32) | 1) * sizeof(uint32_t);
    hipLaunchKernelGGL(transpose_kernel, grid_of((long long)H * n_chunks, kThreads), dim3(kThreads), lds, stream, row_ptr, col_idx,
                       H, nQB, nKB, n_chunks, cap, col_ptr, row_idx, tile_idx);
    return hipGetLastError();
}

}  // namespace ap
