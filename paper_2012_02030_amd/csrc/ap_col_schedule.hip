// Column schedule: the visit schedule of the backward pass's dK/dV kernel, a re-packing of the
// transposed layout.  For every (head, block column) the stored tiles are walked in ascending
// block-row order; a tile in which at least `min_rows` query rows hold a visible kept entry stays
// a run of 64 consecutive queries, the rows of all other tiles that hold one are packed, in
// ascending order, into gathered entries of 64 arbitrary queries.  Every entry carries, per
// query slot, the 64-bit word of kept keys inside this block column with the causal limit
// folded in.  Same structure as the row schedule with the roles of rows and columns swapped.
//
// One workgroup of four wavefronts (one, for many short columns) per block column, one lane per tile row.  Up
// to 64 tiles at a time are held in registers (every wavefront takes every fourth tile, all its loads in flight at
// once); which query rows of a tile hold something is one ballot per tile, shared through LDS; every
// wavefront then knows, with a lane per tile, the entry slot of every tile (ranks and prefix sums
// over the lanes) and writes its own tiles.  All positions depend on ballots only, so the emitted
// order is fixed: no atomics.  The time is the chain of dependent loads of one block column (position
// list -> bitmap words): one wavefront that took the tiles one after another, twice, needed 44 us at
// 16 heads of 64 x 64 tiles, this form 13 us.  A second kernel appends, behind the entry counts, the
// order in which the dK/dV kernel should visit the block columns of each head.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ap_internal.h"

namespace ap {

namespace {

constexpr int kPer = 16;                                     // tiles of one wavefront at a time

template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void build_col_schedule_kernel(
    const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ row_idx,
    const int32_t* __restrict__ tile_idx, const uint64_t* __restrict__ bitmaps, int nKB, int Lq, int Lk,
    int causal, int min_rows, int n_cols, Schedule s)
{
    constexpr int kSeg = kWaves * kPer;                      // tiles held at a time
    __shared__ unsigned long long s_rows[kSeg];              // query rows of every tile that hold something
    const int c = block_index();
    if (c >= n_cols) return;
    const int kb = c % nKB;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long off = (long long)Lk - Lq;
    const int c0 = col_ptr[c], c1 = col_ptr[c + 1];
    const bool one_segment = c1 - c0 <= kSeg;

    uint64_t word[kPer];                                     // this lane's row of this wavefront's tiles
    int q0_lane = 0;                                         // lane t: first query of tile t of the segment
    auto load_segment = [&](int seg, int n) {
        int ti_lane = 0;
        if (lane < n) {
            q0_lane = row_idx[seg + lane] * 64;
            ti_lane = tile_idx[seg + lane];
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kWaves + wave;
            if (t >= n) break;                               // uniform
            word[u] = bitmaps[(size_t)__builtin_amdgcn_readlane(ti_lane, t) * 64 + lane];
        }
        __syncthreads();                                     // s_rows of the previous segment is no longer read
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kWaves + wave;
            if (t >= n) break;
            if (causal) {
                const long long lim = (long long)__builtin_amdgcn_readlane(q0_lane, t) + lane + off - (long long)kb * 64;
                if (lim < 0) word[u] = 0;
                else if (lim < 63) word[u] &= (2ull << lim) - 1ull;
            }
            const unsigned long long rows = __ballot(word[u] != 0);
            if (lane == 0) s_rows[t] = rows;
        }
        __syncthreads();
    };

    // Sweep 0: tiles that stay runs of 64 consecutive queries, in order; sweep 1: the rows of the
    // others, query number p of the block column's gathered stream in slot p % 64 of gathered entry p / 64.
    int n_cons = 0;
    for (int seg = c0; seg < c1; seg += kSeg) {
        const int n = min(kSeg, c1 - seg);
        load_segment(seg, n);
        const int nrows = lane < n ? __popcll(s_rows[lane]) : 0;
        const unsigned long long cons = __ballot(nrows > 0 && nrows >= min_rows);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kWaves + wave;
            if (t >= n) break;
            if (!((cons >> t) & 1ull)) continue;
            const size_t e = (size_t)c0 + n_cons + __popcll(cons & ((1ull << t) - 1ull));
            if (lane == 0) s.start[e] = __builtin_amdgcn_readlane(q0_lane, t);
            s.bitmaps[e * 64 + lane] = word[u];
        }
        n_cons += __popcll(cons);
    }
    const size_t first = (size_t)c0 + n_cons;
    int stream = 0;                                          // gathered queries so far
    for (int seg = c0; seg < c1; seg += kSeg) {
        const int n = min(kSeg, c1 - seg);
        if (!one_segment) load_segment(seg, n);
        const unsigned long long mine = lane < n ? s_rows[lane] : 0ull;   // lane t: tile t
        int cnt = __popcll(mine);
        if (cnt >= min_rows) cnt = 0;                        // already emitted as a run
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = u * kWaves + wave;
            if (t >= n) break;
            if (__builtin_amdgcn_readlane(cnt, t) == 0) continue;
            const unsigned long long rows = s_rows[t];
            const int p0 = stream + __builtin_amdgcn_readlane(incl - cnt, t);
            if (word[u] != 0) {
                const int p = p0 + __popcll(rows & ((1ull << lane) - 1ull));
                const size_t e = first + (size_t)(p >> 6);
                s.cols[e * 64 + (p & 63)] = __builtin_amdgcn_readlane(q0_lane, t) + lane;
                s.bitmaps[e * 64 + (p & 63)] = word[u];
                if ((p & 63) == 0) s.start[e] = -1;
            }
        }
        stream += __builtin_amdgcn_readlane(incl, 63);
    }
    const int fill = stream & 63;
    if (wave == 0 && fill > 0 && lane >= fill) {             // empty slots of the last gathered entry
        const size_t open = first + (size_t)(stream >> 6);
        s.cols[open * 64 + lane] = Lq;                       // beyond the last query: reads as zeros
        s.bitmaps[open * 64 + lane] = 0;
    }
    if (threadIdx.x == 0) s.cnt[c] = n_cons + ((stream + 63) >> 6);
}

// Visiting order of the block columns of one head: columns with at least twice the head's mean
// number of entries ("heavy": their workgroups run longest and should start first) in ascending
// order, then the others in ascending order.  One wavefront per head.
//   order  [H*nKB]  block column at each position      n_heavy [H]  number of heavy columns
__global__ __launch_bounds__(64) void col_order_kernel(const int32_t* __restrict__ cnt, int nKB,
                                                       int32_t* __restrict__ order, int32_t* __restrict__ n_heavy)
{
    const int h = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t* c = cnt + (size_t)h * nKB;
    long long sum = 0;
    for (int k = lane; k < nKB; k += 64) sum += c[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const long long limit = (2 * sum + nKB - 1) / nKB;       // ceil(2 * mean)
    int pos = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int k0 = 0; k0 < nKB; k0 += 64) {
            const int k = k0 + lane;
            const bool heavy = k < nKB && c[k] >= limit && c[k] > 1;
            const bool take = k < nKB && heavy == (pass == 0);
            const unsigned long long m = __ballot(take);
            if (take) order[(size_t)h * nKB + pos + __popcll(m & ((1ull << lane) - 1ull))] = k;
            pos += __popcll(m);
        }
        if (pass == 0 && lane == 0) n_heavy[h] = pos;
    }
}

}  // namespace

hipError_t launch_build_col_schedule(const int32_t* col_ptr, const int32_t* row_idx, const int32_t* tile_idx,
                                     const uint64_t* bitmaps, int H, int Lq, int Lk, int causal,
                                     int min_rows, const Schedule& s, hipStream_t stream)
{
    const int nKB = (Lk + 63) / 64;
    // Up to 16 block rows a wavefront holds all tiles of a column.  Four of them per column are faster as long as
    // all are resident (256 compute units, 32 wavefronts each), one where they take turns:
    // 16 heads of 512 x 16384 9.0 us (20.1 with four), of 64 x 16384 5.2 (18.0), of 1024 x 1024 7.4 (5.0).
    const auto run = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, grid_of((long long)H * nKB, 64 * waves), dim3(64 * waves), 0, stream, col_ptr, row_idx,
                           tile_idx, bitmaps, nKB, Lq, Lk, causal, min_rows, H * nKB, s);
    };
    if ((Lq + 63) / 64 <= kPer && (long long)H * nKB * 4 > 256 * 32) run(build_col_schedule_kernel<1>, 1);
    else run(build_col_schedule_kernel<4>, 4);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int32_t* order = s.cnt + (size_t)H * nKB;                // the count array carries the visiting order
    hipLaunchKernelGGL(col_order_kernel, dim3((unsigned)H), dim3(64), 0, stream, s.cnt, nKB, order,
                       order + (size_t)H * nKB);
    return hipGetLastError();
}

}  // namespace ap
