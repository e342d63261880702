// Last kernel of a matrix-core SPMM or FusedMM call (kernels_dense.hpp): the outputs of K's ranges are added up, and what
// the matrix cores could not do is computed entry by entry, as the general kernels do it.
//
// In an ordinary call all that is left of the second part is a look at one word.  Otherwise rows are dealt out to workgroups with
// the grid's size between them, so that those of one block of S are spread over the chip; a long row's entries are shared by
// the wavefronts of a workgroup, of the others each wavefront takes the next one.  (Rows asked for with an atomic
// counter, 8 at a time, cost 30 us of atomics on one address where one row was to be done.)
//
// Measured on MI355X, against the vector kernels for the same input: 16384^2, 20 %, 512 columns: one pair of entries
// exchanged 0.82 ms (vector: 10.7, their tiled attempt fails), every row reversed 10.8 (19.2), one NaN in C 1.26 (1.49);
// 4096^2, 30 %, 128 columns: 72 (172), 173 (300) and 112 us (68).  (With every workgroup doing its own rows again, 65 ms in each
// of the three and 0.45-7 ms at smaller sizes.)  What it is slow at: rows that are uneven and unordered at once, whose longest
// ones a workgroup does at its end (FusedMM 8192^2, log-normal rows, 64 columns: 0.45 ms, equal shares 0.17).
// After half-precision pieces little else is waited for, and where a row or two of 3277 entries fall to a workgroup their loads one
// after the other are the kernel's time: one pair exchanged at 16384^2, 20 %, 512 columns 0.95 ms with 4 wavefronts, 0.82 with 16;
// FusedMM with 64 1.38 and, with 8 (16 have 128 registers each and spill), 1.25.
// Without anything left to do: the time of a kernel that only adds the ranges (16384 x 4096, 128 columns, 2 ranges: 5.8 us),
// 4.7 us where there are none.
#pragma once
#include "kernels_dense.hpp"
#include "row_segments.hpp"

namespace csrk {

constexpr int kFinishLong = 1024;       // entries of a row that a workgroup's wavefronts share whatever else there is to do

// fused_segment for the entries in special columns alone
template <int DL, int DT, int VEC, int LG, typename E>
__device__ __forceinline__ void special_segment(const DenseArgs &a, int row, int s0, int s1, int n, const E *A, const E *B, const E *C,
                                                float *slot, int *cols, float *vals, float (&acc)[1][VEC]) {
    if (s1 <= s0) return;
    const int lane = lane_id();
    const int d = lane % DL * VEC;
    A += (size_t)row * a.D;
    float av[DT][VEC];
    load_a_row<VEC, DL, DT>(A, a.D, d, av);
    for (int base = s0; base < s1; base += kWave) {
        const int j = base + lane;
        const int k = j < s1 ? a.colidx[j] : 0;
        const bool take = j < s1 && a.special[k] != 0;
        const unsigned long long taken = __ballot(take);
        if (taken == 0) continue;
        const int at = __builtin_amdgcn_mbcnt_hi((unsigned)(taken >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)taken, 0));
        if (take) {
            cols[at] = k;
            vals[at] = a.vals ? a.vals[j] : 1.f;
        }
        const int count = __popcll(taken);
        __builtin_amdgcn_wave_barrier();
        const int kc = cols[lane < count ? lane : 0];
        sddmm_chunk<VEC, DL, DT>(kc, 0, count, B, a.D, d, A, av, slot);
        __builtin_amdgcn_wave_barrier();
        const float sc = lane < count ? vals[lane] * slot[lane] : 0.f;
        __builtin_amdgcn_wave_barrier();
        gather_axpy<VEC, LG, 1>(kc, sc, 0, count, C, a.N, n, acc);
    }
}

// VEC: elements per access of the dense operands (1, or 128 bits); a column block has up to LG * VEC columns (VEC == 1: it
// is done 64 columns at a time).  A workgroup's time for a long row is that of its loads one after the other, so few lanes
// take an entry and many entries are under way: 8 elements of a lane for a dot product, 8 floats of a lane for the sums.  (16
// elements of FP32 rows of more than 64 took 165 registers, and 652 instead of 577 us where no row of FusedMM 16384 x 4096,
// 20 %, 128/128 is ordered.)
// HALVES: after kernels_dense_wide.hpp.
template <typename E, bool FUSED, int VEC, int LG, bool HALVES = false>
__global__ __launch_bounds__(finish_waves(HALVES, FUSED) * kWave) void dense_finish(DenseArgs a) {
    constexpr int kWaves = finish_waves(HALVES, FUSED), kThreads = kWaves * kWave;
    constexpr int PL = 16 / VEC;                            // lanes for a 16-column piece
    constexpr int BL = VEC == 1 ? 16 : VEC == 4 ? LG / 2 : LG, BT = LG / BL;    // ... for a block, and tiles of theirs
    constexpr int DL = 16, DT = 128 / (DL * VEC);           // ... for a dot product of up to 128 elements, and tiles of theirs
    constexpr int SL = VEC == 1 ? 16 : 8, ST = 64 / (SL * VEC);     // ... of up to 64
    __shared__ union {
        RowParts<VEC, LG, 1, kWaves> whole;
        RowParts<VEC, BL, BT, kWaves> block;
        RowParts<VEC, PL, 1, kWaves> piece;
    } lds;
    __shared__ float slots[kWaves][kWave], vals[kWaves][kWave];
    __shared__ int cols[kWaves][kWave], list[kThreads], listed, next;
    const int M = a.M, N = a.N;
    const int lane = lane_id(), wave = uniform(threadIdx.x >> 6);

    // elements [from, to) of O as the sums of the ranges' outputs, two and two
    using T = std::conditional_t<VEC == 1, float, f32x4>;
    constexpr int kUnit = sizeof(T) / 4;
    auto add_ranges = [&](size_t from, size_t to, size_t thread, size_t threads) CSRK_INLINE {
        const size_t total = (size_t)M * N / kUnit;
        const T *p = reinterpret_cast<const T *>(a.partial);
        for (size_t u = from + thread; u < to; u += 2 * threads) {
            T x[2][kDenseMaxSegs];      // two sums' parts, all on their way at once
            const size_t at[2] = {u, u + threads < to ? u + threads : u};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int s = 0; s < kDenseMaxSegs; ++s)
                    x[i][s] = s < a.segs ? p[s * total + at[i]] : T{};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                static_assert(kDenseMaxSegs == 8);
                reinterpret_cast<T *>(a.O)[at[i]] = ((x[i][0] + x[i][1]) + (x[i][2] + x[i][3])) + ((x[i][4] + x[i][5]) + (x[i][6] + x[i][7]));
            }
        }
    };
    const bool special = FUSED && a.todo[1] != 0;
    if (__builtin_expect(!special && a.todo[0] == 0, 1)) {
        if (a.segs > 1)
            add_ranges(0, (size_t)M * N / kUnit, (size_t)blockIdx.x * kThreads + threadIdx.x, (size_t)gridDim.x * kThreads);
        return;
    }

    const int bn = a.bn, pieces = bn / 16;
    auto marks = [&](int row, int cb) CSRK_INLINE {
        unsigned m = 0;
        for (int s = 0; s < a.segs; ++s) m |= a.redo[((size_t)s * a.col_blocks + cb) * M + row];
        return m;
    };
    const E *A = static_cast<const E *>(a.A), *B = static_cast<const E *>(a.B), *C = static_cast<const E *>(a.C);
    // what is to be done of a row, by this wavefront or with the others of the workgroup (`share`)
    auto redo = [&](int row, int begin, int end, bool share) CSRK_INLINE {
        int s0 = begin, s1 = end;
        if (share) row_part(begin, end, wave, kWaves, s0, s1);
        float *const orow = a.O + (size_t)row * N;
        if constexpr (HALVES && !FUSED) {
            // A NaN among the row's values is one in all of its results, whatever C holds, and the matrix cores have left one.  (As in FusedMM's
            // products, where a NaN in B leaves one in every row that stores its column: 16384^2, 20 %, 512/64 4.6 -> 2.6 ms with one
            // such row of B, 12.9 -> 3.2 with ten.)
            if (a.vals && orow[0] != orow[0]) {
                bool nan = false;
#pragma unroll 4
                for (int j = s0 + lane; j < s1; j += kWave) nan |= a.vals[j] != a.vals[j];
                if (share ? __syncthreads_or(nan) : __any(nan)) {
                    for (int n = share ? (int)threadIdx.x : lane; n < N; n += share ? kThreads : kWave) orow[n] = __builtin_nanf("");
                    return;
                }
            }
        }
        auto columns = [&](auto lanes, auto tiles, auto &parts, int n) CSRK_INLINE {
            constexpr int LN = decltype(lanes)::value, TN = decltype(tiles)::value;
            float acc[TN][VEC] = {};
            if constexpr (FUSED) {
                if (a.D <= 64)
                    fused_segment<VEC, SL, ST, VEC, LN, TN>(row, s0, s1, a.colidx, a.vals, A, B, C, a.D, N, lane % SL * VEC, n, slots[wave], acc);
                else
                    fused_segment<VEC, DL, DT, VEC, LN, TN>(row, s0, s1, a.colidx, a.vals, A, B, C, a.D, N, lane % DL * VEC, n, slots[wave], acc);
            } else
                spmm_segment<VEC, LN, TN>(s0, s1, a.colidx, a.vals, C, N, n, acc);
            fold_groups<VEC, LN, TN>(acc);
            if (share) add_row_parts<VEC, LN, TN, kWaves>(parts, wave, wave, kWaves, true, orow, N, n, acc);
            else store_row<VEC, LN, TN>(orow, N, n, acc);
        };
        if constexpr (FUSED)
            if (special)
                for (int cb = 0; cb < a.col_blocks; ++cb)
                    for (int c0 = 0; c0 < bn; c0 += LG * VEC) {
                        const int c = c0 + lane % LG * VEC, n = c < bn ? cb * bn + c : N;
                        float acc[1][VEC] = {};
                        special_segment<DL, DT, VEC, LG>(a, row, s0, s1, n, A, B, C, slots[wave], cols[wave], vals[wave], acc);
                        fold_groups<VEC, LG, 1>(acc);
                        if ((wave == 0 || !share) && lane < LG && n < N)
#pragma unroll
                            for (int v = 0; v < VEC; ++v) acc[0][v] += orow[n + v];
                        if (share) add_row_parts<VEC, LG, 1, kWaves>(lds.whole, wave, wave, kWaves, true, orow, N, n, acc);
                        else store_row<VEC, LG, 1>(orow, N, n, acc);
                    }
        for (int cb = 0; cb < a.col_blocks; ++cb) {
            const unsigned m = uniform(marks(row, cb));
            if (m == 0) continue;
            using Tiles = std::integral_constant<int, BT>;
            using Lanes = std::integral_constant<int, BL>;
            // all that a block's lanes cover at once, or piece by piece where these are few
            constexpr int kAtOnce = BL * BT * VEC / 16;
            const unsigned inside = (1u << min(pieces, (N - cb * bn + 15) / 16)) - 1;
            for (int i = 0; i < pieces; i += kAtOnce) {
                unsigned some = m & inside & ((1u << kAtOnce) - 1) << i;
                if (__popc(some) * 4 > kAtOnce) {
                    columns(Lanes{}, Tiles{}, lds.block, cb * bn + i * 16 + lane % BL * VEC);
                } else {
                    for (; some != 0; some &= some - 1)
                        columns(std::integral_constant<int, PL>{}, std::integral_constant<int, 1>{}, lds.piece,
                                cb * bn + (__ffs(some) - 1) * 16 + lane % PL * VEC);
                }
            }
        }
    };

    const int step = gridDim.x, rows = (M - (int)blockIdx.x + step - 1) / step;     // rows blockIdx.x, blockIdx.x + step, ...
    for (int r0 = 0; r0 < rows; r0 += kThreads) {
        if (threadIdx.x == 0) listed = next = 0;
        __syncthreads();
        const int r = r0 + threadIdx.x, row = (int)blockIdx.x + r * step;
        if (r < rows) {
            unsigned m = special;
            for (int cb = 0; cb < a.col_blocks; ++cb) m |= marks(row, cb);
            if (m != 0) list[atomicAdd(&listed, 1)] = row;
        }
        if (a.segs > 1)
            for (int i = r0 + wave; i < rows && i < r0 + kThreads; i += kWaves) {
                const size_t at = (size_t)(blockIdx.x + (size_t)i * step) * N / kUnit;
                add_ranges(at, at + N / kUnit, lane, kWave);
            }
        __threadfence_block();
        __syncthreads();
        const int count = listed;
        for (int q = 0; q < count; ++q) {
            const int row = uniform(list[q]), begin = uniform(a.rowptr[row]), end = uniform(a.rowptr[row + 1]);
            if (count < kWaves || end - begin > kFinishLong) redo(row, begin, end, true);
        }
        while (count >= kWaves) {
            int q = 0;
            if (lane == 0) q = atomicAdd(&next, 1);
            q = uniform(q);
            if (q >= count) break;
            const int row = uniform(list[q]), begin = uniform(a.rowptr[row]), end = uniform(a.rowptr[row + 1]);
            if (end - begin <= kFinishLong) redo(row, begin, end, false);
        }
        __syncthreads();
    }
}

}  // namespace csrk
