// Row-segment kernels that gather dense rows straight from memory (the general path): every kernel here
// works on segments of rows - a run of stored entries of one row - and differs only in who gets which segment.
//
// Two ways of dealing out the work:
//
//  (1) Equal shares of the stored entries (`*_nnzsplit_kernel`).  Each wavefront ("worker") takes an equal
//      share of S's stored entries, whatever the row lengths are, finds the row its share starts in by a
//      wave-wide search of rowptr and walks the rows it touches.  This is the load balancing for skewed row
//      lengths: a row longer than a share is cut into segments handled by consecutive workers.
//       - SPMM / FusedMM: a worker writes the rows that START inside its share straight to O (if such a row
//         continues into later shares this is its first partial sum), and puts the partial sum of the row
//         that was already running when its share began (its "head") into a scratch row;
//         `combine_heads_kernel` then adds the heads to O in worker order, so the result does not depend on
//         timing.
//       - SDDMM: outputs are per stored entry, segments are disjoint, no combine.
//
//  (2) Whole rows (`*_rows_kernel`, and a branch of the kernels of (1) taken when the row analysis found the
//      rows about equally long): the paper's own decomposition, a row per work-item, with 2 or 4 wavefronts
//      of a workgroup sharing a row where there are few rows (its NT, section "SDDMM").  No search, no heads,
//      no combine step; faster wherever there is nothing to balance.
//
// Paper correspondence: the chunked index stream with look-ahead is the role of the VLC-sized blocks and
// prefetches in the paper's kernels (section "ESIMD Implementation"); the per-row arithmetic is
// Algorithms 1-3.
#pragma once
#include "device_util.hpp"
#include "kernels_ktile.hpp"
#include "row_segments.hpp"

namespace csrk {

// instantiations of the general SPMM kernel whose whole-row branch shares rows between wavefronts whatever M is
template <int VEC, int LG, int T>
constexpr bool kSpmmRowsAnyM = VEC >= 4 && T == 1;

// wavefronts per row when the kernel decides for itself (the whole-row branch of the general SPMM and SDDMM
// kernels): W is the number of wavefronts in the grid
__device__ __forceinline__ int rows_wpr_for(int M, int W) { return 2ll * M > W ? 1 : (4ll * M > W ? 2 : 4); }

template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void spmm_rows_body(int M, int N, const int32_t *__restrict__ rowptr,
                                               const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                               const E *__restrict__ Bmat, float *__restrict__ O, int wpr,
                                               RowParts<VEC, LG, T> &lds) {
    constexpr int TW = LG * VEC;
    const int lane = lane_id();
    const int wv = uniform(threadIdx.x >> 6);
    const int sub = wv % wpr, rows_per_block = kWavesPerBlock / wpr;
    const int n = blockIdx.y * (TW * T) + (lane % LG) * VEC;
    for (long long r0 = (long long)blockIdx.x * rows_per_block; r0 < M; r0 += (long long)gridDim.x * rows_per_block) {
        const long long r = r0 + wv / wpr;
        const bool valid = r < M;
        const int rs = valid ? uniform(rowptr[r]) : 0;
        const int re = valid ? uniform(rowptr[r + 1]) : 0;
        int s0, s1;
        row_part(rs, re, sub, wpr, s0, s1);
        float acc[T][VEC] = {};
        spmm_segment<VEC, LG, T>(s0, s1, colidx, vals, Bmat, N, n, acc);
        fold_groups<VEC, LG, T>(acc);
        if (wpr == 1) {
            if (valid) store_row<VEC, LG, T>(O + (size_t)r * N, N, n, acc);
        } else {
            add_row_parts<VEC, LG, T>(lds, wv, sub, wpr, valid, O + (size_t)(valid ? r : 0) * N, N, n, acc);
        }
    }
}

template <int VEC, int LG, int T, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void spmm_rows_kernel(
    int M, int N, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ vals, const E *__restrict__ Bmat, float *__restrict__ O, int wpr) {
    __shared__ RowParts<VEC, LG, T> lds;
    spmm_rows_body<VEC, LG, T>(M, N, rowptr, colidx, vals, Bmat, O, wpr, lds);
}

template <int VEC, int LG, int T, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void spmm_nnzsplit_kernel(
    int M, int N, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ vals, const E *__restrict__ Bmat, float *__restrict__ O,
    float *__restrict__ head, int32_t *__restrict__ head_row, const int32_t *__restrict__ gate,
    const int32_t *__restrict__ even) {
    constexpr int TW = LG * VEC;
    if (gate && ktile_ok(gate)) return;     // the LDS-tiled kernel has done this call
    const int lane = lane_id();
    const int W = gridDim.x * kWavesPerBlock;
    const int w = uniform(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    const int n = blockIdx.y * (TW * T) + (lane % LG) * VEC;
    if (even && *even != 0) {
        // The row analysis found no row much longer than the mean: nothing to balance, so whole rows are dealt out
        // (1, 2 or 4 wavefronts per row, whatever keeps the wavefronts of the grid busy) - no search for a share's
        // first row, no heads (combine_heads_kernel stands down on the same flag).  Measured 10-60 % faster than
        // the equal-nonzero split on such matrices.
        // (Sharing rows between wavefronts only where it costs no occupancy: not in the 512-wide instantiation,
        // 91 -> 99 VGPRs; that one takes whole rows with more than half as many rows as wavefronts.)
        if constexpr (kSpmmRowsAnyM<VEC, LG, T>) {
            __shared__ RowParts<VEC, LG, T> lds;
            spmm_rows_body<VEC, LG, T>(M, N, rowptr, colidx, vals, Bmat, O, rows_wpr_for(M, W), lds);
            return;
        } else if (2ll * M > W) {
            for (int r = w; r < M; r += W) {
                const int rs = uniform(rowptr[r]);
                const int re = uniform(rowptr[r + 1]);
                float acc[T][VEC] = {};
                spmm_segment<VEC, LG, T>(rs, re, colidx, vals, Bmat, N, n, acc);
                fold_groups<VEC, LG, T>(acc);
                store_row<VEC, LG, T>(O + (size_t)r * N, N, n, acc);
            }
            return;
        }
    }
    const Share sh = make_share(rowptr, M, w, W);
    if (!sh.active) {
        if (blockIdx.y == 0 && lane == 0) head_row[w] = -1;
        return;
    }
    int r = wave_lower_bound(rowptr, M, sh.lo);
    int hr = -1;
    if (sh.lo < sh.nnz) {
        const int start = uniform(rowptr[r]);      // r <= M and rowptr[M] = nnz
        if (start != sh.lo) {                      // share begins inside row r-1
            hr = r - 1;
            float acc[T][VEC] = {};
            spmm_segment<VEC, LG, T>(sh.lo, start < sh.hi ? start : sh.hi, colidx, vals, Bmat, N, n, acc);
            fold_groups<VEC, LG, T>(acc);
            store_row<VEC, LG, T>(head + (size_t)w * N, N, n, acc);
        }
    }
    if (blockIdx.y == 0 && lane == 0) head_row[w] = hr;
    for (; r < M; ++r) {
        const int rs = uniform(rowptr[r]);
        if (!sh.last && rs >= sh.hi) break;
        const int re = uniform(rowptr[r + 1]);
        float acc[T][VEC] = {};
        spmm_segment<VEC, LG, T>(rs, re < sh.hi ? re : sh.hi, colidx, vals, Bmat, N, n, acc);
        fold_groups<VEC, LG, T>(acc);
        store_row<VEC, LG, T>(O + (size_t)r * N, N, n, acc);
    }
}

// O[r, :] += head[w, :] + head[w+1, :] + ... for the run of workers whose head is row r.
// One wavefront per worker, lanes over the output columns; only the first worker of a run does the
// adding, in worker order, so sums are reproducible.  `vec4`: N is a multiple of 4 and O and head
// are 16-byte aligned.
// This is the last kernel of every SPMM / FusedMM call.  If a tiled kernel did the call there are no heads;
// if that kernel's launch was K-split (S > 1) its S partial outputs (`partial`, count4 float4s each) still
// have to be added into O, which this grid then does instead.
__global__ __launch_bounds__(kBlockThreads) void combine_heads_kernel(int M, int N, int W, float *__restrict__ O,
                                                                       const float *__restrict__ head,
                                                                       const int32_t *__restrict__ head_row,
                                                                       const int32_t *__restrict__ gate, int vec4,
                                                                       size_t count4, int S, const float4 *partial,
                                                                       const int32_t *__restrict__ even, int any_m) {
    if (gate && ktile_ok(gate)) {
        if (S > 1) ksplit_reduce(count4, S, partial, reinterpret_cast<float4 *>(O));
        return;
    }
    // the general kernel dealt out whole rows (SPMM: whenever the rows are even; FusedMM: with enough rows too)
    if (even && *even != 0 && (any_m || 2ll * M > W)) return;
    const int w = uniform(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    if (w >= W) return;
    const int r = uniform(head_row[w]);
    if (r < 0) return;
    if (w > 0 && uniform(head_row[w - 1]) == r) return;
    int wend = w + 1;
    while (wend < W && uniform(head_row[wend]) == r) ++wend;
    const int lane = lane_id();
    float *orow = O + (size_t)r * N;
    if (vec4) {
        for (int n = lane * 4; n < N; n += kWave * 4) {
            float s[4];
            load_vec<4>(orow + n, s);
            for (int ww = w; ww < wend; ++ww) {
                float h[4];
                load_vec<4>(head + (size_t)ww * N + n, h);
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += h[v];
            }
            store_vec<4>(orow + n, s);
        }
    } else {
        for (int n = lane; n < N; n += kWave) {
            float s = orow[n];
            for (int ww = w; ww < wend; ++ww) s += head[(size_t)ww * N + n];
            orow[n] = s;
        }
    }
}

// SDDMM with a row per 1, 2 or 4 wavefronts (consecutive parts of the row; outputs are per stored entry, so
// nothing to add up): see spmm_rows_kernel.
template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void sddmm_rows_body(int M, int D, const int32_t *__restrict__ rowptr,
                                                const int32_t *__restrict__ colidx, const float *vals,
                                                const E *__restrict__ A, const E *__restrict__ Bmat, float *P,
                                                int wpr, float *slot) {
    const int lane = lane_id();
    const int wv = uniform(threadIdx.x >> 6);
    const int sub = wv % wpr, rows_per_block = kWavesPerBlock / wpr;
    const int d = (lane % LG) * VEC;
    for (long long r = (long long)blockIdx.x * rows_per_block + wv / wpr; r < M; r += (long long)gridDim.x * rows_per_block) {
        const int rs = uniform(rowptr[r]);
        const int re = uniform(rowptr[r + 1]);
        int s0, s1;
        row_part(rs, re, sub, wpr, s0, s1);
        sddmm_segment<VEC, LG, T>((int)r, s0, s1, colidx, vals, A, Bmat, P, D, d, slot);
    }
}

template <int VEC, int LG, int T, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void sddmm_rows_kernel(
    int M, int D, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx, const float *vals,
    const E *__restrict__ A, const E *__restrict__ Bmat, float *P, int wpr) {
    __shared__ float slots[kWavesPerBlock][kWave];
    sddmm_rows_body<VEC, LG, T>(M, D, rowptr, colidx, vals, A, Bmat, P, wpr, slots[threadIdx.x >> 6]);
}

// P may alias vals, so neither is __restrict__.
template <int VEC, int LG, int T, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void sddmm_nnzsplit_kernel(
    int M, int D, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *vals, const E *__restrict__ A, const E *__restrict__ Bmat, float *P,
    const int32_t *__restrict__ gate, const int32_t *__restrict__ even) {
    __shared__ float slots[kWavesPerBlock][kWave];
    if (gate && ktile_ok(gate)) return;     // the LDS-tiled kernel has done this call
    const int lane = lane_id();
    const int W = gridDim.x * kWavesPerBlock;
    const int wv = threadIdx.x >> 6;
    const int w = uniform(blockIdx.x * kWavesPerBlock + wv);
    const int d = (lane % LG) * VEC;
    if (even && *even != 0) {               // whole rows: see spmm_nnzsplit_kernel
        sddmm_rows_body<VEC, LG, T>(M, D, rowptr, colidx, vals, A, Bmat, P, rows_wpr_for(M, W), slots[wv]);
        return;
    }
    const Share sh = make_share(rowptr, M, w, W);
    if (!sh.active || sh.lo >= sh.nnz) return;
    float *slot = slots[wv];
    // row containing entry lo: the last row that starts at or before lo
    int r = wave_lower_bound(rowptr, M, sh.lo);
    if (uniform(rowptr[r]) != sh.lo) --r;
    for (; r < M; ++r) {
        const int rs = uniform(rowptr[r]);
        if (rs >= sh.hi) break;
        const int re = uniform(rowptr[r + 1]);
        const int s0 = rs > sh.lo ? rs : sh.lo;
        const int s1 = re < sh.hi ? re : sh.hi;
        if (s1 <= s0) continue;
        sddmm_segment<VEC, LG, T>(r, s0, s1, colidx, vals, A, Bmat, P, D, d, slot);
    }
}

// FusedMM with a row per 1, 2 or 4 wavefronts: see spmm_rows_kernel.
template <int VD, int LD, int TD, int VN, int LN, int TN, typename E>
__device__ __forceinline__ void fusedmm_rows_body(int M, int D, int N, const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                                  const E *__restrict__ A, const E *__restrict__ Bmat,
                                                  const E *__restrict__ Cmat, float *__restrict__ O, int wpr,
                                                  float *slot, RowParts<VN, LN, TN> &lds) {
    constexpr int TWN = LN * VN;
    const int lane = lane_id();
    const int wv = uniform(threadIdx.x >> 6);
    const int sub = wv % wpr, rows_per_block = kWavesPerBlock / wpr;
    const int d = (lane % LD) * VD;
    const int n = blockIdx.y * (TWN * TN) + (lane % LN) * VN;
    for (long long r0 = (long long)blockIdx.x * rows_per_block; r0 < M; r0 += (long long)gridDim.x * rows_per_block) {
        const long long r = r0 + wv / wpr;
        const bool valid = r < M;
        const int rs = valid ? uniform(rowptr[r]) : 0;
        const int re = valid ? uniform(rowptr[r + 1]) : 0;
        int s0, s1;
        row_part(rs, re, sub, wpr, s0, s1);
        float acc[TN][VN] = {};
        fused_segment<VD, LD, TD, VN, LN, TN>((int)(valid ? r : 0), s0, s1, colidx, vals, A, Bmat, Cmat, D, N, d, n, slot,
                                              acc);
        fold_groups<VN, LN, TN>(acc);
        if (wpr == 1) {
            if (valid) store_row<VN, LN, TN>(O + (size_t)r * N, N, n, acc);
        } else {
            add_row_parts<VN, LN, TN>(lds, wv, sub, wpr, valid, O + (size_t)(valid ? r : 0) * N, N, n, acc);
        }
    }
}

template <int VD, int LD, int TD, int VN, int LN, int TN, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void fusedmm_rows_kernel(
    int M, int D, int N, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ vals, const E *__restrict__ A, const E *__restrict__ Bmat,
    const E *__restrict__ Cmat, float *__restrict__ O, int wpr) {
    __shared__ float slots[kWavesPerBlock][kWave];
    __shared__ RowParts<VN, LN, TN> lds;
    fusedmm_rows_body<VD, LD, TD, VN, LN, TN>(M, D, N, rowptr, colidx, vals, A, Bmat, Cmat, O, wpr,
                                              slots[threadIdx.x >> 6], lds);
}

template <int VD, int LD, int TD, int VN, int LN, int TN, typename E = float>
__global__ __launch_bounds__(kBlockThreads) void fusedmm_nnzsplit_kernel(
    int M, int D, int N, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ vals, const E *__restrict__ A, const E *__restrict__ Bmat,
    const E *__restrict__ Cmat, float *__restrict__ O, float *__restrict__ head,
    int32_t *__restrict__ head_row, const int32_t *__restrict__ gate, const int32_t *__restrict__ even) {
    __shared__ float slots[kWavesPerBlock][kWave];
    constexpr int TWN = LN * VN;
    if (gate && ktile_ok(gate)) return;
    const int lane = lane_id();
    const int W = gridDim.x * kWavesPerBlock;
    const int wv = threadIdx.x >> 6;
    const int w = uniform(blockIdx.x * kWavesPerBlock + wv);
    const int d = (lane % LD) * VD;
    const int n = blockIdx.y * (TWN * TN) + (lane % LN) * VN;
    float *slot = slots[wv];
    // Whole rows, round robin (see spmm_nnzsplit_kernel) - here only with more than half as many rows as wavefronts
    // and one wavefront per row: sharing rows between wavefronts costs registers that the equal-share branch below,
    // the one skewed matrices take, needs for full occupancy (62 -> 70 VGPRs, 12 % slower on `fused8k_skew`).
    if (even && *even != 0 && 2ll * M > W) {
        for (int r = w; r < M; r += W) {
            const int rs = uniform(rowptr[r]);
            const int re = uniform(rowptr[r + 1]);
            float acc[TN][VN] = {};
            fused_segment<VD, LD, TD, VN, LN, TN>(r, rs, re, colidx, vals, A, Bmat, Cmat, D, N, d, n, slot, acc);
            fold_groups<VN, LN, TN>(acc);
            store_row<VN, LN, TN>(O + (size_t)r * N, N, n, acc);
        }
        return;
    }
    const Share sh = make_share(rowptr, M, w, W);
    if (!sh.active) {
        if (blockIdx.y == 0 && lane == 0) head_row[w] = -1;
        return;
    }
    int r = wave_lower_bound(rowptr, M, sh.lo);
    int hr = -1;
    if (sh.lo < sh.nnz) {
        const int start = uniform(rowptr[r]);
        if (start != sh.lo) {
            hr = r - 1;
            float acc[TN][VN] = {};
            fused_segment<VD, LD, TD, VN, LN, TN>(hr, sh.lo, start < sh.hi ? start : sh.hi, colidx, vals, A, Bmat,
                                                  Cmat, D, N, d, n, slot, acc);
            fold_groups<VN, LN, TN>(acc);
            store_row<VN, LN, TN>(head + (size_t)w * N, N, n, acc);
        }
    }
    if (blockIdx.y == 0 && lane == 0) head_row[w] = hr;
    for (; r < M; ++r) {
        const int rs = uniform(rowptr[r]);
        if (!sh.last && rs >= sh.hi) break;
        const int re = uniform(rowptr[r + 1]);
        float acc[TN][VN] = {};
        fused_segment<VD, LD, TD, VN, LN, TN>(r, rs, re < sh.hi ? re : sh.hi, colidx, vals, A, Bmat, Cmat, D, N, d,
                                              n, slot, acc);
        fold_groups<VN, LN, TN>(acc);
        store_row<VN, LN, TN>(O + (size_t)r * N, N, n, acc);
    }
}

}  // namespace csrk
