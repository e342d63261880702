// Pieces of the kernels that gather dense rows straight from memory: one run of stored entries of one row (a segment) in SPMM,
// SDDMM and FusedMM, and a row shared by the wavefronts of a workgroup.
//
// Column indices and values are streamed in coalesced chunks of 64 (one per lane), the next chunk being loaded while
// the current one is consumed.  A group of LG lanes covers the dense width with VEC floats per lane, so 64/LG entries
// are processed side by side; their dense rows are gathered with one (128-bit when VEC == 4) load per lane, several
// steps' gathers in flight together (gather_axpy).
#pragma once
#include "device_util.hpp"

namespace csrk {

constexpr int kBlockThreads = 256;
constexpr int kWavesPerBlock = kBlockThreads / kWave;

// f(t) for t = t0, t0+stride, ... < t1, in blocks of U statically unrolled calls and a
// one-at-a-time remainder.
template <int U, typename F>
__device__ __forceinline__ void for_unrolled(int t0, int t1, int stride, F &&f) {
    int t = t0;
    for (; t + U * stride <= t1; t += U * stride) {
#pragma unroll
        for (int u = 0; u < U; ++u) f(t + u * stride);
    }
    for (; t < t1; t += stride) f(t);
}

// ---------------------------------------------------------------------------------
// Gather-and-accumulate over the entries [t0, t1) of one chunk (entry t: column in lane t
// of `kc`, scale in lane t of `sc`):
//     acc[tt][v] += sc_t * Mat[kc_t, n + tt*TW + v]
// A group of LG lanes covers the dense width, NPAR = 64/LG entries go side by side.
//
// The gathers of a block of U steps are all requested before the first is used.  That
// only happens if no load sits under a condition (the compiler waits for such a load on
// the spot, which would put the U gathers one after the other): every lane loads in every
// step, with columns beyond N moved to column 0 and steps beyond the chunk's end moved
// to entry t0, and the condition is applied to the multiply-adds instead.
// ---------------------------------------------------------------------------------
template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void gather_axpy(int kc, float sc, int t0, int t1, const E *__restrict__ Mat, int N,
                                            int n, float (&acc)[T][VEC]) {
    constexpr int NPAR = kWave / LG;
    constexpr int TW = LG * VEC;
    constexpr int U = NPAR == 1 ? 8 : 4;         // steps per full block
    constexpr int UR = NPAR == 1 ? 4 : 2;        // steps per block of the remainder
    const int g = lane_id() / LG;
    int off[T];
    bool col_ok[T];
#pragma unroll
    for (int tt = 0; tt < T; ++tt) {
        col_ok[tt] = n + tt * TW < N;
        off[tt] = col_ok[tt] ? n + tt * TW : 0;
    }
    auto block = [&](int t, auto uc) {
        constexpr int UU = decltype(uc)::value;
        float s[UU];
        bool on[UU];
        float b[UU][T][VEC];
#pragma unroll
        for (int u = 0; u < UU; ++u) {
            const int idx = t + u * NPAR + g;
            on[u] = idx >= t0 && idx < t1;
            const int src = on[u] ? idx : t0;
            int k;
            if constexpr (NPAR == 1) {
                const int su = uniform(src);
                k = __builtin_amdgcn_readlane(kc, su);
                s[u] = readlane_f(sc, su);
            } else {
                k = __shfl(kc, src);
                s[u] = __shfl(sc, src);
            }
            const E *row = Mat + (size_t)k * N;
#pragma unroll
            for (int tt = 0; tt < T; ++tt) load_vec<VEC>(row + off[tt], b[u][tt]);
        }
#pragma unroll
        for (int u = 0; u < UU; ++u)
#pragma unroll
            for (int tt = 0; tt < T; ++tt)
                if (on[u] && col_ok[tt]) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[tt][v] = fmaf(s[u], b[u][tt][v], acc[tt][v]);
                }
    };
    int t = t0 - (t0 % NPAR);
    for (; t + U * NPAR <= t1; t += U * NPAR) block(t, std::integral_constant<int, U>{});
    for (; t < t1; t += UR * NPAR) block(t, std::integral_constant<int, UR>{});
}

// ---------------------------------------------------------------------------------
// SPMM segment: acc[t][v] += sum_{j in [s0,s1)} vals[j] * Bmat[colidx[j], n + t*TW + v]
// ---------------------------------------------------------------------------------
template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void spmm_segment(int s0, int s1, const int32_t *__restrict__ colidx,
                                             const float *__restrict__ vals,
                                             const E *__restrict__ Bmat, int N, int n,
                                             float (&acc)[T][VEC]) {
    const int lane = lane_id();
    if (s1 <= s0) return;
    int base = s0 & ~(kWave - 1);
    int j = base + lane;
    bool ok = j >= s0 && j < s1;
    int kc = ok ? colidx[j] : 0;
    float vc = ok ? (vals ? vals[j] : 1.f) : 0.f;
    for (; base < s1; base += kWave) {
        // look-ahead: next chunk of the index/value stream
        const int jn = base + kWave + lane;
        const bool okn = jn < s1;
        const int kn = okn ? colidx[jn] : 0;
        const float vn = okn ? (vals ? vals[jn] : 1.f) : 0.f;
        const int t0 = s0 > base ? s0 - base : 0;
        const int t1 = (s1 - base) < kWave ? (s1 - base) : kWave;
        gather_axpy<VEC, LG, T>(kc, vc, t0, t1, Bmat, N, n, acc);
        kc = kn;
        vc = vn;
    }
}

// Sum the NPAR side-by-side partial rows of a wave into lanes [0, LG).
template <int VEC, int LG, int T>
__device__ __forceinline__ void fold_groups(float (&acc)[T][VEC]) {
#pragma unroll
    for (int off = LG; off < kWave; off <<= 1)
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[tt][v] += __shfl_xor(acc[tt][v], off);
}

template <int VEC, int LG, int T>
__device__ __forceinline__ void store_row(float *dst, int N, int n, const float (&acc)[T][VEC]) {
    constexpr int TW = LG * VEC;
    if (lane_id() < LG) {
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
            if (n + tt * TW < N) store_vec<VEC>(dst + n + tt * TW, acc[tt]);
    }
}

// A row per wavefront - or per 2 or 4 wavefronts of a workgroup (`wpr`), which then take consecutive parts of
// the row and whose partial rows the first of them adds in order through LDS: the paper's own decomposition (a row
// per work-item, NT work-items per row for short matrices; Algorithms 1-3 and section "SDDMM").  No shares, no
// search, no heads and so no combine step: a call is one launch whose wavefronts go through three or four
// dependent memory round trips.  For sparse matrices so small that this chain, not throughput, is the whole
// cost; no balancing of long rows (the host picks it only where a row can hold few chunks).
template <int VEC, int LG, int T, int WAVES = kWavesPerBlock>
struct RowParts {
    static constexpr int kWidth = LG * VEC * T;      // columns one workgroup covers
    float part[WAVES][kWidth];
};

// this wavefront's part [s0, s1) of the row [rs, re)
__device__ __forceinline__ void row_part(int rs, int re, int sub, int wpr, int &s0, int &s1) {
    const long long len = re - rs;
    s0 = rs + (int)(len * sub / wpr);
    s1 = rs + (int)(len * (sub + 1) / wpr);
}

// acc of the `wpr` wavefronts of a row -> O[r, :], added in the order of the parts (wpr > 1 only; all wavefronts
// of the workgroup come through here together)
template <int VEC, int LG, int T, int WAVES>
__device__ __forceinline__ void add_row_parts(RowParts<VEC, LG, T, WAVES> &lds, int wv, int sub, int wpr, bool valid,
                                              float *orow, int N, int n, float (&acc)[T][VEC]) {
    constexpr int TW = LG * VEC;
    const int lane = lane_id();
    const int nl = (lane % LG) * VEC;
    if (sub != 0 && lane < LG) {
#pragma unroll
        for (int tt = 0; tt < T; ++tt) store_vec<VEC>(&lds.part[wv][tt * TW + nl], acc[tt]);
    }
    __syncthreads();
    if (sub == 0 && valid) {
        if (lane < LG) {
            for (int p = 1; p < wpr; ++p)
#pragma unroll
                for (int tt = 0; tt < T; ++tt) {
                    float q[VEC];
                    load_vec<VEC>(&lds.part[wv + p][tt * TW + nl], q);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[tt][v] += q[v];
                }
        }
        store_row<VEC, LG, T>(orow, N, n, acc);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------
// SDDMM chunk: dot products of one row of A with the gathered rows of Bmat for the
// entries of one chunk; results land in `slot[0..64)` (LDS, one slot array per wave)
// ---------------------------------------------------------------------------------
// T > 0: the A row sits in registers (`a`, T tiles of LG*VEC columns).  T == 0: any D,
// tiles are walked at run time and the A row is re-read from memory (it stays in L1).
template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void sddmm_chunk(int kc, int t0, int t1, const E *__restrict__ Bmat, int D,
                                            int d, const E *__restrict__ arow,
                                            const float (&a)[T > 0 ? T : 1][VEC], float *slot) {
    constexpr int NPAR = kWave / LG;
    constexpr int TW = LG * VEC;
    const int lane = lane_id();
    const int g = lane / LG;
    if constexpr (T > 0) {
        // Blocks of U steps whose gathers are all requested before the first dot product starts; loads in every
        // lane and step, conditions on the arithmetic only (see gather_axpy).
        constexpr int U = 4, UR = 2;
        int off[T];
        bool col_ok[T];
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
            col_ok[tt] = d + tt * TW < D;
            off[tt] = col_ok[tt] ? d + tt * TW : 0;
        }
        auto block = [&](int t, auto uc) {
            constexpr int UU = decltype(uc)::value;
            float b[UU][T][VEC];
#pragma unroll
            for (int u = 0; u < UU; ++u) {
                const int idx = t + u * NPAR + g;
                const int src = (idx >= t0 && idx < t1) ? idx : t0;
                const int k = (NPAR == 1) ? __builtin_amdgcn_readlane(kc, uniform(src)) : __shfl(kc, src);
                const E *brow = Bmat + (size_t)k * D;
#pragma unroll
                for (int tt = 0; tt < T; ++tt) load_vec<VEC>(brow + off[tt], b[u][tt]);
            }
#pragma unroll
            for (int u = 0; u < UU; ++u) {
                const int idx = t + u * NPAR + g;
                float part = 0.f;
#pragma unroll
                for (int tt = 0; tt < T; ++tt)
                    if (col_ok[tt]) {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) part = fmaf(a[tt][v], b[u][tt][v], part);
                    }
                part = group_sum<LG>(part);
                if (idx >= t0 && idx < t1 && (lane % LG) == 0) slot[idx] = part;
            }
        };
        int t = t0 - (t0 % NPAR);
        for (; t + U * NPAR <= t1; t += U * NPAR) block(t, std::integral_constant<int, U>{});
        for (; t < t1; t += UR * NPAR) block(t, std::integral_constant<int, UR>{});
    } else {
        for_unrolled<4>(t0 - (t0 % NPAR), t1, NPAR, [&](int t) {
            const int idx = t + g;
            const int k = (NPAR == 1) ? __builtin_amdgcn_readlane(kc, t) : __shfl(kc, idx);
            const bool act = idx >= t0 && idx < t1;
            float part = 0.f;
            if (act) {
                const E *brow = Bmat + (size_t)k * D + d;
                for (int dd = 0; d + dd < D; dd += TW) {
                    float b[VEC], av[VEC];
                    load_vec<VEC>(brow + dd, b);
                    load_vec<VEC>(arow + d + dd, av);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) part = fmaf(av[v], b[v], part);
                }
            }
            part = group_sum<LG>(part);
            if (act && (lane % LG) == 0) slot[idx] = part;
        });
    }
}

template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void load_a_row(const E *__restrict__ arow, int D, int d,
                                           float (&a)[T > 0 ? T : 1][VEC]) {
    constexpr int TW = LG * VEC;
    if constexpr (T > 0) {
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
            if (d + tt * TW < D) {
                load_vec<VEC>(arow + d + tt * TW, a[tt]);
            } else {
#pragma unroll
                for (int v = 0; v < VEC; ++v) a[tt][v] = 0.f;
            }
        }
    } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v) a[0][v] = 0.f;
    }
}

// P[j] = vals[j] * <A[r, :], Bmat[colidx[j], :]> for the stored entries [s0, s1) of row r (Algorithm 1's inner
// loops), a chunk of 64 entries at a time.  P may alias vals.
template <int VEC, int LG, int T, typename E>
__device__ __forceinline__ void sddmm_segment(int r, int s0, int s1, const int32_t *__restrict__ colidx,
                                              const float *vals, const E *__restrict__ A,
                                              const E *__restrict__ Bmat, float *P, int D, int d, float *slot) {
    if (s1 <= s0) return;
    const int lane = lane_id();
    const E *arow = A + (size_t)r * D;
    float a[T > 0 ? T : 1][VEC];
    load_a_row<VEC, LG, T>(arow, D, d, a);
    for (int base = s0 & ~(kWave - 1); base < s1; base += kWave) {
        const int j = base + lane;
        const bool ok = j >= s0 && j < s1;
        const int kc = ok ? colidx[j] : 0;
        const float vc = (ok && vals) ? vals[j] : 1.f;
        const int t0 = s0 > base ? s0 - base : 0;
        const int t1 = (s1 - base) < kWave ? (s1 - base) : kWave;
        sddmm_chunk<VEC, LG, T>(kc, t0, t1, Bmat, D, d, arow, a, slot);
        __builtin_amdgcn_wave_barrier();
        if (ok) P[j] = vc * slot[lane];
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------------
// FusedMM: per chunk, the SDDMM stage leaves the 64 scores in LDS slots, each lane
// picks up "its" score (scaled by vals) into a register, and the SPMM stage consumes
// them from there; scores never reach device memory (Algorithm 3's `arow`).
// Dot stage uses (VD, LD, TD) over D, the accumulate stage (VN, LN, TN) over N.
// ---------------------------------------------------------------------------------
template <int VD, int LD, int TD, int VN, int LN, int TN, typename E>
__device__ __forceinline__ void fused_segment(int row, int s0, int s1, const int32_t *__restrict__ colidx,
                                              const float *__restrict__ vals, const E *__restrict__ A,
                                              const E *__restrict__ Bmat, const E *__restrict__ Cmat,
                                              int D, int N, int d, int n, float *slot, float (&acc)[TN][VN]) {
    if (s1 <= s0) return;
    const int lane = lane_id();
    const E *arow = A + (size_t)row * D;
    float a[TD > 0 ? TD : 1][VD];
    load_a_row<VD, LD, TD>(arow, D, d, a);
    for (int base = s0 & ~(kWave - 1); base < s1; base += kWave) {
        const int j = base + lane;
        const bool ok = j >= s0 && j < s1;
        const int kc = ok ? colidx[j] : 0;
        const float vc = (ok && vals) ? vals[j] : 1.f;
        const int t0 = s0 > base ? s0 - base : 0;
        const int t1 = (s1 - base) < kWave ? (s1 - base) : kWave;
        sddmm_chunk<VD, LD, TD>(kc, t0, t1, Bmat, D, d, arow, a, slot);
        __builtin_amdgcn_wave_barrier();
        const float sc = ok ? vc * slot[lane] : 0.f;
        __builtin_amdgcn_wave_barrier();
        gather_axpy<VN, LN, TN>(kc, sc, t0, t1, Cmat, N, n, acc);
    }
}

}  // namespace csrk
