// Matrix-core SDDMM in slabs of scores: all calls but FP32 ones of more than 64 elements without stored values (sddmm_in_slabs, dense.hip).
//
// A workgroup owns 64 rows of S and goes through its range of K in slabs of 256 columns.  Four of its wavefronts (one on each SIMD)
// compute a slab's scores, all 64 x 256 of them, into one of two buffers in LDS, while the other 8 or 12 pick the stored entries'
// scores out of the buffer before: one barrier per slab.  The two kinds have nothing else in common, and that is the point:
//
// - The scorers keep the 64 rows of A in registers (48 of 128 with dot products of up to 32 FP32 elements) and read B's fragments from
//   memory, 16 rows of B for 4 blocks of 16 rows of S.  A wavefront with 16 rows of its own, as in kernels_dense.hpp, would need four
//   times the reads of B, which would be from LDS then and at its limit (123 of 128 bytes per cycle and CU at the cores' full rate).
// - The handlers take a row at a time, a lane per entry, in chunks of 64 entries that begin at multiples of 64: every load and store is
//   256 aligned bytes, and none is made twice.  A chunk stays in registers over as many slabs as its columns span (2.5 at 10 %), its
//   results beside it, and is stored when its last column has passed; the next one has been loaded meanwhile.  A wavefront that
//   waited for B's fragments as well would wait for its entries, which are behind them in the same queue (both jobs in all of 16
//   wavefronts: 179 us with the entries of every slab loaded anew, which the address units then limit, and 214 in chunks).
//
// A lane knows by itself whether its column lies in the slab, so nothing is counted or searched.  What that cannot see shows where the
// chunk is stored: an entry whose column was in a slab that has passed has no result (infinity stands in its place), and a score that
// is no number in the range of floats, because a piece could not hold a value of its row or column, is none either.  Such a row stops
// at that chunk, of which nothing is stored, and is computed entry by entry from there by the wavefronts that are done.  No entry is
// stored twice, and no value read after its entry was stored, so P may be the array that holds the values.
//
// Measured on MI355X, tiled vector kernel or the matrix-core kernel of 16 lanes per row / this: 32768 x 8192, D = 32 10 % 148.5 / 120.9 us
// (the time of its bytes at the rate of a large copy: 68), 20 % 281 / 176 (135), D = 16 30 % 425 / 250; 16384^2, 20 %, D = 64 303 / 233
// (137); 4096^2, 30 %, D = 64 45.7 / 26; bfloat16 16384 x 8192, 10 %, D = 32 73 / 39, 20 %, D = 64 173 / 78, D = 128 190 / 94.  Error against
// FP64 in the 2-norm at D = 32 / 64 4.4e-8 / 4.8e-8 (vector kernels 1.06e-7 / 1.47e-7).
// FP32 dot products of more than 64 elements need more registers for A than a scorer has: two scorers have one half of the steps each
// and two the other, in slabs of 128 columns, and the handlers add the halves' products with the entry's value.  Kernel of 16 lanes per
// row / this: 4096^2, 30 %, D = 128 40.3 / 34.5 us; 16384^2, 20 %, D = 128 480 / 367; 8192^2, 15 %, D = 72 98 / 86; log-normal rows, 10 %, D = 128
// 136 / 95.  Error against FP64 5.3e-8 / 5.1e-8, of data of one sign 4.7e-8 / 3.8e-8 (the halves' sum in one accumulator after the
// other: 9.9e-8; added before the multiplication 5.5e-8).
// What bounds it: at 10 % and D = 32 neither kind alone (scorers 88 us, handlers 89, of which 19 for the call and each workgroup's
// first loads) but both on one SIMD, whose matrix cores are busy for 42 % of the cycles; from 20 % on the handlers, at the rate of
// memory (150 us without the scores at 20 %).  With D = 64 B does not fit an L2 and its fragments are late (151 us without them): the
// rows of A leave registers for two tiles of them.
// Registers: FP32 kernels of more than 32 elements are at the 168 that 12 wavefronts leave, and spill 2 (up to 64 elements), 1 (up to 96)
// and 6 (more).  In their loops the first read one word per slab back from memory, half of the scorers of the last four words of
// A; at 4096^2, 30 %, D = 128 the matrix cores are busy for 39 % of the cycles.
#pragma once
#include "kernels_dense.hpp"

namespace csrk {

constexpr int kSlabRows = 64, kSlabCols = 256;

// Handlers: as many as 16 wavefronts leave where 128 registers hold the scorers' operands (32768 x 8192, 10 %, D = 32: 133 us with 8, 129
// with 12).  Fragments ahead: a tile of FP32 with D = 32 takes 400 cycles, and B's are 1000 away (two tiles: 141 us, four: 133).
template <int DS, int P>
struct SlabCfg {
    // FP32 of more than 64 elements: half of the scorers compute the first two steps' products, the others those of the rest, in slabs of
    // half the columns; the handlers add the two.
    static constexpr int kParts = DS * P > 6 ? 2 : 1;
    static constexpr int kRows = kSlabRows, kCols = kSlabCols / kParts;
    static constexpr int kScorers = 4, kHandlers = DS * P <= 3 ? 12 : 8;
    static constexpr int kThreads = (kScorers + kHandlers) * kWave;
    static constexpr int kRow = (kCols + 4) * 4, kPart = kRows * kRow, kBuffer = kParts * kPart;
    static constexpr int kHandled = (kRows + kHandlers - 1) / kHandlers;    // rows whose entries a wavefront handles: every kHandlers-th
    // 16-row fragments of B under way or in use
    static constexpr int kAhead = DS * P <= 3 ? 4 : 2;
    // (the words that a wavefront without a last row reads lie behind the second buffer)
    static constexpr int kOffRest = 2 * kBuffer + (kHandled * kHandlers - kRows) * kRow;
    static constexpr int kBytes = kOffRest + kRows * 8 + 16;
    static_assert(kBytes <= 160 * 1024, "LDS of a gfx950 CU");
};

// Scores of 16 rows of B (a step per fragment) with NR * 16 rows of A, transposed; see dense_scores for the order of the sums.
// `between(i, n)`: called n times, between the products.
template <int DS, int P, int NR, typename F>
__device__ __forceinline__ void slab_scores(const bf16x8 (&b)[DS][P], const bf16x8 (*af)[DS][P], f32x4 (&s)[NR], F between) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 part[NR][DS];
    if constexpr (P == 1) {
#pragma unroll
        for (int d = 0; d < DS; ++d) {
#pragma unroll
            for (int r = 0; r < NR; ++r) part[r][d] = mfma(b[d][0], af[r][d][0], zero);
            between(d, DS);
        }
    } else {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int d = 0; d < DS; ++d) part[r][d] = zero;
        int i = 0;
#pragma unroll
        for (int d = 0; d < DS; ++d)
#pragma unroll
            for (int pb = P - 1; pb >= 0; --pb)
#pragma unroll
                for (int pa = P - 1 - pb; pa >= 0; --pa) {
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        f32x4 &to = part[r][pa + pb ? DS - 1 : d];
                        to = mfma(b[d][pb], af[r][d][pa], to);
                    }
                    between(i++, DS * 6);
                }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if constexpr (DS == 1) s[r] = part[r][0];
        if constexpr (DS == 2) s[r] = part[r][0] + part[r][1];
        if constexpr (DS == 3) s[r] = part[r][0] + part[r][1] + part[r][2];
        if constexpr (DS == 4) s[r] = (part[r][0] + part[r][1]) + (part[r][2] + part[r][3]);
    }
}

// The scores of all of the range's slabs, into the two buffers in turn.
// PART: of the dot products; `wave`: of its scorers.
template <int ALL, int P, int PART>
__device__ __forceinline__ void slab_produce(const DenseArgs &a, const DenseJob &job, int wave, char *dlds) {
    using L = SlabCfg<ALL, P>;
    constexpr int D0 = PART * 2, DS = L::kParts == 1 ? ALL : PART == 0 ? 2 : ALL - 2;       // steps from D0 on
    constexpr int NT = L::kCols / 16 / (L::kScorers / L::kParts), RT = L::kRows / 16, NB = L::kAhead, NR = ALL == 1 ? 4 : 2;
    const int lane = lane_id();
    // B's fragments: 16 rows each, from memory to registers (rows past the last prepared one read as zeros)
    const unsigned b_end = (unsigned)((a.K + 31) / 32) * 2u * ALL * P * 1024u;
    const DenseView bview = dense_view(a.Bp, b_end);
    bf16x8 b[NB][DS][P];
    auto issue = [&](int k0, int t) CSRK_INLINE {
        const unsigned want = (unsigned)((k0 + t / NT * L::kCols) / 16 + wave * NT + t % NT) * (ALL * P * 1024u), at = want < b_end ? want : b_end;
#pragma unroll
        for (int d = 0; d < DS; ++d)
#pragma unroll
            for (int p = 0; p < P; ++p)
                b[t % NB][d][p] = __builtin_bit_cast(bf16x8, load_f32x4(bview, lane * 16u + ((D0 + d) * P + p) * 1024u, at));
    };
#pragma unroll
    for (int t = 0; t < (ALL == 1 ? NB - 1 : NB); ++t) issue(job.kb, t);
    bf16x8 af[RT][DS][P];
#pragma unroll
    for (int r = 0; r < RT; ++r) dense_load_a<DS, P, ALL>(a, job.row0 + r * 16, af[r], D0);
    // (waits for them here, not in the loop, where it would be for B's as well)
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int d = 0; d < DS; ++d)
#pragma unroll
            for (int p = 0; p < P; ++p) asm volatile("" : "+v"(af[r][d][p]));
    char *const to = dlds + PART * L::kPart + (lane & 15) * L::kRow + wave * NT * 64 + (lane >> 4) * 16;
    auto write = [&](unsigned buf, int t, int r, f32x4 x) CSRK_INLINE {
        *reinterpret_cast<f32x4 *>(to + buf + r * 16 * L::kRow + t * 64) = x;
    };
    unsigned buf = 0;
    if constexpr (ALL == 1) {
        // a tile's scores are written, and its fragments' registers loaded anew, between the products of the tile behind it
        f32x4 score[2][RT];
        for (int k0 = job.kb; k0 < job.ke; k0 += L::kCols, buf ^= L::kBuffer) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int was = (t + NT - 1) % NT;
                slab_scores<DS, P, RT>(b[t % NB], af, score[t & 1], [&](int i, int n) CSRK_INLINE {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = i * (RT + 1) / n; j < (i + 1) * (RT + 1) / n; ++j) {
                        if (j < RT) write(t ? buf : buf ^ L::kBuffer, was, j, score[was & 1][j]);
                        else issue(t ? k0 : k0 - L::kCols, was + NB);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if (t == 0 && k0 > job.kb) __syncthreads();
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) write(buf ^ L::kBuffer, NT - 1, r, score[(NT - 1) & 1][r]);
        __syncthreads();
    } else {
        for (int k0 = job.kb; k0 < job.ke; k0 += L::kCols, buf ^= L::kBuffer) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int r = 0; r < RT; r += NR) {
                    f32x4 score[NR];
                    slab_scores<DS, P, NR>(b[t % NB], af + r, score, [](int, int) CSRK_INLINE {});
#pragma unroll
                    for (int i = 0; i < NR; ++i) write(buf, t, r + i, score[i]);
                }
                issue(k0, t + NB);
                __builtin_amdgcn_sched_barrier(0);      // (or the next tile's products wait for its loads in front of this one's)
            }
            __syncthreads();
        }
    }
    __syncthreads();
}

template <int DS, int P>
__global__ __launch_bounds__((SlabCfg<DS, P>::kThreads)) void dense_slab_kernel(DenseArgs a) {
    using L = SlabCfg<DS, P>;
    using E = std::conditional_t<P == 3, float, bf16_t>;
    constexpr int KT = L::kCols, NR = L::kHandled;
    extern __shared__ __attribute__((aligned(16))) char dlds[];
    const int lane = lane_id();
    const int wave = uniform(threadIdx.x >> 6) - L::kScorers;
    const DenseJob job = dense_job<L::kRows>(a);
    int2 *const rest = reinterpret_cast<int2 *>(dlds + L::kOffRest);
    int *const next = reinterpret_cast<int *>(rest + L::kRows);
    bool some = false;
    if (wave < 0) {
        const int scorer = wave + L::kScorers;
        if (L::kParts == 1 || scorer < L::kScorers / 2) slab_produce<DS, P, 0>(a, job, scorer, dlds);
        else if constexpr (L::kParts == 2) slab_produce<DS, P, 1>(a, job, scorer - L::kScorers / 2, dlds);
    } else {
        const int M = a.M;
        // Positions are relative to the line of 64 entries that the workgroup's first one lies in.
        const int e0 = job.e0 & ~(kWave - 1), skip = job.e0 - e0;
        const int blk_end = uniform(a.rowptr[job.row0 + L::kRows < M ? job.row0 + L::kRows : M]), nnz = uniform(a.rowptr[M]);
        const int padded = (blk_end + kWave - 1) & ~(kWave - 1);
        const unsigned bytes = (unsigned)((padded < nnz ? padded : nnz) - e0) * 4u;
        const DenseView civ = dense_view(a.colidx + e0, bytes);
        const DenseView vav = dense_view(a.vals ? (const void *)(a.vals + e0) : (const void *)(a.colidx + e0), a.vals ? bytes : 0u);
        const DenseView pview = dense_view(a.O + e0, (unsigned)(blk_end - e0) * 4u);
        const unsigned lane4 = lane * 4u;
        // A row's chunk: 64 entries that begin at a multiple of 64, those of them that are the row's.  Lane r has row r's words: where the
        // chunk begins (in bytes), its first entry, the entries from there to the row's end, and the chunk's last column.  Columns
        // are byte offsets in a row of scores.
        int at = 0, first = 0, left = 0, last = 0x7fffffff;
        int ec[NR], en[NR];
        float ev[NR], vn[NR], res[NR], res2[L::kParts == 2 ? NR : 1];
        const float none = float_of(0x7f800000u);
        auto load_cols = [&](int p) CSRK_INLINE { return (int)__builtin_amdgcn_raw_buffer_load_b32(civ.rsrc, lane4 + (unsigned)p, 0, 0); };
        auto load_vals = [&](int p) CSRK_INLINE { return float_of(__builtin_amdgcn_raw_buffer_load_b32(vav.rsrc, lane4 + (unsigned)p, 0, 0)); };
        const int my_row = lane * L::kHandlers + wave;
        if (my_row < L::kRows) {
            const int2 range = dense_row_range(a, job, my_row);
            first = (range.x + skip) & (kWave - 1);
            at = (range.x + skip - first) * 4;
            left = range.y > range.x ? first + range.y - range.x : 0;
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int p = __builtin_amdgcn_readlane(at, r);
            ec[r] = load_cols(p) * 4;
            en[r] = load_cols(p + kWave * 4);
            ev[r] = load_vals(p);
            vn[r] = load_vals(p + kWave * 4);
            res[r] = none;
            if constexpr (L::kParts == 2) res2[r] = 0.f;
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int n = __builtin_amdgcn_readlane(left, r);
            const int end = __builtin_amdgcn_readlane(ec[r], ((n < kWave ? n : kWave) - 1) & (kWave - 1));
            asm("v_writelane_b32 %0, %1, %2" : "+v"(last) : "s"(n > 0 ? end : 0x7fffffff), "n"(r));
            asm volatile("" : "+v"(ec[r]));     // (waits for it here, not in the loop)
        }
        // (bfloat16, 16384 x 8192, 10 %, D = 32: 48 -> 39 us; at 20 % level)
        __builtin_amdgcn_s_setprio(1);
        unsigned from = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)dlds + wave * L::kRow;
        int buf = L::kBuffer;
        __syncthreads();
        for (int k0 = job.kb; k0 < job.ke; k0 += KT, from += buf, buf = -buf) {
            typedef __attribute__((address_space(3))) float lds_float;
            float x[NR], y[L::kParts == 2 ? NR : 1];
            int to[NR], in[NR];
            const int before = k0 * 4 - (int)from, end_at = (int)from + KT * 4 - 4;
            auto look = [&](int r) CSRK_INLINE {
                to[r] = ec[r] - before;
                // (lanes with columns of other slabs all read the first or the last word)
                asm("v_med3_i32 %0, %1, %2, %3" : "=v"(in[r]) : "v"(to[r]), "s"(from), "v"(end_at));
                x[r] = *(const lds_float *)(uintptr_t)(unsigned)(in[r] + r * (L::kHandlers * L::kRow));
                if constexpr (L::kParts == 2) y[r] = *(const lds_float *)(uintptr_t)(unsigned)(in[r] + L::kPart + r * (L::kHandlers * L::kRow));
            };
            // the entries of row r's chunk that lie in the slab
            auto take = [&](int r) CSRK_INLINE {
                asm volatile("" : "+v"(x[r]));
                res[r] = to[r] == in[r] ? x[r] : res[r];
                if constexpr (L::kParts == 2) asm volatile("" : "+v"(y[r]));
                if constexpr (L::kParts == 2) res2[r] = to[r] == in[r] ? y[r] : res2[r];
            };
            // the rows whose chunk is done
            auto through = [&]() CSRK_INLINE { return (unsigned)__ballot(last < (k0 + KT) * 4); };
#pragma unroll
            for (int r = 0; r < NR; ++r) look(r);
#pragma unroll
            for (int r = 0; r < NR; ++r) take(r);
            unsigned more = through();
            while (more) {
#pragma unroll
                for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(en[r]), "+v"(ev[r]), "+v"(vn[r]));
                // rows whose chunk or the next one has other entries than theirs
                const unsigned edges = (unsigned)__ballot(first != 0 || left < 2 * kWave);
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (more >> r & 1) {
                        const int p = __builtin_amdgcn_readlane(at, r);
                        int end = __builtin_amdgcn_readlane(en[r], kWave - 1) * 4;
                        float size = __builtin_fabsf(res[r]), y = res[r] * DenseScale<P, false>::kScoreBack;
                        if constexpr (L::kParts == 2) {
                            // (the halves' sum in the multiplication: one rounding less, and the error of this kernel's scores no larger
                            // than that of sums in one wavefront.  These calls have stored values.  One that is infinite, or that takes one
                            // half alone out of the range of floats, is for the sum, so a result that is not finite counts as not done;
                            // the sum's product here, where it is needed: 0.4 of 34.5 us at 4096^2, 30 %, D = 128)
                            const float half = res2[r] * DenseScale<P, false>::kScoreBack;
                            y = fmaf(y, ev[r], half * ev[r]);
                            size = __builtin_fabsf(y);
                        } else if (a.vals) {
                            y *= ev[r];
                        }
                        const unsigned long long odd = __ballot(!(size < (L::kParts == 2 ? none : kDenseHuge)));
                        unsigned off = lane4 + (unsigned)p;
                        bool fine = odd == 0;
                        if (__builtin_expect(!fine || (edges >> r & 1), 0)) {
                            const int f = __builtin_amdgcn_readlane(first, r), n = __builtin_amdgcn_readlane(left, r);
                            const unsigned long long mine = (~0ull << f) & (n < kWave ? (1ull << n) - 1 : ~0ull);
                            fine = (odd & mine) == 0;
                            off = __builtin_amdgcn_inverse_ballot_w64(fine ? mine : 0ull) ? off : 0xf0000000u;
                            asm("" : "+v"(off));        // (or there is a branch, and one that makes the row's words vectors)
                            end = __builtin_amdgcn_readlane(en[r], ((n < 2 * kWave ? n : 2 * kWave) - 1) & (kWave - 1)) * 4;
                            // (a row with an entry that is not done stays at the chunk)
                            end = fine && n > kWave ? end : 0x7fffffff;
                            more &= ~(fine ? 0u : 1u << r);
                        }
                        __builtin_amdgcn_raw_buffer_store_b32(bits_of(y), pview.rsrc, off, 0, 0);
                        asm("v_writelane_b32 %0, %1, %2" : "+v"(last) : "s"(end), "n"(r));
                        asm volatile("v_lshlrev_b32 %0, 2, %1" : "=v"(ec[r]) : "v"(en[r]));
                        asm volatile("v_mov_b32 %0, %1" : "=v"(ev[r]) : "v"(vn[r]));
                        res[r] = none;
                        if constexpr (L::kParts == 2) res2[r] = 0.f;
                        en[r] = load_cols(p + 2 * kWave * 4);
                        vn[r] = load_vals(p + 2 * kWave * 4);
                        look(r);
                    }
                const bool done = __builtin_amdgcn_inverse_ballot_w64(more);
                at += done ? kWave * 4 : 0;
                left -= done ? kWave : 0;
                first = done ? 0 : first;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (more >> r & 1) take(r);
                more = through();
            }
            __syncthreads();
        }
        some = left > 0;
        if (my_row < L::kRows) rest[my_row] = some ? make_int2(e0 + (int)((unsigned)at / 4) + first, e0 + (int)((unsigned)at / 4) + left) : make_int2(0, 0);
        if (wave == 0 && lane == 0) *next = 0;
    }
    // what is left of the workgroup's rows, each to the next wavefront that is free
    if (__builtin_expect(!__syncthreads_or(some), 1)) return;
    while (true) {
        int r = 0;
        if (lane == 0) r = atomicAdd(next, 1);
        r = uniform(r);
        if (r >= L::kRows) break;
        dense_sddmm_rest<E>(a, job.row0 + r, uniform(rest[r].x), uniform(rest[r].y), reinterpret_cast<float *>(dlds + (wave + L::kScorers) * L::kRow));
    }
}

}  // namespace csrk
