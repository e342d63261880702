// Matrix-core SPMM and FusedMM for wide outputs: FP32 in two half-precision pieces, 32 rows of S per wavefront.
//
// A float of 24 bits is h + l to 23 bits and a sign, h and l of 11 bits each (Ootomo and Yokota, "Recovering single precision
// accuracy from Tensor Cores while surpassing the FP32 theoretical peak performance", 2022, whose scaling of the smaller piece
// by 2^11 is used here): three products s_h c_h, s_h c_l + s_l c_h instead of the six of three bfloat16 pieces, two thirds of
// the bytes of C in LDS, and half a dozen instructions less for every cell of S, since S's values are split where they are
// scattered and not where they are read.  What that costs:
//
// - Range.  Half precision has exponents from 2^-14 (2^-24) to 2^15.  Magnitudes of 2^16 and more become infinities, which show in
//   every result that they are part of; the pieces of a value from 2^-12 on are off by 2^-23 of it, of a smaller one by up to
//   2^-36.  So operands are multiplied by powers of two: every column of C by its own, which brings its largest value to
//   [2^14, 2^15) (dense_range_kernel); every row of S by its own, after samples of its values and of all of them, which leaves
//   them room upwards (kRowExp); FusedMM's rows of A and B by theirs, and the rows of C by the inverse of B's.  The values below
//   2^-12 are counted for every column of C and row of S (of FusedMM's products).  With n and t of them the error of a result is
//   at most (n + t) (2^-36 + 2^-37) 2^16, so a result of 4 (n + t) and more is off by no more than 2^-21 of its terms'
//   magnitudes; smaller ones, and those that are not finite, are computed again by the finishing kernel, entry by entry.  Of
//   uniform or normal values that is less than one result of a call, by an estimate from these sizes.
// - If more than a twelfth of the output (FusedMM: a thirtieth) would be computed again, the call is done again with six products
//   of bfloat16 pieces (dense_kernel, AGAIN), which have the range of floats: two launches that look at one word otherwise, 4 us
//   each.  At 16384^2, 20 %, 512 columns, FusedMM with dot products of 64, instead of 0.73 and 1.11 ms: all values of C, S and B from a
//   Cauchy distribution 2.0 and 2.6 (entry by entry: 11.3 and 15.5); one value of C 10^9 times the others 1.2 and 2.5 (10^4 times:
//   no more than without); S log-normal with sigma 3 1.4 and 1.8.
// - Rows of few entries: 23 bits instead of 24 show, and they are computed again (kWideShortRow).
// - Rounding of sums.  Products of bfloat16 pieces have 16 bits and mostly add up exactly inside an instruction; these have 22,
//   and long sums are 1.75 times as far from FP64.  So the sums are put away in memory on the way (wide_parts).  Error in the
//   2-norm, operands U[-1,1], six products / this: SPMM 16384^2, 20 %, 512 columns 4.2e-7 / 3.6e-7, 16384 x 8192, 10 % 1.81e-7 /
//   1.64e-7, 6 % 1.34e-7 / 1.28e-7; FusedMM 16384^2, 20 %, 512/64 5.3e-7 / 3.7e-7, 16384 x 8192, 10 %, 512/32 2.44e-7 / 2.24e-7.
//
// A workgroup is 8 wavefronts, 128 rows and CT * 16 columns: a pair of wavefronts shares 32 rows, each has half of the columns
// (two rows' fragments for every read of C's pieces: 2 reads per 6 products; with 16 rows, 2 per 3, the reads bound the kernel).
// Every wavefront scatters 16 rows' entries into the tile that its pair reads.  C's tiles go to LDS directly, three buffers, two
// tiles ahead; S's tiles are scattered two tiles ahead in two buffers; one barrier per tile.
//
// FusedMM's scores stay six products of bfloat16 pieces, each wavefront those of its own 16 rows; times S's values they are
// split in half-precision pieces and passed to the pair through LDS as fragments.
//
// Measured on MI355X, six products of bfloat16 pieces / this: SPMM 16384^2, 20 %, N = 512 1195 / 733 us, 16384 x 8192, 10 %, 512
// 580 / 385, 32768 x 8192, 20 %, 192 503 / 400; FusedMM 16384^2, 20 %, 512/64 1538 / 1110, 16384 x 8192, 10 %, 512/32 674 / 455.
// Of SPMM's 733 the range kernel, the preparation, the two launches that end at once and the finishing kernel are 9 + 13 + 8 + 4.
// Bound by latency: of the 3000 cycles of a tile the matrix cores are busy for
// half; the wavefronts that come second on their SIMD take 770 + 1065 cycles for the products, 670 for S, 200 to ask for
// loads, 215 for the fragments (the first ones wait for them at the barrier).  What gave nothing: S between the matrix
// instructions (780-940 us), four of the wavefronts with S before the products and four behind (756), entries of two halves of
// the range in turn, so that loads are under way for two tiles (908), priorities, 128 columns and 4 wavefronts per SIMD (880).
#pragma once
#include "kernels_dense.hpp"

namespace csrk {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma(f16x8 a, f16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Into how many parts a range of K falls, after each of which but the last one the sums are put away, by the mean entries of a
// row in the range: as few as leave the error in the 2-norm below that of the six products, which grows faster with the entries.
// Both are level at, ranges of 8192 / 16384 columns, operands U[-1,1]: SPMM 4 parts 1470 / 2130 entries, 8 parts 560 / 700, 12
// parts 430; FusedMM 4 parts 530 / 655, 8 parts 250, 12 below 250.  (16384 x 8192, 512 columns, 6 %: six products 1.34e-7, 8 parts
// 1.40e-7 in 470 us, 12 parts 1.28e-7 in 490, 16 1.24e-7 in 535.)  Seven of eight row blocks have one part more, a shorter one in
// front, so that not all put their sums away at the same time.
__device__ __forceinline__ int wide_parts(bool fused, long long nnz, long long rows) {
    return nnz >= (fused ? 700 : 2400) * rows ? 4 : nnz >= (fused ? 300 : 800) * rows ? 8 : 12;
}
// Rows of up to this many entries are computed again as sums of FP32: level at 32 entries (8e-8), with one the pieces' 23 bits are
// three times as far off (7.3e-8 against 2.6e-8 in the 2-norm, 3.3e-7 against 5.9e-8 at most).
constexpr int kWideShortRow = 32;

// DS: 32-element steps of the dot products (0: SPMM)
template <int CT, int DS>
struct WideCfg {
    static constexpr int BN = CT * 16, PW = CT / 2;     // columns of a block, 16-column pieces of a wavefront
    // SPMM: two tiles of S, shared by pairs.  FusedMM: a tile for each wavefront, and two of the products with the scores, as
    // fragments.
    static constexpr int kS = DS == 0 ? kDenseBM * kSRow : kDenseWaves * 2048;
    static constexpr int kC = CT * 2048;                // bytes of a tile of C
    static constexpr int kBufs = DS == 0 ? 3 : 2;
    static constexpr int kIssue = kC / (kDenseThreads * 16);
    static constexpr int kB = DS * 3 * 2048;            // ... and of B
    static constexpr int kIssueB = (kB + kDenseThreads * 16 - 1) / (kDenseThreads * 16);
    static constexpr int kOffS = kBufs * kC;
    static constexpr int kOffRaw = kOffS + 2 * kS;
    static constexpr int kOffB = kOffRaw + (DS == 0 ? 0 : kDenseWaves * kSWave);
    static constexpr int kOffCount = kOffB + 2 * kIssueB * kDenseThreads * 16;
    static constexpr int kOffMarks = kOffCount + kDenseWaves * 4;
    static constexpr int kOffCols = kOffMarks + 3 * kDenseBM * 4;
    static constexpr int kBytes = kOffCols + BN * 8;
    static_assert(CT % 4 == 0 && kBytes <= 160 * 1024, "LDS of a gfx950 CU");
};
// What a row's largest value is expected to be brought to (FusedMM: times the scores' expected size): the largest of 1024 of all of
// S's values, or of 16 of the row's if that is more; where the row's is below the other by more than 2^kRowOwn, rows differ in
// size, and it is 2^kRowAbove times the row's.  Samples are four values in a row for each lane of a quad: 32 places of one value
// each took 9 us at 16384^2, 20 %, 512 columns, for a cache line each.
constexpr int kRowExp = 8, kRowOwn = 8, kRowAbove = 3;
constexpr unsigned kGolden = 2654435769u;
// FusedMM: what the exponent of S's values is lowered by: dot products of D elements of up to 2^9 each are about sqrt(D) times as
// large as one of their terms
__device__ __forceinline__ int wide_score_exponent(int D) { return 2 * kDotExp + 1 + (33 - __clz(D)) / 2; }
// Results below this for each value that the pieces of their row of S and column of C do not hold in full are computed again.
constexpr float kTinyUnit = 4.f;
constexpr int kNoTiny = -(1 << 28);     // of a row or column whose results are zeros

// Largest exponents of C's columns, by parts of K; FusedMM: of the rows of C divided by the powers of two that B's are multiplied
// by, which the first column group's workgroups leave for the preparation.  One workgroup more samples S's values.  Bound by the
// latency of memory: 9 us for the 33 MB of 16384 x 512 (12 with half as many parts).
__global__ __launch_bounds__(256) void dense_range_kernel(DenseArgs a) {
    constexpr int kChunk = 256;
    const DenseScales scales(a);
    __shared__ int most[4][64], row_exps[kChunk];
    const int lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const int groups = a.n_tiles / 4, group = blockIdx.x % groups, part = blockIdx.x / groups, col = group * 64 + lane;
    const int rows = (a.K + kRangeParts - 1) / kRangeParts, end = (part + 1) * rows < a.K ? (part + 1) * rows : a.K;
    const float *src = static_cast<const float *>(a.C) + (col < a.N ? col : a.N - 1);
    int m = -kZeros;
    if (blockIdx.x == groups * kRangeParts) {
        // the largest of 1024 of S's values, from places that follow no pattern (multiples of the golden section)
        unsigned x = a.vals ? 0u : bits_of(1.f);
        const unsigned n = (unsigned)a.rowptr[a.M];
        if (a.vals && n > 0)
#pragma unroll
            for (int i = 0; i < 4; ++i) x = larger(x, finite_magnitude(a.vals[__umulhi((threadIdx.x * 4u + i) * kGolden, n)]));
#pragma unroll
        for (int d = kWave / 2; d > 0; d /= 2) x = larger(x, __shfl_xor(x, d));
        if (lane == 0) most[0][wave] = (int)x;
        __syncthreads();
        if (threadIdx.x == 0) a.todo[3] = max(max(most[0][0], most[0][1]), max(most[0][2], most[0][3]));
        return;
    }
    for (int k0 = part * rows; k0 < end; k0 += kChunk) {
        const int stop = k0 + kChunk < end ? k0 + kChunk : end;
        if (a.d_steps) {
            const float *B = static_cast<const float *>(a.B) + (lane < a.D ? lane : a.D - 1);
            __syncthreads();
            for (int r = wave * (kChunk / 4); r < (wave + 1) * (kChunk / 4) && k0 + r < stop; r += 8) {
                unsigned x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = finite_magnitude(B[(size_t)(k0 + r + i < stop ? k0 + r + i : stop - 1) * a.D]);
#pragma unroll
                for (int d = kWave / 2; d > 0; d /= 2)
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[i] = larger(x[i], __shfl_xor(x[i], d));
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (lane == 0) row_exps[r + i] = x[i] == 0 ? kZeros : exponent_to(x[i], kDotExp);
            }
            __syncthreads();
            if (group == 0 && k0 + (int)threadIdx.x < stop) scales.b_exps[k0 + threadIdx.x] = row_exps[threadIdx.x];
        }
        constexpr int kRows = 16;       // under way at a time
        for (int k = k0 + wave; k < stop; k += 4 * kRows) {
            float x[kRows];
#pragma unroll
            for (int i = 0; i < kRows; ++i) x[i] = src[(size_t)(k + 4 * i < stop ? k + 4 * i : stop - 1) * a.N];
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const unsigned b = finite_magnitude(x[i]);
                const int row = a.d_steps ? row_exps[(k + 4 * i < stop ? k + 4 * i : stop - 1) - k0] : 0;
                m = b == 0 || row == kZeros ? m : max(m, (int)larger(b >> 23, 1u) - row);
            }
        }
    }
    most[wave][lane] = m;
    __syncthreads();
    if (wave == 0) {
        m = max(max(most[0][lane], most[1][lane]), max(most[2][lane], most[3][lane]));
        scales.c_most[(size_t)part * a.n_tiles * 16 + col] = col < a.N ? m : -kZeros;
        if (part == 0) scales.c_exps[2 * col + 1] = 0;
    }
}

template <int CT, int DS>
__global__ __launch_bounds__(kDenseThreads, 2) void dense_wide_kernel(DenseArgs a) {
    using L = WideCfg<CT, DS>;
    constexpr bool kFused = DS > 0;
    constexpr int PW = L::PW;
    extern __shared__ __attribute__((aligned(16))) char dlds[];
    const int M = a.M, K = a.K, N = a.N;
    const int lane = lane_id();
    const int wave = uniform(threadIdx.x >> 6);
    const DenseJob job = dense_job(a);
    const DenseScales scales(a);
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)dlds;

    // part i of C's tile to LDS (tiles past the last one read as zeros: the uniform part of the address stops at the view's end)
    const unsigned c_step = (unsigned)a.n_tiles * 2048u, c_end = (unsigned)((K + kDenseK - 1) / kDenseK) * c_step;
    const DenseView cview = dense_view(a.Cp, c_end);
    const unsigned c_off = (unsigned)job.cb * L::kC + threadIdx.x * 16u;
    auto to_lds = [&](const DenseView &view, unsigned off, unsigned step, unsigned end, int k0, unsigned to, int i) CSRK_INLINE {
        const unsigned tile = (unsigned)(k0 / kDenseK) * step, at = (tile < end ? tile : end) + i * kDenseThreads * 16;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(to + wave * 1024u + i * kDenseThreads * 16), "v"(off), "s"(view.rsrc), "s"(at) : "memory");
    };
    auto issue_c = [&](int k0, int buf, int i) CSRK_INLINE { to_lds(cview, c_off, c_step, c_end, k0, lds0 + buf * L::kC, i); };
    const unsigned b_end = (unsigned)((K + kDenseK - 1) / kDenseK) * L::kB;
    const DenseView bview = dense_view(a.Bp, kFused ? b_end : 0u);
    const unsigned b_off = threadIdx.x * 16u < (unsigned)L::kB ? threadIdx.x * 16u : 0xf0000000u;
    auto issue_b = [&](int k0, int buf, int i) CSRK_INLINE {
        to_lds(bview, L::kIssueB * kDenseThreads * 16 == L::kB || i == 0 || threadIdx.x * 16u < L::kB % (kDenseThreads * 16u) ? b_off : 0xf0000000u, L::kB,
               b_end, k0, lds0 + L::kOffB + buf * (L::kIssueB * kDenseThreads * 16), i);
    };
#pragma unroll
    for (int i = 0; i < (L::kBufs - 1) * L::kIssue; ++i) issue_c(job.kb + i / L::kIssue * kDenseK, i / L::kIssue, i % L::kIssue);
#pragma unroll
    for (int i = 0; i < 2 * L::kIssueB; ++i) issue_b(job.kb + i / L::kIssueB * kDenseK, i / L::kIssueB, i % L::kIssueB);
    // which pieces of which rows are to be computed again (every workgroup's last word), the exponents of the rows' results, the
    // values that pieces do not hold in full
    unsigned *const marks = reinterpret_cast<unsigned *>(dlds + L::kOffMarks);
    int *const row_exps = reinterpret_cast<int *>(marks + kDenseBM), *const row_tiny = row_exps + kDenseBM;
    if (threadIdx.x < kDenseBM) marks[threadIdx.x] = 0;
    // the columns' exponents and such values
    int2 *const columns = reinterpret_cast<int2 *>(dlds + L::kOffCols);
    if (threadIdx.x < L::BN) {
        const int2 c = reinterpret_cast<const int2 *>(scales.c_exps)[job.cb * L::BN + threadIdx.x];
        columns[threadIdx.x] = c.x != kZeros ? c : make_int2(0, c.y >= kNotFinite ? c.y : kNoTiny);
    }
    bf16x8 af[kFused ? DS : 1][3];
    if constexpr (kFused) dense_load_a<DS, 3>(a, job.row0 + wave * kDenseRows, af);

    Entries<true, !kFused> e;
    int several;                // rows with more than one entry
    {
        const unsigned bytes = dense_entry_bytes(a, job);
        e.cols = dense_view(job.ci, bytes);
        e.vals = dense_view(a.vals ? (const void *)(a.vals + job.e0) : (const void *)job.ci, a.vals ? bytes : 0u);
        e.q4 = (lane & 3) * 4;
        e.ke = job.ke;
        e.bad = 0;
        const int2 range = dense_row_range(a, job, wave * kDenseRows + (lane >> 2));
        e.pos = range.x;
        e.end = range.y;
        several = (int)__popcll(__ballot(range.y - range.x > 1)) / 4;
        e.load();
        const unsigned all = (unsigned)uniform(a.todo[3]);
        unsigned most = all;
        const int len = range.y - range.x;
        if (a.vals) {
            const int places = len > 4 ? len - 3 : len > 0 ? 1 : 0;
            const f32x4 x = load_f32x4(e.vals, (unsigned)(range.x + (int)__umulhi((unsigned)lane * kGolden, (unsigned)places)) * 4u, 0);
            most = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) most = larger(most, j < len ? finite_magnitude(x[j]) : 0u);
            most = larger(most, __shfl_xor(most, 1));
            most = larger(most, __shfl_xor(most, 2));
            const bool own = most != 0 && (int)(all >> 23) - (int)(most >> 23) > kRowOwn;
            most = own ? most + ((unsigned)kRowAbove << 23) : larger(most, all);
        }
        int value_exponent = exponent_to(most, kFused ? kRowExp - wide_score_exponent(a.D) : kRowExp);
        value_exponent = value_exponent < -126 ? -126 : value_exponent;
        e.scale = power_of_two(value_exponent);
        e.one = a.vals ? 0.f : e.scale;
        e.full_key = tiny_key(ldexpf(1.f, kFullExp - value_exponent));
        e.tiny = 0;
        const int r = wave * kDenseRows + (lane >> 2);
        // (Rows without entries: results of zero are what they should be.  FusedMM, values scaled so far down that the smallest
        // normal float would become a zero: all of the row's.)
        if ((lane & 3) == 0) {
            row_tiny[r] = len == 0 ? kNoTiny : kFused && value_exponent < -23 ? len : 0;
            if constexpr (kFused) value_exponent += scales.a_exps[job.row0 + r < M ? job.row0 + r : M - 1];
            row_exps[r] = value_exponent;
        }
    }
    char *const swave = dlds + (kFused ? L::kOffRaw : L::kOffS) + wave * kSWave;
    const unsigned row_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)(swave + (lane >> 2) * kSRow);
    const unsigned dump = kDenseK * 4u + (lane & 3) * 4u;
    char *const zero_at = swave + (lane >> 3) * kSRow + (lane & 7) * 16;
    auto bring = [&](int k0, int buf) CSRK_INLINE {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<f32x4 *>(zero_at + (kFused ? 0 : buf * L::kS) + i * 8 * kSRow) = z;
        e.row_at = row_at + (kFused ? 0 : buf * L::kS);
        e.dump = e.row_at + dump;
        e.template place<true>(k0, false);
    };

    // 32 rows of S as fragments: [rows / 16][larger and smaller pieces]
    const int pair = wave >> 1, half = wave & 1;
    const char *const sfrag = dlds + L::kOffS + (kFused ? pair * 4096 + lane * 16 : (pair * 32 + (lane & 15)) * kSRow + (lane >> 4) * 16);
    f16x8 s[2][2];
    auto fetch = [&](int buf) CSRK_INLINE {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if constexpr (kFused) {
#pragma unroll
                for (int p = 0; p < 2; ++p) s[r][p] = *reinterpret_cast<const f16x8 *>(sfrag + buf * L::kS + (r * 2 + p) * 1024);
            } else {
                u32x4 x[2], h, l;
#pragma unroll
                for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const u32x4 *>(sfrag + buf * L::kS + r * 16 * kSRow + i * 64);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    h[i] = lower_halves(x[i >> 1][(i & 1) * 2], x[i >> 1][(i & 1) * 2 + 1]);
                    l[i] = upper_halves(x[i >> 1][(i & 1) * 2], x[i >> 1][(i & 1) * 2 + 1]);
                }
                s[r][0] = __builtin_bit_cast(f16x8, h);
                s[r][1] = __builtin_bit_cast(f16x8, l);
            }
        }
    };
    // FusedMM: the wavefront's own 16 rows times their scores, as fragments for its pair
    const char *const own = swave + (lane & 15) * kSRow + (lane >> 4) * 16, *const bfrag = dlds + L::kOffB + lane * 16;
    char *const frag_to = dlds + L::kOffS + wave * 2048 + lane * 16;
    int tiny = 0;               // products that their pieces do not hold in full
    auto score = [&](int buf) CSRK_INLINE {
#pragma clang fp contract(off)
        if constexpr (kFused) {
            f32x4 x[2], p[2];
            dense_scores<DS, 3>(bfrag + buf * (L::kIssueB * kDenseThreads * 16), af, p);
            u32x4 h, l;
            unsigned least = ~0u;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = *reinterpret_cast<const f32x4 *>(own + i * 64);
                p[i] *= x[i];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const unsigned u = half_pieces(p[i][2 * j]), v = half_pieces(p[i][2 * j + 1]);
                    h[2 * i + j] = lower_halves(u, v);
                    l[2 * i + j] = upper_halves(u, v);
                    const unsigned y = tiny_key(p[i][2 * j]), z = tiny_key(p[i][2 * j + 1]);
                    least = y < least ? y : least;
                    least = z < least ? z : least;
                }
            }
            if (__builtin_expect(__any(least < tiny_key(power_of_two(kFullExp))), 0))
#pragma unroll
                for (int j = 0; j < 8; ++j) tiny += tiny_key(p[j >> 2][j & 3]) < tiny_key(power_of_two(kFullExp)) ? 1 : 0;
            *reinterpret_cast<u32x4 *>(frag_to + buf * L::kS) = h;
            *reinterpret_cast<u32x4 *>(frag_to + buf * L::kS + 1024) = l;
        }
    };
    const char *const cfrag = dlds + half * (PW * 2048) + lane * 16;
    auto piece = [&](int buf, int t, f16x8 (&b)[2]) CSRK_INLINE {
#pragma unroll
        for (int p = 0; p < 2; ++p) b[p] = *reinterpret_cast<const f16x8 *>(cfrag + buf * L::kC + (t * 2 + p) * 1024);
    };
    f32x4 acc[2][PW], low[2][PW];       // the products of the larger pieces, the others times 2^11
    auto clear = [&]() CSRK_INLINE {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int t = 0; t < PW; ++t) acc[r][t] = low[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();

    auto say = [&](unsigned again) CSRK_INLINE {
        const int t = threadIdx.x, row = job.row0 + t;
        // (the upper half of the word: pieces that bfloat16 pieces would not leave)
        int pieces = row < M ? (int)__popc(again >> 16) : 0;
        if (__any(pieces != 0)) {
#pragma unroll
            for (int d = kWave / 2; d > 0; d /= 2) pieces += __shfl_xor(pieces, d);
            if (t % kWave == 0) atomicAdd(&a.todo[2], pieces);
        }
        if (t < kDenseBM && row < M) {
            const int entries = a.rowptr[row + 1] - a.rowptr[row];
            if (entries > 0 && entries <= kWideShortRow) again = 0xffffu;
            a.redo[((size_t)job.seg * a.col_blocks + job.cb) * M + row] = (uint16_t)again;
            // (plain stores of the same word: see kernels_dense.hpp)
            if (again != 0) a.todo[0] = 1;
        }
        if constexpr (kFused)
            for (int i = blockIdx.x * kDenseThreads + t; i < a.b_blocks; i += gridDim.x * kDenseThreads)
                if (a.special_met[i] != 0) a.todo[1] = 1;
    };

    // The results, scaled: what is put away in memory, and what has been.
    float *const out = (a.segs > 1 ? a.partial + (size_t)job.seg * M * N : a.O) + (size_t)job.row0 * N;
    const unsigned ld_b = (unsigned)N * 4u;
    const DenseView oview = dense_view(out, (unsigned)(M - job.row0 < kDenseBM ? M - job.row0 : kDenseBM) * ld_b);
    // lane l holds column l & 15 of each 16-column piece, rows 4 (l / 16) + i; rows past M and columns past N fall outside the view
    auto column_at = [&](int t) CSRK_INLINE {
        const int l = lane_id_again(), col = job.cb * L::BN + (half * PW + t) * 16 + (l & 15);
        unsigned o = col < N ? (unsigned)(l >> 4) * 4u * ld_b + (unsigned)col * 4u : 0xf0000000u;
        asm("" : "+v"(o));      // (otherwise: a branch for every use)
        return o;
    };
    auto row_offset = [&](int r, int i) CSRK_INLINE { return (unsigned)(pair * 32 + r * 16 + i) * ld_b; };
    auto result = [&](int r, int t, int i) CSRK_INLINE { return fmaf(low[r][t][i], 1.f / kHalfLow, acc[r][t][i]); };
    auto add_earlier = [&]() CSRK_INLINE {
        constexpr int T = kFused ? 1 : 2;       // pieces at a time (FusedMM has no more registers)
#pragma unroll
        for (int g = 0; g < PW; g += T) {
            float y[2][T][4];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const unsigned o = column_at(g + t);
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        y[r][t][i] = float_of(__builtin_amdgcn_raw_buffer_load_b32(oview.rsrc, o, row_offset(r, i), 0));
            }
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[r][g + t][i] = y[r][t][i] + result(r, g + t, i);
                        low[r][g + t][i] = 0.f;
                    }
        }
    };

    bring(job.kb, 0);
    e.rest(job.kb);
    if constexpr (!kFused) {
        bring(job.kb + kDenseK, 1);
        e.rest(job.kb + kDenseK);
    }
    i32x4 *const counts = reinterpret_cast<i32x4 *>(dlds + L::kOffCount);
    {
        unsigned long long rows = e.bad | e.bad >> 1;
        rows = (rows | rows >> 2) & 0x1111111111111111ull;
        if (lane == 0) reinterpret_cast<int *>(counts)[wave] = 2 * (int)__popcll(rows) - several;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    {
        // (half of the rows with more than one entry out of order: see kernels_dense.hpp)
        const i32x4 n = counts[0] + counts[1];
        if (uniform(n[0] + n[1] + n[2] + n[3]) > 0) return say(0xffffu);
    }
    if constexpr (kFused) score(0);
    else fetch(0);
    __syncthreads();
    int cbuf = 0, put_away = 0;
    // tiles until the sums are put away (neighbouring workgroups at different times: all at once, 872 instead of 834 us)
    const int parts = wide_parts(kFused, uniform(a.rowptr[M]), (long long)a.segs * M);
    const int part = ((job.ke - job.kb + kDenseK - 1) / kDenseK + parts - 1) / parts;
    int until = part - part * (job.row0 / kDenseBM % 8) / 8;
    for (int k0 = job.kb, t = 0;;) {
        // tiles up to where the sums are put away
        const int stop = k0 + until * kDenseK < job.ke ? k0 + until * kDenseK : job.ke;
        for (; k0 < stop; k0 += kDenseK, t ^= 1) {
            // multiplies tile k0, scatters the one after the next (FusedMM: the next one)
            constexpr int kNext = L::kBufs - 1;
            if constexpr (kFused) fetch(t);
            constexpr int kAhead = kFused ? 1 : 2;      // pieces of C read ahead (FusedMM has no registers for more)
            f16x8 b[kAhead + 1][2];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) piece(cbuf, i, b[i]);
            const int c2 = kFused ? cbuf ^ 1 : cbuf + 2 < 3 ? cbuf + 2 : cbuf - 1;
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                __builtin_amdgcn_sched_barrier(0);
                if (i + kAhead < PW) piece(cbuf, i + kAhead, b[(i + kAhead) % (kAhead + 1)]);
                const f16x8(&c)[2] = b[i % (kAhead + 1)];
#pragma unroll
                for (int r = 0; r < 2; ++r) acc[r][i] = mfma(s[r][0], c[0], acc[r][i]);
#pragma unroll
                for (int r = 0; r < 2; ++r) low[r][i] = mfma(s[r][1], c[0], low[r][i]);
#pragma unroll
                for (int r = 0; r < 2; ++r) low[r][i] = mfma(s[r][0], c[1], low[r][i]);
                if (i == 1) {
                    bring(k0 + kNext * kDenseK, t);
                    e.rest(k0 + kNext * kDenseK);
                }
                // (in the last steps: next to S's loads they cost 40-70 us more)
                if (i >= PW - L::kIssue) issue_c(k0 + kNext * kDenseK, c2, i - (PW - L::kIssue));
                if (kFused && i >= 1 && i <= L::kIssueB) issue_b(k0 + 2 * kDenseK, t, i - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kFused) score(t ^ 1);
            else fetch(t ^ 1);
            // SPMM: all loads but the entries (2) and the parts of C's tile after the next one: the next one's are in LDS
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kFused ? 0 : L::kIssue + 2) : "memory");
            __syncthreads();
            cbuf = cbuf == kNext ? 0 : cbuf + 1;
        }
        if (k0 >= job.ke) break;
        if (put_away) add_earlier();
        put_away = 1;
        until = part;
#pragma unroll
        for (int ct = 0; ct < PW; ++ct) {
            const unsigned o = column_at(ct);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32(bits_of(result(r, ct, i)), oview.rsrc, o, row_offset(r, i), 0);
        }
        clear();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // (LDS must not be written to behind the workgroup's end)
    if (put_away) add_earlier();
    const int at = lane_id_again();
    if constexpr (kFused) {
        tiny += __shfl_xor(tiny, 16);
        tiny += __shfl_xor(tiny, 32);
        if (at < kDenseRows && tiny != 0) row_tiny[wave * kDenseRows + at] += tiny;
    } else {
        int n = e.tiny;
        n += __shfl_xor(n, 1);
        n += __shfl_xor(n, 2);
        if ((at & 3) == 0 && n != 0) row_tiny[wave * kDenseRows + (at >> 2)] += 4 * n;
    }
    const unsigned long long unused = __ballot(e.pos < e.end) | e.bad;
    if (__builtin_expect(unused != 0, 0) && at < kDenseRows && ((unsigned)(unused >> at * 4) & 0xfu) != 0)
        atomicOr(&marks[wave * kDenseRows + at], 0xffffu);
    __syncthreads();
    auto column_of = [&](int t) CSRK_INLINE { return columns[(half * PW + t) * 16 + (at & 15)]; };
    // four rows' words
    auto rows_of = [&](const int *words, int r) CSRK_INLINE { return *reinterpret_cast<const i32x4 *>(words + pair * 32 + r * 16 + (at >> 4) * 4); };
    auto odd_result = [&](float y, int tinies) CSRK_INLINE { return !(fabsf(y) < kDenseHuge) || fabsf(y) < kTinyUnit * (float)tinies; };
    bool odd = false;
#pragma unroll
    for (int t = 0; t < PW; ++t) {
        const unsigned o = column_at(t);
        const int2 c = column_of(t);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const i32x4 exps = rows_of(row_exps, r), tinies = rows_of(row_tiny, r);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float y = result(r, t, i);
                odd |= odd_result(y, c.y + tinies[i]);
                __builtin_amdgcn_raw_buffer_store_b32(bits_of(ldexpf(y, -(exps[i] + c.x))), oview.rsrc, o, row_offset(r, i), 0);
            }
        }
    }
    if (__builtin_expect(__any(odd), 0))
#pragma unroll
        for (int t = 0; t < PW; ++t) {
            const bool inside = column_at(t) != 0xf0000000u;
            const int2 c = column_of(t);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const i32x4 tinies = rows_of(row_tiny, r);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool odd = inside && odd_result(result(r, t, i), c.y + tinies[i]);
                    const unsigned long long again = __ballot(odd), other = __ballot(odd && c.y < kNotFinite);
                    if ((at & 15) == 0 && (again >> at & 0xffffu) != 0)
                        atomicOr(&marks[pair * 32 + r * 16 + (at >> 4) * 4 + i], ((other >> at & 0xffffu) != 0 ? 0x10001u : 1u) << (half * PW + t));
                }
            }
        }
    __syncthreads();
    say(threadIdx.x < kDenseBM ? marks[threadIdx.x] : 0u);
}

}  // namespace csrk
