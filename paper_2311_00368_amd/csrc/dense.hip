// Host side of the matrix-core kernels: how a call is cut into workgroups, and its launches.
#include "dense.hpp"

#include <atomic>

#include "kernels_dense_sddmm.hpp"
#include "kernels_dense_wide.hpp"

namespace csrk {

// SDDMM in slabs of scores (kernels_dense_sddmm.hpp): all but FP32 dot products of more than 64 elements without stored values.
// Those are the sum of two wavefronts' halves; where a value is multiplied by, that takes one rounding less and the error is 0.95
// (both signs) and 0.82 (one sign) of the other kernel's, without it is 1.05-1.08.
bool sddmm_in_slabs(const DenseShape &s) { return s.bf16 || s.D <= 64 || !s.ones; }

namespace {

constexpr int kMaxWidth = 2048, kMaxDot = 128, kMaxK = 1 << 20;
// (the extent of a buffer view is a 32-bit byte count, and the kernels give 0xf0000000 as an offset that is outside)
constexpr size_t kView = 0xe0000000ull;
constexpr int kMaxRows = 1 << 26;
constexpr long long kMaxGroups = 1 << 22;

// Ranges of K from this length on are done in half-precision pieces where blocks of 192 or 256 columns of FP32 are the best
// choice (narrower blocks add up their sums on the way and are the more exact).  Shorter ranges would have to put their sums away
// after fewer tiles for an error no larger than that of the six products of bfloat16 (at 8192^2, log-normal rows, 256 columns, in
// ranges of 2048, 1.36e-7 against 1.41e-7 in the 2-norm with 8 parts, which take 4 us each; kernels_dense_wide.hpp has the figures
// of longer ranges).  A tile takes 1.4-1.5 us, FusedMM's 2.1.
constexpr int kHalvesK = 8192;
constexpr double kHalvesTileUs = 1.5, kHalvesFusedTileUs = 2.1;

int sddmm_rows(const DenseShape &s) { return sddmm_in_slabs(s) ? kSlabRows : kDenseBM; }

size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }
size_t up32(int x) { return ((size_t)x + 31) / 32 * 32; }

int prepare_blocks(size_t units) {
    // one unit of 8 values per thread: a call's latency counts here (two: 1-2 us more)
    const size_t blocks = (units + 255) / 256;
    return (int)(blocks > 1024 ? 1024 : blocks);
}

// where everything lies in the scratch area
struct Layout {
    size_t c, b, a, todo, met, special, redo, cuts, partial, bytes;
    int n_tiles, c_blocks, b_blocks, a_blocks;
    Layout(const DenseShape &s, const DenseConfig &cfg) {
        const bool halves = cfg.halves;
        const size_t pieces = s.bf16 ? 2 : 6;       // bytes of a prepared value
        const int bn = cfg.ct * 16;
        n_tiles = s.op == kDenseSddmm ? 0 : (s.N + bn - 1) / bn * cfg.ct;
        const size_t d = (size_t)cfg.ds * 32, k = up32(s.K), octs = cfg.ds == 3 ? 16 : cfg.ds * 4;
        c_blocks = prepare_blocks(k / 8 * n_tiles * 16);
        if (halves && c_blocks > n_tiles / 4) c_blocks = c_blocks / (n_tiles / 4) * (n_tiles / 4);
        b_blocks = prepare_blocks(k * octs);
        a_blocks = prepare_blocks(up32(s.M) * octs);
        size_t at = 0;
        auto take = [&](size_t n) {
            const size_t was = at;
            at += padded(n);
            return was;
        };
        c = take(k * n_tiles * 16 * pieces);
        // (whole tiles of 64 columns)
        b = take((k + 32) * d * pieces);
        a = take(up32(s.M) * d * pieces);
        todo = take(halves ? DenseScales::bytes(n_tiles, s.K, s.M) : 8);
        met = take(s.op == kDenseFused ? (size_t)b_blocks * 4 : 0);
        special = take(s.op == kDenseFused ? k : 0);
        redo = take(s.op != kDenseSddmm ? (size_t)cfg.segs * (n_tiles / cfg.ct) * s.M * 2 : 0);
        cuts = take(cfg.segs > 1 ? (size_t)(cfg.segs - 1) * s.M * 4 : 0);
        partial = take(cfg.segs > 1 && s.op != kDenseSddmm ? (size_t)cfg.segs * s.M * s.N * 4 : 0);
        bytes = at;
    }
};

template <int P>
DenseKernel spmm_kernel(int ct) {
#define CSRK_DENSE_CASE(CT) \
    if (ct == CT) return {dense_kernel<CT, 0, P>, DenseCfg<CT, 0, P>::kBytes};
    CSRK_DENSE_CT(CSRK_DENSE_CASE)
#undef CSRK_DENSE_CASE
    return {nullptr, 0};
}

DenseKernel wide_kernel(int ct, int ds) {
#define CSRK_DENSE_CASE(DS) \
    if (ct == 12 && ds == DS) return {dense_wide_kernel<12, DS>, WideCfg<12, DS>::kBytes}; \
    if (ct == 16 && ds == DS) return {dense_wide_kernel<16, DS>, WideCfg<16, DS>::kBytes};
    CSRK_DENSE_CASE(0)
    CSRK_DENSE_CASE(1)
    CSRK_DENSE_CASE(2)
#undef CSRK_DENSE_CASE
    return {nullptr, 0};
}

DenseKernel again_kernel(int ct, int ds) {
    if (ds > 0) return dense_again_fused_f32(ct, ds);
    if (ct == 12) return {dense_kernel<12, 0, 3, true>, DenseCfg<12, 0, 3>::kBytes};
    if (ct == 16) return {dense_kernel<16, 0, 3, true>, DenseCfg<16, 0, 3>::kBytes};
    return {nullptr, 0};
}

DenseKernel sddmm_kernel(const DenseShape &s, int ds) {
    if (!sddmm_in_slabs(s) && ds == 3) return {dense_sddmm_kernel<3>, DenseSddmmCfg<3>::kBytes, kDenseThreads};
    if (!sddmm_in_slabs(s) && ds == 4) return {dense_sddmm_kernel<4>, DenseSddmmCfg<4>::kBytes, kDenseThreads};
#define CSRK_SLAB_CASE(DS, P) \
    if (ds == DS && s.bf16 == (P == 1)) return {dense_slab_kernel<DS, P>, SlabCfg<DS, P>::kBytes, SlabCfg<DS, P>::kThreads};
    CSRK_SLAB_CASE(1, 3)
    CSRK_SLAB_CASE(2, 3)
    CSRK_SLAB_CASE(3, 3)
    CSRK_SLAB_CASE(4, 3)
    CSRK_SLAB_CASE(1, 1)
    CSRK_SLAB_CASE(2, 1)
    CSRK_SLAB_CASE(3, 1)
    CSRK_SLAB_CASE(4, 1)
#undef CSRK_SLAB_CASE
    return {nullptr, 0, 0};
}

// Time of a workgroup for 32 columns of K, in us, with a CU to itself.  Read off MI355X timings: FP32 SPMM 1.03 us with 2
// pieces (32768 x 8192), 1.08 with 4, 1.7 with 8, 2.7 with 16 (16384 x 16384); FusedMM with 2 / 4 steps of the dot product
// 2.0 / 2.9 with 8 pieces; bfloat16 1.1 with 8 and 1.55 with 16.
double tile_us(const DenseShape &s, int ct, int ds) {
    if (s.op == kDenseSddmm) return 0.75 + 0.2 * ds;
    if (s.bf16) return 0.65 + 0.056 * ct + 0.05 * ds;
    return 0.6 + 0.13 * ct + 0.27 * ds;
}

}  // namespace

// Time of an SDDMM call in slabs, in us: per call, and for every round of workgroups to begin and end it, per slab of 256 columns, and
// by the slab's density.  Fitted to 3600 random calls of M 512-32768, K 512-16384, 6-35 %, D 16-128 on MI355X, which scatter by 5-13 %
// around it.
bool sddmm_slab_us(const DenseShape &s, const DenseConfig &c, int cus, double density, double *us) {
    struct Cost {
        double call, round, slab, entries;
    };
    static constexpr Cost f32[] = {{5.2, 5.5, 1.12, 5.5}, {5.0, 7.1, 2.24, 4.9}, {5.4, 7.1, 4.1, 3.3}, {5.4, 8.0, 4.7, 2.6}};
    static constexpr Cost bf16[] = {{4.1, 6.3, 0.60, 6.0}, {5.2, 5.6, 0.82, 5.8}, {5.5, 5.9, 0.98, 5.1}, {4.8, 5.7, 1.71, 5.8}};
    if (s.op != kDenseSddmm || !sddmm_in_slabs(s)) return false;
    const Cost t = s.bf16 ? bf16[c.ds - 1] : f32[c.ds - 1];
    const long long rounds = ((s.M + kSlabRows - 1) / kSlabRows * (long long)c.segs + cus - 1) / cus;
    *us = t.call + (double)rounds * (t.round + c.seg_k / kSlabCols * (t.slab + t.entries * density));
    return true;
}

bool dense_config(const DenseShape &s, int cus, DenseConfig *out) {
    if (s.M < 1 || s.M > kMaxRows || s.K < 32 || s.K > kMaxK) return false;
    if (s.op != kDenseSddmm && (s.N < 1 || s.N > kMaxWidth)) return false;
    if (s.op != kDenseSpmm && (s.D < 1 || s.D > kMaxDot)) return false;
    const size_t pieces = s.bf16 ? 2 : 6;
    if ((up32(s.K) + 64) * (size_t)(s.N + 256) * pieces >= kView || (up32(s.K) + 128) * 128 * pieces >= kView) return false;
    const bool slabs = s.op == kDenseSddmm && sddmm_in_slabs(s);
    const int bm = s.op == kDenseSddmm ? sddmm_rows(s) : kDenseBM;
    const long long row_blocks = (s.M + bm - 1) / bm;
    DenseConfig best{};
    best.us = 1e30;
    DenseConfig c{};
    c.ds = s.op == kDenseSpmm ? 0 : (s.D + 31) / 32;
    const int tiles = (s.K + 31) / 32;
    static constexpr int widths[] = {2, 3, 4, 5, 6, 8, 12, 16};
    for (int ct : widths) {
        if (s.op == kDenseSddmm && ct != 2) continue;
        if (s.op == kDenseFused && c.ds > 2 && ct > 8) continue;
        const int col_blocks = s.op == kDenseSddmm ? 1 : (s.N + ct * 16 - 1) / (ct * 16);
        for (int segs = 1; segs <= kDenseMaxSegs; ++segs) {
            // ranges of whole tiles (of 64 columns; slabs), of at least 128 columns
            const int step = slabs ? kSlabCols / 32 : 2;
            const int seg_tiles = ((tiles + segs - 1) / segs + step - 1) / step * step;
            if (segs > 1 && (seg_tiles < 4 || (tiles + seg_tiles - 1) / seg_tiles != segs)) continue;
            const long long wgs = row_blocks * col_blocks * segs;
            if (wgs > kMaxGroups) continue;
            const long long rounds = (wgs + cus - 1) / cus;
            // a launch of 8 us all told, 4 us to begin and end each workgroup, the ranges' outputs written and read again
            double us = 8.0 + (double)rounds * (seg_tiles * tile_us(s, ct, c.ds) + 4.0);
            if (segs > 1 && s.op != kDenseSddmm) us += 3.0 + (double)(segs + 1) * s.M * (double)s.N * 4.0 / 4.0e6;
            c.segs = segs;
            c.seg_k = seg_tiles * 32;
            sddmm_slab_us(s, c, cus, 0.15, &us);        // (how dense S is is not known here)
            if (us < best.us) {
                best = c;
                best.ct = ct;
                best.us = us;
            }
        }
    }
    if (best.ct == 0) return false;
    if (s.op != kDenseSddmm && !s.bf16 && best.ct > 8 && best.seg_k >= kHalvesK) {
        const long long rounds = (row_blocks * ((s.N + best.ct * 16 - 1) / (best.ct * 16)) * best.segs + cus - 1) / cus;
        best.halves = true;
        best.us -= (double)rounds * (best.seg_k / 32 * (tile_us(s, best.ct, best.ds) - (best.ds ? kHalvesFusedTileUs : kHalvesTileUs)) - 24.0);
    }
    const Layout l(s, best);
    best.bytes = l.bytes;
    if (!slabs) best.us += (double)l.partial / 2.0e6;           // the operands' preparation
    *out = best;
    return true;
}

hipError_t dense_run(const DenseShape &s, const DenseConfig &c, const int32_t *rowptr, const int32_t *colidx, const float *vals,
                     const void *A, const void *B, const void *C, float *out, void *scratch, hipStream_t stream) {
    const Layout l(s, c);
    char *base = static_cast<char *>(scratch);
    DenseArgs a{};
    a.M = s.M;
    a.K = s.K;
    a.N = s.op == kDenseSddmm ? 0 : s.N;
    a.D = s.op == kDenseSpmm ? 0 : s.D;
    const int bm = s.op == kDenseSddmm ? sddmm_rows(s) : kDenseBM;
    a.row_blocks = (s.M + bm - 1) / bm;
    a.col_blocks = s.op == kDenseSddmm ? 1 : l.n_tiles / c.ct;
    a.segs = c.segs;
    a.seg_k = c.seg_k;
    a.n_tiles = l.n_tiles;
    a.bn = c.ct * 16;
    a.d_steps = c.ds;
    a.c_blocks = l.c_blocks;
    a.b_blocks = l.b_blocks;
    a.a_blocks = l.a_blocks;
    a.rowptr = rowptr;
    a.colidx = colidx;
    a.vals = vals;
    a.A = A;
    a.B = B;
    a.C = C;
    a.Ap = base + l.a;
    a.Bp = base + l.b;
    a.Cp = base + l.c;
    a.O = out;
    a.partial = reinterpret_cast<float *>(base + l.partial);
    if (s.op == kDenseFused) {
        a.special = reinterpret_cast<uint8_t *>(base + l.special);
        a.special_met = reinterpret_cast<int32_t *>(base + l.met);
    }
    if (s.op != kDenseSddmm) a.todo = reinterpret_cast<int32_t *>(base + l.todo);
    a.redo = reinterpret_cast<uint16_t *>(base + l.redo);
    a.cuts = reinterpret_cast<int32_t *>(base + l.cuts);

    const DenseKernel k = c.halves              ? wide_kernel(c.ct, c.ds)
                          : s.op == kDenseSpmm  ? (s.bf16 ? spmm_kernel<1>(c.ct) : spmm_kernel<3>(c.ct))
                          : s.op == kDenseSddmm ? sddmm_kernel(s, c.ds)
                                                : (s.bf16 ? dense_fused_kernel_bf16(c.ct, c.ds) : dense_fused_kernel_f32(c.ct, c.ds));
    const DenseKernel again = c.halves ? again_kernel(c.ct, c.ds) : DenseKernel{nullptr, 0, 0};
    if (!k.fn || (c.halves && !again.fn)) return hipErrorInvalidValue;
    {
        // once per kernel and device (harmless if two threads do it)
        static std::atomic<uint64_t> done[3][3][17][5];
        int dev = 0;
        if (hipError_t e = hipGetDevice(&dev)) return e;
        std::atomic<uint64_t> &seen = done[s.op][s.bf16 ? 1 : c.halves || (s.op == kDenseSddmm && !sddmm_in_slabs(s)) ? 2 : 0][c.ct][c.ds];
        const uint64_t bit = 1ull << (dev & 63);
        if (!(seen.load(std::memory_order_acquire) & bit)) {
            for (const DenseKernel &one : {k, again})
                if (one.fn)
                    if (hipError_t e = hipFuncSetAttribute((const void *)one.fn, hipFuncAttributeMaxDynamicSharedMemorySize, one.lds_bytes)) return e;
            seen.fetch_or(bit, std::memory_order_release);
        }
    }
    const int prepare = a.c_blocks + a.b_blocks + a.a_blocks + (a.segs > 1 ? (a.M + kDenseCutRows - 1) / kDenseCutRows : 0);
    if (c.halves) hipLaunchKernelGGL(dense_range_kernel, dim3(a.n_tiles / 4 * kRangeParts + 1), dim3(256), 0, stream, a);
    if (s.bf16) hipLaunchKernelGGL(dense_prepare_kernel<bf16_t>, dim3(prepare), dim3(256), 0, stream, a);
    else if (c.halves) hipLaunchKernelGGL((dense_prepare_kernel<float, true>), dim3(prepare), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(dense_prepare_kernel<float>, dim3(prepare), dim3(256), 0, stream, a);
    const dim3 jobs((unsigned)a.row_blocks * a.col_blocks * a.segs);
    hipLaunchKernelGGL(k.fn, jobs, dim3(k.threads), k.lds_bytes, stream, a);
    if (c.halves) {
        // (few workgroups to find that there is nothing to do; no cuts)
        DenseArgs b = a;
        b.c_blocks = b.c_blocks < 192 ? b.c_blocks : 192;
        b.b_blocks = b.b_blocks < 32 ? b.b_blocks : 32;
        b.a_blocks = b.a_blocks < 32 ? b.a_blocks : 32;
        hipLaunchKernelGGL((dense_prepare_kernel<float, false, true>), dim3(b.c_blocks + (b.d_steps ? b.b_blocks + b.a_blocks : 0)), dim3(256), 0, stream, b);
        hipLaunchKernelGGL(again.fn, jobs, dim3(kDenseThreads), again.lds_bytes, stream, b);
    }
    if (s.op != kDenseSddmm) {
        const int unit = s.bf16 ? 8 : 4;
        uintptr_t at = reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(C);
        if (s.op == kDenseFused) at |= reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B);
        const bool vec = a.N % unit == 0 && a.D % unit == 0 && (at & 15u) == 0;
        const DenseKernel f = dense_finish_kernel(s.bf16, s.op == kDenseFused, vec, c.ct, c.halves);
        if (!f.fn) return hipErrorInvalidValue;
        // not many more workgroups than the chip holds at a time (2048 of FusedMM's: 6.8 instead of 5.8 us for the sums of
        // 16384 x 4096, 128 columns, in 2 ranges), and with long rows to do again some to choose from; of 8 and 16 wavefronts two
        // are on a CU
        const int rows = a.segs > 1 && a.N < 1024 ? 1024 / a.N : 1;
        const int blocks = (a.M + rows - 1) / rows, most = c.halves ? 512 : s.op == kDenseFused ? 1536 : 1280;
        hipLaunchKernelGGL(f.fn, dim3(blocks < most ? blocks : most), dim3(finish_waves(c.halves, s.op == kDenseFused) * 64), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace csrk
