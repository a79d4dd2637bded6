// Selective-load GEMM (Sec. 4.4): Y[m,:] = X[kept_idx[m],:] . W^T (+ bias).  The kept rows are read
// straight from the [S,C] input inside the A-tile load -- a kept row is C contiguous elements, so the
// indexed load is as coalesced as a dense one and no compacted copy of X ever exists.
//
// This file holds the launches and the choice of the output tiles; the kernels are gather_gemm_large.hip (256 x 256, bf16),
// gather_gemm_mid.hip (256, 192, 128 or 64 x 128, bf16) and gather_gemm_small.hip (64 x 64; binary32).
#include "gather_gemm.hpp"

namespace lemo {

// Which tiles a product is cut into: the first `head_cols` columns into `head` tiles, the others into `rest` tiles.
//
// The larger the tile the faster per flop, but tiles come in rounds of 256, one per CU, and a round lasts nearly as long for one
// tile as for all: with few tiles, or just past a full round, smaller ones win although they move more bytes per flop.
// The time of n tiles of a kind over k slabs of 64 elements of the contraction, in us, is taken as
//   a + full (b k + e) + (c + d f) k + e f          full whole rounds, the last one filled to f (nothing if f = 0)
// with a the launch, b a slab in a full round, c ... c + d in the last one (c: if it is the first, if there are rounds before), e
// what a round costs besides (loads before, stores after).  `along` (X W^T) and `mixed` (input gradients, whose weights pass through the transposing read) are
// fitted to the six kinds over M = 50 ... 12000 with the widths and contractions of layers of 256 to 4096 (N or K up to 14336), 1000 products
// each, operands from HBM; the kind chosen costs 0.05 % over the best one on average, 5 % at worst (X W^T, M = 112, N = 256, K = 768: 64 x 64) and in one
// input gradient 8 % (M = 575, N = 2048, K = 8192: 64 x 128).  `across` is fitted to 66 weight gradients of layers of 256 to 4096, M = 64 ... 5000; its kinds
// are those whose rows are whole contraction-major regions.
// e.g. us for 256 x 256 / 256 x 128 / 192 x 128 / 128 x 128 / 64 x 128 / 64 x 64:  M = 100, N = K = 4096  - / 46 / 42 / 35 / 28 / 15;
// M = 128, N = 11008, K = 4096  73 / 46 / 43 / 42 / 32 / 42;   M = 504, N = 11008, K = 4096  79 / 56 / 80 / 76 / 83 / 106;
// M = 1500, N = K = 4096  81 / 56 / 50 / 76 / - / 97;   M = 3280, N = K = 4096  93 / 110 / 131 / 136 / - / 196;   input gradient M = 1500,
// 4096 columns, contraction 11008  203 / 153 / 134 / 195 / - / 251;   M = 256, N = K = 256  9.6 / 7.7 / 6.9 / 5.7 / 4.8 / 5.7, its input
// gradient 13.3 / 9.3 / 8.2 / 6.6 / 5.5 / 5.7;   M = 1000, N = K = 768  19.8 / 15.6 / 13.4 / 11.0 / 8.7 / 8.2, its input gradient 23.7 / 16.9 /
// 14.3 / 11.7 / 9.3 / 8.4.  The two kinds between (192 x 128: M = 1500 above is 256 tiles of it; 64 x 128: half of 128 x 128's time where those leave
// half of the CUs without one) are worth 5 % on average.
// Products that fill whole rounds with one of the larger kinds may take another for the columns behind them.  The launches follow each
// other and the times add, but for what the second one's start hides behind the first one's end: with 2 us for that, 46 products for which it matters cost
// 0.6 % over the better choice on average (with none 1.3 %, with 5 1.2 %).
// binary32: 128 x 128 tiles, or 32 x 32 ones with the contraction split over four waves up to 192 of the former (us, 128 x 128 /
// 32 x 32: M = 200, N = K = 768 33 / 7.3; 96 tiles, M = 500, N = 3072, K = 768 36 / 32; 160, M = 640, N = 4096, K = 1024 45 / 60; 192,
// M = 700, N = K = 4096 158 / 204; 256, M = 1024, N = 4096, K = 1024 52 / 85).  By time the line would lie at 128; but the four partial
// sums of the small tiles are nearer to 64 bits (2.9e-7 against 4.9e-7), so what they served before the large ones became
// faster they still serve.
struct GgPlan { int head_cols; GgTile head, rest; };
struct GgFit { GgTile tile; int rows, cols; double a, b, c[2], d, e; };
static GgPlan gg_plan(long long M, int N, int K, int layout, lemo_dtype_t dt) {
    static constexpr GgFit along[] = {{GG_T256, 256, 256, 6.43, 1.405, {1.004, 0.998}, 0.347, 5.76}, {GG_T256x128, 256, 128, 4.76, 0.812, {0.735, 0.655}, 0.129, 5.19},
                                      {GG_T192x128, 192, 128, 4.36, 0.673, {0.617, 0.573}, 0.091, 4.24}, {GG_T128, 128, 128, 3.62, 0.529, {0.498, 0.461}, 0.068, 3.01},
                                      {GG_T64x128, 64, 128, 3.19, 0.388, {0.359, 0.307}, 0.040, 1.78}, {GG_T64, 64, 64, 4.59, 0.226, {0.223, 0.207}, 0.012, 1.27}};
    static constexpr GgFit mixed[] = {{GG_T256, 256, 256, 8.34, 1.429, {0.919, 1.011}, 0.472, 11.79}, {GG_T256x128, 256, 128, 6.15, 0.819, {0.658, 0.701}, 0.178, 7.01},
                                      {GG_T192x128, 192, 128, 4.82, 0.672, {0.583, 0.600}, 0.087, 6.43}, {GG_T128, 128, 128, 4.71, 0.534, {0.486, 0.542}, 0.040, 3.94},
                                      {GG_T64x128, 64, 128, 3.86, 0.409, {0.404, 0.411}, 0.008, 2.24}, {GG_T64, 64, 64, 4.45, 0.272, {0.264, 0.156}, 0.017, 1.33}};
    static constexpr GgFit across[] = {{GG_T256, 256, 256, 5.6, 1.51, {1.16, 1.16}, 0.14, 7.1}, {GG_T256x128, 256, 128, 5.0, 0.94, {0.75, 0.75}, 0.13, 5.0},
                                       {GG_T128, 128, 128, 3.2, 0.59, {0.56, 0.56}, 0.02, 3.6}, {GG_T64, 64, 64, 4.4, 0.18, {0.17, 0.17}, 0.30, 4.2}};
    if (dt == LEMO_F32) {
        const double n128 = (double)((M + 127) / 128) * (double)(((long long)N + 127) / 128);
        return {0, GG_T128, n128 <= 192 ? GG_T64 : GG_T128};
    }
    const GgFit* fits = layout == GG_TN ? across : layout == GG_NN ? mixed : along;
    const int kinds = layout == GG_TN ? 4 : 6, heads = kinds / 2;  // heads: the kinds that may come before another one
    const double meets = layout == GG_TN ? 0. : 2.;                // the second launch starts as the first one ends
    const double k = K / 64.;
    auto time = [&](const GgFit& f, long long cols) {
        const double n = (double)((M + f.rows - 1) / f.rows) * (double)((cols + f.cols - 1) / f.cols);
        const double full = (double)(long long)(n / 256), part = n / 256 - full;
        return f.a + full * (f.b * k + f.e) + (part == 0 ? 0. : (f.c[full > 0] + f.d * part) * k + f.e * part);
    };
    GgPlan best{0, GG_T256, GG_T256};
    double least = time(fits[0], N);
    for (int t = 1; t < kinds; ++t)
        if (time(fits[t], N) < least) { least = time(fits[t], N); best.rest = fits[t].tile; }
    for (int h = 0; h < heads; ++h) {
        const long long tm = (M + fits[h].rows - 1) / fits[h].rows, rounds = tm * ((N + fits[h].cols - 1) / fits[h].cols) / 256;
        const long long cols = rounds * 256 / tm * fits[h].cols;  // columns whose tiles fit whole rounds
        if (cols <= 0 || cols >= N) continue;
        for (int t = h + 1; t < kinds; ++t) {
            const double both = time(fits[h], cols) + time(fits[t], N - cols) - meets;
            if (both < least) { least = both; best = {(int)cols, fits[h].tile, fits[t].tile}; }
        }
    }
    return best;
}

static int launch_tiles(const GgParams& p, lemo_dtype_t dt, bool add, int layout, GgTile tile, hipStream_t st) {
    if (dt == LEMO_F32 || tile == GG_T64) return launch_gather_gemm_small(p, dt, add, layout, tile, st);
    if (tile == GG_T256) return launch_gather_gemm_large(p, add, layout, st);
    return launch_gather_gemm_mid(p, add, layout, tile, st);
}

static int prepare_tiles(lemo_dtype_t dt, bool add, int layout) {
    int rc = prepare_gather_gemm_small(dt, add, layout);
    if (rc == 0 && dt == LEMO_BF16) rc = prepare_gather_gemm_mid(add, layout);
    if (rc == 0 && dt == LEMO_BF16) rc = prepare_gather_gemm_large(add, layout);
    return rc;
}

template <bool ADD, int LAYOUT>
static int launch_gg(const GgParams& p, lemo_dtype_t dt, hipStream_t st) {
    constexpr long long ROWS = 1ll << 24;  // a launch holds 2^32 threads: more rows than this are taken in turns
    if (LAYOUT != GG_TN && p.M > ROWS) {
        const int esz = dt == LEMO_BF16 ? 2 : 4;
        for (long long m = 0; m < p.M; m += ROWS) {
            GgParams part = p;
            part.M = p.M - m < ROWS ? p.M - m : ROWS;
            if (p.idx) part.idx = p.idx + m;
            else { part.A = static_cast<const char*>(p.A) + m * p.lda * esz; part.a_bytes -= (unsigned)(m * p.lda * esz); }
            if (ADD && p.oidx) {
                part.oidx = p.oidx + m;
            } else {
                part.Y = static_cast<char*>(p.Y) + m * p.ldy * esz;
                if (ADD) { part.out_rows -= m; part.y_bytes -= (unsigned)(m * p.ldy * esz); }
            }
            const int rc = launch_gg<ADD, LAYOUT>(part, dt, st);
            if (rc) return rc;
        }
        return 0;
    }
    const int unready = prepare_tiles(dt, ADD, LAYOUT);
    if (unready) return unready;
    const GgPlan plan = gg_plan(p.M, p.N, p.K, LAYOUT, dt);
    GgParams rest = p;
    if (plan.head_cols > 0) {  // (never binary32)
        GgParams head = p;
        head.N = plan.head_cols;
        const int rc = launch_tiles(head, dt, ADD, LAYOUT, plan.head, st);
        if (rc) return rc;
        // the same product on the columns behind: bases move by head_cols columns, the spans that begin there shrink by as much
        const long long c = plan.head_cols;
        rest.N -= plan.head_cols;
        rest.B = static_cast<const bf16_t*>(p.B) + (LAYOUT == GG_NT ? c * p.ldb : c);
        rest.Y = static_cast<bf16_t*>(p.Y) + c;
        if (p.bias) rest.bias = static_cast<const bf16_t*>(p.bias) + c;
        if (LAYOUT == GG_TN) rest.b_bytes -= (unsigned)c * 2u;
        if (ADD) rest.y_bytes -= (unsigned)c * 2u;
    }
    return launch_tiles(rest, dt, ADD, LAYOUT, plan.rest, st);
}

static unsigned span_bytes(long long rows, long long ld, long long cols, lemo_dtype_t dt) {  // host checked: fits 32 bits
    return (unsigned)(((rows - 1) * ld + cols) * (dt == LEMO_BF16 ? 2 : 4));
}

int launch_gather_gemm(const void* X, long long S, long long ldx, const int* idx, long long M, const void* W, long long ldw,
                       const void* bias, void* Y, long long ldy, int C, int N, lemo_dtype_t dt, hipStream_t st) {
    if (M == 0) return 0;
    return launch_gg<false, GG_NT>({X, W, bias, Y, idx, nullptr, ldx, ldw, ldy, M, 0, C, N, 0, 0, span_bytes(S, ldx, C, dt), 0, 0}, dt, st);
}

int launch_gather_gemm_add(const void* X, long long S, long long ldx, const int* idx, long long M, const void* W, long long ldw,
                           const void* bias, void* R, long long ldr, long long out_rows, const int* oidx, int C, int N,
                           lemo_dtype_t dt, hipStream_t st) {
    if (M == 0) return 0;
    return launch_gg<true, GG_NT>({X, W, bias, R, idx, oidx, ldx, ldw, ldr, M, out_rows, C, N, 0, 0, span_bytes(S, ldx, C, dt), 0,
                                   span_bytes(out_rows, ldr, N, dt)}, dt, st);
}

// Input gradient of Y = X[idx] W^T:  dX[oidx[m], c] += sum_n dY[m, n] W[n, c], W as stored ([N, C], contraction-major
// for this product).  bf16.  dY [M, N] compact rows; dX [out_rows, C].
int launch_gather_gemm_dx(const void* dY, long long ldy, long long M, const void* W, long long ldw, void* dX, long long lddx, long long out_rows,
                          const int* oidx, int C, int N, hipStream_t st) {
    if (M == 0) return 0;
    return launch_gg<true, GG_NN>({dY, W, nullptr, dX, nullptr, oidx, ldy, ldw, lddx, M, out_rows, /*contraction*/ N, /*columns*/ C, 0, 0,
                                   span_bytes(M, ldy, N, LEMO_BF16), 0, span_bytes(out_rows, lddx, C, LEMO_BF16)}, LEMO_BF16, st);
}

int prepare_gather_gemm_dw(lemo_dtype_t dt) {  // binary32 may also take transposed copies, as rows along the contraction
    const int rc = prepare_tiles(dt, false, GG_TN);
    return rc || dt == LEMO_BF16 ? rc : prepare_tiles(dt, false, GG_NT);
}

// Weight gradient dW[n, c] = sum_m dY[m, n] X[idx[m], c], both operands read as they are stored (contraction-major),
// the kept rows of X picked inside the B-tile load.
int launch_gather_gemm_dw_direct(const void* dY, long long ldy, const void* X, long long S, long long ldx, const int* idx, long long M, void* dW,
                                 long long lddw, int C, int N, lemo_dtype_t dt, hipStream_t st) {
    return launch_gg<false, GG_TN>({dY, X, nullptr, dW, idx, nullptr, ldy, ldx, lddw, /*output rows*/ N, 0, /*contraction*/ (int)M, /*columns*/ C, 0, 0,
                                    span_bytes(M, ldy, N, dt), span_bytes(S, ldx, C, dt), 0}, dt, st);
}

}  // namespace lemo
