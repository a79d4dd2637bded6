// Selective-load GEMM (Sec. 4.4): Y[m,:] = X[kept_idx[m],:] . W^T (+ bias).  The kept rows are read
// straight from the [S,C] input inside the A-tile load -- a kept row is C contiguous elements, so the
// indexed load is as coalesced as a dense one and no compacted copy of X ever exists.
//
// This file holds the launches and the choice of the output tiles; the kernels are gather_gemm_large.hip (256 x 256, bf16)
// and gather_gemm_small.hip.
#include "gather_gemm.hpp"

namespace lemo {

// Which tiles a product is cut into: the first `cols256` columns into 256 x 256 tiles, the others into `rest` tiles.
//
// The large tile is the fastest per flop but comes in rounds of 256, one per CU, and a round lasts as long for one tile
// as for (nearly) all: with few tiles, or just past a full round, smaller ones win although they move more bytes per
// flop.  The choice is the least of these times, in us, for a contraction of k slabs of 128 bytes; the constants are
// fits to M = 64 ... 9856, N = 256 ... 14336, K = 256 ... 11008, in a stream of other work (within a fourth of what was
// measured; with the operands in the caches already, the smaller tiles take up to 40 % less than this):
//   256 x 256  6 + k (1.5 per full round + 1.5 for a last one over half full, 1.15 otherwise)
//   128 x 128  4 + (k + 3) (0.6 up to 256 tiles -- one per CU --, then n/512 + 0.25, at least 0.95)
//   64 x 64    4 + (2 + 0.25 k) per 256 tiles
//   256 x 256 for the columns that fill whole rounds, 128 x 128 for the rest: the sum (the launches follow each other)
// e.g. M = 256, N = K = 4096: 80 / 32 / 17.5 us; M = 256, N = 11008, K = 4096: 82 / 45 / 58; M = 1500, N = K = 4096: 85 /
// 59 / 97; M = 3280, N = 11008, K = 4096: 282 / 292 / 565, and 9856 rows of it 705 / 815 / 1610.  Between 256 x 256 and
// 128 x 128 the line is known to a fifth: M = 2000, N = 4096, K = 11008 takes the large tiles, 191 / 176 / 270.
// Weight gradients (GG_TN): both operands pass the transposing read, which the 128 x 128 tile pays twice as often; it
// takes over where the large tiles leave half the CUs idle (256 x 256 / 128 x 128, N = 4096: C = 1024, 64 large tiles, 700
// tokens 28 / 14.5 us; 4000 tokens, C = 2048, 128 tiles 113 / 78, C = 2304, 144 tiles 113 / 107, C = 3072, 192 tiles 115 / 112,
// C = 4096, 256 tiles 133 / 145; N = 11008, C = 4096, 9856 tokens: 862 / 1317).
// binary32: the products are bound by MFMA issue at any tile size, so only the fill counts: 128 x 128, or 32 x 32 tiles
// with the contraction split over four waves, up to 192 of the former (M = 200, N = K = 768: 51 / 11.6 us; 96 tiles, M = 500,
// N = 3072, K = 768: 54 / 32; 160, M = 640, N = 4096, K = 1024: 69 / 59; 192, M = 768: 69.5 / 68.6; 256, M = 1024: 71 / 87; dW of 700
// tokens, 4096 x 1024, 256 tiles: 54 / 81).  Past 256 a second round that is nearly empty would favour the small tiles again
// (288 tiles, M = 1500, N = 3072, K = 768: 97 / 80); with more rounds the two are alike (1032 tiles, M = 1500, N = 11008, K = 4096:
// 1193 / 1201, which 256 x 256 tiles took 1852 for).
struct GgPlan { int cols256; GgTile rest; };
static GgPlan gg_plan(long long M, int N, int K, int layout, lemo_dtype_t dt) {
    auto tiles = [&](int b, int n) { return (double)((M + b - 1) / b) * (double)((n + b - 1) / b); };
    const double n256 = tiles(256, N), n128 = tiles(128, N), n64 = tiles(64, N);
    if (dt == LEMO_F32) return {0, n128 <= 192 ? GG_T64 : GG_T128};
    const double k = K / 64.;
    auto t256 = [&](double n) {
        const double full = (double)(long long)(n / 256), rem = n - 256 * full;
        return 6 + k * (1.5 * full + (rem == 0 ? 0. : rem <= 128 ? 1.15 : 1.5));
    };
    auto t128 = [&](double n) { return 4 + (k + 3) * (n <= 256 ? 0.6 : n / 512 + 0.25 > 0.95 ? n / 512 + 0.25 : 0.95); };
    auto t64 = [&](double n) { return 4 + (2 + 0.25 * k) * (double)((long long)(n + 255) / 256); };
    if (layout == GG_TN) {
        if (n256 > 128) return {N, GG_T128};
        return {0, t64(n64) < t128(n128) ? GG_T64 : GG_T128};
    }
    GgPlan best{N, GG_T128};
    double t = t256(n256);
    const long long tm = (M + 255) / 256, rounds = (long long)n256 / 256;
    const long long cols = rounds * 256 / tm * 256;  // columns whose tiles fit whole rounds
    if (rounds > 0 && cols > 0 && cols < N) {
        const double mixed = t256((double)tm * (double)(cols / 256)) + t128(tiles(128, N - (int)cols));
        if (mixed < t) { t = mixed; best = {(int)cols, GG_T128}; }
    }
    if (t128(n128) < t) { t = t128(n128); best = {0, GG_T128}; }
    if (t64(n64) < t) best = {0, GG_T64};
    return best;
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
    const GgPlan plan = gg_plan(p.M, p.N, p.K, LAYOUT, dt);
    if (plan.cols256 >= p.N) return launch_gather_gemm_large(p, ADD, LAYOUT, st);  // (never binary32)
    GgParams rest = p;
    if (plan.cols256 > 0) {
        GgParams head = p;
        head.N = plan.cols256;
        const int rc = launch_gather_gemm_large(head, ADD, LAYOUT, st);
        if (rc) return rc;
        // the same product on the columns behind: bases move by cols256 columns, the output's span shrinks by as much
        // (bf16, and not GG_TN, whose b_bytes would move as well)
        const long long c = plan.cols256;
        rest.N -= plan.cols256;
        rest.B = static_cast<const bf16_t*>(p.B) + (LAYOUT == GG_NT ? c * p.ldb : c);
        rest.Y = static_cast<bf16_t*>(p.Y) + c;
        if (p.bias) rest.bias = static_cast<const bf16_t*>(p.bias) + c;
        if (ADD) rest.y_bytes -= (unsigned)c * 2u;
    }
    return launch_gather_gemm_small(rest, dt, ADD, LAYOUT, plan.rest, st);
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

// Weight gradient dW[n, c] = sum_m dY[m, n] X[idx[m], c], both operands read as they are stored (contraction-major),
// the kept rows of X picked inside the B-tile load.
int launch_gather_gemm_dw_direct(const void* dY, long long ldy, const void* X, long long S, long long ldx, const int* idx, long long M, void* dW,
                                 long long lddw, int C, int N, lemo_dtype_t dt, hipStream_t st) {
    return launch_gg<false, GG_TN>({dY, X, nullptr, dW, idx, nullptr, ldy, ldx, lddw, /*output rows*/ N, 0, /*contraction*/ (int)M, /*columns*/ C, 0, 0,
                                    span_bytes(M, ldy, N, dt), span_bytes(S, ldx, C, dt), 0}, dt, st);
}

}  // namespace lemo
