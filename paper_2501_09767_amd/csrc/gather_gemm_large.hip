// The selective-load GEMM (and its in-place-add and gradient forms, see gather_gemm.hip) on 256 x 256 output tiles, bf16.
//
// Eight waves, two per SIMD, in a 2 x 4 grid: a wave computes a 64 x 32 block in each quadrant of the tile.  The contraction
// advances 128 bytes per slab.  Each operand's slab is two regions (its halves of 128 rows) in one of two LDS stages; regions
// are filled by LDS-direct loads and read into registers one quarter of a slab ahead:
//   quarter 1  A half 0 x the B half that is there already;     read: the other half of B
//   quarter 2  A half 0 x the other half of B;                  read: half 1 of A, over the fragments just used
//   quarter 3  A half 1 x the other half of B;                  read: that half of B of the next slab, likewise
//   quarter 4  A half 1 x the first half of B;                  read: half 0 of A of the next slab, likewise
// so the next slab starts with the B half this one ended its third quarter with, and the halves change roles slab by slab.  A
// region is asked for again half a slab after it was read, for the slab after next, and has a whole slab's time to arrive (one barrier
// per half slab; asked for with one barrier per slab and 0.9 slabs' time: 766 us against 743 at the first size below).
//
// What bounds it: the power the matrix cores draw on operands that switch.  16 x 16 x 32 MFMAs move half the accumulator
// bytes per flop that 32 x 32 x 16 ones do and the chip grants them a higher clock (same schedule: 760 / 821 us); consecutive
// MFMAs share an operand (the tiles of a quarter are walked back and forth, 752 / 758); the matrix cores are busy 81 % of the
// cycles at 1.65 GHz (profiled), and what is missing is lost at the barriers (7 %: 700 us with them taken out).
// Measured, us (four waves of 128 x 128 per tile with 32 x 32 MFMAs, slabs through registers, were before):
//   X W^T          8192 x 8192 x 8192: 742 (1.48 PFLOP/s), before 811;   9856 x 11008 x 4096: 645 / 706;  3280 x 4096 x 4096: 85 / 97
//   input gradient 8192 x 8192 x 8192: 775 / 845;   9856 x 11008 x 4096: 690 / 762
//   weight grad.   8192 x 8192 x 8192: 800 / 987;   9856 x 11008 x 4096: 688 / 869;   3280 x 11008 x 4096: 278 / 357
// Tried: four waves of 128 x 128 in this scheme (the compiler moves the 256 accumulators about: 987); counters in LDS, written
// ahead of the wait, in the barriers' place (793).
#include <mutex>

#include "gather_gemm.hpp"

namespace lemo {

constexpr int LG_BM = 256, LG_BN = 256;
constexpr int LG_KB = 128;               // bytes of the contraction per slab
constexpr int LG_KROWS = LG_KB / 2;      // rows of a contraction-major slab
constexpr int LG_REGION = 128 * LG_KB;   // one operand's half of a slab: 128 rows of 128 bytes, or 64 contraction rows of 256 bytes
constexpr int LG_STAGE = 2 * LG_REGION;  // rows (columns of the output) 0-127, 128-255
constexpr int LG_OPER = 2 * LG_STAGE;    // two stages of A, then two of B: 64 KB, the reach of an LDS read's immediate offset
constexpr int LG_TOK = 2 * LG_OPER;     // (GG_TN) token rings: per wave 4 slabs of 64 indices
constexpr int LG_EP = LG_BN * 2 + 16;    // epilogue: LDS pitch of a row of bf16, ...
constexpr int LG_EPF = LG_BN * 4 + 16;   // ... of binary32 (128 rows at a time)

constexpr int LG_WAVES = 8, LG_THREADS = 64 * LG_WAVES, LG_WN = 4;  // waves, along the columns
constexpr int LG_TA = 4, LG_TB = 2;      // 16-row tiles of a wave per half of A, of B
constexpr int LG_NLD = LG_REGION / (16 * LG_THREADS);  // loads per thread and region
constexpr int LG_LDS_LOOP = LG_TOK + LG_WAVES * 1024;
constexpr int LG_LDS_EPI = LG_BM * LG_EP > 128 * LG_EPF ? LG_BM * LG_EP : 128 * LG_EPF;
constexpr int LG_LDS = LG_LDS_LOOP > LG_LDS_EPI ? LG_LDS_LOOP : LG_LDS_EPI;
static_assert(LG_LDS <= 160 * 1024, "a workgroup's LDS");

template <bool ADD, int LAYOUT>
__global__ __launch_bounds__(LG_THREADS, 1) void gather_gemm_large_kernel(GgParams p) {
    constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    constexpr int TA = LG_TA, TB = LG_TB, NL = LG_NLD, T = LG_THREADS;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    int tm, tn;
    if (!gg_tile(blockIdx.x, p.tiles_m, p.tiles_n, 4, tm, tn)) return;
    const long long m0 = (long long)tm * LG_BM;
    const int n0 = tn * LG_BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / LG_WN, wn = wave % LG_WN;
    const bf16_t* A = static_cast<const bf16_t*>(p.A);
    const bf16_t* B = static_cast<const bf16_t*>(p.B);
    const unsigned lda_bytes = (unsigned)p.lda * 2, ldb_bytes = (unsigned)p.ldb * 2;  // host: both < 2^23
    const int K = p.K, kbytes = K * 2;
    const int nk = (K + LG_KROWS - 1) / LG_KROWS;

    // Loads.  Unit u = i * T + tid of a region is its LDS bytes [16 u, 16 u + 16); the lane asks for the piece that belongs there.
    // Rows along the contraction, 8 pieces: piece p of row r at p ^ (r / 2 % 8), so that one piece of 16 rows meets all banks.
    // Contraction-major rows, 16 pieces of 8 columns: at p ^ kswz(r); a half-wave of a transposing read takes rows 0-3 and 8-11
    // (+ 4, + 16), two pieces each.  The hardware range check sees the per-thread offset only: rows past an operand's end fail it
    // (or are clamped to the last one, A), pieces past the end of the contraction are given an offset at the descriptor's size in
    // both operands and arrive as zeros; the scalar offset moves along a row.
    auto kswz = [](int r) { return ((r & 3) | ((r >> 3) & 1) << 2) << 1; };
    const int kpos = ((tid & 7) ^ ((tid >> 4) & 7)) * 16;
    const int krow = tid >> 4, kcol = ((tid & 15) ^ kswz(krow)) * 16;
    unsigned a_voff[2][NL], b_voff[2][NL];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int row = r * 128 + i * (T / 8) + (tid >> 3), kr = i * (T / 16) + krow;
            if constexpr (A_KMAJOR) {
                a_voff[r][i] = kr * lda_bytes + r * 256 + kcol;
            } else {
                const long long m = min(m0 + row, p.M - 1);
                const unsigned tok = p.idx ? (unsigned)p.idx[m] : (unsigned)m;
                a_voff[r][i] = tok * lda_bytes + kpos;
            }
            if constexpr (LAYOUT == GG_NT) b_voff[r][i] = row * ldb_bytes + kpos;
            else if constexpr (LAYOUT == GG_NN) b_voff[r][i] = kr * ldb_bytes + r * 256 + kcol;
            else b_voff[r][i] = (unsigned)n0 * 2 + r * 256 + kcol;
        }
    // (GG_NT) this tile's rows of B
    const int b_rows = min(LG_BN, p.N - n0);
    const unsigned bn_bytes = (b_rows - 1) * ldb_bytes + kbytes;
    // contraction-major operand: from the slab's first row (and the tile's first column) to the operand's end, which refuses
    // the rows past it (host: the operand spans < 2^31 bytes)
    auto kmajor_rsrc = [&](const bf16_t* col0, unsigned ld_bytes, unsigned cols, int kt) {
        const bool live = kt < nk;
        const unsigned off = live ? (unsigned)(kt * LG_KROWS) * ld_bytes : 0u;
        const unsigned size = live ? (unsigned)(K - 1) * ld_bytes + cols * 2 - off : 0u;
        return raw_rsrc(reinterpret_cast<const char*>(col0) + off, size);
    };
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset_of(smem) + wave * 1024);
    const unsigned lds_tok = __builtin_amdgcn_readfirstlane(lds_offset_of(smem) + LG_TOK + wave * 1024);
    const u32x4 idx_rsrc = raw_rsrc(p.idx, p.idx ? (long long)K * 4 : 0);
    auto issue_tokens = [&](int kt) {  // indices of slab kt into the wave's ring
        if constexpr (LAYOUT == GG_TN) lds_direct_b32(idx_rsrc, lds_tok + (kt & 3) * 256, kt * (LG_KROWS * 4) + lane * 4);
    };
    struct Slab { u32x4 a, b; int soff; unsigned stage; bool in_k; };
    auto slab_of = [&](int kt) {
        Slab s;
        s.soff = kt * LG_KB;
        s.in_k = kpos < kbytes - s.soff;
        s.stage = lds0 + (kt & 1) * LG_STAGE;
        s.a = A_KMAJOR ? kmajor_rsrc(A + m0, lda_bytes, (unsigned)(p.M - m0), kt) : raw_rsrc(A, p.a_bytes);
        s.b = LAYOUT == GG_NN ? kmajor_rsrc(B + n0, ldb_bytes, (unsigned)(p.N - n0), kt)
                              : raw_rsrc(LAYOUT == GG_NT ? B + (long long)n0 * p.ldb : B, LAYOUT == GG_NT ? bn_bytes : p.b_bytes);
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // uniform values; the assembly wants them in scalar registers
            s.a[e] = __builtin_amdgcn_readfirstlane(s.a[e]);
            s.b[e] = __builtin_amdgcn_readfirstlane(s.b[e]);
        }
        return s;
    };
    unsigned tok[LAYOUT == GG_TN ? NL : 1];
    auto read_tokens = [&](int kt) {  // the rows of B of slab kt
        if constexpr (LAYOUT == GG_TN) {
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int kr = i * (T / 16) + krow, k = kt * LG_KROWS + kr;
                const unsigned row = p.idx ? *reinterpret_cast<const unsigned*>(smem + LG_TOK + wave * 1024 + (kt & 3) * 256 + kr * 4) : (unsigned)k;
                tok[i] = k < K ? row * ldb_bytes : p.b_bytes;  // (a row past the end: at or past the descriptor's size with any column)
            }
        }
    };
    auto load_a = [&](const Slab& s, int r, int i) {
        const unsigned dst = s.stage + r * LG_REGION + i * (T * 16);
        if constexpr (A_KMAJOR) lds_direct_b128(s.a, dst, (int)a_voff[r][i]);
        else lds_direct_b128(s.a, dst, (int)(s.in_k ? a_voff[r][i] : p.a_bytes), s.soff);
    };
    auto load_b = [&](const Slab& s, int r, int i) {
        const unsigned dst = s.stage + LG_OPER + r * LG_REGION + i * (T * 16);
        if constexpr (LAYOUT == GG_TN) lds_direct_b128(s.b, dst, (int)(tok[i] == p.b_bytes ? tok[i] : tok[i] + b_voff[r][i]));
        else if constexpr (LAYOUT == GG_NN) lds_direct_b128(s.b, dst, (int)b_voff[r][i]);
        else lds_direct_b128(s.b, dst, (int)(s.in_k ? b_voff[r][i] : bn_bytes), s.soff);
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // fragment (16-row tile t of a region, chunk c of the slab); the transposing read: see gather_gemm.hpp
    const int l16 = lane & 15, quad = lane >> 4;  // MFMA operands: lane holds row l16 of a 16-row tile, elements 8 quad .. + 7 of a chunk of 32
    const int swz = (l16 >> 1) & 7;
    const int trow = 8 * quad + (l16 >> 2);  // this lane's row of a transposing read
    const int tr_base = trow * 256 + (lane & 1) * 8, tr_piece = (lane & 3) >> 1, tr_swz = kswz(trow);
    auto frag = [&](const char* region, bool kmajor, int t, int c) {
        if (!kmajor) return *reinterpret_cast<const u32x4*>(region + t * 16 * LG_KB + l16 * LG_KB + (((4 * c + quad) ^ swz) << 4));
        const char* at = region + tr_base + c * 32 * 256 + (((t * 2 + tr_piece) ^ tr_swz) << 4);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at + 4 * 256));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        return u32x4{l2.x, l2.y, h2.x, h2.y};
    };

    f32x4 acc[2][TA][2][TB];  // [half of A][tile][half of B][tile]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int j = 0; j < TB; ++j) acc[a][i][b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // fragments: the current half of A, both halves of B
    u32x4 fa[2][TA], fb[2][2][TB];
    auto read_a = [&](int st, int r, int c, int i) { fa[c][i] = frag(smem + st * LG_STAGE + r * LG_REGION, A_KMAJOR, wm * TA + i, c); };
    auto read_b = [&](int st, int r, int c, int j) { fb[r][c][j] = frag(smem + LG_OPER + st * LG_STAGE + r * LG_REGION, B_KMAJOR, wn * TB + j, c); };

    constexpr int NM = 2 * TA * TB;  // MFMAs of a quarter
    // One quarter of a slab: the MFMAs of (half AH of A) x (half BH of B), `mem(q, c, i, j)` behind MFMA q, which is of chunk c
    // and tile (i, j).  The source order is the issue order.
    auto quarter = [&](auto ah, auto bh, bool by_columns, auto mem) {
        constexpr int AH = decltype(ah)::value, BH = decltype(bh)::value;
#pragma unroll
        for (int q = 0; q < NM; ++q) {  // the tiles back and forth, row by row or column by column: neighbours share a fragment
            const int c = q / (TA * TB), w = q % (TA * TB), u = by_columns ? w / TA : w / TB, v = by_columns ? w % TA : w % TB;
            const int back = by_columns ? TA - 1 - v : TB - 1 - v, t = u & 1 ? back : v, i = by_columns ? t : u, j = by_columns ? u : t;
            __builtin_amdgcn_sched_barrier(0);
            // (the operands exchanged: a lane holds one row of the output, four consecutive columns of it)
            acc[AH][i][BH][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[BH][c][j]), __builtin_bit_cast(bf16x8, fa[c][i]), acc[AH][i][BH][j], 0, 0, 0);
            mem(q, c, i, j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    auto load_region = [&](const Slab& s, bool a, int r) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (a) load_a(s, r, i); else load_b(s, r, i);
        }
    };

    // What would have been asked for in the halves before: {B 0} {A 0, B 1} of slab 0, {A 1 of 0, B 1 of 1}, {A 0, B 0 of 1}
    if constexpr (LAYOUT == GG_TN) {
        for (int kt = 0; kt < 4; ++kt) issue_tokens(kt);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
    }
    {
        const Slab s0 = slab_of(0), s1 = slab_of(1);
        read_tokens(0);
        load_region(s0, false, 0);
        load_region(s0, true, 0);
        load_region(s0, false, 1);
        load_region(s0, true, 1);
        read_tokens(1);
        load_region(s1, false, 1);
        load_region(s1, true, 0);
        load_region(s1, false, 0);
        read_tokens(2);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(5 * NL));
    barrier();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int j = 0; j < TB; ++j) read_b(0, 0, c, j);
#pragma unroll
        for (int i = 0; i < TA; ++i) read_a(0, 0, c, i);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * NL));
    __builtin_amdgcn_s_waitcnt(LGKMCNT0);

    // Waves of one SIMD do not take turns: one of them goes first (X W^T 752 -> 742 us at 8192^3, the gradients no change)
    if constexpr (LAYOUT == GG_NT)
        if (wave < LG_WAVES / 2) __builtin_amdgcn_s_setprio(1);
    // Slab kt, kt & 1 == PAR.  Halves of a slab begin with a barrier, before which every wave has seen to it that the regions
    // read in this half have landed (its own part: all loads but the last IN_FLIGHT, which complete in order) and that it
    // has read what this half's loads overwrite: all but the fragments read in the quarter before.
    constexpr int IN_FLIGHT = 3 * NL;
    auto slab = [&](int kt, auto par_tag) {
        constexpr int PAR = decltype(par_tag)::value, F = PAR, L = PAR ^ 1;
        using IF = std::integral_constant<int, F>;
        using IL = std::integral_constant<int, L>;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(IN_FLIGHT));
        __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(A_KMAJOR ? 15 : 2 * TA));
        barrier();
        const Slab s1 = slab_of(kt + 1), s2 = slab_of(kt + 2);
        quarter(I0{}, IF{}, false, [&](int q, int c, int i, int j) {
            if (q < 2 * TB) read_b(PAR, L, q / TB, q % TB);
            if (q < 2 * NL) {
                if (q < NL) load_a(s1, 1, q); else load_b(s2, F, q - NL);
            }
        });
        quarter(I0{}, IL{}, false, [&](int q, int c, int i, int j) {
            if (q % TB == TB - 1) read_a(PAR, 1, c, i);
        });
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(IN_FLIGHT));
        barrier();
        if constexpr (LAYOUT == GG_TN) issue_tokens(kt + 4);
        quarter(I1{}, IL{}, true, [&](int q, int c, int i, int j) {
            if (q % TA == TA - 1) read_b(PAR ^ 1, L, c, j);
            if (q < 2 * NL) {
                if (q < NL) load_a(s2, 0, q); else load_b(s2, L, q - NL);
            }
        });
        if constexpr (LAYOUT == GG_TN) read_tokens(kt + 3);
        quarter(I1{}, IF{}, false, [&](int q, int c, int i, int j) {
            if (q % TB == TB - 1) read_a(PAR ^ 1, 0, c, i);
        });
    };
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        slab(kt, I0{});
        slab(kt + 1, I1{});
    }
    if (kt < nk) slab(kt, I0{});
    if constexpr (LAYOUT == GG_NT) __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // requests past the end write (zeros) to the stages, too
    __builtin_amdgcn_s_waitcnt(LGKMCNT0);
    __syncthreads();

    // Epilogue, through LDS: whole rows of 16-byte pieces, 8 consecutive columns per lane.  In-place add: binary32, half of the tile
    // at a time, what the rows hold already asked for ahead through a range-checked descriptor (rows that are not to be written get
    // an offset past its end).  acc[a][i][b][j][r] is row a*128 + (wm*TA + i)*16 + l16, column b*128 + (wn*TB + j)*16 + 4*quad + r of the tile.
    const bool vec_ok = p.ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(p.Y) & 15u) == 0;
    const int piece = lane & 31, rsub = lane >> 5;  // 32 lanes per row, 8 columns each
    const int ncol = n0 + piece * 8;
    if (p.bias) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int n = n0 + b * 128 + (wn * TB + j) * 16 + 4 * quad + r;
                    const float bv = n < p.N ? bf16_to_f32(static_cast<const uint16_t*>(p.bias)[n]) : 0.f;
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int i = 0; i < TA; ++i) acc[a][i][b][j][r] += bv;
                }
    }
    if constexpr (ADD) {
        constexpr int ROWS = 128 / LG_WAVES, PASSES = ROWS / 2;  // rows a wave finishes per half of the tile
        const bool col_vec = vec_ok && ncol + 8 <= p.N;
        const __amdgpu_buffer_rsrc_t y_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.Y, 0, (int)p.y_bytes, 0x00020000);
        const unsigned NONE = p.y_bytes, ldy_bytes = (unsigned)p.ldy * 2;
        unsigned off[2][PASSES];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int q = 0; q < PASSES; ++q) {
                const long long m = m0 + a * 128 + wave * ROWS + q * 2 + rsub;
                const long long row = p.oidx ? (long long)p.oidx[min(m, p.M - 1)] : m;
                const bool ok = (m < p.M) & (ncol < p.N) & (row >= 0) & (row < p.out_rows);
                off[a][q] = ok ? (unsigned)row * ldy_bytes + (unsigned)ncol * 2u : NONE;
            }
        u32x4 old[2][PASSES];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int q = 0; q < PASSES; ++q)
                old[a][q] = __builtin_amdgcn_raw_buffer_load_b128(y_rsrc, (int)(col_vec ? off[a][q] : NONE), 0, 0);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (a) __syncthreads();
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int j = 0; j < TB; ++j)
                        *reinterpret_cast<f32x4*>(smem + ((wm * TA + i) * 16 + l16) * LG_EPF + (b * 128 + (wn * TB + j) * 16 + 4 * quad) * 4) = acc[a][i][b][j];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PASSES; ++q) {
                if (off[a][q] == NONE) continue;
                const char* at = smem + (wave * ROWS + q * 2 + rsub) * LG_EPF + piece * 32;
                const f32x4 lo = *reinterpret_cast<const f32x4*>(at), hi = *reinterpret_cast<const f32x4*>(at + 16);
                const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                uint16_t* dst = reinterpret_cast<uint16_t*>(static_cast<char*>(p.Y) + off[a][q]);
                if (col_vec) {
                    u32x4 out;
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[e] = pack_bf16x2_hw(v[2 * e] + bf16lo_to_f32(old[a][q][e]), v[2 * e + 1] + bf16hi_to_f32(old[a][q][e]));
                    *reinterpret_cast<u32x4*>(dst) = out;
                } else {  // ragged right edge or unaligned rows: element by element
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (ncol + e < p.N) dst[e] = (uint16_t)(pack_bf16x2_hw(v[e] + bf16_to_f32(dst[e]), 0.f) & 0xffffu);
                }
            }
        }
    } else {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int j = 0; j < TB; ++j) {
                        const f32x4& v = acc[a][i][b][j];
                        *reinterpret_cast<uint2*>(smem + (a * 128 + (wm * TA + i) * 16 + l16) * LG_EP + (b * 128 + (wn * TB + j) * 16 + 4 * quad) * 2) =
                            make_uint2(pack_bf16x2_hw(v[0], v[1]), pack_bf16x2_hw(v[2], v[3]));
                    }
        __syncthreads();
        constexpr int ROWS = LG_BM / LG_WAVES;
#pragma unroll 4
        for (int q = 0; q < ROWS / 2; ++q) {
            const int row = wave * ROWS + q * 2 + rsub;
            const long long m = m0 + row;
            const u32x4 v = *reinterpret_cast<const u32x4*>(smem + row * LG_EP + piece * 16);
            if (m >= p.M) continue;
            uint16_t* dst = static_cast<uint16_t*>(p.Y) + m * p.ldy + ncol;
            if (vec_ok && ncol + 8 <= p.N) {
                *reinterpret_cast<u32x4*>(dst) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (ncol + e < p.N) dst[e] = (uint16_t)(v[e >> 1] >> ((e & 1) * 16));
            }
        }
    }
}

template <bool ADD, int LAYOUT>
static int launch_large(GgParams p, hipStream_t st) {
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gather_gemm_large_kernel<ADD, LAYOUT>), hipFuncAttributeMaxDynamicSharedMemorySize, LG_LDS);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    p.tiles_m = (int)((p.M + LG_BM - 1) / LG_BM);
    p.tiles_n = (p.N + LG_BN - 1) / LG_BN;
    const int per_xcd = (p.tiles_m * p.tiles_n + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((gather_gemm_large_kernel<ADD, LAYOUT>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(LG_THREADS), LG_LDS, st, p);
    return (int)hipGetLastError();
}

int launch_gather_gemm_large(const GgParams& p, bool add, int layout, hipStream_t st) {
    if (layout == GG_TN) return launch_large<false, GG_TN>(p, st);
    if (layout == GG_NN) return launch_large<true, GG_NN>(p, st);
    return add ? launch_large<true, GG_NT>(p, st) : launch_large<false, GG_NT>(p, st);
}

}  // namespace lemo
