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
#include "gather_gemm_regions.hpp"

namespace lemo {

constexpr int LG_BM = 256, LG_BN = 256;
constexpr int LG_STAGE = 2 * RG_BYTES;   // regions: rows (columns of the output) 0-127, 128-255
constexpr int LG_OPER = 2 * LG_STAGE;    // two stages of A, then two of B: 64 KB, the reach of an LDS read's immediate offset
constexpr int LG_TOK = 2 * LG_OPER;      // (GG_TN) token rings
constexpr int LG_EP = LG_BN * 2 + 16;    // epilogue: LDS pitch of a row of bf16, ...
constexpr int LG_EPF = LG_BN * 4 + 16;   // ... of binary32 (128 rows at a time)
constexpr int LG_WN = 4;                 // waves along the columns
constexpr int LG_TA = 4, LG_TB = 2;      // 16-row tiles of a wave per half of A, of B
constexpr int LG_LDS_EPI = LG_BM * LG_EP > 128 * LG_EPF ? LG_BM * LG_EP : 128 * LG_EPF;
constexpr int LG_LDS = LG_TOK + RG_TOK > LG_LDS_EPI ? LG_TOK + RG_TOK : LG_LDS_EPI;
static_assert(LG_LDS <= 160 * 1024, "a workgroup's LDS");

template <bool ADD, int LAYOUT>
__global__ __launch_bounds__(RG_THREADS, 1) void gather_gemm_large_kernel(GgParams p) {
    constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    constexpr int TA = LG_TA, TB = LG_TB, NL = RG_NLD;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    int tm, tn;
    if (!gg_tile(blockIdx.x, p.tiles_m, p.tiles_n, 4, tm, tn)) return;
    const long long m0 = (long long)tm * LG_BM;
    const int n0 = tn * LG_BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / LG_WN, wn = wave % LG_WN;
    const int l16 = lane & 15, quad = lane >> 4;
    using Loads = RgLoads<LAYOUT, 4, 4>;
    using Slab = typename Loads::Slab;
    Loads ld(p, m0, n0, tid, smem + LG_TOK + wave * 1024);
    const int nk = ld.nk;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset_of(smem) + wave * 1024);
    auto load_a = [&](const Slab& s, int kt, int r, int i) { ld.load_a(s, 2 * r + i, lds0 + (kt & 1) * LG_STAGE); };
    auto load_b = [&](const Slab& s, int kt, int r, int i) { ld.load_b(s, 2 * r + i, lds0 + LG_OPER + (kt & 1) * LG_STAGE); };

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
    auto read_a = [&](int st, int r, int c, int i) { fa[c][i] = rg_fragment(smem + st * LG_STAGE + r * RG_BYTES, A_KMAJOR, wm * TA + i, c, lane); };
    auto read_b = [&](int st, int r, int c, int j) { fb[r][c][j] = rg_fragment(smem + LG_OPER + st * LG_STAGE + r * RG_BYTES, B_KMAJOR, wn * TB + j, c, lane); };

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
            rg_mma(acc[AH][i][BH][j], fa[c][i], fb[BH][c][j]);
            mem(q, c, i, j);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    auto load_region = [&](const Slab& s, int kt, bool a, int r) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (a) load_a(s, kt, r, i); else load_b(s, kt, r, i);
        }
    };

    // What would have been asked for in the halves before: {B 0} {A 0, B 1} of slab 0, {A 1 of 0, B 1 of 1}, {A 0, B 0 of 1}
    if constexpr (LAYOUT == GG_TN) {
        for (int kt = 0; kt < 4; ++kt) ld.issue_tokens(kt, lane);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
    }
    {
        const Slab s0 = ld.slab(0), s1 = ld.slab(1);
        ld.read_tokens(0);
        load_region(s0, 0, false, 0);
        load_region(s0, 0, true, 0);
        load_region(s0, 0, false, 1);
        load_region(s0, 0, true, 1);
        ld.read_tokens(1);
        load_region(s1, 1, false, 1);
        load_region(s1, 1, true, 0);
        load_region(s1, 1, false, 0);
        ld.read_tokens(2);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(5 * NL));
    rg_barrier();
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
        if (wave < RG_WAVES / 2) __builtin_amdgcn_s_setprio(1);
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
        rg_barrier();
        const Slab s1 = ld.slab(kt + 1), s2 = ld.slab(kt + 2);
        quarter(I0{}, IF{}, false, [&](int q, int c, int i, int j) {
            if (q < 2 * TB) read_b(PAR, L, q / TB, q % TB);
            if (q < 2 * NL) {
                if (q < NL) load_a(s1, PAR ^ 1, 1, q); else load_b(s2, PAR, F, q - NL);
            }
        });
        quarter(I0{}, IL{}, false, [&](int q, int c, int i, int j) {
            if (q % TB == TB - 1) read_a(PAR, 1, c, i);
        });
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(IN_FLIGHT));
        rg_barrier();
        ld.issue_tokens(kt + 4, lane);
        quarter(I1{}, IL{}, true, [&](int q, int c, int i, int j) {
            if (q % TA == TA - 1) read_b(PAR ^ 1, L, c, j);
            if (q < 2 * NL) {
                if (q < NL) load_a(s2, PAR, 0, q); else load_b(s2, PAR, L, q - NL);
            }
        });
        ld.read_tokens(kt + 3);
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
        constexpr int ROWS = 128 / RG_WAVES, PASSES = ROWS / 2;  // rows a wave finishes per half of the tile
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
        constexpr int ROWS = LG_BM / RG_WAVES;
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
static int prepare_large() {
    static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&gather_gemm_large_kernel<ADD, LAYOUT>), LG_LDS}});
    return err;
}

template <bool ADD, int LAYOUT>
static int launch_large(GgParams p, hipStream_t st) {
    p.tiles_m = (int)((p.M + LG_BM - 1) / LG_BM);
    p.tiles_n = (p.N + LG_BN - 1) / LG_BN;
    const int per_xcd = (p.tiles_m * p.tiles_n + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((gather_gemm_large_kernel<ADD, LAYOUT>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(RG_THREADS), LG_LDS, st, p);
    return (int)hipGetLastError();
}

int prepare_gather_gemm_large(bool add, int layout) {
    if (layout == GG_TN) return prepare_large<false, GG_TN>();
    if (layout == GG_NN) return prepare_large<true, GG_NN>();
    return add ? prepare_large<true, GG_NT>() : prepare_large<false, GG_NT>();
}

int launch_gather_gemm_large(const GgParams& p, bool add, int layout, hipStream_t st) {
    if (layout == GG_TN) return launch_large<false, GG_TN>(p, st);
    if (layout == GG_NN) return launch_large<true, GG_NN>(p, st);
    return add ? launch_large<true, GG_NT>(p, st) : launch_large<false, GG_NT>(p, st);
}

}  // namespace lemo
