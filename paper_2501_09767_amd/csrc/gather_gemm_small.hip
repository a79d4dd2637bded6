// The selective-load GEMM (and its in-place-add and gradient forms, see gather_gemm.hip) on 64 x 64 output tiles (bf16, for
// products of few tiles) and, in binary32, on 128 x 128, 32 x 32 and 16 x 16 ones.
//
// A wave computes a block of 32 x 32 MFMA tiles from slabs of 128 bytes of the contraction; two shapes:
//   GW = 1  every wave has its own slabs: 64 x 64 output tile, the four waves take every fourth slab of the contraction
//           each and their partial tiles are added, in wave order, through LDS at the end.  No barrier in the main loop.
//           Bound by the latency of the loads: 128 KB per CU are in flight, all its LDS holds (M = 256, N = K = 4096: 17.5 us with
//           the operands in the caches, 20.8 from HBM).  binary32, whose MFMAs take 16 times as long, is bound by those instead
//           and takes 32 x 32 or 16 x 16 blocks, for four times the workgroups or 16 (splitting an operand for one tile costs as much as it saves).
//   GW = 4  (binary32) the four waves of a workgroup share a slab: 128 x 128 output tile, 64 x 64 per wave, two workgroups per
//           CU (70 KB of LDS each).  The products are three-part splits on the bf16 matrix cores (lemo_common.hpp); a slab costs a
//           wave 352 instructions of splitting and 16 for the largest operands beside 1536 cycles of MFMAs, 2240 cycles where binary32
//           MFMAs took 4096.  Sums that the splits may not give are formed again from those (form_again).  us, binary32
//           MFMAs / now: 1500 x 11008 x 4096 1188 / 784 (2.02 rounds run as 3), 1024 x 4096 x 1024 71 / 54, 10000 x 768 x 3072 359 /
//           249, weight gradient 8192 x 2048 of 300 tokens 95 / 78; error against 64 bits 1.1e-6 / 1.0e-6, 5.7e-7 / 4.9e-7, 9.9e-7 /
//           8.6e-7, 3.1e-7 / 2.6e-7.  The first product without the largest operands 770, with the smallest as well, which would spare
//           form_again its look for them, 825; with many sums of exactly zero (whole numbers, which the chip multiplies faster)
//           617, with that look 815; one row of small values 1283, all rows 2350, not a number throughout 2218.  Sums of one or two
//           products are nearer to 64 bits from binary32 MFMAs, and take those.
// Slabs arrive by LDS-direct loads, two per group in flight, and the registers are the third buffer: the MFMA fragments
// of the next slab are read during the first MFMAs of the current one, which frees its LDS stage for the slab after next.
// Measured beside this (M = 256, N = K = 4096 with 64 x 64 tiles, 17.5 us): a ring of four half-slabs with the loads spread over all
// MFMAs 21.6 (64-byte row segments halve what an L2 delivers), a ring of two slabs without the registers' lookahead 19.1;
// 16 x 16 x 32 MFMAs, which pay in the larger tiles, change nothing here (20.6 / 20.9 from HBM).
#include "gather_gemm.hpp"

namespace lemo {

constexpr int SG_THREADS = 256;
constexpr int SG_KB = 128;          // bytes of the contraction per slab

constexpr int SPLIT_LEAST = 3;      // terms of a sum from which splits are no further from 64 bits than binary32 MFMAs

// WT = MFMA tiles per wave and direction, of E x E
template <int GW, int ESZ, int WT, int E = 32> struct SgGeo {
    static constexpr int W = GW == 4 ? 2 : 1;       // waves of a group per output direction
    static constexpr int WB = E * WT;               // rows and columns of a wave's block
    static constexpr int BM = WB * W, BN = WB * W;  // output tile
    static constexpr int GROUPS = 4 / GW;           // the slabs are dealt out to the groups in turn
    static constexpr int OPER = WB * W * SG_KB;     // bytes of one operand's slab
    static constexpr int STAGE = 2 * OPER;
    static constexpr int NLD = OPER / (GW * 1024);  // LDS-direct loads per thread, operand and slab
    static constexpr int TOK = GROUPS * 2 * STAGE;  // (GG_TN) token rings: per wave 4 slabs of 64 indices
    static constexpr int EP = WB * 4 + 16;          // epilogue: LDS pitch of a row of a wave's block of floats
    static constexpr int EPI = 4 * WB * EP;
    static constexpr int LDS = TOK + 4096 > EPI ? TOK + 4096 : EPI;
    static constexpr int KROWS = SG_KB / ESZ;       // contraction-major slab: rows,
    static constexpr int PIECES = WB * W * ESZ / 16;     // 16-byte pieces per row
    static constexpr int CHUNK = E == 16 ? 64 : 32;      // bytes of the contraction of one fragment; its MFMA tile per lane: rows,
    static constexpr int CHUNKS = SG_KB / CHUNK, REGS = E * E / 64;  // registers
    // position of 16-byte piece p of row r (the loads fill consecutive LDS bytes, so conflicts are avoided by exchanging
    // pieces inside a row).  Rows along the contraction, 128 bytes: p ^ (r / 2 % 8) spreads one piece of 16 rows over all
    // banks.  Contraction-major rows: the transposing read (16 bit) takes 4 rows x 4 pieces at a time; of binary32 rows, which
    // are read element by element, the two half-waves take rows 4 apart, 8 pieces each.
    __device__ static constexpr int swz(int r) { return (r >> 1) & 7; }
    __device__ static constexpr int kswz(int r) { return WT == 1 ? 0 : ESZ == 4 ? ((r >> 2) & 1) << 3 : ((r >> 1) & 1) << 2; }
};

// SPLIT: products from three-part splits
template <typename T, bool ADD, int LAYOUT, int GW, int WT, bool SPLIT, int E = 32>
__global__ __launch_bounds__(SG_THREADS, GW == 4 ? 2 : 1) void gather_gemm_small_kernel(GgParams p) {
    constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    constexpr int ESZ = (int)sizeof(T);
    static_assert(ESZ == 4 || (WT == 2 && GW == 1), "the 16-bit transposing read is laid out for 64 x 64 tiles");
    static_assert(E == 32 || (ESZ == 4 && GW == 1 && WT == 1 && !SPLIT), "16 x 16 tiles: small binary32 products");
    using G = SgGeo<GW, ESZ, WT, E>;
    using Tile = std::conditional_t<E == 16, f32x4, f32x16>;
    constexpr int GROUPS = G::GROUPS, NLD = G::NLD;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    int tm, tn;
    if (!gg_tile(blockIdx.x, p.tiles_m, p.tiles_n, 8, tm, tn)) return;
    const long long m0 = (long long)tm * G::BM;
    const int n0 = tn * G::BN;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / GW, wg = wave % GW, gtid = tid % (64 * GW);
    const int wm = wg >> 1, wn = wg & 1;
    const T* A = static_cast<const T*>(p.A);
    const T* B = static_cast<const T*>(p.B);
    const unsigned lda_bytes = (unsigned)p.lda * ESZ, ldb_bytes = (unsigned)p.ldb * ESZ;  // host: both < 2^23
    const int K = p.K, kbytes = K * ESZ;  // (along-the-contraction operands: bytes of a row)
    const int nk = A_KMAJOR ? (K + G::KROWS - 1) / G::KROWS : (kbytes + SG_KB - 1) / SG_KB;

    // Per-thread byte offsets of the loads.  The range check (raw_rsrc): rows past an
    // operand's end fail it (or are clamped to the last one, A), pieces past the end of the contraction are given an
    // offset at the descriptor's size in both operands and arrive as zeros; the scalar offset moves along a row, whose valid pieces pass with it.
    auto kpos = [&](int i) { return ((gtid & 7) ^ G::swz(i * 8 * GW + (gtid >> 3))) * 16; };  // of piece i in a row's slab
    unsigned a_voff[NLD], b_voff[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int u = i * 64 * GW + gtid, krow = u / G::PIECES, kcol = ((u % G::PIECES) ^ G::kswz(krow)) * 16;
        if constexpr (A_KMAJOR) {
            a_voff[i] = krow * lda_bytes + kcol;
        } else {
            const long long m = min(m0 + u / 8, p.M - 1);
            const unsigned row = p.idx ? (unsigned)p.idx[m] : (unsigned)m;
            a_voff[i] = row * lda_bytes + kpos(i);  // host: the operand spans < 2^32 bytes
        }
        if constexpr (LAYOUT == GG_NT) b_voff[i] = (u / 8) * ldb_bytes + kpos(i);
        else if constexpr (LAYOUT == GG_NN) b_voff[i] = krow * ldb_bytes + kcol;
        else b_voff[i] = (unsigned)n0 * ESZ + kcol;  // + the token's row, per slab
    }
    const int b_rows = min(G::BN, p.N - n0);
    const unsigned bn_bytes = (b_rows - 1) * ldb_bytes + kbytes;  // (GG_NT) this tile's rows of B
    // contraction-major operand: from the slab's first row (and the tile's first column) to the operand's end, which
    // refuses the rows past it (host: the operand spans < 2^31 bytes)
    auto kmajor_rsrc = [&](const T* col0, unsigned ld_bytes, unsigned cols, int kt) {
        const bool live = kt < nk;
        const unsigned off = live ? (unsigned)(kt * G::KROWS) * ld_bytes : 0u;
        const unsigned size = live ? (unsigned)(K - 1) * ld_bytes + cols * ESZ - off : 0u;
        return raw_rsrc(reinterpret_cast<const char*>(col0) + off, size);
    };
    const unsigned lds_g = lds_offset_of(smem) + group * 2 * G::STAGE + wg * 1024;
    const unsigned lds_tok = lds_offset_of(smem) + G::TOK + wave * 1024;
    const u32x4 idx_rsrc = raw_rsrc(p.idx, p.idx ? (long long)K * 4 : 0);
    auto issue_tokens = [&](int it) {  // indices of the group's slab `it` into its ring entry
        if constexpr (LAYOUT == GG_TN) lds_direct_b32(idx_rsrc, lds_tok + (it & 3) * 256, (it * GROUPS + group) * (G::KROWS * 4) + lane * 4);
    };
    // one of the 2 * NLD loads of the group's slab `it`: A pieces first, then B pieces
    struct Slab { u32x4 a, b; int soff, left; unsigned a_none, b_none, stage; };
    auto slab_of = [&](int it) {
        const int kt = it * GROUPS + group;
        Slab s;
        const bool live = kt < nk;
        s.soff = live ? kt * SG_KB : 0;
        s.left = kbytes - s.soff;
        s.stage = lds_g + (it & 1) * G::STAGE;
        s.a_none = live ? p.a_bytes : 0u;
        s.b_none = !live ? 0u : LAYOUT == GG_NT ? bn_bytes : p.b_bytes;
        s.a = A_KMAJOR ? kmajor_rsrc(A + m0, lda_bytes, (unsigned)(p.M - m0), kt) : raw_rsrc(A, s.a_none);
        s.b = LAYOUT == GG_NN ? kmajor_rsrc(B + n0, ldb_bytes, (unsigned)(p.N - n0), kt) : raw_rsrc(LAYOUT == GG_NT ? B + (long long)n0 * p.ldb : B, s.b_none);
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // uniform values; the assembly wants them in scalar registers
            s.a[e] = __builtin_amdgcn_readfirstlane(s.a[e]);
            s.b[e] = __builtin_amdgcn_readfirstlane(s.b[e]);
        }
        s.soff = __builtin_amdgcn_readfirstlane(s.soff);
        s.stage = __builtin_amdgcn_readfirstlane(s.stage);
        return s;
    };
    auto load_a = [&](const Slab& s, int i) {
        if constexpr (A_KMAJOR) lds_direct_b128(s.a, s.stage + i * GW * 1024, (int)a_voff[i]);
        else lds_direct_b128(s.a, s.stage + i * GW * 1024, (int)(kpos(i) < s.left ? a_voff[i] : s.a_none), s.soff);
    };
    unsigned tok[LAYOUT == GG_TN ? NLD : 1];
    auto read_tokens = [&](int it) {  // the rows of B of slab `it`: their byte offsets, past the end for tokens past the end
        if constexpr (LAYOUT == GG_TN) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                const int krow = (i * 64 * GW + gtid) / G::PIECES, k = (it * GROUPS + group) * G::KROWS + krow;
                const unsigned row = p.idx ? *reinterpret_cast<const unsigned*>(smem + G::TOK + wave * 1024 + (it & 3) * 256 + krow * 4) : (unsigned)k;
                tok[i] = k < K ? row * ldb_bytes + b_voff[i] : p.b_bytes;
            }
        }
    };
    auto load_b = [&](const Slab& s, int i) {
        if constexpr (LAYOUT == GG_TN) lds_direct_b128(s.b, s.stage + G::OPER + i * GW * 1024, (int)tok[i]);
        else if constexpr (LAYOUT == GG_NN) lds_direct_b128(s.b, s.stage + G::OPER + i * GW * 1024, (int)b_voff[i]);
        else lds_direct_b128(s.b, s.stage + G::OPER + i * GW * 1024, (int)(kpos(i) < s.left ? b_voff[i] : s.b_none), s.soff);
    };
    constexpr int BATCH = 2 * NLD + (LAYOUT == GG_TN ? 1 : 0);  // vector-memory operations per slab
    // after a wait: every wave of the group has come this far, and no access to LDS moves across
    auto group_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (GW == 4) __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // fragment (subtile i of the wave's rows, chunk c of the slab) of an operand.  E = 16: lane q * 16 + r has row r and a quarter of the chunk's
    // 16 elements, 4 q .. + 3 of rows along the contraction, q, 4 + q, ... (other banks) of contraction-major ones
    const int lrow = lane % E, part = lane / E;
    const int trow = 8 * half + ((l32 & 15) >> 2);
    auto frag = [&](const char* region, bool kmajor, int w, int i, int c) {
        if (!kmajor) {
            const int row = (w * WT + i) * E + lrow;
            return *reinterpret_cast<const u32x4*>(region + row * SG_KB + (((G::CHUNK / 16 * c + part) ^ G::swz(row)) << 4));
        }
        if constexpr (ESZ == 4) {  // binary32: an MFMA takes one element per lane, rows 8c + 4 * half + {0..3} of its own column
            const int col = (w * WT + i) * E + lrow, row = E == 16 ? 16 * c + part : 8 * c + 4 * half;
            const char* at = region + row * (G::PIECES * 16) + (((col >> 2) ^ G::kswz(row)) << 4) + (col & 3) * 4;
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const unsigned*>(at + e * (E == 16 ? 4 : 1) * G::PIECES * 16);
            return v;
        }
        const int piece = (w * 8 + i * 4 + (l32 >> 4) * 2 + ((l32 & 3) >> 1)) ^ G::kswz(trow);
        const char* at = region + (trow + c * 16) * (G::PIECES * 16) + piece * 16 + (l32 & 1) * 8;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at + 4 * G::PIECES * 16));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        return u32x4{l2.x, l2.y, h2.x, h2.y};
    };
    char* const stages = smem + group * 2 * G::STAGE;
    // (GW = 4: the tiles of one of two waves with the same rows, or columns, are exchanged, so that tile 0 of both waves is all of them)
    auto a_frag = [&](int st, int i, int c) { return frag(stages + st * G::STAGE, A_KMAJOR, wm, i ^ wn, c); };
    auto b_frag = [&](int st, int i, int c) { return frag(stages + st * G::STAGE + G::OPER, B_KMAJOR, wn, i ^ wm, c); };

    Tile acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = Tile{0};
    auto mma = [&](Tile& d, const u32x4& a, const u32x4& b) {
        if constexpr (E == 16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), d, 0, 0, 0);
        } else {
            mma_chunk<T>(d, a, b);
        }
    };
    float most[2] = {0.f, 0.f};  // (splits) largest magnitude in the lane's row of tile 0 of the wave's rows, of its columns
    auto drain = [&]() {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // requests past the end write (zeros) to the stages, too
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    // The product from the operands' own MFMAs.
    auto product = [&]() {
    u32x4 fa[2][G::CHUNKS][WT], fb[2][G::CHUNKS][WT];  // fragments of two slabs

    const int nit = (nk + GROUPS - 1) / GROUPS;  // slabs per group; the last may lie past the end (zeros)
    issue_tokens(0);
    issue_tokens(1);
    if constexpr (LAYOUT == GG_TN) {  // (the ring is the wave's own)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const Slab s = slab_of(it);
        read_tokens(it);
#pragma unroll
        for (int i = 0; i < NLD; ++i) load_a(s, i);
#pragma unroll
        for (int i = 0; i < NLD; ++i) load_b(s, i);
        issue_tokens(it + 2);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(BATCH));  // slab 0 (and the indices of slab 2)
    group_barrier();
#pragma unroll
    for (int c = 0; c < G::CHUNKS; ++c)
#pragma unroll
        for (int i = 0; i < WT; ++i) {
            fa[0][c][i] = a_frag(0, i, c);
            fb[0][c][i] = b_frag(0, i, c);
        }
    __builtin_amdgcn_s_waitcnt(LGKMCNT0);
    group_barrier();
    {
        const Slab s = slab_of(2);
        read_tokens(2);
#pragma unroll
        for (int i = 0; i < NLD; ++i) load_a(s, i);
#pragma unroll
        for (int i = 0; i < NLD; ++i) load_b(s, i);
        issue_tokens(4);
    }
    // Slab `it` of the group (it & 1 == PAR), its fragments in set PAR; slab it+1 has been asked for into stage PAR^1,
    // slab it+2 into stage PAR.  First half of the MFMAs: read slab it+1's fragments; then, every wave of the group
    // having read them, the second half: ask for slab it+3 into the same stage.
    constexpr int NMMA = G::CHUNKS * WT * WT;
    auto step = [&](int it, auto par_tag) {
        constexpr int PAR = decltype(par_tag)::value, NXT = PAR ^ 1;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(BATCH));
        group_barrier();
        const Slab s = slab_of(it + 3);
#pragma unroll
        for (int q = 0; q < NMMA; ++q) {  // MFMA q of the slab: chunk q / (WT * WT)
            const int c = q / (WT * WT), i = q / WT % WT, j = q % WT;
            __builtin_amdgcn_sched_barrier(0);
            mma(acc[i][j], fa[PAR][c][i], fb[PAR][c][j]);
            if (q < NMMA / 2) {
#pragma unroll
                for (int f = q * G::CHUNKS * WT / (NMMA / 2); f < (q + 1) * G::CHUNKS * WT / (NMMA / 2); ++f) {
                    fa[NXT][f / WT][f % WT] = a_frag(NXT, f % WT, f / WT);
                    fb[NXT][f / WT][f % WT] = b_frag(NXT, f % WT, f / WT);
                }
            }
            if (q == NMMA / 2) {
                read_tokens(it + 3);
                __builtin_amdgcn_s_waitcnt(LGKMCNT0);
                group_barrier();
            }
            if (q >= NMMA / 2) {
#pragma unroll
                for (int k = (q - NMMA / 2) * 2 * NLD / (NMMA / 2); k < (q + 1 - NMMA / 2) * 2 * NLD / (NMMA / 2); ++k) {
                    if (k < NLD) load_a(s, k);
                    else load_b(s, k - NLD);
                }
                if (q == NMMA - 1) issue_tokens(it + 5);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int it = 0;
    for (; it + 1 < nit; it += 2) {
        step(it, I0{});
        step(it + 1, I1{});
    }
    if (it < nit) step(it, I0{});
    drain();
    };

    // (SPLIT) The product from three-part splits.  A slab is two operand chunks of 16 elements; during the 24 MFMAs of one
    // chunk the next one's four operand tiles are split, pair by pair, and the one after that is read.  So slab it has left LDS when
    // its MFMAs begin: its stage is asked for again at once, with one barrier per slab, and has a slab's time to fill.
    auto split_product = [&](auto& acc) {
        u32x4 raw[4][2];   // A's tiles, B's tiles
        Split8 part[2][4];
        auto read_raw = [&](int st, int c16, int o) {
#pragma unroll
            for (int e = 0; e < 2; ++e) raw[o][e] = o < 2 ? a_frag(st, o, 2 * c16 + e) : b_frag(st, o - 2, 2 * c16 + e);
        };
        auto half_slab = [&](auto set_tag, int st, int c16, auto mem) {
            constexpr int SET = decltype(set_tag)::value;
#pragma unroll
            for (int q = 0; q < 4 * SPLIT_TERMS; ++q) {
                const int i = q % 4 / 2, j = i ? 1 - q % 2 : q % 2;
                __builtin_amdgcn_sched_barrier(0);
                mma_split(acc[i][j], part[SET][i], part[SET][2 + j], q / 4);
#pragma unroll
                for (int pr = q * 16 / (4 * SPLIT_TERMS); pr < (q + 1) * 16 / (4 * SPLIT_TERMS); ++pr) {
                    split_pair(part[SET ^ 1][pr / 4], pr % 4, raw[pr / 4][pr % 4 / 2]);
                    if (pr / 4 % 2 == 0) most_of_pair(most[pr / 8], pr % 4, raw[pr / 4][pr % 4 / 2]);
                    if (pr % 4 == 3) read_raw(st, c16, pr / 4);
                }
                mem(q);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        issue_tokens(0);
        issue_tokens(1);
        if constexpr (LAYOUT == GG_TN) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const Slab s = slab_of(it);
            read_tokens(it);
#pragma unroll
            for (int i = 0; i < NLD; ++i) load_a(s, i);
#pragma unroll
            for (int i = 0; i < NLD; ++i) load_b(s, i);
            issue_tokens(it + 2);
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(BATCH));
        group_barrier();
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            read_raw(0, 0, o);
            part[0][o] = split_f32(raw[o][0], raw[o][1]);
            if (o % 2 == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) most_of_pair(most[o / 2], e, raw[o][e / 2]);
            }
            read_raw(0, 1, o);
        }
        auto step = [&](int it, auto par_tag) {
            constexpr int PAR = decltype(par_tag)::value, NXT = PAR ^ 1;
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_waitcnt(LGKMCNT0);
            group_barrier();
            const Slab s = slab_of(it + 2);
            read_tokens(it + 2);
            half_slab(I0{}, NXT, 0, [&](int q) {
                if (q % 3 == 1) {
                    if (q / 3 < NLD) load_a(s, q / 3);
                    else load_b(s, q / 3 - NLD);
                }
            });
            issue_tokens(it + 4);
            half_slab(I1{}, NXT, 1, [&](int) {});
        };
        int it = 0;
        for (; it + 1 < nk; it += 2) {
            step(it, I0{});
            step(it + 1, I1{});
        }
        if (it < nk) step(it, I0{});
        drain();
    };
    // Sums that the splits do not give, formed again from the operands' own MFMAs: those that are not finite, and small ones of a row
    // and a column of which one has values too small to be split (they lose up to 2^-134 each, so a sum above `slight` times the
    // largest operand does not feel it).  Sum by sum, so that no row depends on its neighbours.
    const float slight = 0x1p-103f * (float)K;
    auto form_again = [&](auto& acc) {
        // f(stage) for every slab, the next one on its way
        auto each_slab = [&](auto f) {
            issue_tokens(0);
            issue_tokens(1);
            auto load = [&](int kt) {
                const Slab s = slab_of(kt);
                read_tokens(kt);
#pragma unroll
                for (int i = 0; i < NLD; ++i) load_a(s, i);
#pragma unroll
                for (int i = 0; i < NLD; ++i) load_b(s, i);
                issue_tokens(kt + 2);
            };
            auto landed = [&]() {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                __builtin_amdgcn_s_waitcnt(LGKMCNT0);
                group_barrier();
            };
            if constexpr (LAYOUT == GG_TN) landed();
            load(0);
#pragma unroll 1
            for (int kt = 0; kt < nk; ++kt) {
                landed();  // and everyone has read the slab before, into whose stage the next one comes
                load(kt + 1);
                f(kt & 1);
            }
            drain();
        };
        unsigned* const of_rows = reinterpret_cast<unsigned*>(smem);  // [half-wave][128], of what a lane knows about tile 0
        unsigned* const of_cols = of_rows + 256;
        auto exchange = [&](unsigned row, unsigned col) {
            of_rows[half * 128 + (wm * WT + wn) * 32 + l32] = row;
            of_cols[half * 128 + (wn * WT + wm) * 32 + l32] = col;
            __syncthreads();
        };
        unsigned again[WT][WT];  // bit r: acc[i][j][r]
        // drops the sums that are not in f(what the lanes know about the sum's row, its column; the sum); false if none is left
        auto keep = [&](auto f) {
            bool any = false;
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j) {
                    const int col = (wn * WT + (j ^ wm)) * 32 + l32;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = (wm * WT + (i ^ wn)) * 32 + acc_row(r, lane);
                        if (!f(of_rows[row], of_rows[128 + row], of_cols[col], of_cols[128 + col], fabsf(acc[i][j][r])) || m0 + row >= p.M || n0 + col >= p.N)
                            again[i][j] &= ~(1u << r);
                    }
                    any |= again[i][j] != 0;
                }
            return __syncthreads_or(any) != 0;
        };
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) again[i][j] = 0xffffu;
        exchange(__float_as_uint(most[0]), __float_as_uint(most[1]));
        if (!keep([&](unsigned r0, unsigned r1, unsigned c0, unsigned c1, float v) {
                const float r = fmaxf(__uint_as_float(r0), __uint_as_float(r1)), c = fmaxf(__uint_as_float(c0), __uint_as_float(c1));
                return !(v < INFINITY) | ((v < slight * fmaxf(r, c)) & (r > 0.f) & (c > 0.f));
            }))
            return;
        unsigned least[2] = {0xffffffffu, 0xffffffffu};  // smallest magnitude but zero, bits * 2 - 1
        each_slab([&](int st) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const u32x4 v = o ? b_frag(st, 0, c) : a_frag(st, 0, c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) least[o] = min(least[o], (v[e] << 1) - 1);
                }
        });
        exchange(least[0], least[1]);
        if (!keep([&](unsigned r0, unsigned r1, unsigned c0, unsigned c1, float v) { return !(v < INFINITY) | (min(min(r0, r1), min(c0, c1)) < SPLIT_WHOLE * 2 - 1); }))
            return;
        f32x16 sum[WT][WT];
        bool tile[WT][WT];  // of the wave
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                sum[i][j] = f32x16{0};
                tile[i][j] = __ballot(again[i][j] != 0) != 0;
            }
        each_slab([&](int st) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < WT; ++i)
#pragma unroll
                    for (int j = 0; j < WT; ++j)
                        if (tile[i][j]) mma_chunk<T>(sum[i][j], a_frag(st, i, c), b_frag(st, j, c));
        });
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = again[i][j] >> r & 1 ? sum[i][j][r] : acc[i][j][r];
    };
    if constexpr (SPLIT) {
        static_assert(ESZ == 4 && GW == 4 && WT == 2 && 2 * NLD == 8, "four operand tiles, a load per three MFMAs");
        split_product(acc);
        // (an infinity does not survive the split: the sum is then not a number)
        float probe = 0.f, low = INFINITY;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    probe = fmaf(acc[i][j][r], 0.f, probe);
                    low = fminf(low, fabsf(acc[i][j][r]));
                }
        if (__syncthreads_or(!(probe == 0.f) | (low < slight * 0x1p20f) | (fmaxf(most[0], most[1]) >= 0x1p20f))) form_again(acc);
    } else {
        product();
    }

    // Epilogue.  Every wave lays its block out in LDS as binary32; rows are then put together (GW = 1: the four
    // partial blocks are added in wave order, each wave finishing a quarter of the rows; GW = 4: each wave its own block), eight
    // consecutive columns of a row per lane, and stored in whole 16-byte pieces.
    constexpr int PARTS = GROUPS, ROWS = G::WB / PARTS;                       // rows a wave finishes
    constexpr int LPR = G::WB / 8, RPP = 64 / LPR, PASSES = (ROWS + RPP - 1) / RPP;  // lanes per row, rows per pass
    const int piece = lane % LPR, rsub = lane / LPR;
    const int row0 = group * ROWS;
    const int ncol = n0 + wn * G::WB + piece * 8;
    const char* first = smem + wg * G::WB * G::EP;  // + part * GW blocks
    constexpr int NV = 8 * ESZ / 16;  // 16-byte pieces of a lane's 8 columns
    const bool vec = p.ldy % (16 / ESZ) == 0 && (reinterpret_cast<uintptr_t>(p.Y) & 15u) == 0 && ncol + 8 <= p.N;
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bv[e] = 0.f;
        if (p.bias && ncol + e < p.N) {
            if constexpr (ESZ == 2) bv[e] = bf16_to_f32(static_cast<const uint16_t*>(p.bias)[ncol + e]);
            else bv[e] = static_cast<const float*>(p.bias)[ncol + e];
        }
    }
    // output rows (ADD: picked by oidx, dropped outside [0, out_rows)), and what they hold already
    long long orow[PASSES];
    u32x4 old[PASSES][NV];
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        const long long m = m0 + wm * G::WB + row0 + q * RPP + rsub;
        orow[q] = ADD && p.oidx ? (long long)p.oidx[min(m, p.M - 1)] : m;
        if (m >= p.M || ncol >= p.N || q * RPP + rsub >= ROWS || (ADD && (orow[q] < 0 || orow[q] >= p.out_rows))) orow[q] = -1;
    }
    if constexpr (ADD) {
        const __amdgpu_buffer_rsrc_t y_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.Y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
        for (int q = 0; q < PASSES; ++q)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const unsigned off = vec && orow[q] >= 0 ? (unsigned)orow[q] * (unsigned)p.ldy * ESZ + (unsigned)ncol * ESZ + v * 16 : p.y_bytes;
                old[q][v] = __builtin_amdgcn_raw_buffer_load_b128(y_rsrc, (int)off, 0, 0);
            }
    }
    char* mine = smem + wave * G::WB * G::EP;
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
#pragma unroll
            for (int r = 0; r < G::REGS; ++r)
                *reinterpret_cast<float*>(mine + ((i ^ wn) * E + (E == 16 ? 4 * part + r : acc_row(r, lane))) * G::EP + ((j ^ wm) * E + lrow) * 4) = acc[i][j][r];
    if constexpr (PARTS > 1) __syncthreads();  // (one group: a wave reads back its own block only)
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        if (orow[q] < 0) continue;
        float v[8];
        const char* at = first + (row0 + q * RPP + rsub) * G::EP + piece * 32;
#pragma unroll
        for (int part = 0; part < PARTS; ++part) {
            const f32x4 lo = *reinterpret_cast<const f32x4*>(at + part * GW * G::WB * G::EP);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(at + part * GW * G::WB * G::EP + 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = part ? v[e] + lo[e] : lo[e];
                v[e + 4] = part ? v[e + 4] + hi[e] : hi[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[e];
        T* dst = static_cast<T*>(p.Y) + orow[q] * p.ldy + ncol;
        if (vec) {
            if constexpr (ESZ == 2) {
                u32x4 out;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float o0 = ADD ? bf16lo_to_f32(old[q][0][e]) : 0.f, o1 = ADD ? bf16hi_to_f32(old[q][0][e]) : 0.f;
                    out[e] = ADD ? pack_bf16x2_hw(v[2 * e] + o0, v[2 * e + 1] + o1) : pack_bf16x2_hw(v[2 * e], v[2 * e + 1]);
                }
                *reinterpret_cast<u32x4*>(dst) = out;
            } else {
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    f32x4 out;
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[e] = ADD ? __uint_as_float(old[q][w % NV][e]) + v[w * 4 + e] : v[w * 4 + e];
                    *reinterpret_cast<f32x4*>(dst + w * 4) = out;
                }
            }
        } else {  // ragged right edge or unaligned rows: element by element
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (ncol + e >= p.N) continue;
                if constexpr (ESZ == 2) {
                    uint16_t* d = reinterpret_cast<uint16_t*>(dst) + e;
                    *d = (uint16_t)(pack_bf16x2_hw(ADD ? v[e] + bf16_to_f32(*d) : v[e], 0.f) & 0xffffu);
                } else {
                    float* d = reinterpret_cast<float*>(dst) + e;
                    *d = ADD ? *d + v[e] : v[e];
                }
            }
        }
    }
}

template <typename T, bool ADD, int LAYOUT>
static int prepare_small() {
    constexpr int ESZ = (int)sizeof(T);
    if constexpr (ESZ == 2) {
        static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&gather_gemm_small_kernel<T, ADD, LAYOUT, 1, 2, false>), SgGeo<1, ESZ, 2>::LDS}});
        return err;
    } else {
        static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&gather_gemm_small_kernel<T, ADD, LAYOUT, 1, 1, false>), SgGeo<1, ESZ, 1>::LDS},
                                                 {reinterpret_cast<const void*>(&gather_gemm_small_kernel<T, ADD, LAYOUT, 4, 2, true>), SgGeo<4, ESZ, 2>::LDS}});
        if constexpr (LAYOUT == GG_TN) {
            static const int few = raise_lds_limits({{reinterpret_cast<const void*>(&gather_gemm_small_kernel<T, ADD, LAYOUT, 4, 2, false>), SgGeo<4, ESZ, 2>::LDS}});
            if (few) return few;
        }
        return err;
    }
}

template <typename T, bool ADD, int LAYOUT, int GW, int WT, bool SPLIT = false, int E = 32>
static int launch_small(GgParams p, hipStream_t st) {
    using G = SgGeo<GW, (int)sizeof(T), WT, E>;
    p.tiles_m = (int)((p.M + G::BM - 1) / G::BM);
    p.tiles_n = (p.N + G::BN - 1) / G::BN;
    const int per_xcd = (p.tiles_m * p.tiles_n + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((gather_gemm_small_kernel<T, ADD, LAYOUT, GW, WT, SPLIT, E>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(SG_THREADS), G::LDS, st, p);
    return (int)hipGetLastError();
}

template <typename T, int GW, int WT, bool SPLIT = false, int E = 32>
static int launch_small_form(const GgParams& p, bool add, int layout, hipStream_t st) {
    if (layout == GG_TN) return launch_small<T, false, GG_TN, GW, WT, SPLIT, E>(p, st);
    if constexpr (sizeof(T) == 2)
        if (layout == GG_NN) return launch_small<T, true, GG_NN, GW, WT>(p, st);
    return add ? launch_small<T, true, GG_NT, GW, WT, SPLIT, E>(p, st) : launch_small<T, false, GG_NT, GW, WT, SPLIT, E>(p, st);
}

template <typename T>
static int prepare_small_form(bool add, int layout) {
    if (layout == GG_TN) return prepare_small<T, false, GG_TN>();
    if constexpr (sizeof(T) == 2)
        if (layout == GG_NN) return prepare_small<T, true, GG_NN>();
    return add ? prepare_small<T, true, GG_NT>() : prepare_small<T, false, GG_NT>();
}

int prepare_gather_gemm_small(lemo_dtype_t dt, bool add, int layout) {
    return dt == LEMO_BF16 ? prepare_small_form<bf16_t>(add, layout) : prepare_small_form<float>(add, layout);
}

int launch_gather_gemm_small(const GgParams& p, lemo_dtype_t dt, bool add, int layout, GgTile tile, hipStream_t st) {
    if (dt == LEMO_BF16) return launch_small_form<bf16_t, 1, 2>(p, add, layout, st);
    // binary32 MFMAs bound these, so a CU's time is that of its tiles' areas: four 16 x 16 tiles for one of 32 x 32 spread them better over 256
    // CUs until a CU would have more than two (of 32 x 32 two run side by side).  us, 32 x 32 / 16 x 16 tiles, contraction 64 / 1024:  256 x 256
    // (256 tiles) 4.2 / 3.3, 8.1 / 4.8, its weight gradient 4.5 / 3.7, 9.3 / 5.7;  256 x 512 (512) 4.2 / 3.8, 8.3 / 6.3, 4.5 / 4.2, 9.5 / 8.0;  272 x 512 (544)
    // 4.2 / 4.4, 8.3 / 7.7, 4.5 / 5.1, 9.5 / 10.4;  256 x 768 (768) 4.2 / 4.5, 8.4 / 8.1, 4.5 / 5.2, 9.5 / 11.1.  Errors against 64 bits alike (2.07e-7,
    // 4.93e-7, 1.5e-7, ...).
    const long long n16 = (p.M + 15) / 16 * ((p.N + 15ll) / 16);
    if (tile != GG_T128 && n16 <= 512) return launch_small_form<float, 1, 1, false, 16>(p, add, layout, st);
    if (tile != GG_T128) return launch_small_form<float, 1, 1>(p, add, layout, st);
    // sums of one or two products (only a weight gradient has them, the other forms contract over 4 at least) from binary32 MFMAs:
    // error 2.5e-8 and 3.1e-8 against 3.5e-8 and 3.4e-8 of splits, 8192 x 8192 83 us against 69
    if (layout == GG_TN && p.K < SPLIT_LEAST) return launch_small<float, false, GG_TN, 4, 2>(p, st);
    return launch_small_form<float, 4, 2, true>(p, add, layout, st);
}

}  // namespace lemo
