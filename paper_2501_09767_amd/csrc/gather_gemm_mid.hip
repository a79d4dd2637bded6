// The selective-load GEMM (and its in-place-add and gradient forms, see gather_gemm.hip) on 256 x 128 and 128 x 128 output
// tiles, bf16, for products that leave most CUs without a 256 x 256 tile or its last round nearly empty.
//
// One workgroup of eight waves per CU, in a 4 x 2 grid: a wave computes 32 x 64 of every 128 x 128 region.  Slabs of 128 bytes of
// the contraction pass through a ring of 3 (256 x 128) or 4 stages, filled by LDS-direct loads; the fragments of the next slab are
// read during the MFMAs of the current one, so the registers are one stage more, and a slab needs one barrier: the next slab has
// landed, and everyone has the current one in registers, so its stage can be asked for again.
//
// What bounds it: LDS (a slab of 256 x 128 takes 896 cycles of it for 1024 of MFMAs, of 128 x 128 640 for 512) and what the barrier
// costs; with weights that come from HBM, the latency of the loads (M = 256, N = 11008, K = 4096: 30 us with W in the caches, 41
// without, whether the loads are spread or not, and 50 with a ninth wave that touches the slabs ahead).
// Measured, operands from HBM, us (two workgroups of four waves per CU on 128 x 128 tiles, 64 x 64 per wave, were before):
//   256 x 128  M = 1504: N = K = 4096 55 / 63, N = 4096, K = 11008 149 / 165 (input gradient 149 / 165, weight gradient 159 / 189);
//              M = 3280, N = K = 4096: 101 / 119
//   128 x 128  M = 256, N = 11008, K = 4096: 41.5 / 44.4;  M = N = 256 x 4096: 38 / 41;  M = 768, N = 3072, K = 768: 9.4 / 10.7
#include "gather_gemm_regions.hpp"

namespace lemo {

template <int RA> struct MdGeo {                           // RA: regions of A's rows
    static constexpr int BM = 128 * RA, BN = 128;
    static constexpr int NS = RA == 1 ? 4 : 3;             // stages
    static constexpr int STAGE = (RA + 1) * RG_BYTES;      // A's regions, then B's
    static constexpr int TOK = NS * STAGE;                 // (GG_TN) token rings
    static constexpr int EP = BN * 4 + 16;                 // epilogue: LDS pitch of a row of floats
    static constexpr int LDS_LOOP = TOK + RG_TOK, LDS_EPI = BM * EP;
    static constexpr int LDS = LDS_LOOP > LDS_EPI ? LDS_LOOP : LDS_EPI;
    static_assert(LDS <= 160 * 1024, "a workgroup's LDS");
};

template <bool ADD, int LAYOUT, int RA>
__global__ __launch_bounds__(RG_THREADS, 1) void gather_gemm_mid_kernel(GgParams p) {
    using G = MdGeo<RA>;
    constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    constexpr int TA = 2, TB = 4, NL = RG_NLD, NS = G::NS;  // 16-row tiles of a wave per region of A, of B
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int tm, tn;
    if (!gg_tile(blockIdx.x, p.tiles_m, p.tiles_n, 8 / RA, tm, tn)) return;
    const long long m0 = (long long)tm * G::BM;
    const int n0 = tn * G::BN;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    using Loads = RgLoads<LAYOUT, RA, 1>;
    Loads ld(p, m0, n0, tid, smem + G::TOK + wave * 1024);
    const int nk = ld.nk;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset_of(smem) + wave * 1024);
    constexpr int LOADS = NL * (RA + 1), BATCH = LOADS + (LAYOUT == GG_TN ? 1 : 0);
    constexpr int AHEAD = NS - 1;  // (GG_TN) the indices of a slab are asked for this many slabs ahead of its rows
    auto load = [&](const typename Loads::Slab& s, unsigned stage, int k) {  // load k of a slab
        if (k < NL * RA) ld.load_a(s, k / NL, k % NL, stage + (k / NL) * RG_BYTES);
        else ld.load_b(s, 0, k - NL * RA, stage + RA * RG_BYTES);
    };

    f32x4 acc[RA][TA][TB];
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) acc[a][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 fa[2][RA][2][TA], fb[2][2][TB];  // fragments of two slabs
    constexpr int NF = 2 * (RA * TA + TB);
    auto read = [&](auto set_tag, const char* stage, int f) {  // fragment f of a slab: B's, then A's
        constexpr int SET = decltype(set_tag)::value;
        if (f < 2 * TB) { fb[SET][f / TB][f % TB] = rg_fragment(stage + RA * RG_BYTES, B_KMAJOR, wn * TB + f % TB, f / TB, lane); return; }
        f -= 2 * TB;
        const int a = f / (2 * TA), c = f / TA % 2, i = f % TA;
        fa[SET][a][c][i] = rg_fragment(stage + a * RG_BYTES, A_KMAJOR, wm * TA + i, c, lane);
    };

    if constexpr (LAYOUT == GG_TN) {
        for (int kt = 0; kt < 4; ++kt) ld.issue_tokens(kt, lane);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
    }
    // (the batches as the loop issues them: a slab's rows, then the indices of the slab AHEAD, into the entry of a slab that is done)
#pragma unroll
    for (int kt = 0; kt < NS; ++kt) {
        const typename Loads::Slab s = ld.slab(kt);
        ld.read_tokens(kt);
#pragma unroll
        for (int k = 0; k < LOADS; ++k) load(s, lds0 + kt * G::STAGE, k);
        if constexpr (LAYOUT == GG_TN) {
            __builtin_amdgcn_s_waitcnt(LGKMCNT0);
            asm volatile("" ::: "memory");
            ld.issue_tokens(kt + AHEAD, lane);
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 1) * BATCH));
    rg_barrier();
#pragma unroll
    for (int f = 0; f < NF; ++f) read(std::integral_constant<int, 0>{}, smem, f);

    constexpr int NM = 2 * RA * TA * TB;
    int st = 0;  // stage of slab kt
    // Slab kt (kt & 1 == PAR), its fragments in set PAR.  Behind the barrier slab kt + 1 has landed (all batches but the last
    // NS - 2) and stage st is free; the source order is the issue order, neighbouring MFMAs share a fragment.
    auto step = [&](int kt, auto par_tag) {
        constexpr int PAR = decltype(par_tag)::value;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * BATCH));
        __builtin_amdgcn_s_waitcnt(LGKMCNT0);
        rg_barrier();
        const typename Loads::Slab s = ld.slab(kt + NS);
        const int nxt = st + 1 == NS ? 0 : st + 1;
        const char* next = smem + nxt * G::STAGE;
        const unsigned free_stage = lds0 + st * G::STAGE;
        if constexpr (LAYOUT == GG_TN) ld.read_tokens(kt + NS);
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const int a = q / (2 * TA * TB), c = q / (TA * TB) % 2, w = q % (TA * TB), i = w / TB, j = i & 1 ? TB - 1 - w % TB : w % TB;
            __builtin_amdgcn_sched_barrier(0);
            rg_mma(acc[a][i][j], fa[PAR][a][c][i], fb[PAR][c][j]);
#pragma unroll
            for (int f = q * NF / (NM * 3 / 4); f < (q + 1) * NF / (NM * 3 / 4); ++f)
                if (f < NF) read(std::integral_constant<int, PAR ^ 1>{}, next, f);
#pragma unroll
            for (int k = q * LOADS / (NM / 2); k < (q + 1) * LOADS / (NM / 2); ++k)
                if (k < LOADS) load(s, free_stage, k);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (LAYOUT == GG_TN) ld.issue_tokens(kt + NS + AHEAD, lane);
        st = nxt;
    };
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        step(kt, std::integral_constant<int, 0>{});
        step(kt + 1, std::integral_constant<int, 1>{});
    }
    if (kt < nk) step(kt, std::integral_constant<int, 0>{});
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // requests past the end write (zeros) to the stages, too
    __builtin_amdgcn_s_waitcnt(LGKMCNT0);
    __syncthreads();

    // Epilogue, through LDS as binary32: whole rows of 16-byte pieces, 8 consecutive columns per lane, one rounding.  In-place add:
    // what the rows hold is asked for ahead (rows that are not to be written get an offset past the descriptor's end).
    const bool vec_ok = p.ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(p.Y) & 15u) == 0;
    constexpr int ROWS = G::BM / RG_WAVES, PASSES = ROWS / 4;  // rows a wave finishes, 4 at a time
    const int piece = lane & 15, rsub = lane >> 4;
    const int ncol = n0 + piece * 8;
    const bool col_vec = vec_ok && ncol + 8 <= p.N;
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = p.bias && ncol + e < p.N ? bf16_to_f32(static_cast<const uint16_t*>(p.bias)[ncol + e]) : 0.f;
    long long orow[PASSES];
    u32x4 old[PASSES];
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        const long long m = m0 + wave * ROWS + q * 4 + rsub;
        orow[q] = ADD && p.oidx ? (long long)p.oidx[min(m, p.M - 1)] : m;
        if (m >= p.M || ncol >= p.N || (ADD && (orow[q] < 0 || orow[q] >= p.out_rows))) orow[q] = -1;
    }
    if constexpr (ADD) {
        const __amdgpu_buffer_rsrc_t y_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.Y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
        for (int q = 0; q < PASSES; ++q) {
            const unsigned off = col_vec && orow[q] >= 0 ? (unsigned)orow[q] * (unsigned)p.ldy * 2u + (unsigned)ncol * 2u : p.y_bytes;
            old[q] = __builtin_amdgcn_raw_buffer_load_b128(y_rsrc, (int)off, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
                *reinterpret_cast<f32x4*>(smem + (a * 128 + (wm * TA + i) * 16 + l16) * G::EP + ((wn * TB + j) * 16 + 4 * quad) * 4) = acc[a][i][j];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        if (orow[q] < 0) continue;
        const char* at = smem + (wave * ROWS + q * 4 + rsub) * G::EP + piece * 32;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(at), hi = *reinterpret_cast<const f32x4*>(at + 16);
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = lo[e] + bv[e]; v[e + 4] = hi[e] + bv[e + 4]; }
        uint16_t* dst = static_cast<uint16_t*>(p.Y) + orow[q] * p.ldy + ncol;
        if (col_vec) {
            u32x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                out[e] = ADD ? pack_bf16x2_hw(v[2 * e] + bf16lo_to_f32(old[q][e]), v[2 * e + 1] + bf16hi_to_f32(old[q][e])) : pack_bf16x2_hw(v[2 * e], v[2 * e + 1]);
            *reinterpret_cast<u32x4*>(dst) = out;
        } else {  // ragged right edge or unaligned rows: element by element
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (ncol + e < p.N) dst[e] = (uint16_t)(pack_bf16x2_hw(ADD ? v[e] + bf16_to_f32(dst[e]) : v[e], 0.f) & 0xffffu);
        }
    }
}

template <bool ADD, int LAYOUT>
static int prepare_mid() {
    static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&gather_gemm_mid_kernel<ADD, LAYOUT, 1>), MdGeo<1>::LDS},
                                             {reinterpret_cast<const void*>(&gather_gemm_mid_kernel<ADD, LAYOUT, 2>), MdGeo<2>::LDS}});
    return err;
}

template <bool ADD, int LAYOUT, int RA>
static int launch_mid(GgParams p, hipStream_t st) {
    using G = MdGeo<RA>;
    p.tiles_m = (int)((p.M + G::BM - 1) / G::BM);
    p.tiles_n = (p.N + G::BN - 1) / G::BN;
    const int per_xcd = (p.tiles_m * p.tiles_n + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((gather_gemm_mid_kernel<ADD, LAYOUT, RA>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(RG_THREADS), G::LDS, st, p);
    return (int)hipGetLastError();
}
template <int RA>
static int launch_mid_form(const GgParams& p, bool add, int layout, hipStream_t st) {
    if (layout == GG_TN) return launch_mid<false, GG_TN, RA>(p, st);
    if (layout == GG_NN) return launch_mid<true, GG_NN, RA>(p, st);
    return add ? launch_mid<true, GG_NT, RA>(p, st) : launch_mid<false, GG_NT, RA>(p, st);
}

int prepare_gather_gemm_mid(bool add, int layout) {
    if (layout == GG_TN) return prepare_mid<false, GG_TN>();
    if (layout == GG_NN) return prepare_mid<true, GG_NN>();
    return add ? prepare_mid<true, GG_NT>() : prepare_mid<false, GG_NT>();
}

int launch_gather_gemm_mid(const GgParams& p, bool add, int layout, GgTile tile, hipStream_t st) {
    return tile == GG_T128 ? launch_mid_form<1>(p, add, layout, st) : launch_mid_form<2>(p, add, layout, st);
}

}  // namespace lemo
