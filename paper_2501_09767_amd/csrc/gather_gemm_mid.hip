// The selective-load GEMM (and its in-place-add and gradient forms, see gather_gemm.hip) on output tiles of 256, 192, 128 or 64
// rows x 128 columns, bf16, for products that leave most CUs without a 256 x 256 tile or its last round nearly empty.
//
// One workgroup of eight waves per CU, in a 4 x 2 grid: a wave computes a quarter of the rows x 64 columns.  Slabs of 128 bytes of
// the contraction pass through a ring of 4 stages (256 x 128: 3), filled by LDS-direct loads; the fragments of the next slab are
// read during the MFMAs of the current one, so the registers are one stage more, and a slab needs one barrier: the next slab has
// landed, and everyone has the current one in registers, so its stage can be asked for again.
//
// What bounds it: LDS (a slab of 256 x 128 takes 896 cycles of it for 1024 of MFMAs, of 128 x 128 640 for 512) and what the barrier
// costs; with weights that come from HBM, what a CU gets: 55 to 60 GB/s of rows of both operands, however many stages
// are in flight (3 or 4 alike; loads spread or not; tiles starting at different slabs alike; a ninth wave that touches the slabs ahead 50 us
// against 41, M = 256, N = 11008, K = 4096), so that fewer rows per tile on more CUs win there.
// Measured, operands from HBM, us (the kind before it in brackets):
//   256 x 128  M = 1504: N = 4096, K = 11008 149;  weight gradient 159;  M = 3280, N = K = 4096: 101
//   192 x 128  M = 1500: N = K = 4096 50 (256 x 128: 56), input gradient of 11008 x 4096 134 (153);  M = 522, N = 8192, K = 2048 25.7 (27.6)
//   128 x 128  M = 256, N = 11008, K = 4096: 42;  M = 768, N = 3072, K = 768: 9.4
//   64 x 128   M = 128, N = 11008, K = 4096: 32 (128 x 128: 42);  M = 500, N = K = 4096 30 (37);  M = 408, N = 3072, K = 768 8.0 (9.7)
// (128 x 64 does as well as 64 x 128.  128 x 96 gained 7 % in X W^T where 64 x 128 loses, M = 256, N = 11008; it is not built: B's rows are loaded 64 at a time.)
#include "gather_gemm_regions.hpp"

namespace lemo {

template <int LAYOUT, int UA> struct MdGeo {               // UA: the tile's rows / 64
    static constexpr int BM = 64 * UA, BN = 128;
    static constexpr int A_BYTES = BM * RG_KB, STAGE = A_BYTES + RG_BYTES;  // A's rows, then B's region
    static constexpr int TOKENS = LAYOUT == GG_TN ? RG_TOK : 0;
    static constexpr int NS = UA == 4 ? 3 : 4;             // stages
    static constexpr int TOK = NS * STAGE;                 // (GG_TN) token rings
    static constexpr int EP = BN * 4 + 16;                 // epilogue: LDS pitch of a row of floats
    static constexpr int LDS_LOOP = TOK + TOKENS, LDS_EPI = BM * EP;
    static constexpr int LDS = LDS_LOOP > LDS_EPI ? LDS_LOOP : LDS_EPI;
    static_assert(LDS <= 160 * 1024, "a workgroup's LDS");
};

template <bool ADD, int LAYOUT, int UA>
__global__ __launch_bounds__(RG_THREADS, 1) void gather_gemm_mid_kernel(GgParams p) {
    using G = MdGeo<LAYOUT, UA>;
    constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    constexpr int TA = UA, TB = 4, NS = G::NS;  // 16-row tiles of a wave of A, of B
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int tm, tn;
    if (!gg_tile(blockIdx.x, p.tiles_m, p.tiles_n, UA <= 2 ? 16 / UA : 4, tm, tn)) return;
    const long long m0 = (long long)tm * G::BM;
    const int n0 = tn * G::BN;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // 16-row tile i of the wave, among the tile's: contraction-major rows come in regions of 128, of which a wave takes 32
    auto a_tile = [&](int i) { return A_KMAJOR ? i / 2 * 8 + wm * 2 + i % 2 : wm * TA + i; };
    using Loads = RgLoads<LAYOUT, UA, 2>;
    Loads ld(p, m0, n0, tid, smem + G::TOK + wave * 1024);
    const int nk = ld.nk;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_offset_of(smem) + wave * 1024);
    constexpr int LOADS = UA + 2, BATCH = LOADS + (LAYOUT == GG_TN ? 1 : 0);
    constexpr int AHEAD = NS - 1;  // (GG_TN) the indices of a slab are asked for this many slabs ahead of its rows
    auto load = [&](const typename Loads::Slab& s, unsigned stage, int k) {  // load k of a slab
        if (k < UA) ld.load_a(s, k, stage);
        else ld.load_b(s, k - UA, stage + G::A_BYTES);
    };

    f32x4 acc[TA][TB];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 fa[2][2][TA], fb[2][2][TB];  // fragments of two slabs
    constexpr int NF = 2 * (TA + TB);
    auto read = [&](auto set_tag, const char* stage, int f) {  // fragment f of a slab: B's, then A's
        constexpr int SET = decltype(set_tag)::value;
        if (f < 2 * TB) { fb[SET][f / TB][f % TB] = rg_fragment(stage + G::A_BYTES, B_KMAJOR, wn * TB + f % TB, f / TB, lane); return; }
        f -= 2 * TB;
        const int c = f / TA, t = a_tile(f % TA);
        fa[SET][c][f % TA] = A_KMAJOR ? rg_fragment(stage + t / 8 * RG_BYTES, true, t % 8, c, lane) : rg_fragment(stage, false, t, c, lane);
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

    constexpr int NM = 2 * TA * TB;
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
            const int c = q / (TA * TB), w = q % (TA * TB), i = w / TB, j = i & 1 ? TB - 1 - w % TB : w % TB;
            __builtin_amdgcn_sched_barrier(0);
            rg_mma(acc[i][j], fa[PAR][c][i], fb[PAR][c][j]);
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
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
            *reinterpret_cast<f32x4*>(smem + (a_tile(i) * 16 + l16) * G::EP + ((wn * TB + j) * 16 + 4 * quad) * 4) = acc[i][j];
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

template <bool ADD, int LAYOUT, int UA> constexpr LdsLimit mid_limit() {
    return {reinterpret_cast<const void*>(&gather_gemm_mid_kernel<ADD, LAYOUT, UA>), MdGeo<LAYOUT, UA>::LDS};
}
template <bool ADD, int LAYOUT>
static int prepare_mid() {
    static const int err = [] {
        if constexpr (LAYOUT == GG_TN) return raise_lds_limits({mid_limit<ADD, LAYOUT, 2>(), mid_limit<ADD, LAYOUT, 4>()});
        else return raise_lds_limits({mid_limit<ADD, LAYOUT, 1>(), mid_limit<ADD, LAYOUT, 2>(), mid_limit<ADD, LAYOUT, 3>(), mid_limit<ADD, LAYOUT, 4>()});
    }();
    return err;
}

template <bool ADD, int LAYOUT, int UA>
static int launch_mid(GgParams p, hipStream_t st) {
    using G = MdGeo<LAYOUT, UA>;
    p.tiles_m = (int)((p.M + G::BM - 1) / G::BM);
    p.tiles_n = (p.N + G::BN - 1) / G::BN;
    const int per_xcd = (p.tiles_m * p.tiles_n + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((gather_gemm_mid_kernel<ADD, LAYOUT, UA>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(RG_THREADS), G::LDS, st, p);
    return (int)hipGetLastError();
}
template <int UA>
static int launch_mid_form(const GgParams& p, bool add, int layout, hipStream_t st) {
    if (layout == GG_TN) {
        if constexpr (UA % 2 == 0) return launch_mid<false, GG_TN, UA>(p, st);
        else return (int)hipErrorInvalidValue;  // (its plans know whole regions of rows only)
    }
    if (layout == GG_NN) return launch_mid<true, GG_NN, UA>(p, st);
    return add ? launch_mid<true, GG_NT, UA>(p, st) : launch_mid<false, GG_NT, UA>(p, st);
}

int prepare_gather_gemm_mid(bool add, int layout) {
    if (layout == GG_TN) return prepare_mid<false, GG_TN>();
    if (layout == GG_NN) return prepare_mid<true, GG_NN>();
    return add ? prepare_mid<true, GG_NT>() : prepare_mid<false, GG_NT>();
}

int launch_gather_gemm_mid(const GgParams& p, bool add, int layout, GgTile tile, hipStream_t st) {
    switch (tile) {
        case GG_T256x128: return launch_mid_form<4>(p, add, layout, st);
        case GG_T192x128: return launch_mid_form<3>(p, add, layout, st);
        case GG_T128: return launch_mid_form<2>(p, add, layout, st);
        default: return launch_mid_form<1>(p, add, layout, st);
    }
}

}  // namespace lemo
