// The head sums and tile maxima of score_blocks.hip (bf16) where there are more than 256 rectangles.
//
// The same 128 x 128 rectangles on four waves of 64 x 64, two workgroups per CU: 8 fragment reads from LDS per 32 x 32 pairs
// where waves of 32 x 64 take 12, and the two waves of a SIMD wait at different barriers.  A stage of whole head rows would be 64 KB
// and need 64 fragment registers more than there are; so the operands come in slabs of 128 bytes of the row (half a head at D = 128, a
// head at D = 64; 32 KB) through two stages, and a slab's fragments are refilled in place, each behind the last MFMA that takes
// it, with the next slab's.  At D = 128 the logit tiles of a wave stand half done between its two slabs: the first slab's MFMAs
// go chunk by chunk over all of them, the second one finishes them two at a time, and a pair's exponentials are issued two pairs
// later (those of the last two pairs, which have registers of their own by then, among the next head's first MFMAs).  The product
// is K Q^T, so that a lane owns a query column and needs a row statistic per subtile of 16 queries.  One barrier per slab: behind
// it the next slab has landed and this one is in everyone's registers, so the slab after the next is asked for.
//
// What bounds it: the power that the matrix cores and the exponentials draw (16384 tokens, 32 heads: 1292 us at 1.80 GHz; with 32 x 32
// MFMAs a tenth less cycles, but at 1.63 GHz; 256 x 128 rectangles, which take a quarter less from L2, 1341 at 1.85).
// Both kernels, us per call with the row statistics given: 32 heads, D = 128, causal 4096 tokens 117 / 106, 8192 426 / 331, 32768
// 6040 / 4990; 16 heads, D = 64 4096 52 / 47, 16000 565 / 424; 6001, full 98 / 82.
#include "score_blocks.hpp"

namespace lemo {

template <int D> struct SGeo {
    static constexpr int SLABS = D / 64;                              // per head
    static constexpr int Q_BYTES = 128 * 128, STAGE = 2 * Q_BYTES, NS = 2;
    static constexpr int LSE_BASE = NS * STAGE, LSE_BYTES = 128 * 4;  // ring of four heads' row statistics
    static constexpr int LDS = LSE_BASE + 4 * LSE_BYTES;
    static constexpr int THREADS = 256, NLOAD = STAGE / (16 * THREADS), NLOAD_Q = NLOAD / 2;
};

// MODE as in tilemax_kernel
template <int D, int MODE>
__global__ __launch_bounds__(256, 2) void tilemax_slab_kernel(BlockParams p) {
    using G = SGeo<D>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    const int id = blockIdx.x % NUM_XCD * p.per_xcd + blockIdx.x / NUM_XCD;
    if (blockIdx.x / NUM_XCD >= p.per_xcd || id >= p.count) return;
    int tq, tk;
    sb_rectangle(id, p.nt, causal, tq, tk);
    const int S = p.S, q0 = tq * 128, k0 = tk * 128;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave >> 1, wk = wave & 1;  // the wave's 64 queries, 64 keys
    const float c2 = p.c2;
    const bf16_t* Qb = static_cast<const bf16_t*>(p.Q);
    const bf16_t* Kb = static_cast<const bf16_t*>(p.K);
    const unsigned group = (unsigned)(p.H / p.H_kv);

    // Unit u = i * 256 + tid of a slab is its LDS bytes [16 u, 16 u + 16): row u / 8 (queries, then keys), position u % 8, which
    // holds piece (u % 8) ^ (row / 2 % 8), so that one piece of 16 rows meets all banks.  The descriptor ends with the
    // last row, so that rows past the end fail the range check (raw_rsrc) and arrive as zeros; the scalar offset moves along a row.
    const unsigned q_row_bytes = (unsigned)p.q_ts * 2u, k_row_bytes = (unsigned)p.k_ts * 2u;  // host: < 2^24
    unsigned voff[G::NLOAD];
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
        const unsigned row = (unsigned)((i < G::NLOAD_Q ? i : i - G::NLOAD_Q) * 32 + (tid >> 3));
        voff[i] = row * (i < G::NLOAD_Q ? q_row_bytes : k_row_bytes) + (unsigned)((tid & 7) ^ ((tid >> 4) & 7)) * 16u;
    }
    const unsigned l_voff = (unsigned)min(q0 + (tid & 127), S - 1) * 4u;  // rows past the end reuse the last row's (left out at the end)
    const unsigned lds0 = lds_offset_of(smem) + (unsigned)wave * 1024u, lds_l = lds_offset_of(smem) + G::LSE_BASE + (unsigned)(wave & 1) * 256u;
    u32x4 aim_q, aim_k, aim_l;  // descriptors of the head whose slabs are asked for; past the last one of length zero: all is refused
    auto aim = [&](int hh) {
        const bool live = hh < p.H;
        const int h = min(hh, p.H - 1), g = (int)((unsigned)h / group);
        aim_q = raw_rsrc(reinterpret_cast<const char*>(Qb + (long long)h * p.q_hs) + (long long)q0 * q_row_bytes, live ? (long long)(S - q0 - 1) * q_row_bytes + 2 * D : 0);
        aim_k = raw_rsrc(reinterpret_cast<const char*>(Kb + (long long)g * p.k_hs) + (long long)k0 * k_row_bytes, live ? (long long)(S - k0 - 1) * k_row_bytes + 2 * D : 0);
        if (MODE == 0) aim_l = raw_rsrc(p.lse2 + (size_t)h * S, live ? (long long)S * 4 : 0);
    };
    // load n of slab s of head hh into ring stage `stage`; the row statistics are the last load of a head's first slab
    auto issue_one = [&](int n, int hh, int s, unsigned stage) {
        if (n < G::NLOAD) lds_direct_b128(n < G::NLOAD_Q ? aim_q : aim_k, lds0 + stage + n * (G::THREADS * 16), (int)voff[n], s * 128);
        else if (MODE == 0 && s == 0 && n == G::NLOAD) lds_direct_b32(aim_l, lds_l + (unsigned)(hh & 3) * G::LSE_BYTES, (int)l_voff);
    };

    // A wave's 4 x 4 tiles of 16 x 16 (query subtile i, key subtile j): a lane holds query column l16, keys 4 quad .. + 3
    f32x4 sum[4][4];  // head sums
#pragma unroll
    for (int t = 0; t < 16; ++t) sum[t >> 2][t & 3] = f32x4{0.f, 0.f, 0.f, 0.f};
    float nl[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};  // minus the row statistics of the lane's queries, of the head that is being added
    u32x4 qf[4][2], kf[4][2];  // fragments: [subtile][chunk of 32 of the slab]
    const int q_at = (wq * 64 + l16) * 128, k_at = G::Q_BYTES + (wk * 64 + l16) * 128;
    const int f_at[2] = {(quad ^ (l16 >> 1)) << 4, ((4 + quad) ^ (l16 >> 1)) << 4};
    auto read_q = [&](const char* stage, int s, int c) { qf[s][c] = *reinterpret_cast<const u32x4*>(stage + q_at + f_at[c] + s * 2048); };
    auto read_k = [&](const char* stage, int s, int c) { kf[s][c] = *reinterpret_cast<const u32x4*>(stage + k_at + f_at[c] + s * 2048); };
    auto read_nl = [&](int h) {
        if (MODE != 0) return;
        const float* at = reinterpret_cast<const float*>(smem + G::LSE_BASE + (h & 3) * G::LSE_BYTES) + wq * 64 + l16;
#pragma unroll
        for (int i = 0; i < 4; ++i) nl[i] = -at[i * 16];
    };
    // element r of a logit tile into its head sum
    auto add = [&](int i, int j, const f32x4& raw, int r) {
        if (MODE == 0) sum[i][j][r] += __builtin_amdgcn_exp2f(fmaf(raw[r], c2, nl[i]));
        else sum[i][j][r] += fmaxf(raw[r], 0.f);
    };
    auto mma = [&](f32x4& d, const f32x4& from, int i, int j, int c) {
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[j][c]), __builtin_bit_cast(bf16x8, qf[i][c]), from, 0, 0, 0);
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

    // slabs 0 and 1 (of head 0, or of heads 0 and 1)
    aim(0);
#pragma unroll
    for (int n = 0; n <= G::NLOAD; ++n) issue_one(n, 0, 0, 0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) { read_q(smem, s, c); read_k(smem, s, c); }
    if (G::SLABS == 1) aim(1);
#pragma unroll
    for (int n = 0; n <= G::NLOAD; ++n) issue_one(n, G::SLABS == 1 ? 1 : 0, G::SLABS == 1 ? 0 : 1, G::STAGE);
    aim(G::SLABS == 1 ? 2 : 1);

    f32x4 acc[4][4], carry[4];  // carry: tiles (3, 2), (3, 3), (3, 0), (3, 1) of the head before
#pragma unroll
    for (int t = 0; t < 4; ++t) carry[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    unsigned st = 0;  // LDS offset of the ring stage whose slab is in the registers
    // before the MFMAs of a slab: the next one has landed, this wave's reads have returned
    auto enter = [&] {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __builtin_amdgcn_s_waitcnt(LGKMCNT0);
        __syncthreads();
    };
    for (int h = 0; h < p.H; ++h) {
        if constexpr (G::SLABS == 2) {
            // first slab: chunk by chunk over all tiles; every second MFMA an exponential of the head before's last four
            enter();
            const char* next = smem + (st ^ G::STAGE);
#pragma unroll
            for (int m = 0; m < 32; ++m) {
                const int c = m / 16, i = m / 4 % 4, j = i & 1 ? 3 - m % 4 : m % 4;  // neighbours share a fragment
                fence();
                mma(acc[i][j], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j], i, j, c);
                issue_one(m, h + 1, 0, st);
                if (m % 4 == 3) read_q(next, i, c);
                if (i == 3) read_k(next, j, c);
                if (m % 2 == 0) add(3, (m / 8) ^ 2, carry[m / 8], m / 2 % 4);
                if (m == 31) read_nl(h);
            }
            fence();
            st ^= G::STAGE;
        }
        // last (or only) slab: two tiles at a time, the exponentials of the two before the last between their MFMAs
        enter();
        const char* next = smem + (st ^ G::STAGE);
#pragma unroll
        for (int m = 0; m < 32; ++m) {
            const int P = m / 4, i = P / 2, jp = (P ^ i) & 1, c = m / 2 % 2, j = 2 * jp + m % 2;
            fence();
            f32x4& d = i == 3 ? carry[(j ^ 2)] : acc[i][j];
            if (c == 0) mma(d, G::SLABS == 2 ? acc[i][j] : f32x4{0.f, 0.f, 0.f, 0.f}, i, j, c);
            else mma(d, d, i, j, c);
            issue_one(m, G::SLABS == 2 ? h + 1 : h + 2, G::SLABS - 1, st);
            if (m == G::NLOAD + 1) aim(G::SLABS == 2 ? h + 2 : h + 3);
            if (P % 2 == 1 && m % 4 == 1) read_q(next, i, 0);
            if (P % 2 == 1 && m % 4 == 3) read_q(next, i, 1);
            if (i == 3 && m % 4 == 2) { read_k(next, 2 * jp, 0); read_k(next, 2 * jp + 1, 0); }
            if (i == 3 && m % 4 == 3) { read_k(next, 2 * jp, 1); read_k(next, 2 * jp + 1, 1); }
            const int e = m % 4 * 2;  // two of the eight elements of a pair
            if (P >= 2) {
                const int pi = (P - 2) / 2, pj = 2 * (((P - 2) ^ pi) & 1) + e / 4;
                add(pi, pj, acc[pi][pj], e % 4);
                add(pi, pj, acc[pi][pj], e % 4 + 1);
            } else if (G::SLABS == 1) {
                const int pj = 2 * (1 - P) + e / 4;
                add(3, pj, carry[pj ^ 2], e % 4);
                add(3, pj, carry[pj ^ 2], e % 4 + 1);
                if (m == 7) read_nl(h);
            }
        }
        fence();
        st ^= G::STAGE;
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) add(3, (m / 4) ^ 2, carry[m / 4], m % 4);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // (requests past the last head, of length zero, still write zeros to LDS)

    // maximum of every 32 x 32 tile over the pairs that are admitted
    const bool excl = (p.flags & LEMO_EXCLUDE_SELF) != 0;
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int i0 = q0 + wq * 64 + qs * 32, j0 = k0 + wk * 64 + ks * 32;
            float m = 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = i0 + (t >> 1) * 16 + l16, j = j0 + (t & 1) * 16 + 4 * quad + r;
                    const bool ok = (i < S) & (j < S) & (!causal | (j <= i)) & (!excl | (i != j));
                    m = fmaxf(m, ok ? sum[2 * qs + (t >> 1)][2 * ks + (t & 1)][r] : 0.f);
                }
#pragma unroll
            for (int sh = 32; sh >= 1; sh >>= 1) m = fmaxf(m, __shfl_xor(m, sh));
            const int ti = i0 / 32, tj = j0 / 32;
            if (lane == 0 && ti < p.nt32 && tj < p.nt32) p.tilemax[(size_t)ti * p.nt32 + tj] = m * p.out_scale;
        }
}

template <int D>
static int prepare_slabs() {
    static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&tilemax_slab_kernel<D, 0>), SGeo<D>::LDS},
                                             {reinterpret_cast<const void*>(&tilemax_slab_kernel<D, 1>), SGeo<D>::LDS}});
    return err;
}
int prepare_tilemax_slabs(int d) { return d == 128 ? prepare_slabs<128>() : prepare_slabs<64>(); }

template <int D, int MODE>
static int launch_slabs(const BlockParams& p, hipStream_t st) {
    using G = SGeo<D>;
    hipLaunchKernelGGL((tilemax_slab_kernel<D, MODE>), dim3((unsigned)(p.per_xcd * NUM_XCD)), dim3(G::THREADS), G::LDS, st, p);
    return (int)hipGetLastError();
}
int launch_tilemax_slabs(const BlockParams& p, int d, int mode, hipStream_t st) {
    if (d == 128) return mode ? launch_slabs<128, 1>(p, st) : launch_slabs<128, 0>(p, st);
    return mode ? launch_slabs<64, 1>(p, st) : launch_slabs<64, 0>(p, st);
}

}  // namespace lemo
