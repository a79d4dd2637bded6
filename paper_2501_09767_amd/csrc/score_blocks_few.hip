// The head sums and tile maxima of score_blocks.hip for few rectangles (bf16): short sequences, and the last round of longer ones.
//
// A workgroup owns a 64 x 64 quarter of a rectangle, or a 32 x 32 piece, and its waves (four, eight) share out the heads: a wave forms the
// whole quarter for its heads from operands of its own (32 KB of LDS at D = 128, filled by LDS-direct loads while the head before
// is worked on from registers; no barrier in the loop), and the partial sums meet in LDS at the end.  A quarter then takes a
// quarter of the steps, where tilemax_kernel walks all heads one after the other: that one needs half the bytes per
// flop and keeps two waves on a SIMD (32 heads, D = 128: 256 rectangles in 39 us, 64 as quarters in 19), but with few rectangles its
// time is one walk of all heads whatever their number.
// What bounds it: the latency of a step (quarters: one wave per SIMD, 4 us for the launch, then 2 us per step of loads, 32 reads of LDS,
// 32 MFMAs and 64 exponentials per lane, overlapped only in parts).  Pieces halve the steps and the bytes a CU takes in, and two
// waves share a SIMD; but they load twice the bytes per flop, so they pay while all of them run at once.
#include <type_traits>

#include "score_blocks.hpp"

namespace lemo {

template <int D, int N32> struct FGeo {  // N32: subtiles of 32 rows along an edge
    static constexpr int EDGE = 32 * N32, TILES = N32 * N32, WAVES = N32 == 2 ? 4 : 8, THREADS = 64 * WAVES;
    static constexpr int SIDE = 128 / EDGE, PIECES = SIDE * SIDE;  // of a rectangle
    static constexpr int ROWB = D * 2, NCH = ROWB / 32, CPR = ROWB / 16;
    static constexpr int OPER = EDGE * ROWB;          // one operand's rows
    static constexpr int NLD = OPER / 1024, RPI = 1024 / ROWB;  // loads per operand and head, rows of one
    static constexpr int PERIOD = D == 128 ? 4 : 2;   // of the loads' exchange of pieces
    static constexpr int BUF = 2 * OPER + 256;        // a wave's: Q rows, K rows, row statistics
    static constexpr int SUMS = WAVES * TILES * 16 * 64 * 4;  // partial sums: [wave][tile][register][lane]
    static constexpr int LDS = WAVES * BUF > SUMS + 4 * WAVES ? WAVES * BUF : SUMS + 4 * WAVES;
    __device__ static constexpr int swz(int row) { return CPR >= 16 ? (row & 15) : ((row >> 1) & (CPR - 1)); }
};

// MODE as in tilemax_kernel.  The pieces of the rectangles first .. first + rest - 1.
template <int D, int MODE, int N32>
__global__ __launch_bounds__((FGeo<D, N32>::THREADS), 1) void tilemax_few_kernel(BlockParams p, int first, int rest) {
    using G = FGeo<D, N32>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    const int per_xcd = (G::PIECES * rest + NUM_XCD - 1) / NUM_XCD;  // a die takes neighbouring pieces
    const int id = blockIdx.x % NUM_XCD * per_xcd + blockIdx.x / NUM_XCD;
    if (blockIdx.x / NUM_XCD >= per_xcd || id >= G::PIECES * rest) return;
    int tq, tk;
    sb_rectangle(first + id / G::PIECES, p.nt, causal, tq, tk);
    tq = G::SIDE * tq + id / G::SIDE % G::SIDE;
    tk = G::SIDE * tk + id % G::SIDE;
    if (tq * G::EDGE >= p.S || tk * G::EDGE >= p.S || (causal && tk > tq)) return;
    const int S = p.S, q0 = tq * G::EDGE, k0 = tk * G::EDGE;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float c2 = p.c2;
    const bf16_t* Qb = static_cast<const bf16_t*>(p.Q);
    const bf16_t* Kb = static_cast<const bf16_t*>(p.K);
    const unsigned group = (unsigned)(p.H / p.H_kv);

    // load i of an operand fills 1 KB of consecutive LDS bytes: rows i * RPI + lane / CPR, position lane % CPR, which holds piece
    // (lane % CPR) ^ swz(row); range-checked, rows past the end arrive as zeros
    const int q_row_bytes = (int)p.q_ts * 2, k_row_bytes = (int)p.k_ts * 2;  // host: < 2^24
    int q_off[G::PERIOD], k_off[G::PERIOD];
#pragma unroll
    for (int i = 0; i < G::PERIOD; ++i) {
        const int row = lane / G::CPR, piece = (lane % G::CPR) ^ G::swz(i * G::RPI + row);
        q_off[i] = row * q_row_bytes + piece * 16;
        k_off[i] = row * k_row_bytes + piece * 16;
    }
    char* const buf = smem + wave * G::BUF;
    const unsigned lds = __builtin_amdgcn_readfirstlane(lds_offset_of(buf));
    const int l_off = min(q0 + lane, S - 1) * 4;  // rows past the end reuse the last row's statistics (left out at the end)
    auto issue = [&](int h) {
        const char* qh = reinterpret_cast<const char*>(Qb + (long long)h * p.q_hs) + (long long)q0 * q_row_bytes;
        const char* kh = reinterpret_cast<const char*>(Kb + (long long)((unsigned)h / group) * p.k_hs) + (long long)k0 * k_row_bytes;
        const u32x4 qd = raw_rsrc(qh, (long long)(S - q0 - 1) * q_row_bytes + G::ROWB), kd = raw_rsrc(kh, (long long)(S - k0 - 1) * k_row_bytes + G::ROWB);
#pragma unroll
        for (int i = 0; i < G::NLD; ++i) lds_direct_b128(qd, lds + i * 1024, q_off[i % G::PERIOD] + i * G::RPI * q_row_bytes);
#pragma unroll
        for (int i = 0; i < G::NLD; ++i) lds_direct_b128(kd, lds + G::OPER + i * 1024, k_off[i % G::PERIOD] + i * G::RPI * k_row_bytes);
        if (MODE == 0) lds_direct_b32(raw_rsrc(p.lse2 + (size_t)h * S, (long long)S * 4), lds + 2 * G::OPER, l_off);
    };

    f32x16 sum[N32][N32];  // [query subtile][key subtile], of this wave's heads
#pragma unroll
    for (int t = 0; t < G::TILES; ++t) sum[t / N32][t % N32] = f32x16{0};
    if (wave < p.H) issue(wave);
    for (int h = wave; h < p.H; h += G::WAVES) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
        u32x4 qf[N32][G::NCH], kf[N32][G::NCH];
        float nl[N32][16];  // row statistics of the lane's rows 8 gq + 4 half + {0..3}, negated
#pragma unroll
        for (int s = 0; s < N32; ++s) {
            const char* row = buf + (s * 32 + l32) * G::ROWB;
#pragma unroll
            for (int c = 0; c < G::NCH; ++c) {
                qf[s][c] = *reinterpret_cast<const u32x4*>(row + (((2 * c + half) ^ G::swz(l32)) << 4));
                kf[s][c] = *reinterpret_cast<const u32x4*>(row + G::OPER + (((2 * c + half) ^ G::swz(l32)) << 4));
            }
            if (MODE == 0) {
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(buf + 2 * G::OPER + (s * 32 + gq * 8 + half * 4) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) nl[s][gq * 4 + e] = -v[e];
                }
            }
        }
        // the buffer is the wave's own: once its reads have returned, the next head may land in it
        __builtin_amdgcn_s_waitcnt(LGKMCNT0);
        asm volatile("" ::: "memory");
        if (h + G::WAVES < p.H) issue(h + G::WAVES);
        f32x16 prev = {0};
        auto add = [&](int t, int r) {  // element r of tile t
            f32x16& s = sum[t / N32][t % N32];
            if (MODE == 0) s[r] += __builtin_amdgcn_exp2f(fmaf(prev[r], c2, nl[t / N32][r]));
            else s[r] += fmaxf(prev[r], 0.f);
        };
#pragma unroll
        for (int t = 0; t < G::TILES; ++t) {  // the tile before is added between this one's MFMAs
            f32x16 acc = {0};
#pragma unroll
            for (int c = 0; c < G::NCH; ++c) {
                __builtin_amdgcn_sched_barrier(0);
                mma_chunk<bf16_t>(acc, qf[t / N32][c], kf[t % N32][c]);  // acc[query row][key col]
                if (t > 0) {
#pragma unroll
                    for (int r = c * 16 / G::NCH; r < (c + 1) * 16 / G::NCH; ++r) add(t - 1, r);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            prev = acc;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) add(G::TILES - 1, r);
    }

    // a wave puts its share of the tiles' registers together: the partial sums in wave order, then the maximum over the pairs that are
    // admitted (quarters: wave w takes tile w)
    constexpr int SHARE = 16 * G::TILES / G::WAVES;
    float* const sums = reinterpret_cast<float*>(smem);
    __syncthreads();  // every wave is done with its buffer
#pragma unroll
    for (int t = 0; t < G::TILES; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) sums[((wave * G::TILES + t) * 16 + r) * 64 + lane] = sum[t / N32][t % N32][r];
    __syncthreads();
    const bool excl = (p.flags & LEMO_EXCLUDE_SELF) != 0;
    const int tile = wave * SHARE / 16, r0 = wave * SHARE % 16;
    const int i0 = q0 + tile / N32 * 32, j0 = k0 + tile % N32 * 32, j = j0 + l32;
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < SHARE; ++e) {
        const int r = r0 + e;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < G::WAVES; ++w) v += sums[((w * G::TILES + tile) * 16 + r) * 64 + lane];
        const int i = i0 + acc_row(r, lane);
        const bool ok = (i < S) & (j < S) & (!causal | (j <= i)) & (!excl | (i != j));
        m = fmaxf(m, ok ? v : 0.f);
    }
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) m = fmaxf(m, __shfl_xor(m, sh));
    if constexpr (SHARE < 16) {
        float* const parts = sums + G::SUMS / 4;
        if (lane == 0) parts[wave] = m;
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int w = 1; w < G::WAVES; ++w) m = fmaxf(m, parts[w]);
    }
    const int ti = i0 / 32, tj = j0 / 32;
    if (lane == 0 && ti < p.nt32 && tj < p.nt32) p.tilemax[(size_t)ti * p.nt32 + tj] = m * p.out_scale;
}

template <int D>
static int prepare_few() {
    static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&tilemax_few_kernel<D, 0, 1>), FGeo<D, 1>::LDS},
                                             {reinterpret_cast<const void*>(&tilemax_few_kernel<D, 1, 1>), FGeo<D, 1>::LDS},
                                             {reinterpret_cast<const void*>(&tilemax_few_kernel<D, 0, 2>), FGeo<D, 2>::LDS},
                                             {reinterpret_cast<const void*>(&tilemax_few_kernel<D, 1, 2>), FGeo<D, 2>::LDS}});
    return err;
}
int prepare_tilemax_few(int d) { return d == 128 ? prepare_few<128>() : prepare_few<64>(); }

template <int D, int MODE, int N32>
static int launch_few(const BlockParams& p, int first, int rest, hipStream_t st) {
    using G = FGeo<D, N32>;
    const int per_xcd = (G::PIECES * rest + NUM_XCD - 1) / NUM_XCD;
    hipLaunchKernelGGL((tilemax_few_kernel<D, MODE, N32>), dim3((unsigned)(per_xcd * NUM_XCD)), dim3(G::THREADS), G::LDS, st, p, first, rest);
    return (int)hipGetLastError();
}
template <int D, int N32>
static int launch_few_mode(const BlockParams& p, int mode, int first, int rest, hipStream_t st) {
    return mode ? launch_few<D, 1, N32>(p, first, rest, st) : launch_few<D, 0, N32>(p, first, rest, st);
}

int launch_tilemax_few(const BlockParams& p, int d, int mode, int first, int rest, hipStream_t st) {
    // Pieces where each has a CU of its own (D = 64: 66 KB of LDS, half a CU).  us per call with the row statistics given, quarters / pieces,
    // 32 heads, D = 128: 3 rectangles 20.4 / 11.1, 10 21.4 / 12.4, 16 (no mask) 21.6 / 13.1, 36 23.2 / 28.0, 512 and 16 100.7 / 93.8, 512 and
    // 49 103.4 / 114.4; D = 64, 16 heads 10 11.5 / 7.9, 21 (12 heads) 10.9 / 9.2, 36 12.6 / 13.6, 512 and 16 44.1 / 41.4.
    const bool small = rest <= (d == 128 ? 16 : 32);
    if (d == 128) return small ? launch_few_mode<128, 1>(p, mode, first, rest, st) : launch_few_mode<128, 2>(p, mode, first, rest, st);
    return small ? launch_few_mode<64, 1>(p, mode, first, rest, st) : launch_few_mode<64, 2>(p, mode, first, rest, st);
}

}  // namespace lemo
