// The scoring sweeps of score.hip in binary32.
//
// The logits come from three-part splits on the bf16 matrix cores (split_f32, mma_split in lemo_common.hpp): 6 MFMAs of 32 x 32 x 16
// where binary32 MFMAs take 16 times the cycles for 16 elements.  The resident operand is split once; a wave splits its streamed
// subtile once per stage, between the MFMAs that use it.  The waves of a workgroup share resident rows (KS = 4, d = 128: 2; of eight waves twice as many), so
// that no two of them split the same rows and a stage is one subtile per wave; the statistics are those of score.hip's shared rows.
//
// What bounds it: issue.  A 32 x 32 tile of 64 elements (d = 64) is 768 cycles of MFMAs, 176 instructions of splitting over the NRT
// tiles that use them, and the fma, exp2 and add of each logit; one subtile per barrier leaves the rest uncovered (about 1700
// cycles a tile on a full chip).  Measured, both sweeps and the head mean, us, before (binary32 MFMAs) / now, causal:
//   d = 64    1024 tokens, 4 heads 32.8 / 28.1;  3000, 4: 91.7 / 65.2;  1024, 12: 39.1 / 29.6;  5000, 16: 478 / 307
//   d = 128   1000 tokens, 32 heads 117 / 76;  2500, 32: 475 / 329;  1500, 16, no mask: 220 / 151
// and as far from 64 bits within what draws of this number tell apart (scores, relative 2-norm, binary32 MFMAs / now, mean of 24 to
// 200 draws and of the paired differences with their standard error):
//   d = 64    1024 tokens, 4 heads 4.99e-8 / 4.63e-8 (-3.5 +- 1.3 e-9);  3000, 4 5.03e-8 / 4.86e-8 (-1.7 +- 1.0);  300, 12 6.22e-8 / 5.86e-8
//             (-3.6 +- 1.8);  5000, 16 6.33e-8 / 6.30e-8 (-0.2 +- 1.8);  1024, 12, no mask 6.44e-8 / 6.21e-8 (-2.3 +- 1.6)
//   d = 128   1000 tokens, 16 heads 6.57e-8 / 6.56e-8 (-0.1 +- 1.9);  2500, 32 8.85e-8 / 8.54e-8 (-3.1 +- 1.9);  5000, 32 8.63e-8 / 8.78e-8
//             (+1.5 +- 3.0);  700, 16, no mask 6.27e-8 / 6.13e-8 (-1.4 +- 1.8)
// Tried (5000 tokens, 16 heads, d = 64): two waves per row with two subtiles each 580 us, whole rows 397, one resident subtile
// per wave 341.
//
// A sum that is not finite -- an infinity does not survive the split -- is formed again from binary32 MFMAs before anything is stored;
// blocks whose logits would feel what small values lose to the split (needs_whole) take those at once.
#include "score_sweeps.hpp"

namespace lemo {

// smallest magnitude but zero (as bits * 2 - 1) and largest (NaN is passed over)
struct Extent {
    unsigned least = 0xffffffffu;
    float most = 0.f;
    __device__ __forceinline__ void take(const u32x4& v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) least = min(least, (v[e] << 1) - 1);
        most_of_pair(most, 0, v);
        most_of_pair(most, 1, v);
    }
    __device__ __forceinline__ bool small() const { return least < SPLIT_WHOLE * 2 - 1; }
};
// One 32-row subtile as MFMA operand: resident (split once, from the block's rows in a stage) and streamed.  Lane half h of operand
// chunk c holds the 16 bytes h of the row's 32-byte chunks 2c and 2c + 1.
template <typename G> struct Resident32 {
    Split8 f[G::NCH / 2];
    __device__ __forceinline__ void read(const char* sbuf, int sub, int l32, int half, Extent& extent) {
        u32x4 raw[G::NCH];
        read_frags<G>(raw, sbuf, sub, l32, half);
#pragma unroll
        for (int c = 0; c < G::NCH; ++c) extent.take(raw[c]);
#pragma unroll
        for (int c = 0; c < G::NCH / 2; ++c) f[c] = split_f32(raw[2 * c], raw[2 * c + 1]);
    }
};
// Does the block need whole operands from the start?  A value below 2^-110 loses up to 2^-134 to the split, and a logit feels
// that if the other operand is beyond `limit` (logits of base 2: c2 * D * 2^-134 * limit = 2^-32).  The resident rows are at hand; only
// if they have such values are the streamed rows [first, last) looked through.  `flags`: a word of LDS per wave.  Both sweeps and the
// head mean, us without / with it: 1024 tokens, 4 heads of 64 28.7 / 28.9; 1000, 32 heads of 128 75.6 / 76.6; 2500, 32 331 / 333.
template <typename G, int D>
__device__ __forceinline__ bool needs_whole(const Extent& resident, float c2, const float* base, long long tok_stride, long long head_off, int first,
                                            int last, int tid, int wave, int* flags) {
    const float limit = 0x1p102f / (c2 * (float)D);
    bool look = __any(resident.small() | (resident.most > limit));
    if constexpr (G::KS < G::WAVES) {  // (otherwise all waves hold the same rows; __syncthreads_or took 0.4 us of each sweep)
        if (tid % WAVE == 0) flags[wave] = look;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < G::WAVES; ++w) look |= flags[w] != 0;
    }
    if (!look) return false;
    Extent streamed;
#pragma unroll 1
    for (int row = first + tid / G::CPR; row < last; row += G::ROWS_PER_LOAD) streamed.take(load_piece(base, tok_stride, head_off, row, last, tid % G::CPR * 16));
    const bool small = __syncthreads_or(resident.small()), large = __syncthreads_or(resident.most > limit);
    const bool other_small = __syncthreads_or(streamed.small()), other_large = __syncthreads_or(streamed.most > limit);
    return (small & other_large) | (large & other_small);
}
template <typename G> struct Streamed32 {
    static constexpr int NM = G::NCH / 2 * SPLIT_TERMS;  // MFMAs per tile
    const char* row;   // (the pieces of a row are exchanged)
    int half, swz;
    u32x4 raw[2][2];   // of the operand chunk that is split next, and of the one behind it
    Split8 f[G::NCH / 2];
    __device__ __forceinline__ u32x4 piece(int c) const { return *reinterpret_cast<const u32x4*>(row + (((2 * c + half) ^ swz) << 4)); }
    __device__ __forceinline__ void read(const char* sbuf, int sub, int l32, int h) {
        row = sbuf + (sub * 32 + l32) * G::ROWB;
        half = h;
        swz = G::swz(l32);
        raw[0][0] = piece(0);
        raw[0][1] = piece(1);
    }
    // MFMA q of a tile (streamed rows x resident columns); the subtile's first tile splits the operand on its way.  The products of the
    // leading parts come last: what the others round is then a rounding of sums
    // 2^-8 as large (chunk by chunk: 4.9e-8 from 64 bits instead of 4.5e-8 at 1024 tokens, 4 heads, same time).
    __device__ __forceinline__ void mma(int q, f32x16& acc, const Resident32<G>& r, bool first) {
        constexpr int LOW = SPLIT_TERMS - 1, LEAD = G::NCH / 2 * LOW;
        if (q >= LEAD) return mma_split(acc, f[q - LEAD], r.f[q - LEAD], LOW);
        const int c = q / LOW;
        if (first && q % LOW == 0) {
            f[c] = split_f32(raw[c & 1][0], raw[c & 1][1]);
            if (c + 1 < G::NCH / 2) { raw[(c + 1) & 1][0] = piece(2 * c + 2); raw[(c + 1) & 1][1] = piece(2 * c + 3); }
        }
        mma_split(acc, f[c], r.f[c], q % LOW);
    }
    // the same tile from binary32 MFMAs, the resident operand read again
    __device__ __forceinline__ void mma_whole(f32x16& acc, const float* base, long long tok_stride, long long head_off, int at, int nrows) const {
#pragma unroll 1
        for (int c = 0; c < G::NCH; ++c) mma_chunk<float>(acc, piece(c), load_piece(base, tok_stride, head_off, at, nrows, c * 32 + half * 16));
    }
};

// Sweep 1 (see rowstats_kernel): lse2 of every query row.
template <int D, int NRT, int KS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (Geo<float, D, NRT, KS, WAVES>::MIN_WG)) void rowstats_f32_kernel(ScoreParams p) {
    using G = Geo<float, D, NRT, KS, WAVES>;
    static_assert(KS > 1 && G::SHARE == 1, "one subtile per wave and stage");
    constexpr int NM = Streamed32<G>::NM;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    int h, qb;
    decode_block(p.order, p.H, p.n_query_blocks, h, qb);
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    if (causal) qb = p.n_query_blocks - 1 - qb;  // late query blocks see the most keys: start them first
    const int g = (int)(((long long)h * p.H_kv) / p.H);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* Qb = static_cast<const float*>(p.Q);
    const float* Kb = static_cast<const float*>(p.K);
    const long long q_off = (long long)h * p.q_hs, k_off = (long long)g * p.k_hs;
    const int S = p.S;
    const float c2 = p.c2;
    const int q0 = qb * G::BLOCK;             // first query of the workgroup
    const int part = wave % KS;               // this wave's subtile of a stage
    const int qw0 = q0 + wave / KS * G::RES;  // first query of this wave

    // key stages [0, nstage): under a causal mask only keys up to the block's last query matter
    const int q_last = min(q0 + G::BLOCK, S) - 1;
    const int nstage = (causal ? q_last : S - 1) / G::TILE + 1;
    const char* k_head = reinterpret_cast<const char*>(Kb + k_off);  // wave-uniform
    const int k_row_bytes = (int)p.k_ts * 4;                        // host guarantees < 2^24
    int st_voff[G::NLOAD];
    stage_offsets<G>(st_voff, k_row_bytes, tid);
    const unsigned lds_w = lds_offset_of(smem) + (unsigned)wave * 1024u;

    // the queries pass through the second stage, while the first stage of keys arrives
    Resident32<G> qf[NRT];
    Extent extent;
    load_resident<G>(reinterpret_cast<const char*>(Qb + q_off), (int)p.q_ts * 4, q0, S, lds_w + G::STAGE_BYTES, tid);
    stage_load<G>(st_voff, stage_desc<G>(k_head, k_row_bytes, 0, S, true), lds_w);
    stage_settle();
    __syncthreads();
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) qf[qt].read(smem + G::STAGE_BYTES, (qw0 - q0) / 32 + qt, l32, half, extent);
    stage_settle();

    float2* const shares = reinterpret_cast<float2*>(smem + 2 * G::STAGE_BYTES);                // [wave][half][RES]
    float* const refs = reinterpret_cast<float*>(smem + 2 * G::STAGE_BYTES + G::MERGE_BYTES);  // [wave][RES]
    float lse;            // the result: lse2 of query qw0 + lane % RES
    const int lq = lane % G::RES;
    // workgroup-uniform: which pass this is
    bool frozen = !needs_whole<G, D>(extent, c2, Kb, p.k_ts, k_off, 0, causal ? q_last + 1 : S, tid, wave, reinterpret_cast<int*>(shares));
    for (;;) {
    float m[NRT], l[NRT];  // statistics of the queries qw0 + qt*32 + l32 this lane keeps
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) { m[qt] = -INFINITY; l[qt] = 0.f; }
    f32x16 carry;          // the last tile of the pipeline, not yet summed (of the last query subtile); -inf: none
#pragma unroll
    for (int r = 0; r < 16; ++r) carry[r] = -INFINITY;

    if (!frozen) {
        stage_load<G>(st_voff, stage_desc<G>(k_head, k_row_bytes, 0, S, true), lds_w);
        stage_settle();
    }
    for (int t = 0; t < nstage; ++t) {
        __syncthreads();  // stage t is complete; every wave is done reading stage t-1
        const bool more = t + 1 < nstage;
        const u32x4 next_desc = stage_desc<G>(k_head, k_row_bytes, (t + 1) * G::TILE, S, more);
        const unsigned next_lds = lds_w + ((t + 1) & 1) * G::STAGE_BYTES;
        if (t == 1) {  // the shares' common reference (none: no share met a key of the first stage it may use)
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) {
                float top = -INFINITY;
#pragma unroll
                for (int w = 0; w < KS; ++w) top = fmaxf(top, refs[(wave - part + w) * G::RES + qt * 32 + l32]);
                l[qt] *= __builtin_amdgcn_exp2f(m[qt] - (top == -INFINITY ? 0.f : top));
                m[qt] = top;
            }
        }
        // wave-uniform classification of this share of keys against the wave's queries [qw0, qw0+RES-1]
        const int kmin = t * G::TILE + part * 32;
        const bool skip = causal && kmin > qw0 + G::RES - 1;  // every key lies after every query
        const bool hot = frozen && t > 0 && (causal ? kmin + 31 <= qw0 : kmin + 31 < S);
        const char* sbuf = smem + (t & 1) * G::STAGE_BYTES;
        if (more && !hot) stage_load<G>(st_voff, next_desc, next_lds);  // (the hot path spreads them over its tiles)
        Streamed32<G> kf;
        if (hot) {
            // frozen reference: exp/sum of the previous tile between the MFMAs of tile qt; each stage's sum begins at zero, since
            // terms below 2^-24 of what they are added to are lost
            float nm[NRT], l1[NRT], l2[NRT];
#pragma unroll
            for (int q = 0; q < NRT; ++q) {
                m[q] = m[q] == -INFINITY ? 0.f : m[q];  // nothing seen yet: take 0 as the reference
                nm[q] = -m[q];
                l1[q] = 0.f;
                l2[q] = 0.f;
            }
            kf.read(sbuf, part, l32, half);
            f32x16 prev = carry;
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) {
                const int pq = (qt + NRT - 1) % NRT;  // query subtile of the tile before
                f32x16 acc = {0};
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < NM; ++c) {
                    rowstat_frozen_slice<NM>(c, prev, c2, nm[pq], l1[pq], l2[pq]);
                    kf.mma(c, acc, qf[qt], qt == 0);  // acc[key row][query col]
                    if (c == 1) stage_load_slot<G>(st_voff, next_desc, next_lds, qt, NRT);
                    __builtin_amdgcn_sched_barrier(0);
                }
                prev = acc;
            }
            carry = prev;
#pragma unroll
            for (int q = 0; q < NRT; ++q) l[q] += l1[q] + l2[q];
        } else if (!skip) {
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) l[qt] = frozen_sum(l[qt]);
            rowstat_update(carry, c2, m[NRT - 1], l[NRT - 1]);  // drain the pipeline
#pragma unroll
            for (int r = 0; r < 16; ++r) carry[r] = -INFINITY;
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) {
                // this 32x32 tile: keys [kmin, kmin+31] against queries [qmin, qmin+31] (wave-uniform tests)
                const int qmin = qw0 + qt * 32;
                if (causal && kmin > qmin + 31) continue;  // every key lies after every query
                f32x16 acc = {0};
                kf.read(sbuf, part, l32, half);
                if (!frozen) {
                    kf.mma_whole(acc, Qb, p.q_ts, q_off, qmin + l32, S);
                } else {
#pragma unroll
                    for (int c = 0; c < NM; ++c) kf.mma(c, acc, qf[qt], true);
                }
                const bool all_allowed = causal ? (kmin + 31 <= qmin) : (kmin + 31 < S);
                if (!all_allowed) {
                    // key j may be used by query i iff j <= lim(i): i itself under the causal mask, S-1 otherwise
                    const int lim = causal ? qmin + l32 : S - 1;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = kmin + acc_row(r, lane) <= lim ? acc[r] : -INFINITY;
                }
                rowstat_update(acc, c2, m[qt], l[qt]);
            }
        }
        if (t == 0 && more) {
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) refs[wave * G::RES + qt * 32 + l32] = fmaxf(m[qt], __shfl_xor(m[qt], 32));
        }
        stage_settle();
    }
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) l[qt] = frozen_sum(l[qt]);
    rowstat_update(carry, c2, m[NRT - 1], l[NRT - 1]);

    // the half-waves and the KS waves hold disjoint keys of the same queries: every partial sum is rescaled once, to the largest
    // reference of all, then lse2 = m + log2(l)
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) shares[(wave * 2 + half) * G::RES + qt * 32 + l32] = make_float2(m[qt], l[qt]);
    __syncthreads();
    float2 v[2 * KS];
#pragma unroll
    for (int w = 0; w < 2 * KS; ++w) v[w] = shares[((wave - part) * 2 + w) * G::RES + lq];  // the same order in every wave
    float top = v[0].x, sum = 0.f;
#pragma unroll
    for (int w = 1; w < 2 * KS; ++w) top = fmaxf(top, v[w].x);
    const float ms = top == -INFINITY ? 0.f : top;
#pragma unroll
    for (int w = 0; w < 2 * KS; ++w) sum += v[w].y * __builtin_amdgcn_exp2f(v[w].x - ms);
    lse = add_log2(top, sum);
    const bool bad = qw0 + lq < S && !isfinite(lse);
    // every wave is past its last read of the stages here as well, so a second pass may refill them (KS = WAVES: all waves have the same rows)
    if (!frozen || !(KS == WAVES ? __any(bad) : __syncthreads_or(bad))) break;
    frozen = false;
    }
    const int q = qw0 + lq;
    if (lane < G::RES && part == 0 && q < S) p.lse2[(size_t)h * S + q] = lse;
}

// Sweep 2 (see colsum_kernel): column sums (and the diagonal) of the probabilities, one key block per workgroup.
template <int D, int NRT, int KS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (Geo<float, D, NRT, KS, WAVES>::MIN_WG)) void colsum_f32_kernel(ScoreParams p) {
    using G = Geo<float, D, NRT, KS, WAVES>;
    constexpr int NM = Streamed32<G>::NM;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* const sLbase = reinterpret_cast<float*>(smem + 2 * G::STAGE_BYTES);

    int h, kb;
    decode_block(p.order, p.H, p.n_query_blocks, h, kb);
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    const int S = p.S;
    const float c2 = p.c2;
    const int key0 = kb * G::BLOCK;
    const int kend = (int)min((long long)S, (long long)key0 + G::BLOCK);  // exclusive

    const int g = (int)(((long long)h * p.H_kv) / p.H);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* Qb = static_cast<const float*>(p.Q);
    const float* Kb = static_cast<const float*>(p.K);
    const long long q_off = (long long)h * p.q_hs, k_off = (long long)g * p.k_hs;
    const float* lse = p.lse2 + (size_t)h * S;
    const int part = wave % KS;                 // this wave's subtile of a stage
    const int kw0 = key0 + wave / KS * G::RES;  // first key of this wave

    // query stages run from the end of the sequence DOWN to the first stage that can see this block
    const int t_hi = (S - 1) / G::TILE;
    const int t_lo = causal ? key0 / G::TILE : 0;
    const char* q_head = reinterpret_cast<const char*>(Qb + q_off);  // wave-uniform
    const int q_row_bytes = (int)p.q_ts * 4;                        // host guarantees < 2^24
    int st_voff[G::NLOAD];
    stage_offsets<G>(st_voff, q_row_bytes, tid);
    const unsigned lds_w = lds_offset_of(smem) + (unsigned)wave * 1024u;
    // row statistics of a stage: thread tid < TILE owns row tid; beyond the end +inf, so that p = exp2(-inf) = 0
    auto fetch_l = [&](int t) { return tid < G::TILE ? lse[min(t * G::TILE + tid, S - 1)] : 0.f; };
    auto fix_l = [&](int t, float v) { return t * G::TILE + tid < S ? -v : -INFINITY; };  // stored negated: p = exp2(s*c2 + nl)

    // the keys pass through the second stage, while the first stage of queries arrives
    Resident32<G> kf[NRT];
    Extent extent;
    load_resident<G>(reinterpret_cast<const char*>(Kb + k_off), (int)p.k_ts * 4, key0, S, lds_w + G::STAGE_BYTES, tid);
    stage_load<G>(st_voff, stage_desc<G>(q_head, q_row_bytes, t_hi * G::TILE, S, true), lds_w);
    stage_settle();
    __syncthreads();
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) kf[kt].read(smem + G::STAGE_BYTES, (kw0 - key0) / 32 + kt, l32, half, extent);
    stage_settle();

    float col[NRT], dg[NRT];  // column kw0 + kt*32 + l32
    float2* const shares = reinterpret_cast<float2*>(smem + 2 * G::STAGE_BYTES + 2 * G::TILE * (int)sizeof(float));  // [wave][RES]
    // workgroup-uniform: which pass this is
    bool whole = needs_whole<G, D>(extent, c2, Qb, p.q_ts, q_off, t_lo * G::TILE, S, tid, wave, reinterpret_cast<int*>(shares));
    for (;;) {
    float pre_l = 0.f;
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) { col[kt] = 0.f; dg[kt] = 0.f; }
    f32x16 carry = {0};  // the last tile of the pipeline, not yet summed (of the last key subtile); nl = -inf: none
    float carry_nl[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) carry_nl[r] = -INFINITY;

    if (whole) stage_load<G>(st_voff, stage_desc<G>(q_head, q_row_bytes, t_hi * G::TILE, S, true), lds_w);
    pre_l = fetch_l(t_hi);
    if (tid < G::TILE) sLbase[tid] = fix_l(t_hi, pre_l);
    stage_settle();
    int buf = 0;
    for (int t = t_hi; t >= t_lo; --t, buf ^= 1) {
        __syncthreads();
        const bool more = t > t_lo;
        const u32x4 next_desc = stage_desc<G>(q_head, q_row_bytes, (t - 1) * G::TILE, S, more);
        const unsigned next_lds = lds_w + (buf ^ 1) * G::STAGE_BYTES;
        if (more) pre_l = fetch_l(t - 1);
        const int qmin = t * G::TILE + part * 32;                            // this wave's subtile: queries [qmin, qmin + 31]
        const bool on_diag = qmin <= kw0 + G::RES - 1 && qmin + 31 >= kw0;  // they meet the diagonal band of this wave
        const bool skip = (causal && qmin + 31 < kw0) || qmin >= S;         // every query lies before every key, or past the end
        const char* sbuf = smem + buf * G::STAGE_BYTES;
        const float* lbuf = sLbase + buf * G::TILE;
        const bool hot = !on_diag && !skip && !whole;
        if (more && !hot) stage_load<G>(st_voff, next_desc, next_lds);  // (the hot path spreads them over its tiles)
        Streamed32<G> qf;
        float nl[16];
        if (hot) {
            // exp/sum of the previous tile between the MFMAs of tile kt
            float s1[NRT], s2[NRT];  // summed stage by stage
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) { s1[kt] = 0.f; s2[kt] = 0.f; }
            qf.read(sbuf, part, l32, half);
            read_nl(nl, lbuf, part, half);
            f32x16 prev = carry;
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) {
                const int pk = (kt + NRT - 1) % NRT;  // key subtile of the tile before
                f32x16 acc = {0};
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < NM; ++c) {
                    if (kt == 0) colsum_slice<NM>(c, prev, carry_nl, c2, s1[pk], s2[pk]);  // the carried tile has its own rows
                    else colsum_slice<NM>(c, prev, nl, c2, s1[pk], s2[pk]);
                    qf.mma(c, acc, kf[kt], kt == 0);  // acc[query row][key col]
                    if (c == 1) stage_load_slot<G>(st_voff, next_desc, next_lds, kt, NRT);
                    __builtin_amdgcn_sched_barrier(0);
                }
                prev = acc;
            }
            carry = prev;
#pragma unroll
            for (int r = 0; r < 16; ++r) carry_nl[r] = nl[r];
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) col[kt] += s1[kt] + s2[kt];
        } else if (!skip) {
            col[NRT - 1] += colsum_tile(carry, carry_nl, c2);  // drain the pipeline
#pragma unroll
            for (int r = 0; r < 16; ++r) carry_nl[r] = -INFINITY;
            read_nl(nl, lbuf, part, half);
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) {
                // this 32x32 tile: queries [qmin, qmin+31] against keys [kmin, kmin+31] (wave-uniform tests)
                const int kmin = kw0 + kt * 32;
                if (causal && qmin + 31 < kmin) continue;  // every query lies before every key
                f32x16 acc = {0};
                qf.read(sbuf, part, l32, half);
                if (whole) {
                    qf.mma_whole(acc, Kb, p.k_ts, k_off, kmin + l32, kend);
                } else {
#pragma unroll
                    for (int c = 0; c < NM; ++c) qf.mma(c, acc, kf[kt], true);
                }
                if (qmin > kmin + 31 || qmin + 31 < kmin) {  // off the diagonal: nothing to mask, no self term
                    col[kt] += colsum_tile(acc, nl, c2);
                } else {
                    const int my_k = kmin + l32;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int q = qmin + acc_row(r, lane);
                        float pr = __builtin_amdgcn_exp2f(fmaf(acc[r], c2, nl[r]));
                        if (causal && q < my_k) pr = 0.f;
                        if (q == my_k) dg[kt] = pr;
                        sum += pr;
                    }
                    col[kt] += sum;
                }
            }
        }
        if (more && tid < G::TILE) sLbase[(buf ^ 1) * G::TILE + tid] = fix_l(t - 1, pre_l);
        stage_settle();
    }
    col[NRT - 1] += colsum_tile(carry, carry_nl, c2);
    bool bad = false;  // (the zeros that fill up the last block aside: a normaliser far below 0 takes them past all limits)
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) bad |= kw0 + kt * 32 + l32 < kend && !isfinite(col[kt]);
    // (every wave is past its last read of the stages)
    if (whole || !__syncthreads_or(bad)) break;
    whole = true;
    }

#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) {
        col[kt] += __shfl_xor(col[kt], 32);
        dg[kt] += __shfl_xor(dg[kt], 32);
        shares[wave * G::RES + kt * 32 + l32] = make_float2(col[kt], dg[kt]);
    }
    __syncthreads();
    if (part != 0) return;
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) {
        const float2 all = add_shares<G>(shares + wave * G::RES + kt * 32 + l32);
        col[kt] = all.x;
        dg[kt] = all.y;
        const int key = kw0 + kt * 32 + l32;
        if (half == 0 && key < kend) {
            p.colsum[(size_t)h * S + key] = col[kt];
            p.diag[(size_t)h * S + key] = dg[kt];
        }
    }
}

template <int D, int NRT, int KS, int WAVES>
static int prepare_f32() {
    using G = Geo<float, D, NRT, KS, WAVES>;
    static const int err = raise_lds_limits({{reinterpret_cast<const void*>(&rowstats_f32_kernel<D, NRT, KS, WAVES>), G::LDS_ROWSTATS},
                                             {reinterpret_cast<const void*>(&colsum_f32_kernel<D, NRT, KS, WAVES>), G::LDS_COLSUM}});
    return err;
}

template <int D, int NRT, int KS, int WAVES>
static int launch_f32(const ScoreParams& p_in, int which, hipStream_t st) {
    using G = Geo<float, D, NRT, KS, WAVES>;
    static_assert(G::LONGEST_PITCH >= (PITCH_END - 4) * 4 || (D == 64 && WAVES == 8), "a stage reaches all its rows at every pitch");
    ScoreParams p = p_in;
    p.n_query_blocks = (p.S + G::BLOCK - 1) / G::BLOCK;
    const unsigned grid = (unsigned)(p.H * p.n_query_blocks);  // as many key blocks
    if (which & 1) hipLaunchKernelGGL((rowstats_f32_kernel<D, NRT, KS, WAVES>), dim3(grid), dim3(G::THREADS), G::LDS_ROWSTATS, st, p);
    if (which & 2) hipLaunchKernelGGL((colsum_f32_kernel<D, NRT, KS, WAVES>), dim3(grid), dim3(G::THREADS), G::LDS_COLSUM, st, p);
    return (int)hipGetLastError();
}

int prepare_sweeps_f32(int d) { return d == 128 ? first_error(prepare_f32<128, 1, 2, 4>, prepare_f32<128, 1, 4, 8>) : first_error(prepare_f32<64, 1, 4, 4>, prepare_f32<64, 2, 4, 4>, prepare_f32<64, 1, 8, 8>); }

int launch_sweeps_f32(const ScoreParams& p, int d, int which, hipStream_t st) {
    const long long blocks256 = (long long)p.H * ((p.S + 255) / 256);
    // Eight waves, twice the sharers of a row and twice the rows of a stage, one workgroup per CU: where the CUs then have at most one, or
    // the longest block decides.  us a sweep, four / eight: d = 64 1024 tokens, 4 heads 13.2 / 11.6, 500, 16 9.0 / 8.7, 400, 4 8.8 / 8.6, 384, 4 (a stage and a
    // half) 7.5 / 8.2, 300, 4 7.6 / 8.2, 3000, 4 32 / 25, 4000, 4 41 / 38, 1024, 12 13.5 / 16, full 2000, 4 22.5 / 19.4, 2500, 4 37 / 41.5; d = 128 400, 8 17.7 / 17.8,
    // 500, 16 19 / 17.5, 1000, 16 33 / 28.5, 2000, 12 62 / 52, 1000, 32 38 / 39, full 700, 16 24.6 / 23.5.
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    if (d == 128 && p.S >= 384 && (blocks256 <= 64 || (causal && blocks256 <= 128 && p.S >= 1500))) return launch_f32<128, 1, 4, 8>(p, which, st);
    // (d = 64: their 256 rows of a stage must be within reach, up to 8.4 MB of pitch)
    const bool reach = (p.q_ts > p.k_ts ? p.q_ts : p.k_ts) * 4 <= Geo<float, 64, 1, 8, 8>::LONGEST_PITCH;
    if (d == 64 && reach && p.S > 384 && (blocks256 <= 32 || (causal && blocks256 <= 64 && p.S >= 3000))) return launch_f32<64, 1, 8, 8>(p, which, st);
    if (d == 128) return launch_f32<128, 1, 2, 4>(p, which, st);
    return blocks256 <= 192 ? launch_f32<64, 1, 4, 4>(p, which, st) : launch_f32<64, 2, 4, 4>(p, which, st);
}

}  // namespace lemo
