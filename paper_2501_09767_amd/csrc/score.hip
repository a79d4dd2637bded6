// Token informativeness (Sec. 4.2, Eq. 1 with the head mean of Eq. 2) on gfx950.
//
// Column sums of softmax(Q K^T) need every row's FINAL normaliser, so Q K^T is swept twice and the
// S x S matrix is never stored (memory linear in S, as Sec. 4.3 requires of the scoring kernel):
//
//   sweep 1  rowstats_kernel   per (head, block of 256 queries or a part of that): keys stream through LDS, the block's
//                              queries stay in registers; an online max/sum per query gives the
//                              base-2 log-sum-exp  lse2[h][i].
//   sweep 2  colsum_kernel     per (head, block of 256 keys or a part of that): the block's keys stay in
//                              registers, queries stream through LDS; p = exp2(s*c2 - lse2[i]) is
//                              added into per-lane column accumulators -- each column is owned by one
//                              workgroup, so there are no atomics and the result is deterministic.
//   reduce   head_mean_kernel  scores[j] = (1/H) sum_h (colsum - [exclude self] diag), fixed order.
//
// Both sweeps compute 32x32 logit tiles with MFMA (bf16: 32x32x16; fp32: score_f32.hip, three-part
// splits on the same instruction).  The product is oriented so that the axis being reduced runs along the accumulator
// REGISTERS of a lane and the axis being kept runs along LANES: sweep 1 computes K.Q^T (lane = query),
// sweep 2 computes Q.K^T (lane = key).  Row and column statistics are then plain in-register chains
// with one cross-lane step at the very end.
//
// Per logit the matrix core spends as many cycles (2*d flops) as the vector ALU does on fma + exp2 + add,
// so the two must run at the same time.  Tiles that need no masking go through a software pipeline:
// while the MFMA chain of tile n runs, the exp/sum work of tile n-1 (kept in a "carry" accumulator)
// is issued between the MFMAs; the instruction order is pinned with scheduling-group barriers.
#include <type_traits>

#include "score_sweeps.hpp"

namespace lemo {

// ------------------------------------------------------------------------------------------------
// Sweep 1: base-2 log-sum-exp of every query row.
// ------------------------------------------------------------------------------------------------

// First pass, frozen reference: the running maximum is tracked through the first stage (and through every masked
// tile); from then on unmasked tiles add exp2(s*c2 - m) against the maximum frozen at that point, which saves the
// maximum search and the rescale.  Waves that share rows freeze the maximum of the whole first stage, not of the 32 or 64
// keys of their own share (of which the last tile is still in the carry: a share of one tile would have no reference at
// all): a lower reference is overtaken more often, and against one far above every logit the exponentials are flushed.
// Should a later logit exceed the frozen reference by too much, the sum overflows or passes FROZEN_LIMIT; it is then made
// infinite before it is rescaled, and lse2 comes out non-finite.  A workgroup that finds such a row among its own
// (normally none does) goes through its keys a second time with the running maximum everywhere, before it stores
// anything: no second launch, no extra traffic when there is nothing to repair.
template <int D, int NRT, int KS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (Geo<bf16_t, D, NRT, KS, WAVES>::MIN_WG)) void rowstats_kernel(ScoreParams p) {
    using G = Geo<bf16_t, D, NRT, KS, WAVES>;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    int h, qb;
    decode_block(p.order, p.H, p.n_query_blocks, h, qb);
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    if (causal) qb = p.n_query_blocks - 1 - qb;  // late query blocks see the most keys: start them first
    const int g = (int)(((long long)h * p.H_kv) / p.H);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    // (KS = 1: not made a scalar -- the hot stream then comes out 1 % slower, 22000 tokens, 32 heads, full: 3640 / 3600 us)
    const int wave = KS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const bf16_t* Qb = static_cast<const bf16_t*>(p.Q);
    const bf16_t* Kb = static_cast<const bf16_t*>(p.K);
    const long long q_off = (long long)h * p.q_hs, k_off = (long long)g * p.k_hs;
    const int S = p.S;
    const float c2 = p.c2;
    const int q0 = qb * G::BLOCK;        // first query of the workgroup
    const int part = wave % KS, sub0 = part * G::SHARE;  // this wave's share of a stage: subtiles [sub0, sub0 + SHARE)
    const int qw0 = q0 + wave / KS * G::RES;  // first query of this wave

    // resident operand: this wave's queries as MFMA B fragments
    u32x4 qf[NRT][G::NCH];
    if constexpr (KS == 1) {
#pragma unroll
        for (int qt = 0; qt < NRT; ++qt)
#pragma unroll
            for (int c = 0; c < G::NCH; ++c) qf[qt][c] = load_piece(Qb, p.q_ts, q_off, qw0 + qt * 32 + l32, S, c * 32 + half * 16);
    }

    // key stages [0, nstage): under a causal mask only keys up to the block's last query matter
    const int q_last = min(q0 + G::BLOCK, S) - 1;
    const int nstage = (causal ? q_last : S - 1) / G::TILE + 1;

    const char* k_head = reinterpret_cast<const char*>(Kb + k_off);  // wave-uniform
    const int k_row_bytes = (int)p.k_ts * (int)sizeof(bf16_t);           // host guarantees < 2^24
    int st_voff[G::NLOAD];
    stage_offsets<G>(st_voff, k_row_bytes, tid);
    const unsigned lds_w = lds_offset_of(smem) + (unsigned)__builtin_amdgcn_readfirstlane(wave) * 1024u;

    if constexpr (KS > 1) {  // the queries pass through the second stage, while the first stage of keys arrives
        load_resident<G>(reinterpret_cast<const char*>(Qb + q_off), (int)p.q_ts * (int)sizeof(bf16_t), q0, S, lds_w + G::STAGE_BYTES, tid);
        stage_load<G>(st_voff, stage_desc<G>(k_head, k_row_bytes, 0, S, true), lds_w);
        stage_settle();
        __syncthreads();
#pragma unroll
        for (int qt = 0; qt < NRT; ++qt) read_frags<G>(qf[qt], smem + G::STAGE_BYTES, (qw0 - q0) / 32 + qt, l32, half);
        stage_settle();
    }

    float* const refs = reinterpret_cast<float*>(smem + 2 * G::STAGE_BYTES + G::MERGE_BYTES);  // [wave][RES]
    static_assert(KS == 1 || G::RES == WAVE, "a lane finishes one of the shared rows");
    constexpr int NR = KS > 1 ? 1 : NRT;
    float lse[NR];        // the result: lse2 of query qw0 + qt*32 + l32 (KS > 1: qw0 + lane)
    bool frozen = true;   // wave-uniform (in fact workgroup-uniform): which pass this is
    for (;;) {
    float m[NRT], l[NRT];  // statistics of the queries qw0 + qt*32 + l32 this lane keeps
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) { m[qt] = -INFINITY; l[qt] = 0.f; }

    // carry: the last computed tile whose statistics have not been folded in yet (it belongs to the last
    // query subtile); -inf means "none"
    f32x16 carry;
#pragma unroll
    for (int r = 0; r < 16; ++r) carry[r] = -INFINITY;

    if (KS == 1 || !frozen) {
        stage_load<G>(st_voff, stage_desc<G>(k_head, k_row_bytes, 0, S, true), lds_w);
        stage_settle();
    }
    for (int t = 0; t < nstage; ++t) {
        __syncthreads();  // stage t is complete; every wave is done reading stage t-1
        const bool more = t + 1 < nstage;
        const u32x4 next_desc = stage_desc<G>(k_head, k_row_bytes, (t + 1) * G::TILE, S, more);
        const unsigned next_lds = lds_w + ((t + 1) & 1) * G::STAGE_BYTES;
        if constexpr (KS > 1) {
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
        }
        const int k0 = t * G::TILE;
        // wave-uniform classification of this share of keys against the wave's queries [qw0, qw0+RES-1]
        const int ka = k0 + sub0 * 32, kz = ka + G::SHARE * 32 - 1;  // keys of this wave's share
        const bool skip = causal && ka > qw0 + G::RES - 1;  // every key lies after every query
        const bool clean = causal ? (kz <= qw0) : (kz < S);
        const char* sbuf = smem + (t & 1) * G::STAGE_BYTES;
        const bool hot = clean && frozen && t > 0;
        if (more && !hot) stage_load<G>(st_voff, next_desc, next_lds);  // (the hot path spreads them over its tiles)
        if (hot) {
            // pipelined, frozen reference: exp/sum of the previous tile between the MFMAs of tile (ks, qt)
            // (the sum of a query is kept in two halves, l1 and l2, that the exponentials are added to directly; shared
            // rows begin each stage's sum at zero, since terms below 2^-24 of what they are added to are lost)
            float nm[NRT], l1[NRT], l2[NRT];
#pragma unroll
            for (int q = 0; q < NRT; ++q) {
                m[q] = m[q] == -INFINITY ? 0.f : m[q];  // nothing seen yet: take 0 as the reference
                nm[q] = -m[q];
                l1[q] = KS > 1 ? 0.f : l[q];
                l2[q] = 0.f;
            }
            u32x4 kf[G::NCH];
            read_frags<G>(kf, sbuf, sub0, l32, half);
#pragma unroll
            for (int ks = 0; ks < G::SHARE; ++ks) {
                u32x4 kn[G::NCH];
                f32x16 prev = carry;
#pragma unroll
                for (int qt = 0; qt < NRT; ++qt) {  // tile (ks, qt) while the tile before it is summed
                    const int pq = (qt + NRT - 1) % NRT;  // query subtile of the tile before
                    f32x16 acc = {0};
                    slot_fence();
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) {
                        rowstat_frozen_slice<G::NCH>(c, prev, c2, nm[pq], l1[pq], l2[pq]);
                        mma_chunk<bf16_t>(acc, kf[c], qf[qt][c]);  // acc[key row][query col]
                        if (c == 1) stage_load_slot<G>(st_voff, next_desc, next_lds, ks * NRT + qt, G::SHARE * NRT);
                        if (qt == NRT - 1 && ks + 1 < G::SHARE)
                            kn[c] = *reinterpret_cast<const u32x4*>(&sbuf[G::frag((sub0 + ks + 1) * 32 + l32, c, half)]);
                        slot_fence();
                    }
                    prev = acc;
                }
                carry = prev;
                if (ks + 1 < G::SHARE) {
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) kf[c] = kn[c];
                }
            }
#pragma unroll
            for (int q = 0; q < NRT; ++q) l[q] = KS > 1 ? l[q] + (l1[q] + l2[q]) : l1[q] + l2[q];
        } else if (clean) {
            // pipelined, running maximum: the statistics update of the previous tile is issued slice by slice
            // between the MFMAs of tile (ks, qt); fragments of the next key subtile are read during the last chain
            u32x4 kf[G::NCH];
            read_frags<G>(kf, sbuf, sub0, l32, half);
#pragma unroll
            for (int ks = 0; ks < G::SHARE; ++ks) {
                u32x4 kn[G::NCH];
                f32x16 prev = carry;
#pragma unroll
                for (int qt = 0; qt < NRT; ++qt) {
                    const int pq = (qt + NRT - 1) % NRT;
                    f32x16 acc = {0};
                    RowStat st;
                    slot_fence();
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) {
                        rowstat_slice<G::NCH>(c, prev, c2, m[pq], st);
                        mma_chunk<bf16_t>(acc, kf[c], qf[qt][c]);
                        if (qt == NRT - 1 && ks + 1 < G::SHARE)
                            kn[c] = *reinterpret_cast<const u32x4*>(&sbuf[G::frag((sub0 + ks + 1) * 32 + l32, c, half)]);
                        slot_fence();
                    }
                    rowstat_finish(st, m[pq], l[pq]);
                    prev = acc;
                }
                carry = prev;
                if (ks + 1 < G::SHARE) {
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) kf[c] = kn[c];
                }
            }
        } else if (!skip) {
#pragma unroll
            for (int qt = 0; qt < NRT; ++qt) l[qt] = frozen_sum(l[qt]);
            rowstat_update(carry, c2, m[NRT - 1], l[NRT - 1]);  // drain the pipeline before the masked tiles
#pragma unroll
            for (int r = 0; r < 16; ++r) carry[r] = -INFINITY;
#pragma unroll
            for (int ks = 0; ks < G::SHARE; ++ks) {
                u32x4 kf[G::NCH];
                read_frags<G>(kf, sbuf, sub0 + ks, l32, half);
#pragma unroll
                for (int qt = 0; qt < NRT; ++qt) {
                    // this 32x32 tile: keys [kmin, kmin+31] against queries [qmin, qmin+31] (wave-uniform tests)
                    const int kmin = ka + ks * 32, qmin = qw0 + qt * 32;
                    if (causal && kmin > qmin + 31) continue;  // every key lies after every query
                    f32x16 acc = {0};
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) mma_chunk<bf16_t>(acc, kf[c], qf[qt][c]);
                    const bool all_allowed = causal ? (kmin + 31 <= qmin) : (kmin + 31 < S);
                    if (!all_allowed) {
                        // key j may be used by query i iff j <= lim(i): i itself under the causal mask, S-1 otherwise
                        const int lim = causal ? qmin + l32 : S - 1;
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int key = kmin + acc_row(r, lane);
                            acc[r] = key <= lim ? acc[r] : -INFINITY;
                        }
                    }
                    rowstat_update(acc, c2, m[qt], l[qt]);
                }
            }
        }
        if constexpr (KS > 1) {
            if (t == 0 && more) {
                rowstat_update(carry, c2, m[NRT - 1], l[NRT - 1]);  // the last tile counts as well
#pragma unroll
                for (int r = 0; r < 16; ++r) carry[r] = -INFINITY;
#pragma unroll
                for (int qt = 0; qt < NRT; ++qt) refs[wave * G::RES + qt * 32 + l32] = fmaxf(m[qt], __shfl_xor(m[qt], 32));
            }
        }
        stage_settle();
    }
#pragma unroll
    for (int qt = 0; qt < NRT; ++qt) l[qt] = frozen_sum(l[qt]);
    rowstat_update(carry, c2, m[NRT - 1], l[NRT - 1]);

    // the two half-waves hold disjoint key rows of the same queries: merge, then lse2 = m + log2(l)
    // (with KS > 1, so do the KS waves: every partial sum is rescaled once, to the largest reference of all)
    float2* const shares = reinterpret_cast<float2*>(smem + 2 * G::STAGE_BYTES);  // [wave][half][RES]
    if constexpr (KS > 1) {
#pragma unroll
        for (int qt = 0; qt < NRT; ++qt) shares[(wave * 2 + half) * G::RES + qt * 32 + l32] = make_float2(m[qt], l[qt]);
        __syncthreads();
    }
    bool bad = false;
#pragma unroll
    for (int qt = 0; qt < NR; ++qt) {
        constexpr int N = KS > 1 ? 2 * KS : 2;
        float2 v[N];
        if constexpr (KS > 1) {
#pragma unroll
            for (int w = 0; w < N; ++w) v[w] = shares[((wave - part) * 2 + w) * G::RES + lane];  // the same order in every wave
        } else {
            v[0] = make_float2(m[qt], l[qt]);
            v[1] = make_float2(__shfl_xor(m[qt], 32), __shfl_xor(l[qt], 32));
        }
        float top = v[0].x, sum = 0.f;
#pragma unroll
        for (int w = 1; w < N; ++w) top = fmaxf(top, v[w].x);
        const float ms = top == -INFINITY ? 0.f : top;
#pragma unroll
        for (int w = 0; w < N; ++w) sum += v[w].y * __builtin_amdgcn_exp2f(v[w].x - ms);
        lse[qt] = KS > 1 ? add_log2(top, sum) : top + __builtin_amdgcn_logf(sum);
        bad |= qw0 + (KS > 1 ? lane : qt * 32 + l32) < S && !isfinite(lse[qt]);
    }
    // every wave is past its last read of the stages here as well, so a second pass may refill them (KS = WAVES: all waves have the same rows)
    if (!frozen || !(KS == WAVES ? __any(bad) : __syncthreads_or(bad))) break;
    frozen = false;
    }
#pragma unroll
    for (int qt = 0; qt < NR; ++qt) {
        const int q = qw0 + (KS > 1 ? lane : qt * 32 + l32);
        if ((KS > 1 || half == 0) && part == 0 && q < S) p.lse2[(size_t)h * S + q] = lse[qt];
    }
}

// ------------------------------------------------------------------------------------------------
// Sweep 2: column sums (and the diagonal) of the probabilities, one key block per workgroup.
// ------------------------------------------------------------------------------------------------

template <int D, int NRT, int KS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (Geo<bf16_t, D, NRT, KS, WAVES>::MIN_WG)) void colsum_kernel(ScoreParams p) {
    using G = Geo<bf16_t, D, NRT, KS, WAVES>;
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
    const int wave = KS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const bf16_t* Qb = static_cast<const bf16_t*>(p.Q);
    const bf16_t* Kb = static_cast<const bf16_t*>(p.K);
    const long long q_off = (long long)h * p.q_hs, k_off = (long long)g * p.k_hs;
    const float* lse = p.lse2 + (size_t)h * S;
    const int part = wave % KS, sub0 = part * G::SHARE;  // this wave's share of a stage: subtiles [sub0, sub0 + SHARE)
    const int kw0 = key0 + wave / KS * G::RES;  // first key of this wave

    // resident operand: this wave's keys as MFMA B fragments (zero beyond the block's end)
    u32x4 kf[NRT][G::NCH];
    if constexpr (KS == 1) {
#pragma unroll
        for (int kt = 0; kt < NRT; ++kt)
#pragma unroll
            for (int c = 0; c < G::NCH; ++c) kf[kt][c] = load_piece(Kb, p.k_ts, k_off, kw0 + kt * 32 + l32, kend, c * 32 + half * 16);
    }

    float col[NRT], col2[NRT], dg[NRT];  // column kw0 + kt*32 + l32 (its sum kept in two halves, col and col2)
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) { col[kt] = 0.f; col2[kt] = 0.f; dg[kt] = 0.f; }

    // query stages run from the end of the sequence DOWN to the first stage that can see this block, so
    // that all key blocks of a head walk the same query rows at about the same time (shared through L2)
    const int t_hi = (S - 1) / G::TILE;
    const int t_lo = causal ? key0 / G::TILE : 0;

    const char* q_head = reinterpret_cast<const char*>(Qb + q_off);  // wave-uniform
    const int q_row_bytes = (int)p.q_ts * (int)sizeof(bf16_t);           // host guarantees < 2^24
    int st_voff[G::NLOAD];
    stage_offsets<G>(st_voff, q_row_bytes, tid);
    const unsigned lds_w = lds_offset_of(smem) + (unsigned)__builtin_amdgcn_readfirstlane(wave) * 1024u;
    float pre_l = 0.f;
    // row statistics of a stage: thread tid < TILE owns row tid; beyond the end +inf, so that p = exp2(-inf) = 0
    auto fetch_l = [&](int t) { return tid < G::TILE ? lse[min(t * G::TILE + tid, S - 1)] : 0.f; };
    auto fix_l = [&](int t, float v) { return t * G::TILE + tid < S ? -v : -INFINITY; };  // stored negated: p = exp2(s*c2 + nl)

    // carry: last computed tile not yet summed (always a tile of the last key subtile); nl = -inf means "none"
    f32x16 carry = {0};
    float carry_nl[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) carry_nl[r] = -INFINITY;

    if constexpr (KS > 1)  // the keys pass through the second stage
        load_resident<G>(reinterpret_cast<const char*>(Kb + k_off), (int)p.k_ts * (int)sizeof(bf16_t), key0, S, lds_w + G::STAGE_BYTES, tid);
    stage_load<G>(st_voff, stage_desc<G>(q_head, q_row_bytes, t_hi * G::TILE, S, true), lds_w);
    pre_l = fetch_l(t_hi);
    if (tid < G::TILE) sLbase[tid] = fix_l(t_hi, pre_l);
    stage_settle();
    if constexpr (KS > 1) {
        __syncthreads();
#pragma unroll
        for (int kt = 0; kt < NRT; ++kt) read_frags<G>(kf[kt], smem + G::STAGE_BYTES, (kw0 - key0) / 32 + kt, l32, half);
        stage_settle();
    }
    int buf = 0;
    for (int t = t_hi; t >= t_lo; --t, buf ^= 1) {
        __syncthreads();
        const bool more = t > t_lo;
        const u32x4 next_desc = stage_desc<G>(q_head, q_row_bytes, (t - 1) * G::TILE, S, more);
        const unsigned next_lds = lds_w + (buf ^ 1) * G::STAGE_BYTES;
        if (more) pre_l = fetch_l(t - 1);
        const int i0 = t * G::TILE;
        const int ia = i0 + sub0 * 32, iz = ia + G::SHARE * 32 - 1;   // queries of this wave's share
        const bool on_diag = ia <= kw0 + G::RES - 1 && iz >= kw0;    // they meet the diagonal band of this wave
        const bool skip = causal && iz < kw0;                        // every query lies before every key
        const char* sbuf = smem + buf * G::STAGE_BYTES;
        const float* lbuf = sLbase + buf * G::TILE;
        // (eight waves: no subtile past the end is touched, so that their longer stages meet no more zeros in the place of queries)
        bool hot = !on_diag && !skip;
        if constexpr (WAVES > 4) hot = hot && ia + (G::SHARE - 1) * 32 < S;
        if (more && !hot) stage_load<G>(st_voff, next_desc, next_lds);  // (the hot path spreads them over its tiles)
        if (hot) {
            // pipelined: exp/sum of the previous tile is issued slice by slice between the MFMAs of tile
            // (qs, kt); fragments and row statistics of the next query subtile are read during the last chain
            u32x4 qf[G::NCH];
            float nl[16];
            float s1[NRT], s2[NRT];  // as in sweep 1: shared rows sum stage by stage
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) {
                s1[kt] = KS > 1 ? 0.f : col[kt];
                s2[kt] = KS > 1 ? 0.f : col2[kt];
            }
            read_frags<G>(qf, sbuf, sub0, l32, half);
            read_nl(nl, lbuf, sub0, half);
#pragma unroll
            for (int qs = 0; qs < G::SHARE; ++qs) {
                u32x4 qn[G::NCH];
                float nn[16];
                f32x16 prev = carry;
#pragma unroll
                for (int kt = 0; kt < NRT; ++kt) {  // tile (qs, kt) while the tile before it is summed
                    const int pk = (kt + NRT - 1) % NRT;  // key subtile of the tile before
                    f32x16 acc = {0};
                    slot_fence();
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) {
                        if (kt == 0) colsum_slice<G::NCH>(c, prev, carry_nl, c2, s1[pk], s2[pk]);  // the carried tile has its own rows
                        else colsum_slice<G::NCH>(c, prev, nl, c2, s1[pk], s2[pk]);
                        mma_chunk<bf16_t>(acc, qf[c], kf[kt][c]);  // acc[query row][key col]
                        if (c == 1) stage_load_slot<G>(st_voff, next_desc, next_lds, qs * NRT + kt, G::SHARE * NRT);
                        if (kt == NRT - 1 && qs + 1 < G::SHARE) {
                            qn[c] = *reinterpret_cast<const u32x4*>(&sbuf[G::frag((sub0 + qs + 1) * 32 + l32, c, half)]);
                            if (c < 4) {
                                const f32x4 v = *reinterpret_cast<const f32x4*>(&lbuf[(sub0 + qs + 1) * 32 + c * 8 + half * 4]);
                                nn[c * 4 + 0] = v[0]; nn[c * 4 + 1] = v[1]; nn[c * 4 + 2] = v[2]; nn[c * 4 + 3] = v[3];
                            }
                        }
                        slot_fence();
                    }
                    prev = acc;
                }
                carry = prev;
#pragma unroll
                for (int r = 0; r < 16; ++r) carry_nl[r] = nl[r];
                if (qs + 1 < G::SHARE) {
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) qf[c] = qn[c];
#pragma unroll
                    for (int r = 0; r < 16; ++r) nl[r] = nn[r];
                }
            }
#pragma unroll
            for (int kt = 0; kt < NRT; ++kt) {
                col[kt] = KS > 1 ? col[kt] + s1[kt] : s1[kt];
                col2[kt] = KS > 1 ? col2[kt] + s2[kt] : s2[kt];
            }
        } else if (!skip) {
            col[NRT - 1] += colsum_tile(carry, carry_nl, c2);  // drain the pipeline before the masked tiles
#pragma unroll
            for (int r = 0; r < 16; ++r) carry_nl[r] = -INFINITY;
#pragma unroll
            for (int qs = 0; qs < G::SHARE; ++qs) {
                u32x4 qf[G::NCH];
                float nl[16];
                read_frags<G>(qf, sbuf, sub0 + qs, l32, half);
                read_nl(nl, lbuf, sub0 + qs, half);
#pragma unroll
                for (int kt = 0; kt < NRT; ++kt) {
                    // this 32x32 tile: queries [qmin, qmin+31] against keys [kmin, kmin+31] (wave-uniform tests)
                    const int qmin = ia + qs * 32, kmin = kw0 + kt * 32;
                    if (causal && qmin + 31 < kmin) continue;  // every query lies before every key
                    if constexpr (WAVES > 4)
                        if (qmin >= S) continue;
                    f32x16 acc = {0};
#pragma unroll
                    for (int c = 0; c < G::NCH; ++c) mma_chunk<bf16_t>(acc, qf[c], kf[kt][c]);
                    if (qmin > kmin + 31 || qmin + 31 < kmin) {  // off the diagonal: nothing to mask, no self term
                        col[kt] += colsum_tile(acc, nl, c2);
                    } else {
                        const int my_k = kmin + l32;
                        float part = 0.f;
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int q = qmin + acc_row(r, lane);
                            float pr = __builtin_amdgcn_exp2f(fmaf(acc[r], c2, nl[r]));
                            if (causal && q < my_k) pr = 0.f;
                            if (q == my_k) dg[kt] = pr;
                            part += pr;
                        }
                        col[kt] += part;
                    }
                }
            }
        }
        if (more && tid < G::TILE) sLbase[(buf ^ 1) * G::TILE + tid] = fix_l(t - 1, pre_l);
        stage_settle();
    }
    col[NRT - 1] += colsum_tile(carry, carry_nl, c2);

    float2* const shares = reinterpret_cast<float2*>(smem + 2 * G::STAGE_BYTES + 2 * G::TILE * (int)sizeof(float));  // [wave][RES]
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) {
        col[kt] += col2[kt];
        col[kt] += __shfl_xor(col[kt], 32);
        dg[kt] += __shfl_xor(dg[kt], 32);
        if constexpr (KS > 1) shares[wave * G::RES + kt * 32 + l32] = make_float2(col[kt], dg[kt]);
    }
    if constexpr (KS > 1) {
        __syncthreads();
        if (part != 0) return;
    }
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) {
        if constexpr (KS > 1) {
            const float2 all = add_shares<G>(shares + wave * G::RES + kt * 32 + l32);
            col[kt] = all.x;
            dg[kt] = all.y;
        }
        const int key = kw0 + kt * 32 + l32;
        if (half == 0 && key < kend) {
            p.colsum[(size_t)h * S + key] = col[kt];
            p.diag[(size_t)h * S + key] = dg[kt];
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Head mean (Eq. 2's 1/N_head) with the self term optionally removed (Eq. 1's i != j).
// ------------------------------------------------------------------------------------------------
// Bound by the latency of the loads (2 H of them per token): they are asked for eight heads at a time, and 64-thread
// workgroups spread short sequences over more CUs.  S = 32768, H = 32: 15.4 us with one head at a time.
constexpr int HM_THREADS = 64;
__global__ __launch_bounds__(HM_THREADS) void head_mean_kernel(const float* __restrict__ colsum, const float* __restrict__ diag,
                                                        float* __restrict__ scores, int S, int H, int exclude_self) {
    const int j = blockIdx.x * HM_THREADS + threadIdx.x;
    if (j >= S) return;
    float acc = 0.f;
    for (int h0 = 0; h0 < H; h0 += 8) {
        float c[8], d[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const size_t at = (size_t)min(h0 + e, H - 1) * S + j;
            c[e] = colsum[at];
            d[e] = exclude_self ? diag[at] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (h0 + e < H) acc += exclude_self ? c[e] - d[e] : c[e];
    }
    scores[j] = acc / (float)H;
}

template <int D, int NRT, int KS, int WAVES>
static int limits_of() {
    using G = Geo<bf16_t, D, NRT, KS, WAVES>;
    return raise_lds_limits({{reinterpret_cast<const void*>(&rowstats_kernel<D, NRT, KS, WAVES>), G::LDS_ROWSTATS},
                             {reinterpret_cast<const void*>(&colsum_kernel<D, NRT, KS, WAVES>), G::LDS_COLSUM}});
}
template <int D, int NRT>
static int prepare_sweeps() {
    static const int err = [] {
        const int rc = first_error(limits_of<D, NRT, 1, 4>, limits_of<D, NRT, 2, 4>, limits_of<D, NRT, 4, 4>, limits_of<D, NRT, 1, 8>, limits_of<D, NRT, 4, 8>,
                                   limits_of<D, NRT, 8, 8>);
        if constexpr (D == 128) return rc ? rc : limits_of<D, NRT, 2, 8>();
        return rc;
    }();
    return err;
}

// which: bit 0 = sweep 1 (row statistics), bit 1 = sweep 2 (column sums)
template <int D, int NRT, int KS, int WAVES>
static int launch_sweeps(const ScoreParams& p_in, int which, hipStream_t st) {
    using G = Geo<bf16_t, D, NRT, KS, WAVES>;
    static_assert(G::LONGEST_PITCH >= (PITCH_END - 8) * 2, "a stage reaches all its rows at every pitch");
    ScoreParams p = p_in;
    p.n_query_blocks = (p.S + G::BLOCK - 1) / G::BLOCK;
    const unsigned grid = (unsigned)(p.H * p.n_query_blocks);  // as many key blocks
    if (which & 1) hipLaunchKernelGGL((rowstats_kernel<D, NRT, KS, WAVES>), dim3(grid), dim3(G::THREADS), G::LDS_ROWSTATS, st, p);
    if (which & 2) hipLaunchKernelGGL((colsum_kernel<D, NRT, KS, WAVES>), dim3(grid), dim3(G::THREADS), G::LDS_COLSUM, st, p);
    return (int)hipGetLastError();
}

// How many waves share resident rows (KS).  Large launches take 1: the fewest loads into LDS per flop (32K tokens, 32
// heads, d = 128: 4.04 / 4.50 / 5.46 ms a sweep for KS = 1 / 2 / 4).  With fewer than about two blocks per resident
// workgroup slot the launch is as long as its longest block, and smaller blocks win: by number n of 256-row blocks,
//   d = 128  n = 512 (4096 tokens, 32 heads) 89 / 87 / 108 us, n = 384 (6000, 16 heads) 101 / 86 / 94, n = 256 40 / 30 / 33,
//            n = 128 (1000, 32 heads) 22 / 15 / 14, n = 704 (5500, 32 heads) 134 / 136 / 161
//   d = 64   the vector work per logit weighs twice as much against the loads: n = 2048 (32K tokens, 16 heads) 1.26 / 1.34 /
//            1.50 ms, n = 756 (16000, 12 heads) 289 / 254 / 292 us, n = 240 (5000, 12 heads) 70 / 48 / 43, n = 96 30 / 19 / 16.5
// Without a causal mask all blocks are equally long, and a launch takes as many rounds of 1/KS as its KS n blocks fill the 256
// CUs: shares win only where they leave less of the last round empty, i.e. where 2 n fills an odd number of half rounds
// (rowstats, full attention, us for KS = 1 / 2 / 4; d = 128: n = 32 14 / 11 / 10, n = 128 21 / 16.4 / 18.4, n = 192 28.8 / 31.3 /
// 32.3, n = 256 39.5 / 42.4 / 50.7, n = 384 89.5 / 86.2 / 99.8, n = 448 107 / 122 / 133, n = 512 129 / 144 / 170, n = 576 199 / 194 /
// 213, n = 896 399 / 411 / 485; d = 64: n = 192 23.7 / 24.7 / 22.6, n = 256 30.4 / 30.9 / 35.9, n = 384 66 / 59 / 68, n = 512 88 / 97 /
// 110, n = 640 123 / 118 / 135, n = 768 190 / 204 / 232, n = 896 272 / 270 / 307).
//
// Workgroups of eight waves have a CU each, stages of 256 rows (half the barriers, and the loads of 256 rows serve all eight) and blocks of
// 512 / KS rows.  Under the mask a launch is as long as its longest block or as all of them over 256 CUs: many heads of few tokens are
// better off with the smaller blocks that two workgroups per CU take in turn.  Without a mask it takes as many rounds as its workgroups fill the CUs, and
// 513 to 640 tokens end in a stage that is half empty.  Both sweeps, time with eight waves / with four and the KS above, n = 256-row blocks:
//   d = 128, causal  KS = 8: n = 64 (512 tokens, 32 heads) 0.96, (16384, 1) 0.70, 96 (6000, 4) 0.79, (2000, 12) 0.93, (1500, 16) 0.97,
//                    112 (1949, 14) 0.94, (1792, 16) 1.01, 120 (1500, 20) 1.13, 128 (8192, 4) 0.85, (2048, 16) 1.02
//                    KS = 4: n = 160 (1280, 32) 0.86, 192 (1500, 32) 0.94, 216 (1323, 36) 1.11, 256 (4096, 16) 0.90, (2048, 32) 1.00, (1024, 64) 1.20
//                    KS = 2: n = 432 (2304, 48) 1.00, 448 (7168, 16) 0.93, (1846, 56) 1.08, 512 (8192, 16) 0.96, (2048, 64) 1.04
//                    KS = 1: n = 896 (7168, 32) 0.95, 980 (12345, 20) 0.98, 1024 (8192, 32) 0.98, (4096, 64) 1.04, 1008 (5376, 48: 528
//                    workgroups) 1.04
//   d = 64, causal   KS = 8: n = 64 (16384, 1) 0.71, (2048, 8) 0.80, 80 (1000, 20) 1.01, 112 (3584, 8) 0.84, 128 (4096, 8) 0.92, (2048, 16) 1.03
//                    KS = 4: n = 256 1.06
//   d = 128, full    KS = 8: n = 64 (16384, 1) 0.75, (1000, 16) 0.90, 60 (640, 20) 1.06, (641, 20) 0.93
//                    KS = 4: n = 96 (1500, 16) 0.87, (640, 32) 1.08, 128 (4096, 8) 0.87, (512, 64) 1.02
//                    KS = 2: n = 192 (3000, 16) 0.86, (640, 64) 1.06, 256 (4096, 16) 0.94
//                    KS = 1: n = 448 (7168, 16) 0.95, 512 (4096, 32) 0.95, 896 (7168, 32) 0.95, 1024 (8192, 32) 0.97, 1008 (2304, 112: 560
//                    workgroups) 1.29, (6254, 40: 520) 1.35
//   d = 64, full     KS = 8: n = 64 (16384, 1) 0.71, (1000, 16) 0.90, 60 (640, 20) 1.07;  KS = 4: n = 96 (3000, 8) 0.83, (640, 32) 1.09, 128 (4096,
//                    8) 0.81;  KS = 1: n = 448 (7168, 16) 0.93, 512 (8192, 16) 0.97, 1024 (8192, 32) 1.00, 1008 (2304, 112) 1.38
// Where rows are not shared either way only: whole rows add up less exactly.  Column sums of 16 heads of 64, relative 2-norm from 64 bits with
// KS = 2 / 1: 14336 tokens 7.4e-8 / 1.2e-6, 16384 7.1e-8 / 1.3e-6, 14336 without a mask 9.8e-8 / 4.0e-6.
template <int D, int NRT>
static int launch_sweeps_ks(const ScoreParams& p, long long n, int which, hipStream_t st) {
    const bool causal = (p.flags & LEMO_CAUSAL) != 0;
    if (p.S >= 512 && (causal || p.S == 512 || p.S > 640)) {
        const int longest = D == 128 ? 64 : 80;  // blocks of 64 rows for any length; beyond it, where the longest one decides
        if (n <= (causal ? longest : 64) || (causal && n <= 128 && (D == 128 ? p.H <= 14 : p.S >= 3000))) return launch_sweeps<D, NRT, 8, 8>(p, which, st);
        if (causal ? D == 128 && n > 128 && n <= 256 && p.H <= 32 : n <= 128) return launch_sweeps<D, NRT, 4, 8>(p, which, st);
        if constexpr (D == 128)
            if (causal ? n > 400 && n <= 512 && p.H <= 48 : n <= 256) return launch_sweeps<D, NRT, 2, 8>(p, which, st);
        const long long n512 = (long long)p.H * ((p.S + 511ll) / 512);  // workgroups with KS = 1
        const bool full_rounds = (!causal && n >= 448 && n512 <= 256) || (D == 128 && n >= 896 && n512 <= 512 && (!causal || p.H <= 48));
        if (p.S >= 2048 && full_rounds) return launch_sweeps<D, NRT, 1, 8>(p, which, st);
    }
    if (!causal) {
        if (n <= 64 || (D == 64 && n > 128 && n <= 192)) return launch_sweeps<D, NRT, 4, 4>(p, which, st);
        if ((2 * n + 255) / 256 % 2 == 1 && n <= (D > 64 ? 640 : 1024)) return launch_sweeps<D, NRT, 2, 4>(p, which, st);
        return launch_sweeps<D, NRT, 1, 4>(p, which, st);
    }
    if (n <= (D > 64 ? 128 : 256)) return launch_sweeps<D, NRT, 4, 4>(p, which, st);
    if (n <= (D > 64 ? 640 : 1024)) return launch_sweeps<D, NRT, 2, 4>(p, which, st);
    return launch_sweeps<D, NRT, 1, 4>(p, which, st);
}

int prepare_score(lemo_dtype_t dt, int d) {
    if (dt == LEMO_F32) return prepare_sweeps_f32(d);
    return d == 128 ? prepare_sweeps<128, 2>() : prepare_sweeps<64, 2>();
}

int launch_score(const ScoreParams& p_in, lemo_dtype_t dt, int d, int which, hipStream_t st) {
    ScoreParams p = p_in;
    p.order = head_order(p.H, (p.flags & LEMO_CAUSAL) != 0, 8);
    int rc = 0;
    const long long blocks256 = (long long)p.H * ((p.S + 255) / 256);
    if (which & 3) {
        rc = prepare_score(dt, d);
        if (rc) return rc;
        if (dt == LEMO_BF16 && d == 128) rc = launch_sweeps_ks<128, 2>(p, blocks256, which, st);
        else if (dt == LEMO_BF16 && d == 64) rc = launch_sweeps_ks<64, 2>(p, blocks256, which, st);
        else if (dt == LEMO_F32 && (d == 64 || d == 128)) rc = launch_sweeps_f32(p, d, which, st);
        else return (int)hipErrorInvalidValue;
        if (rc) return rc;
    }
    if (which & 4) {
        hipLaunchKernelGGL(head_mean_kernel, dim3((p.S + HM_THREADS - 1) / HM_THREADS), dim3(HM_THREADS), 0, st, p.colsum, p.diag, p.scores, p.S, p.H,
                           (p.flags & LEMO_EXCLUDE_SELF) ? 1 : 0);
        rc = (int)hipGetLastError();
    }
    return rc;
}

}  // namespace lemo
