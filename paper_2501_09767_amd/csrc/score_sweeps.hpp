// What the two scoring sweeps share in bf16 (score.hip) and binary32 (score_f32.hip): geometry of a workgroup, stage loads, and the
// statistics of a 32 x 32 logit tile in slices that fit between MFMAs.
#pragma once
#include "lemo_common.hpp"

namespace lemo {

// Geometry of one instantiation.  NRT = 32-row MFMA subtiles of the RESIDENT operand a wave keeps in registers:
//   NRT = 2  64 resident rows per wave, 256 per workgroup, two workgroups per CU (two waves per SIMD)
//   NRT = 4  (not built any more) 128 resident rows per wave, 512 per workgroup, one workgroup per CU: every LDS fragment read feeds
//            four MFMA chains instead of two (half the LDS traffic per flop), but a SIMD then has no second wave
//            to run while the first waits at a barrier or on LDS
// Measured on the 32K-token bf16 d=128 layer: NRT = 2 4.20 / 4.25 ms (sweep 1 / sweep 2), NRT = 4 4.45 / 4.57 ms; with
// the stages filled by LDS-direct loads NRT = 2 4.06 ms (sweep 1) against 4.93 ms for NRT = 4 (4.23 ms when NRT = 4 is
// squeezed into half the register file for two workgroups per CU).
//
// KS = waves that share resident rows: KS consecutive waves hold the same rows and take every stage's streamed subtiles
// in shares; their statistics are put together through LDS at the end.  A block is then 1/KS as many rows and takes 1/KS
// as long, at KS times the loads into LDS per flop.
// WAVES = 4, or 8: one workgroup per CU where there are few, and stages of twice the rows.
template <typename T, int D, int NRT_, int KS_, int WAVES_> struct Geo {
    static constexpr int NRT = NRT_, KS = KS_, WAVES = WAVES_, THREADS = 64 * WAVES;
    static constexpr int RES = 32 * NRT;             // resident rows per wave
    static constexpr int BLOCK = WAVES / KS * RES; // resident rows per workgroup
    static constexpr int ROWB = D * (int)sizeof(T);  // bytes per head row
    static constexpr int NCH = ROWB / 32;            // MFMA chunks per row
    static constexpr int CPR = ROWB / 16;            // 16-byte pieces per row
    // LDS rows are not padded (LDS-direct loads fill consecutive bytes): piece p of row r sits at position p ^ swz(r),
    // which spreads any one piece of 16 consecutive rows over 16 distinct bank groups
    static constexpr int STRIDE = ROWB;
    __device__ static constexpr int swz(int row) { return CPR >= 16 ? (row & 15) : ((row >> 1) & (CPR - 1)); }
    // byte offset inside a stage of the fragment piece (chunk c, half) of row `row`
    __device__ static constexpr int frag(int row, int c, int half) { return row * ROWB + (((2 * c + half) ^ swz(row)) << 4); }
    static constexpr int TILE = (ROWB > 256 ? 16 : 32) * WAVES;  // streamed rows per LDS stage (two stages; long enough to hide a global load)
    static constexpr int NSUB = TILE / 32;           // 32-row MFMA subtiles per stage
    static constexpr int SHARE = NSUB / KS;          // of them, those a wave takes
    static constexpr int NLOAD = TILE * CPR / THREADS;  // 16-byte global loads per thread per stage
    static constexpr int ROWS_PER_LOAD = THREADS / CPR; // rows covered by one load of the whole workgroup
    static constexpr int STAGE_BYTES = TILE * STRIDE;
    // Longest pitch of a streamed token, in bytes: stage_offsets and stage_desc have 31 bits, and a row beyond arrives as zeros
    static constexpr long long LONGEST_PITCH = (0x7fffffffLL - ROWB) / (TILE - 1);
    static constexpr int MERGE_BYTES = KS > 1 ? WAVES * RES * 16 : 0;  // two floats per half-wave and resident row
    static constexpr int REF_BYTES = KS > 1 ? WAVES * RES * (int)sizeof(float) : 0;  // a share's maximum of the first stage per row
    static constexpr int LDS_ROWSTATS = 2 * STAGE_BYTES + MERGE_BYTES + REF_BYTES;
    static constexpr int LDS_COLSUM = 2 * STAGE_BYTES + 2 * TILE * (int)sizeof(float) + MERGE_BYTES;
    static constexpr int MIN_WG = WAVES > 4 ? 2 : (ROWB * NRT > 512 || NRT > 2) ? 1 : ROWB > 128 ? 2 : 3;  // waves per SIMD the register budget is set for
    static_assert(TILE * CPR % THREADS == 0, "tile must split evenly over the workgroup");
    static_assert(KS == 1 || (BLOCK <= TILE && NLOAD * BLOCK % TILE == 0), "shared rows are loaded through one stage");
    static_assert(WAVES % KS == 0 && NSUB % KS == 0, "the shares must be whole subtiles");
};

constexpr long long PITCH_END = 1 << 22;  // token pitches are below this many elements, whole 16-byte pieces (host: check_qk)

// 16 bytes at byte offset `byte_off` of row `row` of a [rows, heads, D] tensor, zero beyond `nrows`
template <typename T>
__device__ __forceinline__ u32x4 load_piece(const T* base, long long tok_stride, long long head_off, int row, int nrows, int byte_off) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row < nrows) v = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base + (long long)row * tok_stride + head_off) + byte_off);
    return v;
}

// Stage loads: LDS-direct (no staging registers, no LDS write instructions).  Unit u = i * THREADS + tid of a stage is
// its LDS bytes [16u, 16u + 16) = row u / CPR, position u % CPR; the lane fetches the piece that belongs there.  The
// loads go through a buffer descriptor rebuilt per stage (wave-uniform base = first row of the stage, size = bytes up to
// the end of the last valid row), so pieces of rows beyond the end of the tensor arrive as zeros.
template <typename G>
__device__ __forceinline__ void stage_offsets(int (&voff)[G::NLOAD], int row_bytes, int tid) {
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
        const int u = i * G::THREADS + tid, row = u / G::CPR, piece = (u % G::CPR) ^ G::swz(row);
        voff[i] = row * row_bytes + piece * 16;
    }
}
// descriptor of the stage that starts at row0 (length zero when !live: its loads then fetch nothing)
template <typename G>
__device__ __forceinline__ u32x4 stage_desc(const char* head, int row_bytes, int row0, int nrows, bool live) {
    const long long span = (long long)(nrows - row0 - 1) * row_bytes + G::ROWB;  // bytes from row0 to the end of row nrows-1
    return raw_rsrc(head + (long long)row0 * row_bytes, !live ? 0 : span > 0x7fffffffLL ? 0x7fffffffLL : span);
}
// lds_stage: LDS byte offset of the stage plus 1024 * (wave index), wave-uniform
template <typename G>
__device__ __forceinline__ void stage_load(const int (&voff)[G::NLOAD], u32x4 rsrc, unsigned lds_stage) {
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) lds_direct_b128(rsrc, lds_stage + i * (G::THREADS * 16), voff[i]);
}
// the share of pipeline slot `ti` of `nslots`: issued one slot at a time, the loads do not queue up behind each other
// in the CU's vector-memory pipe (16 cycles per 1 KB instruction) while the wave stands still
template <typename G>
__device__ __forceinline__ void stage_load_slot(const int (&voff)[G::NLOAD], u32x4 rsrc, unsigned lds_stage, int ti, int nslots) {
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i)
        if (i >= ti * G::NLOAD / nslots && i < (ti + 1) * G::NLOAD / nslots) lds_direct_b128(rsrc, lds_stage + i * (G::THREADS * 16), voff[i]);
}
// A wave's resident fragments (row `row0` of the block on), from the block's rows in an LDS stage of the same layout.  For waves
// that share rows: loaded straight from memory, 32 bytes of each of 32 rows at a time and by every sharer, the block's rows
// are 4096 line accesses of a CU (two workgroups, d = 128: 1.8 us of the 4.3 between the start and the first stage), as
// LDS-direct loads a quarter of that or less.  Both sweeps and the head mean, us before / now: bf16 d = 128 1000 tokens, 32 heads 29.2 /
// 25.9, 2048 60.1 / 57.4, 4096 174 / 171; d = 64 2048 tokens, 16 heads 35.1 / 33.2; binary32 d = 64 5000 tokens, 16 heads 318 / 307.
template <typename G>
__device__ __forceinline__ void load_resident(const char* head, int row_bytes, int first, int nrows, unsigned lds_stage, int tid) {
    int voff[G::NLOAD];
    stage_offsets<G>(voff, row_bytes, tid);
    const u32x4 desc = stage_desc<G>(head, row_bytes, first, nrows, true);
#pragma unroll
    for (int i = 0; i < G::NLOAD * G::BLOCK / G::TILE; ++i) lds_direct_b128(desc, lds_stage + i * (G::THREADS * 16), voff[i]);
}
// before the barrier that ends a stage: this wave's loads of the next stage have landed, its reads of this one returned
__device__ __forceinline__ void stage_settle() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_waitcnt(LGKMCNT0);
}
// the NCH fragments of one 32-row subtile of a stage
template <typename G>
__device__ __forceinline__ void read_frags(u32x4 (&f)[G::NCH], const char* sbuf, int sub, int l32, int half) {
#pragma unroll
    for (int c = 0; c < G::NCH; ++c) f[c] = *reinterpret_cast<const u32x4*>(&sbuf[G::frag(sub * 32 + l32, c, half)]);
}

// The scheduler may not move anything across this point: the source order of the pipeline slots below
// (a share of the carried tile's vector work, then the next MFMAs) is the order the wave issues them in.
__device__ __forceinline__ void slot_fence() { __builtin_amdgcn_sched_barrier(0); }

// Online softmax update of one query's (m, l) with the 16 logits a lane holds of one tile, cut into NS
// slices so that it can be issued between the MFMAs of the next tile.  `raw` are unscaled dot products
// (-inf = masked, or "no tile at all"); everything stays finite-safe when all inputs so far are -inf.
struct RowStat {
    float mn, ms, sum0, sum1, corr;
};
template <int NS>
__device__ __forceinline__ void rowstat_slice(int c, const f32x16& raw, float c2, float m, RowStat& st) {
    if (c == 0) {
        float t0 = fmaxf(fmaxf(raw[0], raw[1]), raw[2]);  // v_max3_f32
        float t1 = fmaxf(fmaxf(raw[3], raw[4]), raw[5]);
        float t2 = fmaxf(fmaxf(raw[6], raw[7]), raw[8]);
        float t3 = fmaxf(fmaxf(raw[9], raw[10]), raw[11]);
        float t4 = fmaxf(fmaxf(raw[12], raw[13]), raw[14]);
        t0 = fmaxf(fmaxf(t0, t1), t2);
        t3 = fmaxf(fmaxf(t3, t4), raw[15]);
        st.mn = fmaxf(m, fmaxf(t0, t3) * c2);
        st.ms = st.mn == -INFINITY ? 0.f : st.mn;  // nothing seen yet: keep the exp2 arguments finite
        st.corr = __builtin_amdgcn_exp2f(m - st.ms);
        st.sum0 = 0.f;
        st.sum1 = 0.f;
    } else {
        const int lo = (c - 1) * 16 / (NS - 1), hi = c * 16 / (NS - 1);
#pragma unroll
        for (int r = lo; r < hi; ++r) {
            const float e = __builtin_amdgcn_exp2f(fmaf(raw[r], c2, -st.ms));
            if (r & 1) st.sum1 += e; else st.sum0 += e;
        }
    }
}
__device__ __forceinline__ void rowstat_finish(const RowStat& st, float& m, float& l) {
    l = fmaf(l, st.corr, st.sum0 + st.sum1);
    m = st.mn;
}
// the whole update at once (masked tiles, pipeline drain)
__device__ __forceinline__ void rowstat_update(const f32x16& raw, float c2, float& m, float& l) {
    RowStat st;
#pragma unroll
    for (int c = 0; c < 8; ++c) rowstat_slice<8>(c, raw, c2, m, st);
    rowstat_finish(st, m, l);
}
// The same sum against a FROZEN reference m (no maximum search, no rescaling): exact for any finite m that no logit exceeds
// by too much, which the caller checks before it rescales the sum.  Slice c of NS covers elements [c*16/NS, (c+1)*16/NS).
template <int NS>
__device__ __forceinline__ void rowstat_frozen_slice(int c, const f32x16& raw, float c2, float neg_m, float& s0, float& s1) {
    const int lo = c * 16 / NS, hi = (c + 1) * 16 / NS;
#pragma unroll
    for (int r = lo; r < hi; ++r) {
        const float e = __builtin_amdgcn_exp2f(fmaf(raw[r], c2, neg_m));
        if (r & 1) s1 += e; else s0 += e;
    }
}

// What a sum against a frozen reference may reach before it is rescaled.  A later or another lane's reference brings it down by
// a factor that underflows 126 base-2 units on (the exponential flushes results below 2^-126 to zero); what that drops of a
// smaller sum is below 2^(90-126) of a total that is at least 1 (the largest reference is some key's own logit), far under
// a binary32 rounding for all partial sums of a row together.
constexpr float FROZEN_LIMIT = 0x1p90f;
__device__ __forceinline__ float frozen_sum(float l) { return l >= FROZEN_LIMIT ? INFINITY : l; }  // (NaN stays)
// m + log2(l), rounded once.  v_log_f32 cuts off rather than rounds (mean error half a unit in its last place: -2.3e-7 for l
// of 16 to 64), which every column sum of the row would see; one step of Newton's method gives what it leaves out.
__device__ __forceinline__ float add_log2(float m, float l) {
    const float y = __builtin_amdgcn_logf(l), s = m + y;
    if (!isfinite(s)) return s;
    const float rest = (fmaf(l, __builtin_amdgcn_exp2f(-y), -1.f)) * 1.44269504f;  // log2(l) - y
    const float mm = s - y, lost = (m - mm) + (y - (s - mm));                      // m + y - s
    return s + (lost + rest);
}

// sum over the 16 probabilities a lane holds of one tile, p = exp2(raw * c2 + nl) with nl = -lse2 of the
// row; slice c of NS covers elements [c*16/NS, (c+1)*16/NS) and adds into two partial sums
template <int NS>
__device__ __forceinline__ void colsum_slice(int c, const f32x16& raw, const float (&nl)[16], float c2, float& s0, float& s1) {
    const int lo = c * 16 / NS, hi = (c + 1) * 16 / NS;
#pragma unroll
    for (int r = lo; r < hi; ++r) {
        const float e = __builtin_amdgcn_exp2f(fmaf(raw[r], c2, nl[r]));
        if (r & 1) s1 += e; else s0 += e;
    }
}
__device__ __forceinline__ float colsum_tile(const f32x16& raw, const float (&nl)[16], float c2) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) colsum_slice<8>(c, raw, nl, c2, s0, s1);
    return s0 + s1;
}
// -lse2 of the 16 query rows of subtile `sub` this lane meets (rows 8g + 4*half + 0..3)
__device__ __forceinline__ void read_nl(float (&nl)[16], const float* lbuf, int sub, int half) {
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&lbuf[sub * 32 + gq * 8 + half * 4]);
        nl[gq * 4 + 0] = v[0]; nl[gq * 4 + 1] = v[1]; nl[gq * 4 + 2] = v[2]; nl[gq * 4 + 3] = v[3];
    }
}

// The sums of the KS waves that share a key, from the first one's entry on: in pairs, then in pairs of those, so that eight shares round the whole
// sum once and not seven times.  Column sums, relative 2-norm from 64 bits, mean of 24 draws, one after the other /
// in pairs: eight shares 3000 tokens, 4 heads of 64 6.4e-8 / 5.1e-8, 1500, 8 of 128 6.6e-8 / 5.8e-8; four 6000, 8 of 128 5.8e-8 / 5.6e-8.
template <typename G>
__device__ __forceinline__ float2 add_shares(const float2* share) {
    float2 v[G::KS];
#pragma unroll
    for (int w = 0; w < G::KS; ++w) v[w] = share[w * G::RES];
#pragma unroll
    for (int step = 1; step < G::KS; step *= 2)
#pragma unroll
        for (int w = 0; w < G::KS; w += 2 * step) { v[w].x += v[w + step].x; v[w].y += v[w + step].y; }
    return v[0];
}

int prepare_sweeps_f32(int d);
int launch_sweeps_f32(const ScoreParams& p, int d, int which, hipStream_t st);  // score_f32.hip

}  // namespace lemo
