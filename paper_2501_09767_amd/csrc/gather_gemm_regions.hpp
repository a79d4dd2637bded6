// Loads, LDS layout and fragments of the selective-load GEMM kernels with workgroups of eight waves (bf16): an operand's slab
// (128 bytes of the contraction) comes in regions of 128 rows, 16 KB each, filled by LDS-direct loads.
#pragma once
#include "gather_gemm.hpp"

namespace lemo {

constexpr int RG_WAVES = 8, RG_THREADS = 64 * RG_WAVES;
constexpr int RG_KB = 128;                            // bytes of the contraction per slab
constexpr int RG_KROWS = RG_KB / 2;                   // rows of a contraction-major slab
constexpr int RG_BYTES = 128 * RG_KB;                 // a region: 128 rows of 128 bytes, or 64 contraction rows of 256 bytes
constexpr int RG_NLD = RG_BYTES / (16 * RG_THREADS);  // loads per thread and region
constexpr int RG_TOK = RG_WAVES * 1024;               // (GG_TN) token rings: per wave 4 slabs of 64 indices

// The loads of one thread.  Unit u = i * 512 + tid of a region is its LDS bytes [16 u, 16 u + 16); the lane asks for the piece
// that belongs there.  Rows along the contraction, 8 pieces: piece p of row r at p ^ (r / 2 % 8), so that one piece of 16 rows meets
// all banks.  Contraction-major rows, 16 pieces of 8 columns: at p ^ kswz(r); a half-wave of a transposing read takes rows 0-3
// and 8-11 (+ 4, + 16), two pieces each.  The range check (raw_rsrc): rows past an operand's end
// fail it (or are clamped to the last one, A), pieces past the end of the contraction are given an offset at the descriptor's
// size in both operands and arrive as zeros; the scalar offset moves along a row, whose valid pieces pass with it.
__device__ __forceinline__ constexpr int rg_kswz(int r) { return ((r & 3) | ((r >> 3) & 1) << 2) << 1; }

// Load u of an operand: rows (columns) 64 u .. + 63; contraction-major, half u % 2 of the contraction rows of region u / 2.
template <int LAYOUT, int UA, int UB> struct RgLoads {  // the tile's rows of A, of B, / 64
    static_assert((LAYOUT != GG_TN || UA % 2 == 0) && (LAYOUT == GG_NT || UB % 2 == 0), "contraction-major operands come in whole regions");
    static constexpr bool A_KMAJOR = LAYOUT == GG_TN, B_KMAJOR = LAYOUT != GG_NT;
    const bf16_t *a_base, *b_base;
    const int* idx;
    unsigned lda_bytes, ldb_bytes, a_size, b_size, a_cols, b_cols;
    int K, nk, kpos, krow;
    unsigned a_voff[UA], b_voff[UB], tok[LAYOUT == GG_TN ? RG_NLD : 1];
    const char* ring;
    unsigned lds_ring;
    u32x4 idx_rsrc;

    // token_ring: the wave's 1 KB of LDS
    __device__ __forceinline__ RgLoads(const GgParams& p, long long m0, int n0, int tid, const char* token_ring) {
        lda_bytes = (unsigned)p.lda * 2;  // host: both < 2^23
        ldb_bytes = (unsigned)p.ldb * 2;
        K = p.K;
        nk = (K + RG_KROWS - 1) / RG_KROWS;
        idx = p.idx;
        kpos = ((tid & 7) ^ ((tid >> 4) & 7)) * 16;
        krow = tid >> 4;
        const int kcol = ((tid & 15) ^ rg_kswz(krow)) * 16;
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            if constexpr (A_KMAJOR) {
                a_voff[u] = (u % 2 * (RG_THREADS / 16) + krow) * lda_bytes + u / 2 * 256 + kcol;
            } else {
                const long long m = min(m0 + u * (RG_THREADS / 8) + (tid >> 3), p.M - 1);
                a_voff[u] = (p.idx ? (unsigned)p.idx[m] : (unsigned)m) * lda_bytes + kpos;
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            if constexpr (LAYOUT == GG_NT) b_voff[u] = (u * (RG_THREADS / 8) + (tid >> 3)) * ldb_bytes + kpos;
            else if constexpr (LAYOUT == GG_NN) b_voff[u] = (u % 2 * (RG_THREADS / 16) + krow) * ldb_bytes + u / 2 * 256 + kcol;
            else b_voff[u] = (unsigned)n0 * 2 + u / 2 * 256 + kcol;  // + the token's row, per slab
        }
        a_base = static_cast<const bf16_t*>(p.A) + (A_KMAJOR ? m0 : 0ll);
        b_base = static_cast<const bf16_t*>(p.B) + (LAYOUT == GG_NT ? (long long)n0 * p.ldb : LAYOUT == GG_NN ? (long long)n0 : 0ll);
        a_size = p.a_bytes;
        b_size = LAYOUT == GG_NT ? (min(64 * UB, p.N - n0) - 1) * ldb_bytes + K * 2 : p.b_bytes;  // GG_NT: this tile's rows of B
        a_cols = (unsigned)(p.M - m0);
        b_cols = (unsigned)(p.N - n0);
        ring = token_ring;
        lds_ring = __builtin_amdgcn_readfirstlane(lds_offset_of(token_ring));
        idx_rsrc = raw_rsrc(p.idx, p.idx ? (long long)K * 4 : 0);
    }
    struct Slab { u32x4 a, b; int soff; bool in_k; };
    // contraction-major operand: from the slab's first row (and the tile's first column) to the operand's end, which refuses
    // the rows past it (host: the operand spans < 2^31 bytes)
    __device__ __forceinline__ u32x4 kmajor_rsrc(const bf16_t* col0, unsigned ld_bytes, unsigned cols, int kt) const {
        const bool live = kt < nk;
        const unsigned off = live ? (unsigned)(kt * RG_KROWS) * ld_bytes : 0u;
        const unsigned size = live ? (unsigned)(K - 1) * ld_bytes + cols * 2 - off : 0u;
        return raw_rsrc(reinterpret_cast<const char*>(col0) + off, size);
    }
    __device__ __forceinline__ Slab slab(int kt) const {
        Slab s;
        s.soff = kt * RG_KB;
        s.in_k = kpos < K * 2 - s.soff;
        s.a = A_KMAJOR ? kmajor_rsrc(a_base, lda_bytes, a_cols, kt) : raw_rsrc(a_base, a_size);
        s.b = LAYOUT == GG_NN ? kmajor_rsrc(b_base, ldb_bytes, b_cols, kt) : raw_rsrc(b_base, b_size);
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // uniform values; the assembly wants them in scalar registers
            s.a[e] = __builtin_amdgcn_readfirstlane(s.a[e]);
            s.b[e] = __builtin_amdgcn_readfirstlane(s.b[e]);
        }
        return s;
    }
    // load u; lds: the operand's first region + 1024 * wave
    __device__ __forceinline__ void load_a(const Slab& s, int u, unsigned lds) const {
        if constexpr (A_KMAJOR) lds_direct_b128(s.a, lds + u * (RG_THREADS * 16), (int)a_voff[u]);
        else lds_direct_b128(s.a, lds + u * (RG_THREADS * 16), (int)(s.in_k ? a_voff[u] : a_size), s.soff);
    }
    __device__ __forceinline__ void load_b(const Slab& s, int u, unsigned lds) const {
        if constexpr (LAYOUT == GG_TN) lds_direct_b128(s.b, lds + u * (RG_THREADS * 16), (int)(tok[u % 2] == b_size ? tok[u % 2] : tok[u % 2] + b_voff[u]));
        else if constexpr (LAYOUT == GG_NN) lds_direct_b128(s.b, lds + u * (RG_THREADS * 16), (int)b_voff[u]);
        else lds_direct_b128(s.b, lds + u * (RG_THREADS * 16), (int)(s.in_k ? b_voff[u] : b_size), s.soff);
    }
    // (GG_TN) indices of slab kt into the wave's ring; the rows of B of slab kt, which load_b then takes
    __device__ __forceinline__ void issue_tokens(int kt, int lane) const {
        if constexpr (LAYOUT == GG_TN) lds_direct_b32(idx_rsrc, lds_ring + (kt & 3) * 256, kt * (RG_KROWS * 4) + lane * 4);
    }
    __device__ __forceinline__ void read_tokens(int kt) {
        if constexpr (LAYOUT == GG_TN) {
#pragma unroll
            for (int i = 0; i < RG_NLD; ++i) {
                const int kr = i * (RG_THREADS / 16) + krow, k = kt * RG_KROWS + kr;
                const unsigned row = idx ? *reinterpret_cast<const unsigned*>(ring + (kt & 3) * 256 + kr * 4) : (unsigned)k;
                tok[i] = k < K ? row * ldb_bytes : b_size;  // (a row past the end: at the descriptor's size whatever the column)
            }
        }
    }
};

// MFMA operands (16 x 16 x 32): a lane holds row lane % 16 of a 16-row tile, elements 8 (lane / 16) .. + 7 of a chunk of 32.
// Fragment of tile t of a region, chunk c of the slab; the transposing read: see gather_gemm.hpp.
__device__ __forceinline__ u32x4 rg_fragment(const char* region, bool kmajor, int t, int c, int lane) {
    const int l16 = lane & 15, quad = lane >> 4;
    if (!kmajor) return *reinterpret_cast<const u32x4*>(region + t * 16 * RG_KB + l16 * RG_KB + (((4 * c + quad) ^ ((l16 >> 1) & 7)) << 4));
    const int row = 8 * quad + (l16 >> 2);
    const char* at = region + row * 256 + (lane & 1) * 8 + c * 32 * 256 + (((t * 2 + ((lane & 3) >> 1)) ^ rg_kswz(row)) << 4);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at + 4 * 256));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    return u32x4{l2.x, l2.y, h2.x, h2.y};
}
__device__ __forceinline__ void rg_mma(f32x4& acc, const u32x4& a, const u32x4& b) {
    // the operands exchanged: a lane holds one row of the output (row lane % 16 of A's tile), columns 4 (lane / 16) .. + 3 of B's
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), acc, 0, 0, 0);
}
// no access to LDS moves across; every wave has come this far
__device__ __forceinline__ void rg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace lemo
