// Shared device-side vocabulary of the gfx950 kernels: MFMA fragment types, the 32x32 accumulator
// layout, bf16 conversion, and the parameter blocks the host entry points fill in.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

#include "lemo.h"

namespace lemo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;  // one 16-byte piece; a native vector, so copies are plain loads/stores

struct bf16_t { uint16_t bits; };  // storage tag for bfloat16 (upper half of a binary32)

constexpr int WAVE = 64;
constexpr int NUM_XCD = 8;  // MI355X: 8 accelerator dies, workgroup b is dispatched to die b % 8

// ---- one 32x32 MFMA "chunk": 32 bytes of the contraction axis per operand row ---------------------
// Every lane supplies 16 bytes per operand: lane l holds row (l % 32), bytes [16*(l/32), +16) of the
// chunk.  bf16: one v_mfma_f32_32x32x16_bf16 (16 elements).  fp32: four v_mfma_f32_32x32x2_f32, step t
// contracting element t of the lower half with element 4+t of the upper half; A and B use the same
// assignment, and a dot product does not care in which order its terms are paired off.
template <typename T> __device__ __forceinline__ void mma_chunk(f32x16& acc, const u32x4& a, const u32x4& b);

template <> __device__ __forceinline__ void mma_chunk<bf16_t>(f32x16& acc, const u32x4& a, const u32x4& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ void mma_chunk<float>(f32x16& acc, const u32x4& a, const u32x4& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// Accumulator layout of the 32x32 MFMAs (checked on hardware): register r of lane l is the element in
//   row = 8*(r/4) + 4*(l/32) + (r%4)   (A-operand row),   col = l % 32   (B-operand row).
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---- LDS-direct loads ----------------------------------------------------------------------------
// Every lane fetches 16 (or 4) bytes at its own byte offset `voff` (+ the wave-uniform `soff`) into the buffer; the
// wave's 64 pieces land in consecutive LDS bytes starting at the wave-uniform LDS byte offset `lds_off`.  No registers
// and no LDS write instructions are involved.  Written as assembly so that the compiler does not make every later LDS
// read wait for them; a kernel that uses them awaits completion itself (vmcnt, they complete in issue order) before
// the barrier that publishes the data, and makes sure (lgkmcnt) that its own reads of the target have returned before
// the barrier that releases it.  The LDS offset travels in M0, which is set inside the same statement that uses it (the
// compiler keeps no value of its own in M0 across statements).
__device__ __forceinline__ void lds_direct_b128(u32x4 rsrc, unsigned lds_off, int voff, int soff = 0) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void lds_direct_b32(u32x4 rsrc, unsigned lds_off, int voff, int soff = 0) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// Raw buffer descriptor over [base, base + bytes).  The range check takes the per-thread and the scalar offset together, without wrapping at
// 2^32 (seen on hardware: of 256 bytes, a scalar offset of 128 leaves the first eight 16-byte pieces; of none, none; at sizes and offsets just below 2^32
// likewise).  What it refuses reaches no memory and arrives as zeros, in LDS as well.
__device__ __forceinline__ u32x4 raw_rsrc(const void* base, long long bytes) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(base);
    u32x4 r;
    r[0] = (unsigned)a;
    r[1] = (unsigned)(a >> 32) & 0xffffu;
    r[2] = (unsigned)(bytes < 0xffffffffLL ? (bytes > 0 ? bytes : 0) : 0xffffffffLL);
    r[3] = 0x00020000u;
    return r;
}
// s_waitcnt immediates that wait on one counter only (gfx9 layout: vmcnt in bits 3:0 and 15:14, lgkmcnt in 11:8)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }
constexpr int lgkmcnt_imm(int n) { return n << 8 | 0xC07F; }
constexpr int LGKMCNT0 = lgkmcnt_imm(0);
// LDS byte offset of a pointer into the workgroup's LDS
__device__ __forceinline__ unsigned lds_offset_of(const void* p) { return (unsigned)reinterpret_cast<unsigned long long>(p); }

// ---- bf16 <-> binary32 ----------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bf16lo_to_f32(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// round to nearest, ties to even; NaN stays NaN (quiet)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) { return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16); }
// the same rounding done by the conversion instruction of gfx950 (v_cvt_pk_bf16_f32, nearest-even): one
// instruction for two values, used where conversions are on the critical path
__device__ __forceinline__ uint32_t pack_bf16x2_hw(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// ---- binary32 products on the bf16 matrix cores ---------------------------------------------------
// A binary32 value is the exact sum of three bf16 ones, each the rest rounded to nearest (below 2^-110 it may not be: SPLIT_WHOLE).
// Six of the nine products of two such sums are formed, the smallest first; the other three amount to at most 2^-24 of a product
// (a = b = 1.0038986), 2^-27.5 of it in the mean square over mantissas, with either sign, and the 32 x 32 x 16 MFMA adds 16
// products per rounding of the sum where the binary32 one adds 2.  16 times the rate for 6 products; splitting 8 values takes 44
// instructions.  (Cut off instead of rounded, the rests have their value's sign: scores were then up to twice as far from 64 bits.)
// Infinities do not survive this (infinity times a zero part).  Results that are not finite, or that feel what small values lose,
// have to be formed again with mma_chunk<float>.
struct Split8 { u32x4 part[3]; };  // 8 values in three parts, as MFMA operands
__device__ __forceinline__ void split_pair(Split8& s, int e, const u32x4& from) {  // values 2e and 2e + 1, elements 2 (e % 2) of `from` on
    float v0 = __uint_as_float(from[e % 2 * 2]), v1 = __uint_as_float(from[e % 2 * 2 + 1]);
#pragma unroll
    for (int part = 0; part < 3; ++part) {
        const uint32_t both = pack_bf16x2_hw(v0, v1);
        s.part[part][e] = both;
        v0 -= bf16lo_to_f32(both);
        v1 -= bf16hi_to_f32(both);
    }
}
__device__ __forceinline__ Split8 split_f32(const u32x4& lo, const u32x4& hi) {
    Split8 s;
#pragma unroll
    for (int e = 0; e < 4; ++e) split_pair(s, e, e < 2 ? lo : hi);
    return s;
}
// Bits of 2^-110: below it a value's last part may fall below bf16's smallest number, 2^-133 (the matrix cores take denormal
// numbers as they are), and up to 2^-134 of the value is lost.
constexpr unsigned SPLIT_WHOLE = 17u << 23;
// largest magnitude of the values that split_pair takes (NaN is passed over)
__device__ __forceinline__ void most_of_pair(float& most, int e, const u32x4& from) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(from[e % 2 * 2]), "v"(from[e % 2 * 2 + 1]));
}
constexpr int SPLIT_TERMS = 6;
__device__ __forceinline__ void mma_split(f32x16& acc, const Split8& a, const Split8& b, int term) {
    constexpr int ap[SPLIT_TERMS] = {2, 0, 1, 1, 0, 0}, bp[SPLIT_TERMS] = {0, 2, 1, 0, 1, 0};
    mma_chunk<bf16_t>(acc, a.part[ap[term]], b.part[bp[term]]);
}

// ---- workgroups of per-head kernels ---------------------------------------------------------------
// Block index -> (head, block rank).  Workgroup b runs on die b % 8; when the heads divide evenly a die gets a contiguous
// range of them (the query heads of one GQA group share the die's L2 with their KV head), otherwise (per_xcd = 0) blocks are
// dealt out over all dies: with 12 heads, two dies would be idle.  The heads are cut into groups as even as can be; the
// nblk blocks of a group's heads are walked rank by rank, so that the longest blocks of all of them start first and the
// group ends on short ones; then comes the next group.
struct HeadOrder { int per_xcd, groups; };
// Groups: blocks of equal length (no causal mask) gain nothing from the order and go head by head (dealt out: 8 at a time),
// which keeps the rows that a die streams in its L2.  Under the mask up to `limit` heads of a die are walked together.
// Score, 16384 tokens, 128 heads, us with 1 / 2 / 4 / 8 / 16 heads of a die together: causal 8293 / 7937 / 7815 / 7802 /
// 8395, full 14793 / 14832 / 15022 / 15462 / 16676; 8192 tokens, 32 heads, causal 616 / 573 / 541.  Attention, 3277 kept
// tokens, 128 / 8 heads of 64, causal: 277 / 273 / 260 / 248 / 239; 128-wide heads: see its launch.
inline HeadOrder head_order(int H, bool causal, int limit) {
    const int per_xcd = H % NUM_XCD == 0 ? H / NUM_XCD : 0;
    const int heads = per_xcd ? per_xcd : H, together = (causal ? limit : 1) * (per_xcd ? 1 : NUM_XCD);
    return {per_xcd, heads < (1 << 15) ? (heads + together - 1) / together : 1};  // (the products of decode_block fit 32 bits)
}
__device__ __forceinline__ void decode_block(HeadOrder o, int H, int nblk, int& h, int& rank) {
    const bool dealt = o.per_xcd == 0;
    const int x = dealt ? 0 : blockIdx.x % NUM_XCD, w = dealt ? blockIdx.x : blockIdx.x / NUM_XCD, heads = dealt ? H : o.per_xcd;
    int first = 0, width = heads;
    if (o.groups > 1) {  // group g holds heads [g * heads / groups, (g + 1) * heads / groups)
        const int g = ((w / nblk + 1) * o.groups - 1) / heads;
        first = g * heads / o.groups;
        width = (g + 1) * heads / o.groups - first;
    }
    const int r = w - first * nblk;
    rank = r / width;
    h = x * o.per_xcd + first + (r - rank * width);
}

// ---- host: do [a, a + a_bytes) and [b, b + b_bytes) share a byte? -----------------------------------
inline bool spans_meet(const void* a, long long a_bytes, const void* b, long long b_bytes) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + (uintptr_t)b_bytes && y < x + (uintptr_t)a_bytes;
}

// ---- host: dynamic-LDS limits -------------------------------------------------------------------------
// The limit of a kernel is raised once, which a stream capture cannot hold, and which kernel a call takes depends on its sizes: so
// an entry point raises the limits of all the kernels that calls of one type and head size may take in the first of them
// (prepare_...; function-local statics, safe between threads).
struct LdsLimit { const void* kernel; int bytes; };
inline int raise_lds_limits(std::initializer_list<LdsLimit> kernels) {
    for (const LdsLimit& k : kernels) {
        const hipError_t err = hipFuncSetAttribute(k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes);
        if (err != hipSuccess) return (int)err;
    }
    return 0;
}
template <typename... F> int first_error(F... prepare) {
    int rc = 0;
    ((rc = rc ? rc : prepare()), ...);
    return rc;
}

// ---- parameter blocks -----------------------------------------------------------------------------
struct ScoreParams {
    const void* Q;
    const void* K;
    int S, H, H_kv;
    long long q_ts, q_hs, k_ts, k_hs;  // element strides
    float c2;                          // scale * log2(e): logits are handled in base-2 units
    int n_query_blocks;                // blocks per head (of queries: sweep 1, of keys: sweep 2)
    HeadOrder order;
    unsigned flags;
    float* lse2;    // [H,S] base-2 log-sum-exp of every query row
    float* colsum;  // [H,S]
    float* diag;    // [H,S]
    float* scores;  // [S]
};

struct BlockParams {
    const void* Q;
    const void* K;
    int S, H, H_kv;
    long long q_ts, q_hs, k_ts, k_hs;  // element strides
    float c2;           // probabilities: scale * log2(e)
    float out_scale;    // probabilities: 1/H;  positive logits: scale / H
    unsigned flags;
    const float* lse2;  // [H,S] row statistics (probabilities only)
    float* tilemax;     // [nt32, nt32] maxima of the 32 x 32 tiles
    int nt32;           // ceil(S / 32)
    int nt;             // rectangles per side
    int count, per_xcd; // rectangles, of them on a die
};

// kernel launchers (defined next to their kernels; return hipError_t as int)
int launch_score(const ScoreParams& p, lemo_dtype_t dt, int d, int which, hipStream_t st);  // which: 1 row stats | 2 column sums | 4 head mean
int prepare_score(lemo_dtype_t dt, int d);  // (launch_score does so itself)
int launch_score_blocks(const BlockParams& p, lemo_dtype_t dt, int d, int mode, int b, float* score_blocks, float* token_blocks,
                        hipStream_t st);  // mode 0: probabilities (p.lse2 filled), 1: positive logits
int launch_select(const float* scores, int S, int L, int k, int* kept, hipStream_t st);
int launch_head_mean_select(const float* colsum, const float* diag, int S, int H, int exclude_self, int L, int k, float* scores, int* kept,
                            hipStream_t st);
int launch_empty(hipStream_t st);
int launch_issue_mix(int tiles, unsigned operand_seed, float* sink, int* waves_out, hipStream_t st);
int launch_block_mean(const float* token_blocks, int nb, float* out, hipStream_t st);
int launch_select_threshold(const float* token_blocks, int S, int b, float t_host, const float* t_dev, int* kept, int* kept_count,
                            hipStream_t st);
int launch_gather_gemm_dw(const void* dY, long long ldy, const void* X, long long S, long long ldx, const int* idx, long long M, void* dW,
                          long long lddw, int C, int N, void* workspace, hipStream_t st);
int prepare_gather_gemm_dw(lemo_dtype_t dt);
int launch_zero_matrix(void* p, long long pitch, int row_elems, int rows, lemo_dtype_t dt, hipStream_t st);  // pitch in elements
int launch_kept_attention(const void* Q, const void* K, const void* V, long long S, int H, int H_kv, int d, long long q_ts, long long q_hs,
                          long long k_ts, long long k_hs, long long v_ts, long long v_hs, const int* idx, long long M, float c2,
                          unsigned flags, void* O, long long o_ts, long long o_hs, void* workspace, hipStream_t st);
int launch_scatter(const void* G, long long ldg, const int* idx, long long M, void* dX, long long lddx, long long S,
                   int C, lemo_dtype_t g_dt, lemo_dtype_t dx_dt, int mode, hipStream_t st);
int launch_gather_gemm(const void* X, long long S, long long ldx, const int* idx, long long M, const void* W,
                       long long ldw, const void* bias, void* Y, long long ldy, int C, int N, lemo_dtype_t dt,
                       hipStream_t st);
int launch_gather_gemm_dx(const void* dY, long long ldy, long long M, const void* W, long long ldw, void* dX, long long lddx, long long out_rows,
                          const int* oidx, int C, int N, hipStream_t st);
int launch_gather_gemm_dw_direct(const void* dY, long long ldy, const void* X, long long S, long long ldx, const int* idx, long long M, void* dW,
                                 long long lddw, int C, int N, lemo_dtype_t dt, hipStream_t st);
int launch_gather_gemm_add(const void* X, long long S, long long ldx, const int* idx, long long M, const void* W,
                           long long ldw, const void* bias, void* R, long long ldr, long long out_rows, const int* oidx,
                           int C, int N, lemo_dtype_t dt, hipStream_t st);

}  // namespace lemo
