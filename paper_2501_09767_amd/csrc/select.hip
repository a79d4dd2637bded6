// Per-segment top-k (token-block elimination of Sec. 4.2 with a keep count instead of a threshold).
//
// One workgroup per segment.  The k-th largest score is found by an MSB-first radix select over the
// order-preserving uint32 image of the floats (digits of 11, 11 and 10 bits, LDS histogram), which ends early where the last
// digit's candidates are all kept or fit a wavefront; the kept set is
// then { key > pivot } plus the first (k - #greater) elements with key == pivot in index order, which
// is exactly "ties go to the lower index".  A block-wide prefix sum in index order gives every kept
// element its output slot, so the indices come out ascending without a sort.  Integer work only:
// bit-exact and deterministic.
//
// What bounds it: latency -- the launch, the scores' way from memory, then one barrier after the other.  us per launch
// (an empty one 1.85), four digits of 8 bits through shuffles / now: 1000 tokens, segments of 512 5.4 / 4.1; 32768, 1024 6.9 / 5.1 (all scores
// equal 9.5 / 7.2); 20000, 8192 27.5 / 7.7.
#include <mutex>

#include "lemo_common.hpp"

namespace lemo {

// monotone map float -> uint32 (larger float <=> larger key); -0.0 and +0.0 share a key
__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive prefix sum over the 64 lanes of a wave, on the data-parallel-primitives path: inside rows of 16 lanes, then across
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t plus_dpp(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    v = plus_dpp<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
    v = plus_dpp<0x112, 0xf>(v);
    v = plus_dpp<0x114, 0xf>(v);
    v = plus_dpp<0x118, 0xf>(v);
    v = plus_dpp<0x142, 0xa>(v);         // row_bcast:15 into rows 1 and 3
    return plus_dpp<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
}

// LDS of a selection by T threads.  A kernel clears it, fills keys and the histogram of their first digit (add) behind a barrier, and
// calls select_from_keys.
constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS, SEL_FIRST = 32 - SEL_BITS;
template <int T> struct SelectLds {
    uint32_t hist[SEL_BINS];
    uint32_t candidates[WAVE];
    uint32_t wave_total[T / WAVE];
    uint32_t prefix, need, count, n_candidates;
    __device__ __forceinline__ void clear(int tid) {
        for (int i = tid; i < SEL_BINS / 4; i += T) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void add(uint32_t key) { atomicAdd(&hist[key >> SEL_FIRST], 1u); }
};

// The selection proper, shared by the two kernels below: `keys` [len] (LDS) hold the order keys of one segment, the
// `keep` kept token indices go to kept[out0 ...) in ascending order.  T = threads of the workgroup;
// every thread of the workgroup must call it.  Scans run inside wavefronts with one pass through LDS for the wave totals.
template <int T>
__device__ __forceinline__ void select_from_keys(SelectLds<T>& lds, const uint32_t* keys, int len, int keep, long long out0, int start,
                                                 int* __restrict__ kept) {
    constexpr int BPT = SEL_BINS / T;  // digits per thread, in DESCENDING order: a prefix sum over threads is the suffix sum
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t prefix = 0u, himask = 0u, need = (uint32_t)keep;  // the pivot's known bits; how many are to be taken among those that share them
    for (int shift = SEL_FIRST;;) {
        __syncthreads();
        uint32_t c[BPT], sum = 0u;
#pragma unroll
        for (int b = 0; b < BPT; ++b) { c[b] = lds.hist[SEL_BINS - 1 - tid * BPT - b]; sum += c[b]; }
        uint32_t ge = wave_inclusive_scan(sum);
        if (lane == 63) lds.wave_total[wave] = ge;
        __syncthreads();
        for (int w = 0; w < wave; ++w) ge += lds.wave_total[w];
        if (ge - sum < need && need <= ge) {  // exactly one thread: one of its digits is the pivot's
            uint32_t gt = ge - sum;
#pragma unroll
            for (int b = 0; b < BPT; ++b) {
                if (gt < need && need <= gt + c[b]) {
                    lds.prefix = prefix | (uint32_t)(SEL_BINS - 1 - tid * BPT - b) << shift;
                    lds.need = need - gt;
                    lds.count = c[b];
                    lds.n_candidates = 0u;
                    need = 0u;  // (found)
                }
                gt += c[b];
            }
        }
        __syncthreads();
        prefix = lds.prefix;
        need = lds.need;
        const uint32_t count = lds.count;
        himask = 0xffffffffu << shift;
        if (shift == 0 || count == need) break;  // (all that share the known bits are kept)
        if (count <= WAVE) {  // every wave finds the pivot among the candidates by their ranks
            uint32_t mine = 0u;
            if (count == (uint32_t)len) {  // (a short segment, all in one digit: nothing to pick)
                if (lane < len) mine = keys[lane];
            } else {
                for (int t = tid; t < len; t += T)
                    if ((keys[t] & himask) == prefix) lds.candidates[atomicAdd(&lds.n_candidates, 1u)] = keys[t];
                __syncthreads();
                if ((uint32_t)lane < count) mine = lds.candidates[lane];
            }
            uint32_t gt = 0u;
            for (uint32_t j = 0; j < count; j += 4)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) gt += (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(j + e)) > mine;  // (zeros behind the last are above nothing)
            // the pivot is the least key with fewer than `need` above it, that is the one with the most above it
            uint32_t most = (uint32_t)lane < count && gt < need ? gt + 1 : 0u;
            const uint32_t own = most;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
            const int src = __ffsll((long long)__ballot(own == most)) - 1;
            prefix = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
            need -= (uint32_t)__builtin_amdgcn_readlane((int)gt, src);
            himask = 0xffffffffu;
            break;
        }
        shift = shift > SEL_BITS ? shift - SEL_BITS : 0;
        lds.clear(tid);
        __syncthreads();
        for (int t = tid; t < len; t += T) {
            const uint32_t key = keys[t];
            if ((key & himask) == prefix) atomicAdd(&lds.hist[(key & ~himask) >> shift], 1u);
        }
    }
    const uint32_t pivot = prefix;   // (the known bits of) the key of the k-th largest element
    const uint32_t need_eq = need;   // how many elements equal to the pivot are kept (lowest indices first)

    // compaction in index order: thread t owns the contiguous range [t*per, (t+1)*per)
    const int per = (len + T - 1) / T;
    const int lo = min(len, tid * per), hi = min(len, lo + per);
    uint32_t ngt = 0, neq = 0;
    for (int t = lo; t < hi; ++t) {
        const uint32_t key = keys[t] & himask;
        ngt += key > pivot;
        neq += key == pivot;
    }
    // len <= 32768 so both counts fit 16 bits, as do their prefix sums: one scan carries both
    uint32_t incl = wave_inclusive_scan(ngt | (neq << 16));
    if (lane == 63) lds.wave_total[wave] = incl;  // (everyone has read the totals of the last digit: a barrier ago)
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += lds.wave_total[w];
    uint32_t gt_before = (incl & 0xffffu) - ngt, eq_before = (incl >> 16) - neq;
    for (int t = lo; t < hi; ++t) {
        const uint32_t key = keys[t] & himask;
        if (key > pivot) {
            kept[out0 + gt_before + min(eq_before, need_eq)] = start + t;
            ++gt_before;
        } else if (key == pivot) {
            if (eq_before < need_eq) kept[out0 + gt_before + eq_before] = start + t;
            ++eq_before;
        }
    }
}

// tokens kept in a segment of length len when full segments of length L keep k
__device__ __forceinline__ int segment_keep(int len, int L, int k) {
    if (len == L) return k;
    const long long v = ((long long)k * len + L - 1) / L;
    return (int)max(1ll, min((long long)len, v));
}

// 512 threads, from segments of more than 2048 on 1024 (us with 256 / 512 / 1024: segments of 512 4.2 / 4.1 / 4.8, 1024 5.5 / 5.1 / 6.0, 8192
// 17.7 / 10.3 / 7.7), up to 128 tokens 256 (32768 tokens, us with 256 / 512: segments of 16 4.4 / 6.6, all scores equal 5.0 / 7.7; 64 3.6 / 3.8, 4.5 / 5.4; 128 3.6 /
// 3.6, 4.6 / 4.6; 256 4.0 / 4.0, 4.9 / 4.9)
template <int T>
__global__ __launch_bounds__(T) void select_topk_kernel(const float* __restrict__ scores, int S, int L, int k,
                                                                  int* __restrict__ kept) {
    extern __shared__ uint32_t keys[];  // [len]
    const int seg = blockIdx.x, tid = threadIdx.x;
    const int start = seg * L;  // host guarantees start < S and no overflow
    const int len = min(L, S - start);
    __shared__ __attribute__((aligned(16))) SelectLds<T> lds;
    float ahead = tid < len ? scores[start + tid] : 0.f;  // on its way while the histogram is cleared
    lds.clear(tid);
    __syncthreads();
    for (int t = tid; t < len; t += T) {
        const uint32_t key = order_key(ahead);
        if (t + T < len) ahead = scores[start + t + T];
        keys[t] = key;
        lds.add(key);
    }
    select_from_keys<T>(lds, keys, len, segment_keep(len, L, k), (long long)seg * k /* every earlier segment is full */, start, kept);
}

// Head mean and selection in one launch (one workgroup per segment): the segment's [H, len] slab of per-head column
// sums and diagonals is read once, coalesced along the tokens, the heads are added in ascending order exactly as
// head_mean_kernel adds them (same bits), the scores are written out and their order keys go straight to LDS for the
// selection.  Saves one launch and the round trip of the scores through memory.
constexpr int FUSED_THREADS = 1024;
__global__ __launch_bounds__(FUSED_THREADS) void head_mean_select_kernel(const float* __restrict__ colsum, const float* __restrict__ diag,
                                                                         int S, int H, int exclude_self, int L, int k,
                                                                         float* __restrict__ scores, int* __restrict__ kept) {
    extern __shared__ uint32_t keys[];  // [len]
    const int seg = blockIdx.x, tid = threadIdx.x;
    const int start = seg * L;
    const int len = min(L, S - start);
    __shared__ __attribute__((aligned(16))) SelectLds<FUSED_THREADS> lds;
    lds.clear(tid);
    for (int t = tid; t < len; t += FUSED_THREADS) {
        const float* c = colsum + start + t;
        const float* g = diag + start + t;
        float acc = 0.f;
        int h = 0;
        for (; h + 8 <= H; h += 8) {  // eight heads' loads in flight at a time; the additions stay in head order
            float cv[8], gv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) cv[u] = c[(size_t)(h + u) * S];
            if (exclude_self) {
#pragma unroll
                for (int u = 0; u < 8; ++u) gv[u] = g[(size_t)(h + u) * S];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float v = cv[u];
                if (exclude_self) v -= gv[u];
                acc += v;
            }
        }
        for (; h < H; ++h) {
            float v = c[(size_t)h * S];
            if (exclude_self) v -= g[(size_t)h * S];
            acc += v;
        }
        const float sc = acc / (float)H;
        scores[start + t] = sc;
        keys[t] = order_key(sc);
    }
    __syncthreads();
    for (int t = tid; t < len; t += FUSED_THREADS) lds.add(keys[t]);
    select_from_keys<FUSED_THREADS>(lds, keys, len, segment_keep(len, L, k), (long long)seg * k, start, kept);
}

// nothing: the cost of one launch on a stream (what the microsecond-sized steps of the path are measured against)
__global__ void empty_kernel() {}

// ------------------------------------------------------------------------------------------------
// Threshold selection over token blocks (Sec. 4.2 "Layer-specific Threshold"; Alg. 1 step 1).
// ------------------------------------------------------------------------------------------------

// mean of the token-block scores: one workgroup, per-thread partial sums in index order, fixed-order tree
__global__ __launch_bounds__(256) void block_mean_kernel(const float* __restrict__ token_blocks, int nb, float* __restrict__ out) {
    __shared__ float part[256];
    const int tid = threadIdx.x;
    float s = 0.f;
    for (int n = tid; n < nb; n += 256) s += token_blocks[n];
    part[tid] = s;
    __syncthreads();
    for (int k = 128; k >= 1; k >>= 1) {
        if (tid < k) part[tid] += part[tid + k];
        __syncthreads();
    }
    if (tid == 0) out[0] = part[0] / (float)nb;
}

// One workgroup.  Phase 1: start[n] = number of kept tokens in blocks before n (prefix sum over the kept blocks'
// lengths, carried from chunk to chunk of 1024 blocks).  Phase 2: every token of a kept block writes its own index.
// The scan is one inside the wavefronts and a pass over their totals (us, twenty barriers of a scan through LDS / now: 64 blocks of 64
// 3.7 / 2.4, 1024 of 32 8.7 / 7.4).
constexpr int THR_THREADS = 1024;
__global__ __launch_bounds__(THR_THREADS) void select_threshold_kernel(const float* __restrict__ token_blocks, int S, int b, int nb,
                                                                       float t_host, const float* __restrict__ t_dev,
                                                                       int* __restrict__ kept, int* __restrict__ kept_count) {
    extern __shared__ int start[];  // [nb]; -1 marks a dropped block
    __shared__ int wave_total[THR_THREADS / WAVE];
    const int tid = threadIdx.x, wave = tid / WAVE;
    const float T = t_dev ? t_dev[0] : t_host;
    int base = 0;
    for (int n0 = 0; n0 < nb; n0 += THR_THREADS) {
        const int n = n0 + tid;
        int len = 0;
        if (n < nb && token_blocks[n] >= T) len = min(b, S - n * b);
        const int incl = (int)wave_inclusive_scan((uint32_t)len);
        if (tid % WAVE == WAVE - 1) wave_total[wave] = incl;
        __syncthreads();
        int before = base;
#pragma unroll
        for (int w = 0; w < THR_THREADS / WAVE; ++w) {
            if (w < wave) before += wave_total[w];
            base += wave_total[w];
        }
        if (n < nb) start[n] = len ? before + incl - len : -1;
        __syncthreads();  // (the totals have been read; behind the last chunk: the starts are complete)
    }
    if (tid == 0) kept_count[0] = base;
    for (int j = tid; j < S; j += THR_THREADS) {
        const int n = j / b;
        if (start[n] >= 0) kept[start[n] + (j - n * b)] = j;
    }
}

int launch_block_mean(const float* token_blocks, int nb, float* out, hipStream_t st) {
    hipLaunchKernelGGL(block_mean_kernel, dim3(1), dim3(256), 0, st, token_blocks, nb, out);
    return (int)hipGetLastError();
}

int launch_select_threshold(const float* token_blocks, int S, int b, float t_host, const float* t_dev, int* kept, int* kept_count,
                            hipStream_t st) {
    const int nb = (S + b - 1) / b;  // host checked: nb <= 16384
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {  // 16384 block offsets are 64 KB of dynamic LDS on top of the kernel's static 64 bytes: above the default limit
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_threshold_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 4);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    hipLaunchKernelGGL(select_threshold_kernel, dim3(1), dim3(THR_THREADS), (size_t)nb * sizeof(int), st, token_blocks, S, b, nb, t_host,
                       t_dev, kept, kept_count);
    return (int)hipGetLastError();
}

int launch_empty(hipStream_t st) {
    hipLaunchKernelGGL(empty_kernel, dim3(1), dim3(64), 0, st);
    return (int)hipGetLastError();
}

int launch_head_mean_select(const float* colsum, const float* diag, int S, int H, int exclude_self, int L, int k, float* scores, int* kept,
                            hipStream_t st) {
    const int Leff = L < S ? L : S;
    const int nseg = (S + L - 1) / L;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {  // a 32768-token segment needs 128 KB of dynamic LDS
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&head_mean_select_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 32768 * 4);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    hipLaunchKernelGGL(head_mean_select_kernel, dim3(nseg), dim3(FUSED_THREADS), (size_t)Leff * sizeof(uint32_t), st, colsum, diag, S, H,
                       exclude_self, L, k, scores, kept);
    return (int)hipGetLastError();
}

int launch_select(const float* scores, int S, int L, int k, int* kept, hipStream_t st) {
    const int Leff = L < S ? L : S;
    const int nseg = (S + L - 1) / L;  // L <= 32768 here (keys of one segment live in LDS), no overflow
    static std::once_flag once;
    static int attr_err = 0;
    std::call_once(once, [] {  // a 32768-token segment needs 128 KB of dynamic LDS
        attr_err = raise_lds_limits({{reinterpret_cast<const void*>(&select_topk_kernel<512>), 2048 * 4}, {reinterpret_cast<const void*>(&select_topk_kernel<1024>), 32768 * 4}});
    });
    if (attr_err != 0) return attr_err;
    const size_t lds = (size_t)Leff * sizeof(uint32_t);
    if (Leff <= 128) hipLaunchKernelGGL(select_topk_kernel<256>, dim3(nseg), dim3(256), lds, st, scores, S, L, k, kept);
    else if (Leff <= 2048) hipLaunchKernelGGL(select_topk_kernel<512>, dim3(nseg), dim3(512), lds, st, scores, S, L, k, kept);
    else hipLaunchKernelGGL(select_topk_kernel<1024>, dim3(nseg), dim3(1024), lds, st, scores, S, L, k, kept);
    return (int)hipGetLastError();
}

}  // namespace lemo
