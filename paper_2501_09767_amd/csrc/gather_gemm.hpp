// What the selective-load GEMM kernels share: gather_gemm_large.hip (256 x 256 tiles), gather_gemm_mid.hip (256, 192,
// 128 or 64 x 128), gather_gemm_small.hip (64 x 64; all of binary32).
#pragma once
#include <type_traits>

#include "lemo_common.hpp"

namespace lemo {

// How the operands lie in memory (an MFMA lane always wants 8 consecutive contraction elements of one operand row):
//   GG_NT  A rows and B rows run along the contraction (X[idx] [M,C] against an nn.Linear weight [N,C]); 16-byte reads.
//   GG_NN  A as above; B is stored contraction-major, [C, N] (the same weight used the other way round, as the input
//          gradient needs it).  Its slabs go to LDS as they are, 64 contraction rows at a time, and the fragments
//          come out through the transposing LDS read (ds_read_b64_tr_b16: inside a group of 16 lanes, lane l receives
//          element l % 4 of the 8 bytes addressed by lanes l / 4, 4 + l / 4, 8 + l / 4 and 12 + l / 4 -- with lane
//          4 j + q pointed at row j, column quad q of a 4-row x 16-column block, lane l gets 4 consecutive rows of
//          column l).  Two such reads make one 16-byte fragment: the same bytes from LDS as before, no transposed copy
//          anywhere.
//   GG_TN  both operands contraction-major: A [C, M], B [C, N] with B's rows picked by idx (the weight gradient: the
//          contraction runs over the kept tokens).  GG_NN is bf16 only; binary32 fragments of GG_TN are read element by
//          element, which is what its MFMAs take.
enum { GG_NT = 0, GG_NN = 1, GG_TN = 2 };
typedef __attribute__((ext_vector_type(4))) short s16x4;

// Y (+)= A . B^T over K: the operands in the layouts above, A's rows (GG_TN: B's) picked by idx.
struct GgParams {
    const void* A;
    const void* B;
    const void* bias;  // [N] or null
    void* Y;           // in-place-add form: the residual stream, its rows picked by oidx
    const int* idx;    // or null: rows 0, 1, ...
    const int* oidx;   // likewise
    long long lda, ldb, ldy, M, out_rows;  // pitches in elements
    int K, N, tiles_m, tiles_n;
    unsigned a_bytes, b_bytes, y_bytes;  // spans of the whole operands (b_bytes: GG_TN; y_bytes: in-place add)
};

// Tile of workgroup b: die b % 8 takes a contiguous run of tiles in grouped order (group_m tile rows at a time, column
// by column), so the tiles resident on one die share rows of both operands through its L2.  False: nothing to do.
__device__ __forceinline__ bool gg_tile(int b, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + NUM_XCD - 1) / NUM_XCD;
    const int tile = (b % NUM_XCD) * per_xcd + b / NUM_XCD;
    if (b / NUM_XCD >= per_xcd || tile >= total) return false;
    const int group = tile / (group_m * tiles_n);
    const int first_m = group * group_m;
    const int rows_in_group = min(group_m, tiles_m - first_m);
    const int within = tile - group * group_m * tiles_n;
    tm = first_m + within % rows_in_group;
    tn = within / rows_in_group;
    return true;
}

// Output tiles.  binary32 knows GG_T128 and GG_T64 only, both in gather_gemm_small.hip, the latter 32 x 32 or 16 x 16.
enum GgTile { GG_T256, GG_T256x128, GG_T192x128, GG_T128, GG_T64x128, GG_T64 };
int prepare_gather_gemm_large(bool add, int layout);
int prepare_gather_gemm_mid(bool add, int layout);
int prepare_gather_gemm_small(lemo_dtype_t dt, bool add, int layout);
int launch_gather_gemm_large(const GgParams& p, bool add, int layout, hipStream_t st);               // GG_T256, bf16
int launch_gather_gemm_mid(const GgParams& p, bool add, int layout, GgTile tile, hipStream_t st);    // the kinds of 128 columns, bf16
int launch_gather_gemm_small(const GgParams& p, lemo_dtype_t dt, bool add, int layout, GgTile tile, hipStream_t st);

}  // namespace lemo
