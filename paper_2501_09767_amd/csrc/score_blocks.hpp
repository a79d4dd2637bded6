// The 128 x 128 rectangles of the block-wise scores and the order in which the kernels walk them.
#pragma once
#include "lemo_common.hpp"

namespace lemo {

// Rectangle `id` in the order of walk: bands of four rows from the top, a band's rectangles column by column.  Under a causal mask
// a row ends on the diagonal.  A die takes a run of this order, so that what it works on at a time is a 4 x 8 patch (12 operand
// tiles for 32 rectangles) and all dies have the same share.
__host__ __device__ inline void sb_rectangle(int id, int nt, bool causal, int& tq, int& tk) {
    int band;
    if (causal) {  // bands before band n hold 8 n^2 + 2 n rectangles
        band = (int)((sqrtf(4.f + 32.f * (float)id) - 2.f) * (1.f / 16.f));
        while (8 * (band + 1) * (band + 1) + 2 * (band + 1) <= id) ++band;
        while (band > 0 && 8 * band * band + 2 * band > id) --band;
        id -= 8 * band * band + 2 * band;
    } else {
        band = id / (4 * nt);
        id -= band * 4 * nt;
    }
    const int r0 = band * 4, rows = nt - r0 < 4 ? nt - r0 : 4;
    const int full = causal ? r0 + 1 : nt;  // columns that reach all of the band's rows
    if (id < rows * full) {
        tk = id / rows;
        tq = r0 + id - tk * rows;
        return;
    }
    id -= rows * full;
    int t = 0;  // then the triangle: columns full + t, rows r0 + 1 + t on
    while (id >= rows - 1 - t) { id -= rows - 1 - t; ++t; }
    tk = full + t;
    tq = r0 + 1 + t + id;
}

// The first p.count rectangles of that order (bf16): score_blocks_slabs.hip
int prepare_tilemax_slabs(int d);
int launch_tilemax_slabs(const BlockParams& p, int d, int mode, hipStream_t st);
// Rectangles first .. first + rest - 1 of that order as 64 x 64 quarters or 32 x 32 pieces (bf16): score_blocks_few.hip
int prepare_tilemax_few(int d);
int launch_tilemax_few(const BlockParams& p, int d, int mode, int first, int rest, hipStream_t st);

}  // namespace lemo
