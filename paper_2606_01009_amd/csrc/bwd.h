// What the backward's host side (melt_bwd.hip) and its split-plane products (bwd_split.hip) share.
#pragma once
#include "pack.h"

namespace melt {

constexpr int kRowsDx = 128;       // hop-block rows per dx chunk

// A backward row chunk: up to kRowsDx hop-block rows of one clip.
struct RowChunk {
    int64_t sample_start;   // first sample of row 0 of the chunk
    int64_t sample_end;     // clip end (exclusive)
    int64_t g_row0;         // G row of clip frame b0 (= frame offset of the clip + b0)
    int32_t n_rows;         // rows in this chunk
    int32_t t_lo;           // -b0: chunk-local row index of the clip's frame 0
    int32_t t_hi;           // T_c - b0: chunk-local index one past the clip's last frame
    int32_t pad;
};
static_assert(sizeof(RowChunk) == 40, "RowChunk layout");

// dx on operand planes: whether the plan's geometry fits, its basis layout, the launch
bool dx_split_fits(const Plan &p);
size_t dx_split_pack_bytes(const Plan &p);
PackJob dx_split_job(const Plan &p, void *out);
melt_status launch_dx_split(const Plan &p, const float *G, const RowChunk *rows, const int *n_rows, int64_t est_chunks,
                            int64_t n_frames, float *dx, hipStream_t s);
// dW on operand planes: blocks of dW, and the partial sums of `splits` frame ranges
int dw_split_blocks(const Plan &p);
melt_status launch_dw_split(const Plan &p, const float *G, const int64_t *fstart, const float *wave, int64_t n_frames,
                            int splits, float *part, hipStream_t s);

}  // namespace melt
