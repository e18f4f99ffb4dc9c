// The evaluation kernels' parameters (eval.hip, eval_vec.hip, eval_mat.hip).
#pragma once

#include "askit_impl.h"

namespace askit {

struct ChunkParams {
    const Chunk *chunks;
    int64_t nchunk;
    const int32_t *tpos, *tslot;
    // single problem (MULTI = false)
    const Node *nodes;
    const float *Y, *Xt, *gt, *Xs, *gs;
    const int32_t *skk;
    int smax, dp;
    // batch (MULTI = true)
    const EvalInst *inst;
    int32_t *queue;
    int persistent;
    // weights and output
    const float *Wt, *Wsk;     // single: the problem's; batch: shared buffers (instance offsets)
    float *part;
    int R, r0, rb;             // columns [r0, r0 + rb) in this pass
    int mode;                  // tiled form: eval_mode
    float sc;                  // its FP16 split's coordinate scale (batch: each instance's)
    int d;                     // dimensions without padding (batch: each instance's)
};

// One pass of cm columns (vector units: 1 or 4; matrix: 32 or 64) over the
// chunks of problems with dp <= 64; vh: per-source bandwidths.
void launch_eval_tile_vec(const ChunkParams &p, int cm, bool multi, bool vh, unsigned grid, hipStream_t s);
void launch_eval_tile_mat(const ChunkParams &p, int cm, bool multi, bool vh, unsigned grid, hipStream_t s);

}  // namespace askit
