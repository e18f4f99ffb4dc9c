// Evaluation passes of 32 and 64 columns (contraction on the matrix cores).
#include "eval_tile.h"

namespace askit {

void launch_eval_tile_mat(const ChunkParams &p, int cm, bool multi, bool vh, unsigned grid, hipStream_t s)
{
    if (cm == 32) launch_eval_tile<32>(p, multi, vh, grid, s);
    else launch_eval_tile<64>(p, multi, vh, grid, s);
}

}  // namespace askit
