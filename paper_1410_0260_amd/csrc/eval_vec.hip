// Evaluation passes of 1 and 4 columns (contraction on the vector units).
#include "eval_tile.h"

namespace askit {

void launch_eval_tile_vec(const ChunkParams &p, int cm, bool multi, bool vh, unsigned grid, hipStream_t s)
{
    if (cm == 1) launch_eval_tile<1>(p, multi, vh, grid, s);
    else launch_eval_tile<4>(p, multi, vh, grid, s);
}

}  // namespace askit
