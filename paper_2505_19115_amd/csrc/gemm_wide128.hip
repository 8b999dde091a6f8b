#include "gemm_wide.h"

namespace nvfp4 {

bool launch_gemm_wide128(const TileArgs &P, GemmTile tile, int out_dt, hipStream_t st)
{
    return launch_wide_tile<128, false>(P, tile, out_dt, st);  // (a contraction in blocks of 128 is whole K tiles)
}

void launch_gemm_wide_mixed128(const TileArgs &P, const WideMix &X, int out_dt, hipStream_t st) { launch_wide_mixed<128>(P, X, out_dt, st); }

}  // namespace nvfp4
