#include "gemm_wide.h"

namespace nvfp4 {

bool launch_gemm_wide32(const TileArgs &P, GemmTile tile, int out_dt, hipStream_t st)
{
    return P.K % wide::KT ? launch_wide_tile<32, true>(P, tile, out_dt, st) : launch_wide_tile<32, false>(P, tile, out_dt, st);
}

void launch_gemm_wide_mixed32(const TileArgs &P, const WideMix &X, int out_dt, hipStream_t st) { launch_wide_mixed<32>(P, X, out_dt, st); }

}  // namespace nvfp4
