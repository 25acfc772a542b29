// The MFMA GEMM (gemm_tile.h), EPI 3.  One of them to a source file, so that they compile side by side.
#include "gemm_tile.h"

namespace clv {
void launch_tile_qkv(const TileGemmQkv& g, const TileForm& t, int wgs, hipStream_t st) { launch_tile<3>(g, t, wgs, st); }
}  // namespace clv
