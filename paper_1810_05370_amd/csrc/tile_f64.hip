// Two-kernel transforms instantiated for double arithmetic.
#include "tile_impl.hpp"

namespace tumor {
template void launch_tile_inv<double>(int, const TileInvArgs&, const void*, hipStream_t);
template void launch_tile_xelast<double>(int, const TileXArgs&, const void*, hipStream_t);
template void launch_tile_fwd<double>(int, const TileFwdArgs&, const void*, hipStream_t);
template int tile_fwd_blocks<double>(int);
}  // namespace tumor
