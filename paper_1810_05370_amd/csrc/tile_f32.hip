// Two-kernel transforms instantiated for float arithmetic.
#include "tile_impl.hpp"

namespace tumor {
template void launch_tile_inv<float>(int, const TileInvArgs&, const void*, hipStream_t);
template void launch_tile_xelast<float>(int, const TileXArgs&, const void*, hipStream_t);
template void launch_tile_fwd<float>(int, const TileFwdArgs&, const void*, hipStream_t);
template int tile_fwd_blocks<float>(int);
}  // namespace tumor
