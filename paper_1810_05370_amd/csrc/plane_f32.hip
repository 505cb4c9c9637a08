// Small grids' Krylov iterations instantiated for float arithmetic.
#include "plane_impl.hpp"

namespace tumor {
template void launch_plane<float>(int, bool, int, const PlaneArgs&, const void*, hipStream_t);
template void launch_plane_start<float>(int, bool, const void*, const double (&)[kMaxSys], int, const PlaneArgs&,
                                     SolveScalars*, hipStream_t);
template void launch_plane_final<float>(int, bool, void*, const double (&)[kMaxSys], int, const PlaneArgs&,
                                     const SolveScalars*, hipStream_t);
template void launch_plane_coefs<float>(int, int, const void* const*, void* const*, hipStream_t);
}  // namespace tumor
