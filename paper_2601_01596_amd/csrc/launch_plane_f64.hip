// Dispatch of the plane pass, double instantiations.
#include "kernels_plane.hpp"

namespace ffcz {

template <int LY, int H>
static hipError_t go_plane(const PlaneArgs<double>& a, int64_t nb, hipStream_t s) {
  if constexpr (plane_fits<double>(LY, H)) {
    hipLaunchKernelGGL((plane_kernel<double, LY, H>), dim3((unsigned)nb), dim3(PlaneGeom<LY, H>::NT), 0, s, a);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}
template <int LY>
static hipError_t go_plane_h(int H, const PlaneArgs<double>& a, int64_t nb, hipStream_t s) {
  switch (H) {
    case 8: return go_plane<LY, 8>(a, nb, s);
    case 16: return go_plane<LY, 16>(a, nb, s);
    case 32: return go_plane<LY, 32>(a, nb, s);
    case 64: return go_plane<LY, 64>(a, nb, s);
    case 128: return go_plane<LY, 128>(a, nb, s);
    case 256: return go_plane<LY, 256>(a, nb, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_plane_f64(int Ly, int H, const void* args, int64_t nb, hipStream_t s) {
  const PlaneArgs<double>& a = *static_cast<const PlaneArgs<double>*>(args);
  switch (Ly) {
    case 16: return go_plane_h<16>(H, a, nb, s);
    case 32: return go_plane_h<32>(H, a, nb, s);
    case 64: return go_plane_h<64>(H, a, nb, s);
    case 128: return go_plane_h<128>(H, a, nb, s);
    case 256: return go_plane_h<256>(H, a, nb, s);
    case 512: return go_plane_h<512>(H, a, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ffcz
