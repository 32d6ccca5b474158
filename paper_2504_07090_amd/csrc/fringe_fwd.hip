// Forward fringe contraction: launcher and kernel instantiations (fringe.hpp).
#include "fringe.hpp"

namespace bv {

void launch_fringe_fwd(const vis_field* f, const float* img, const float* fwhm, float2* vu,
                       hipStream_t st) {
#define BV_CALL_FWD(DD) fwd_d<DD>(f, img, fwhm, vu, st)
  BV_DISPATCH_EXTENT(f->extent, BV_CALL_FWD);
#undef BV_CALL_FWD
}

int fringe_tile_extent(int e) {
  return e <= 2 ? 2 : e <= 4 ? 4 : e <= 6 ? 6 : e <= 8 ? 8 : e <= 12 ? 12 : 16;
}

}  // namespace bv
