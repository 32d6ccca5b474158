// Adjoint fringe contraction: launcher and kernel instantiations (fringe.hpp).
#include "fringe.hpp"

namespace bv {

void launch_fringe_adj(const vis_field* f, const float* img, const float* fwhm, const float* gco,
                       float* dimg, float* f_part, hipStream_t st, float* dfull) {
#define BV_CALL_ADJ(DD) adj_d<DD>(f, img, fwhm, gco, dimg, dfull, f_part, st)
  BV_DISPATCH_EXTENT(f->extent, BV_CALL_ADJ);
#undef BV_CALL_ADJ
}

}  // namespace bv
