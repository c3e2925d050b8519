// The fused stage with two ghost layers: the HLLC instances.
#include "fused_stage.h"

namespace amrvac {

hipError_t launch_fused_hllc(hipStream_t s, const GridConst& G, const Tables& T, const JobScalars& J,
                              const FusedTune& tune, const void* in, const void* base, void* out, double w,
                              const PhysConst& P, DevStatus* st, const JobCfl* cfl, void* freg) {
  return launch_fused_flux<FLUX_HLLC>(s, G, T, J, tune, in, base, out, w, P, st, cfl, freg);
}

}  // namespace amrvac
