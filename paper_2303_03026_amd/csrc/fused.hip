// The fused stage with two ghost layers: the HLL instances and the dispatch
// on the flux (the kernel is in fused_stage.h; the HLLC and HLLD instances
// are built in fused_hllc.hip and fused_hlld.hip).
#include "fused_stage.h"

namespace amrvac {

hipError_t launch_fused_stage(hipStream_t s, const GridConst& G, const Tables& T, const JobScalars& J,
                              const FusedTune& tune, const void* in, const void* base, void* out, double w,
                              const PhysConst& P, DevStatus* st, const JobCfl* cfl, void* freg) {
  if (P.flux == FLUX_HLLC) return launch_fused_hllc(s, G, T, J, tune, in, base, out, w, P, st, cfl, freg);
  if (P.flux == FLUX_HLLD) return launch_fused_hlld(s, G, T, J, tune, in, base, out, w, P, st, cfl, freg);
  return launch_fused_flux<FLUX_HLL>(s, G, T, J, tune, in, base, out, w, P, st, cfl, freg);
}

}  // namespace amrvac
