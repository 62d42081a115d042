// lbm_twostep_cl.hip -- the three-step kernel for the edge tiles of a lattice
// on the learned closure (three_step_tile with CL), one instance per storage
// format, shape and collision model, in a translation unit of its own.
#include <hip/hip_runtime.h>

#include "lbm_threestep.h"

namespace lbm {

hipError_t launch_three_step_closure(const LatDesc& L, int parity, int id, hipStream_t s) {
  switch (L.store) {
    case ST_F64: return launch_three_s<ST_F64, true>(L, parity, id, s, 2);
    case ST_F32: return launch_three_s<ST_F32, true>(L, parity, id, s, 2);
    case ST_F16: return launch_three_s<ST_F16, true>(L, parity, id, s, 2);
    case ST_BF16: return launch_three_s<ST_BF16, true>(L, parity, id, s, 2);
  }
  return hipErrorInvalidValue;
}

// Edge tiles of a march of `ty` tile rows (8 or 12, the rows of LBM_THREE_MARCH).
template <int S>
static hipError_t launch_march_ring_s(const LatDesc& L, int parity, int ty, hipStream_t s) {
  if (ty == 8) return launch_march_ring_t<S, 8>(L, parity, s);
  if (ty == 12) return launch_march_ring_t<S, 12>(L, parity, s);
  return hipErrorInvalidValue;
}
hipError_t launch_march_ring_closure(const LatDesc& L, int parity, int ty, hipStream_t s) {
  switch (L.store) {
    case ST_F64: return launch_march_ring_s<ST_F64>(L, parity, ty, s);
    case ST_F32: return launch_march_ring_s<ST_F32>(L, parity, ty, s);
    case ST_F16: return launch_march_ring_s<ST_F16>(L, parity, ty, s);
    case ST_BF16: return launch_march_ring_s<ST_BF16>(L, parity, ty, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
