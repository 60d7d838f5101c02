// F32 kernels of the OptCC executor (see optcc_launch.hpp): one GPU per
// server; servers of 2-4 GPUs; servers of more than 8 GPUs (general lane).
// Servers of 5-8 GPUs: optcc_kern_f32_g58.hip.
#include "optcc_launch.hpp"

namespace optcc {

hipError_t launch_f32(const kern::KArgs &a, bool servers, bool two, hipStream_t st,
                     int *occ) {
  if (!servers) return kern::launch<kern::F32, false, 0>(a, two, st, occ);
  if (a.g >= 2 && a.g <= 4) return kern::launch_fixed_g<kern::F32, 2, 3, 4>(a, two, st, occ);
  if (a.g >= 5 && a.g <= 8) return launch_f32_g58(a, two, st, occ);
  return kern::launch<kern::F32, true, 0>(a, two, st, occ);
}

}  // namespace optcc
