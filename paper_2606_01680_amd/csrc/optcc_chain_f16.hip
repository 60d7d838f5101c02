// F16 kernels of the OptCC executor for whole AllReduces with one GPU per
// server (see optcc_chain.hpp).
#include "optcc_launch.hpp"

namespace optcc {

hipError_t launch_chain_f16(const kern::ChainArgs &a, const kern::ChainShape &s, hipStream_t st) {
  return kern::launch_chain<kern::F16>(a, s, st);
}

}  // namespace optcc
