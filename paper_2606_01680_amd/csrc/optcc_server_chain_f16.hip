// F16 kernels of the OptCC executor for whole AllReduces with several GPUs
// per server (see optcc_server_chain.hpp).
#include "optcc_launch.hpp"

namespace optcc {

hipError_t launch_server_chain_f16(const kern::ServerChainArgs &a, int g, const kern::ChainShape &s,
                                 hipStream_t st) {
  return kern::launch_server_chain<kern::F16>(a, g, s, st);
}

}  // namespace optcc
