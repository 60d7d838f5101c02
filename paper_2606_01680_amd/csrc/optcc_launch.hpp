// Kernel launches of the OptCC executor: the kernel variants of one element
// type and the choice among them.  Each optcc_kern_*.hip instantiates one
// element type; optcc_exec.hip calls them through launch_f32/bf16/i32/f16.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "optcc_chain.hpp"
#include "optcc_kernels.hpp"
#include "optcc_server_chain.hpp"

namespace optcc {
namespace kern {

// Launch the kernel variant K, or, when occ is not NULL, only report how many
// of its workgroups one CU holds at this launch's dynamic LDS (no launch).
#define OPTCC_LAUNCH_OR_QUERY(K)                                                         \
  do {                                                                                  \
    if (occ)                                                                            \
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(occ, K, kThreads,            \
                                                          (size_t)a.occ_lds);           \
    hipLaunchKernelGGL(K, grid, block, (unsigned)a.occ_lds, st, a);                     \
    return hipGetLastError();                                                           \
  } while (0)

template <class D, bool S, int G>
hipError_t launch(const KArgs &a, bool two, hipStream_t st, int *occ) {
  if constexpr (!S && Streams<D>::value)
    if (a.kept) return launch<Kept<D>, S, G>(a, two, st, occ);
  constexpr int W16 = 16 / (int)sizeof(typename D::S);
  const int64_t grid64 = std::min<int64_t>(a.ntiles, a.grid > 0 ? (int64_t)a.grid : (int64_t)1 << 30);
  const dim3 grid((unsigned)std::max<int64_t>(grid64, 1)), block(kThreads);
  if constexpr (sizeof(typename D::S) == 4) {  // two vectors per lane: 32-bit types only
    if (two) OPTCC_LAUNCH_OR_QUERY((optcc_exec_kernel<D, W16, 2, S, G>));
    if constexpr (!S && G == 0) {  // long chains with large messages: the wider hop window
      if (a.wide_window) OPTCC_LAUNCH_OR_QUERY((optcc_exec_kernel<D, W16, 1, S, G, kHopWindowWide>));
    }
  }
  OPTCC_LAUNCH_OR_QUERY((optcc_exec_kernel<D, W16, 1, S, G>));
}

// Several GPUs per server: the kernel with the local ring
// fixed at compile time when g is one of Gs (else hipErrorInvalidValue).
template <class D, int... Gs>
hipError_t launch_fixed_g(const KArgs &a, bool two, hipStream_t st, int *occ) {
  hipError_t err = hipErrorInvalidValue;
  (void)((a.g == Gs ? (err = launch<D, true, Gs>(a, two, st, occ), true) : false) || ...);
  return err;
}

// Launch of a chain kernel (optcc_chain.hpp): bytes per lane access, cache
// policy, workgroup size, dynamic LDS bytes reserved per workgroup (not used
// by the kernel; it limits the workgroups per CU) and the log2 of the runs of
// workgroups taken side by side.
struct ChainShape {
  int bytes;
  ChainPolicy pol;
  int threads, lds, runs;
};

template <class D, int B, int H, ChainPolicy POL>
hipError_t launch_chain_variant(const ChainArgs &a, const ChainShape &s, hipStream_t st) {
  if (s.threads > chain_threads(B, H)) return hipErrorInvalidValue;
  ChainArgsOf<chain_ptrs(H)> k;
  static_cast<ChainHead &>(k) = a;
  std::memcpy(k.ptr, a.ptr, sizeof(k.ptr));
  hipLaunchKernelGGL((optcc_chain_kernel<D, B / (int)sizeof(typename D::S), H, POL>),
                     dim3((unsigned)a.per_run << a.runs), dim3((unsigned)s.threads),
                     (unsigned)s.lds, st, k);
  return hipGetLastError();
}
// The kernel with the fewest registers that hold the chain.
template <class D, int B, ChainPolicy POL, int H, int... Hs>
hipError_t launch_chain_held(const ChainArgs &a, const ChainShape &s, hipStream_t st) {
  if (a.pp <= H) return launch_chain_variant<D, B, H, POL>(a, s, st);
  if constexpr (sizeof...(Hs) > 0) return launch_chain_held<D, B, POL, Hs...>(a, s, st);
  else return hipErrorInvalidValue;
}
// Every combination that chain_rule (optcc_exec.hip) chooses.
template <class D>
hipError_t launch_chain(const ChainArgs &a, const ChainShape &s, hipStream_t st) {
  constexpr bool k32 = sizeof(typename D::S) == 4;
  if (s.bytes == 4) {
    if (s.pol == kResident) return launch_chain_held<D, 4, kResident, 8, 16, 32, 64, 128>(a, s, st);
    if (s.pol == kStreaming) return launch_chain_held<D, 4, kStreaming, 8, 16, 32, 64, 128>(a, s, st);
    if constexpr (k32) return launch_chain_held<D, 4, kMixed, 64, 128>(a, s, st);
    else return launch_chain_held<D, 4, kMixed, 128>(a, s, st);
  } else if (s.bytes == 8) {
    if (s.pol == kResident) return launch_chain_held<D, 8, kResident, 8>(a, s, st);
    if constexpr (k32) return launch_chain_held<D, 8, kStreaming, 8>(a, s, st);
  } else {
    if (s.pol == kMixed) return launch_chain_held<D, 16, kMixed, 8, 16>(a, s, st);
    if constexpr (k32) return launch_chain_held<D, 16, kStreaming, 8>(a, s, st);
    else if (s.pol == kResident) return launch_chain_held<D, 16, kResident, 8, 16>(a, s, st);
  }
  return hipErrorInvalidValue;
}

// Several GPUs per server: the kernel with the fewest registers that hold
// every rank, NSs healthy servers at most.
template <class D, int G, ChainPolicy POL, int NS, int... NSs>
hipError_t launch_server_held(const ServerChainArgs &a, const ChainShape &s, hipStream_t st) {
  if (a.pp <= NS) {
    constexpr int kBytes = 4;
    if (s.threads > server_threads(kBytes, G, NS)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((optcc_server_kernel<D, kBytes / (int)sizeof(typename D::S), G, NS, POL>),
                       dim3((unsigned)a.per_run << a.runs), dim3((unsigned)s.threads),
                       (unsigned)s.lds, st, a);
    return hipGetLastError();
  }
  if constexpr (sizeof...(NSs) > 0) return launch_server_held<D, G, POL, NSs...>(a, s, st);
  else return hipErrorInvalidValue;
}
template <class D>
hipError_t launch_server_chain(const ServerChainArgs &a, int g, const ChainShape &s,
                               hipStream_t st) {
#define OPTCC_SERVER_CASE(POL, G, ...) \
  if (s.pol == POL && g == G) return launch_server_held<D, G, POL, __VA_ARGS__>(a, s, st)
  OPTCC_SERVER_CASE(kResident, 2, 7, 15, 31, 63);
  OPTCC_SERVER_CASE(kResident, 4, 3, 7, 15, 31);
  OPTCC_SERVER_CASE(kResident, 8, 3, 7, 15);
  OPTCC_SERVER_CASE(kMixed, 2, 7, 15, 31, 63);
  OPTCC_SERVER_CASE(kMixed, 4, 3, 7, 15, 31);
  OPTCC_SERVER_CASE(kMixed, 8, 3, 7, 15);
  OPTCC_SERVER_CASE(kStreaming, 2, 7, 15, 23);  // up to 48 ranks
  OPTCC_SERVER_CASE(kStreaming, 4, 3, 7, 11);
  OPTCC_SERVER_CASE(kStreaming, 8, 3, 5);
#undef OPTCC_SERVER_CASE
  return hipErrorInvalidValue;
}

}  // namespace kern

hipError_t launch_chain_f32(const kern::ChainArgs &a, const kern::ChainShape &s, hipStream_t st);
hipError_t launch_chain_bf16(const kern::ChainArgs &a, const kern::ChainShape &s, hipStream_t st);
hipError_t launch_chain_i32(const kern::ChainArgs &a, const kern::ChainShape &s, hipStream_t st);
hipError_t launch_chain_f16(const kern::ChainArgs &a, const kern::ChainShape &s, hipStream_t st);
hipError_t launch_server_chain_f32(const kern::ServerChainArgs &a, int g, const kern::ChainShape &s,
                                   hipStream_t st);
hipError_t launch_server_chain_bf16(const kern::ServerChainArgs &a, int g,
                                    const kern::ChainShape &s, hipStream_t st);
hipError_t launch_server_chain_i32(const kern::ServerChainArgs &a, int g, const kern::ChainShape &s,
                                   hipStream_t st);
hipError_t launch_server_chain_f16(const kern::ServerChainArgs &a, int g, const kern::ChainShape &s,
                                   hipStream_t st);

// One element type each (optcc_kern_<type>.hip: one GPU per server, and
// servers of 2-4 GPUs or any other size; optcc_kern_<type>_g58.hip: servers
// of 5-8 GPUs, split off so that the files compile in parallel): servers
// selects the several-GPUs-per-server lane, two the two-vectors-per-lane variant.  With occ not NULL nothing is launched: *occ
// receives the number of workgroups of the chosen variant one CU holds.
hipError_t launch_f32(const kern::KArgs &a, bool servers, bool two, hipStream_t st,
                      int *occ = nullptr);
hipError_t launch_bf16(const kern::KArgs &a, bool servers, bool two, hipStream_t st,
                       int *occ = nullptr);
hipError_t launch_i32(const kern::KArgs &a, bool servers, bool two, hipStream_t st,
                      int *occ = nullptr);
hipError_t launch_f16(const kern::KArgs &a, bool servers, bool two, hipStream_t st,
                      int *occ = nullptr);
hipError_t launch_f32_g58(const kern::KArgs &a, bool two, hipStream_t st, int *occ);
hipError_t launch_bf16_g58(const kern::KArgs &a, bool two, hipStream_t st, int *occ);
hipError_t launch_i32_g58(const kern::KArgs &a, bool two, hipStream_t st, int *occ);
hipError_t launch_f16_g58(const kern::KArgs &a, bool two, hipStream_t st, int *occ);

}  // namespace optcc
