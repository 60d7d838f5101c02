// Device code of whole AllReduces with G GPUs per server (App. E): every
// server's collects and the chain are held in registers, as optcc_chain.hpp
// does with one GPU per server (same accesses, same waves, same bound: HBM).
//
// A wave loads every rank's value of its elements, runs the collects of all
// servers, the chain over the leaders and the straggler server's fold in
// place, and then stores, rank by rank, the partials that the rank's steps
// write (none for the far end of a collect, one for the GPUs between, the
// collect's and the hop's for a leader) and right after them the global sum.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "optcc_chain.hpp"

namespace optcc {
namespace kern {

constexpr int kServerChainMaxRanks = 128;  // most ranks held in registers

struct ServerChainArgs {
  int64_t n;         // elements per rank
  uint32_t nq, k;    // quanta per rank, segments per part
  int32_t pp;        // healthy servers
  int32_t runs, per_run, waves;  // as in ChainHead
  uint32_t lp, lq;   // quanta of the shorter parts and segments
  ChainDiv by_nq, by_g, by_k;
  ChainDiv by_lp[2];  // parts of lp and lp + 1 quanta
  ChainSeg seg[2];    // segments of lq and lq + 1 quanta (no P2P chunk)
  // Per server (healthy in ring order, then the straggler) its GPUs by local
  // index from G - 1 down to 0, twice: the collect order of part i, positions
  // G - 1 .. 0 of its local ring, is the G entries from (G - i) mod G.
  uint64_t ptr[2 * kServerChainMaxRanks];
};
typedef const OPTCC_CONST_AS ServerChainArgs *ServerArgsPtr;

// Where a quantum lies: its part, schedule type, section and the first quantum
// past that section.
struct ServerPlace {
  int part, type, j;
  uint32_t end;
};
template <int G>
__device__ __forceinline__ ServerPlace server_place_of(ServerArgsPtr a, uint32_t q) {
  ServerPlace r;
  const uint32_t part = divide((q + 1) * G - 1, &a->by_nq);
  const uint32_t p0 = divide(part * a->nq, &a->by_g);
  const uint32_t lp = divide((part + 1) * a->nq, &a->by_g) - p0;
  const uint32_t u = q - p0;
  const uint32_t c = divide((u + 1) * a->k - 1, &a->by_lp[lp > a->lp ? 1 : 0]);
  const uint32_t s0 = divide(c * lp, &a->by_k), s1 = divide((c + 1) * lp, &a->by_k);
  const OPTCC_CONST_AS ChainSeg *sg = &a->seg[s1 - s0 > a->lq ? 1 : 0];
  const uint32_t x = u - s0, big = sg->nbig * (sg->qbase + 1);
  r.part = (int)part;
  r.type = c & 1 ? 2 : 1;  // patterns A and C: type 1, B and D: type 2
  if (x < big) {
    r.j = (int)divide(x, &sg->by_big);
    r.end = p0 + s0 + ((uint32_t)r.j + 1) * (sg->qbase + 1);
  } else {
    const uint32_t i = divide(x - big, &sg->by_small);
    r.j = (int)(sg->nbig + i);
    r.end = p0 + s0 + big + (i + 1) * sg->qbase;
  }
  return r;
}

// A server's G rank pointers in collect order.
template <int G>
struct ServerPtrs {
  uint64_t p[G];
};
template <int G>
__device__ __forceinline__ ServerPtrs<G> load_server(PtrTable t) {
  ServerPtrs<G> r;
#pragma unroll
  for (int c = 0; c < G; ++c) r.p[c] = t[c];
#pragma unroll
  for (int c = 0; c < G; ++c) asm volatile("" : "+s"(r.p[c]));
  return r;
}

// f(t) for t in [T, n) of at most NS servers, t a compile-time constant in f.
template <int T, int NS, class F>
__device__ __forceinline__ void servers_from(int n, F &f) {
  if constexpr (T < NS) {
    if (T < n) {
      f(Hop<T>());
      OPTCC_BLOCK_MARK(2000 + T);
      servers_from<T + 1, NS>(n, f);
    }
  }
}
template <int T0, int NS, class F>
__device__ __forceinline__ void each_server(int n, F f) {
  servers_from<T0, NS>(fresh(n), f);
}

// Every step of one section's elements for the lanes that are active here.
// tab: the pointer table rotated to the part's collect order.
template <class D, int W, int G, int NS, ChainPolicy POL>
__device__ __forceinline__ void server_piece(PtrTable tab, int j, int pp, bool type1, int64_t off,
                                             uint32_t lane) {
  using V = Held<D, W>;
  constexpr bool kNtL = POL != kResident, kNtM = POL == kStreaming, kNtF = POL != kResident;
  // entry of chain position t (healthy server R[j + t]) in collect order
  auto at = [&](PtrTable b, int t) __attribute__((always_inline)) {
    const int h = j + t;
    return b + (h >= pp ? h - pp : h) * (2 * G);
  };
  V x[NS * G], xs[G];
  {
    const ServerPtrs<G> s = load_server<G>(tab + pp * (2 * G));
#pragma unroll
    for (int c = 0; c < G; ++c) xs[c] = cload<D, W, kNtL>(s.p[c], off, lane);
  }
  {
    const PtrTable b = fresh(tab);
    each_server<0, NS>(pp, [&](auto t) __attribute__((always_inline)) {
      const ServerPtrs<G> s = load_server<G>(at(b, t));
#pragma unroll
      for (int c = 0; c < G; ++c) x[t * G + c] = cload<D, W, kNtL>(s.p[c], off, lane);
    });
  }
  V v, start;  // the chain's running value; its value after the first server
  if (!type1) {  // slot 0: N3 collect on the straggler server
#pragma unroll
    for (int c = 1; c < G; ++c) xs[c] = add_held<D, W, kFixed>(xs[c], xs[c - 1]);
  }
  each_server<0, NS>(pp, [&](auto t) __attribute__((always_inline)) {  // slot 1: N1 collects
#pragma unroll
    for (int c = 1; c < G; ++c)
      x[t * G + c] = add_held<D, W, kFixed>(x[t * G + c], x[t * G + c - 1]);
    const V &lead = x[t * G + G - 1];
    if constexpr (t == 0) {
      v = lead;
      if (!type1) v = add_held<D, W, kFixed>(v, xs[G - 1]);  // slot 2: S3 into the chain start
      start = v;
    } else {
      v = add_held<D, W, kFixed>(lead, v);  // slot 3: S1 hop
    }
  });
  if (type1) {  // slots 4 and 5: S2 and the N2 fold along the straggler's ring
#pragma unroll
    for (int c = G - 1; c >= 0; --c) {
      v = add_held<D, W, kFixed>(xs[c], v);
      xs[c] = v;
    }
  }
  const V sum = v;
  {
    const PtrTable b = fresh(tab);
    V hop = start;
    each_server<0, NS>(pp, [&](auto t) __attribute__((always_inline)) {
      const ServerPtrs<G> s = load_server<G>(at(b, t));
      cstore<D, W, kNtF>(s.p[0], off, lane, sum);  // slot 9
#pragma unroll
      for (int c = 1; c < G - 1; ++c) {
        cstore<D, W, kNtM>(s.p[c], off, lane, x[t * G + c]);
        OPTCC_STEP_ORDER();
        cstore<D, W, kNtF>(s.p[c], off, lane, sum);
        OPTCC_STEP_ORDER();
      }
      const V &lead = x[t * G + G - 1];
      cstore<D, W, kNtM>(s.p[G - 1], off, lane, lead);
      OPTCC_STEP_ORDER();
      if constexpr (t > 0) hop = add_held<D, W, kFixed>(lead, hop);
      if (t > 0 || !type1) {
        cstore<D, W, kNtM>(s.p[G - 1], off, lane, hop);
        OPTCC_STEP_ORDER();
      }
      // slots 7 and 8; without the straggler's fold the holder's hop is the sum
      if (type1 || t + 1 < pp) cstore<D, W, kNtF>(s.p[G - 1], off, lane, sum);
      OPTCC_STEP_ORDER();
    });
  }
  {  // the straggler server: slots 0 and 10-11, or 4-6
    const ServerPtrs<G> s = load_server<G>(fresh(tab) + pp * (2 * G));
    cstore<D, W, kNtF>(s.p[0], off, lane, sum);
#pragma unroll
    for (int c = 1; c < G; ++c) {
      cstore<D, W, kNtM>(s.p[c], off, lane, xs[c]);
      OPTCC_STEP_ORDER();
      cstore<D, W, kNtF>(s.p[c], off, lane, sum);
      OPTCC_STEP_ORDER();
    }
  }
}

template <class D, int W, int G, int NS, ChainPolicy POL>
__device__ __forceinline__ void server_span(ServerArgsPtr a, uint32_t q, uint32_t qe, int64_t x,
                                            int l, uint32_t ql, bool whole) {
  constexpr int64_t kEs = sizeof(typename D::S);
  const uint32_t lane = (uint32_t)(l * W * kEs);
  while (q < qe) {
    const ServerPlace s = server_place_of<G>(a, q);
    const PtrTable tab = a->ptr + (s.part ? G - s.part : 0);
    if (whole && ql >= q && ql < s.end)
      server_piece<D, W, G, NS, POL>(tab, s.j, a->pp, s.type == 1, x * kEs, lane);
    q = s.end;
  }
}

constexpr int server_threads(int bytes, int g, int ns) { return chain_threads(bytes, g * (ns + 1)); }

template <class D, int W, int G, int NS, ChainPolicy POL>
__global__ __launch_bounds__(server_threads(W * (int)sizeof(typename D::S), G, NS))
void optcc_server_kernel(ServerChainArgs) {
  ServerArgsPtr a = (ServerArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t i = blockIdx.x;
  const uint32_t b = (i & ((1u << a->runs) - 1)) * (uint32_t)a->per_run + (i >> a->runs);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  const uint32_t nq = a->nq;
  const uint64_t q64 = ((uint64_t)b * a->waves + wave) * W;
  if (q64 >= nq) return;
  const uint32_t q = (uint32_t)q64, qe = nq - q < W ? nq : q + W;
  const int64_t x = (int64_t)q * kQuantum;
  server_span<D, W, G, NS, POL>(a, q, qe, x, l, q + (uint32_t)(l * W) / kQuantum,
                                x + l * W + W <= a->n);
  if constexpr (W > 1) {  // the rank vectors' last elements, less than a lane's W
    const int rest = (int)(a->n % W);
    if (qe == nq && rest)
      server_span<D, 1, G, NS, POL>(a, nq - 1, nq, a->n - rest, l, nq - 1, l < rest);
  }
}

}  // namespace kern
}  // namespace optcc
