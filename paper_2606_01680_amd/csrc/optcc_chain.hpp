// Device code of whole AllReduces with one GPU per server: every chain is
// held in registers.  Included through optcc_launch.hpp.
//
// A wave takes 64 lanes x W consecutive elements of one section and runs all
// of its steps: it loads every rank's value first (H registers' worth), runs
// the Stage 1 chain in place, so that register t ends as the partial sum that
// hop t writes, and then stores, rank by rank, the partial and right after it
// the global sum that overwrites it.  All lanes of a wave are in one section,
// so the rank pointers are wave-uniform: they are read from the kernel
// arguments with scalar loads, and an access is a scalar base plus a lane
// offset.
//
// What bounds it: HBM.  The two stores of a rank reach L2 back to back, so
// the line leaves L2 once, with the global sum: HBM writes are 1.00-1.04 of the
// results' bytes (8, 16, 64 and 128 ranks, 2-8 GiB of buffers) where the steps
// write 1.7-2.0 of them.  Storing each partial as its hop runs (ring_lane)
// leaves it in L2 for the rest of the chain, where other waves' lines push
// it out.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "optcc_kernels.hpp"

namespace optcc {
namespace kern {

constexpr int kChainMaxHealthy = 128;  // longest chain held in registers
constexpr int kGroup = 8;  // hops of one straight-line group

// Division of a 32-bit number by an invariant d >= 1 (Granlund and Montgomery,
// "Division by Invariant Integers using Multiplication", 1994, Fig. 4.1):
// five scalar instructions.
struct ChainDiv {
  uint32_t m, s1, s2;
};
// Segments of one length (a plan has at most two, a quantum apart): quanta of
// the point-to-point chunk, of a section (the first nbig have one more) and
// the divisions by qbase + 1 and qbase.
struct ChainSeg {
  uint32_t dq, qbase, nbig;
  ChainDiv by_big, by_small;
};

struct ChainHead {
  int64_t n;         // elements per rank
  uint32_t nq, k;    // quanta per rank, segments
  int32_t pp, m;
  // Keeps runs and per_run apart from the numbers that follow: with one wide load
  // for all of them 16 ranks of 2^26 bf16 elements take 752 us instead of 745.
  int32_t unused;
  // 2^runs contiguous runs of `per_run` workgroups are taken side by side
  int32_t runs, per_run;
  int32_t waves;     // waves per workgroup
  uint32_t ord2;     // bit g mod 4: segment g has ordering 2
  uint32_t wide;     // nq * k does not fit 32 bits: plain 64-bit divisions
  uint32_t lq;       // quanta of the shorter segments, seg[0]
  ChainDiv by_nq, by_k;
  ChainSeg seg[2];
};
// Pointer table: [0, 2 pp) the healthy ranks in ring order, twice, so that a
// chain's ranks R[j], R[j+1], .. are consecutive entries for every j;
// [2 pp, 2 pp + m) the stragglers sorted by slowdown (worst first); a group of
// entries is read past the last one used, so kGroup more are there.
constexpr int kChainStragglers = 16;  // most stragglers the kernel takes
constexpr int chain_ptrs(int h) { return 2 * h + kGroup + kChainStragglers; }
template <int NP>
struct ChainArgsOf : ChainHead {
  uint64_t ptr[NP];
};
using ChainArgs = ChainArgsOf<chain_ptrs(kChainMaxHealthy)>;

// Cache hints: kStreaming marks every access nontemporal, kMixed all but the
// stores of partials, kResident none.
enum ChainPolicy { kStreaming, kMixed, kResident };

#define OPTCC_CONST_AS __attribute__((address_space(4)))
#define OPTCC_GLOBAL_AS __attribute__((address_space(1)))

// W elements of a lane as 1, 2 or 4 dwords (the low half of one for a single
// 16-bit element).  A chain's values are held in this form, two 16-bit
// elements to a register, and unpacked only inside an addition.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <class D, int W>
struct Held {
  static constexpr int kBytes = W * (int)sizeof(typename D::S);
  static constexpr int kWords = kBytes < 4 ? 1 : kBytes / 4;
  uint32_t w[kWords];
};
// Memory accesses of that many bytes, aligned to the element only: gfx950
// takes them at any element alignment.
template <int BYTES, int ALIGN>
struct AccessOf;
#define OPTCC_ACCESS(BYTES, TYPE, ALIGN)            \
  template <>                                       \
  struct AccessOf<BYTES, ALIGN> {                   \
    typedef TYPE T __attribute__((aligned(ALIGN))); \
  };
OPTCC_ACCESS(2, uint16_t, 2)
OPTCC_ACCESS(4, uint32_t, 2)
OPTCC_ACCESS(8, u32x2, 2)
OPTCC_ACCESS(16, u32x4, 2)
OPTCC_ACCESS(4, uint32_t, 4)
OPTCC_ACCESS(8, u32x2, 4)
OPTCC_ACCESS(16, u32x4, 4)
#undef OPTCC_ACCESS

// Of two NaNs a step keeps its destination's: own value + received value, as the
// oracle adds and as a float addition with the own value as first operand does.
// To the compiler a float addition is commutative, and it swaps operands by the
// kind of instruction they come from, so every sum here says how its operands
// stay in place:
//   kFixed   the instruction is written out;
//   kOpaque  an addition whose result the compiler knows nothing about, so that
//            the next one's operands look alike;
//   kPlain   an addition whose operands it leaves alone as it is (16-bit halves
//            of a word, which are shifts on both sides).
// kFixed and kOpaque keep branches that a plain addition's compiler would turn
// into selects; which one costs nothing differs (us, plain -> kFixed): 128 ranks
// fp32 at 2^24 3370 -> 3387 and kOpaque 3368, 16 ranks bf16 at 2^26 744.3 ->
// 748.1, fp16 744.7 -> 742.1, 16 x 4 GPUs fp32 at 2^24 1571 -> 1568.
enum AddOrder { kFixed, kOpaque, kPlain };
template <class D>
constexpr AddOrder kHopOrder = std::is_same<D, F32>::value   ? kOpaque
                               : std::is_same<D, F16>::value ? kFixed
                                                             : kPlain;
template <AddOrder O>
__device__ __forceinline__ float add_in_order(float a, float b) {
  if constexpr (O != kFixed) return a + b;
  float r;
  asm("v_add_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <AddOrder O>
__device__ __forceinline__ uint32_t add_in_order(uint32_t a, uint32_t b) {
  return a + b;
}

// One reduce step with a single source, narrow(widen(a) + widen(b)), on a
// dword: two 16-bit elements or one 32-bit element.
template <class D, AddOrder O>
__device__ __forceinline__ uint32_t add_word(uint32_t a, uint32_t b) {
  if constexpr (std::is_same<D, F32>::value) {
    return __float_as_uint(add_in_order<O>(__uint_as_float(a), __uint_as_float(b)));
  } else if constexpr (std::is_same<D, I32>::value) {
    return a + b;
  } else if constexpr (std::is_same<D, BF16>::value) {
    return BF16::narrow_pair(
        add_in_order<O>(__uint_as_float(a << 16), __uint_as_float(b << 16)),
        add_in_order<O>(__uint_as_float(a & 0xffff0000u), __uint_as_float(b & 0xffff0000u)));
  } else {
    // rounding the sum of two halves to fp32 and then to fp16 gives the same
    // as rounding it once: 24 bits >= 2 * 11 + 2
    static_assert(std::is_same<D, F16>::value && O == kFixed, "element type");
    uint32_t r;
    asm("v_pk_add_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
  }
}
template <class D, int W, AddOrder O = kHopOrder<D>>
__device__ __forceinline__ Held<D, W> add_held(const Held<D, W> &a, const Held<D, W> &b) {
  Held<D, W> r;
  if constexpr (Held<D, W>::kBytes == 2) {
    r.w[0] = D::narrow(add_in_order<O>(D::widen((uint16_t)a.w[0]), D::widen((uint16_t)b.w[0])));
  } else {
#pragma unroll
    for (int i = 0; i < Held<D, W>::kWords; ++i) r.w[i] = add_word<D, O>(a.w[i], b.w[i]);
  }
  if constexpr (O == kOpaque) {
#pragma unroll
    for (int i = 0; i < Held<D, W>::kWords; ++i) asm("" : "+v"(r.w[i]));
  }
  return r;
}
// Sums of several sources: widened values, narrowed once.
template <class D, int W>
__device__ __forceinline__ AccV<D, W> widen_held(const Held<D, W> &a) {
  AccV<D, W> r;
  if constexpr (sizeof(typename D::S) == 4) {
#pragma unroll
    for (int i = 0; i < W; ++i) r.v[i] = D::widen(__builtin_bit_cast(typename D::S, a.w[i]));
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) r.v[i] = D::widen((uint16_t)(a.w[i / 2] >> (i % 2 * 16)));
  }
  return r;
}
// In slot 0 the accumulator stays first as it is; with kFixed its loop costs 8
// ranks of 2^21 fp32 elements 22.07 -> 22.42 us.
template <class D, int W, AddOrder O = kPlain>
__device__ __forceinline__ void accum_held(AccV<D, W> &acc, const Held<D, W> &b) {
  const AccV<D, W> x = widen_held<D, W>(b);
#pragma unroll
  for (int i = 0; i < W; ++i) acc.v[i] = add_in_order<O>(acc.v[i], x.v[i]);
}
template <class D, int W>
__device__ __forceinline__ Held<D, W> narrow_held(const AccV<D, W> &a) {
  Held<D, W> r;
  if constexpr (sizeof(typename D::S) == 4) {
#pragma unroll
    for (int i = 0; i < W; ++i) r.w[i] = __builtin_bit_cast(uint32_t, D::narrow(a.v[i]));
  } else if constexpr (W == 1) {
    r.w[0] = D::narrow(a.v[0]);
  } else {
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
      if constexpr (D::kPairs) r.w[i] = D::narrow_pair(a.v[2 * i], a.v[2 * i + 1]);
      else r.w[i] = (uint32_t)D::narrow(a.v[2 * i]) | (uint32_t)D::narrow(a.v[2 * i + 1]) << 16;
    }
  }
  return r;
}

// A wave-uniform address in scalar registers.  Without this, and without the
// accesses' opaque 32-bit lane offset, the compiler adds the uniform part to
// the lane offset instead: a 64-bit vector add per access, in place of the
// access's own scalar base + lane offset form.
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  asm volatile("" : "+s"(v));
  return v;
}
// Access at `base` (a rank's buffer, wave-uniform) + `off` bytes (uniform) +
// `lane` bytes.
template <class D, int W, bool NT>
__device__ __forceinline__ Held<D, W> cload(uint64_t base, int64_t off, uint32_t &lane) {
  using T = typename AccessOf<Held<D, W>::kBytes, sizeof(typename D::S)>::T;
  const OPTCC_GLOBAL_AS char *b = (const OPTCC_GLOBAL_AS char *)uniform(base + (uint64_t)off);
  asm("" : "+v"(lane));
  const OPTCC_GLOBAL_AS T *p = (const OPTCC_GLOBAL_AS T *)(b + lane);
  T v;
  if constexpr (NT) v = __builtin_nontemporal_load(p);
  else v = *p;
  Held<D, W> r;
  if constexpr (Held<D, W>::kWords == 1) {
    r.w[0] = v;
  } else {
#pragma unroll
    for (int i = 0; i < Held<D, W>::kWords; ++i) r.w[i] = v[i];
  }
  return r;
}
template <class D, int W, bool NT>
__device__ __forceinline__ void cstore(uint64_t base, int64_t off, uint32_t &lane,
                                       const Held<D, W> &x) {
  using T = typename AccessOf<Held<D, W>::kBytes, sizeof(typename D::S)>::T;
  OPTCC_GLOBAL_AS char *b = (OPTCC_GLOBAL_AS char *)uniform(base + (uint64_t)off);
  asm("" : "+v"(lane));
  OPTCC_GLOBAL_AS T *p = (OPTCC_GLOBAL_AS T *)(b + lane);
  T v;
  if constexpr (Held<D, W>::kWords == 1) {
    v = (T)x.w[0];
  } else {
#pragma unroll
    for (int i = 0; i < Held<D, W>::kWords; ++i) v[i] = x.w[i];
  }
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

typedef const OPTCC_CONST_AS uint64_t *PtrTable;

// Forget what the compiler knows about a table pointer, so that it loads the
// entries again (scalar cache) instead of keeping up to 2 H scalar registers.
__device__ __forceinline__ PtrTable fresh(PtrTable p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (PtrTable)v;
}
// The same for a trip count, so that the branches of one phase are not kept
// in scalar registers for the next.
__device__ __forceinline__ int fresh(int n) {
  asm volatile("" : "+s"(n));
  return n;
}
// Keeps a partial's store and the sum's store to the same address, and in
// that order: every step of the schedule writes its destination.
#define OPTCC_STEP_ORDER() asm volatile("" ::: "memory")

// f(t) for t in [T0, min(n, H)), in straight-line groups of kGroup where a
// whole group is below n (one uniform branch per group).  t is a compile-time
// constant in f from the start, so that arrays indexed by it are registers.
template <int T>
struct Hop {
  __device__ constexpr operator int() const { return T; }
};
// Marks the end of a branch's block: blocks that differ in the mark are not
// merged, which would turn the register arrays into indexed scratch memory.
#define OPTCC_BLOCK_MARK(ID) asm volatile("; hop %0" ::"i"(ID))
template <int T, int H, int U = 0, class F>
__device__ __forceinline__ void group_all(F &f) {
  if constexpr (U < kGroup && T + U < H) {
    f(Hop<T + U>());
    group_all<T, H, U + 1>(f);
  }
}
template <int T, int H, int U = 0, class F>
__device__ __forceinline__ void group_some(int n, F &f) {
  if constexpr (U < kGroup && T + U < H) {
    if (T + U < n) {
      f(Hop<T + U>());
      OPTCC_BLOCK_MARK(T + U);
      group_some<T, H, U + 1>(n, f);
    }
  }
}
template <int T, int H, class F>
__device__ __forceinline__ void groups(int n, F &f) {
  if constexpr (T < H) {
    if (T + kGroup <= n) {
      group_all<T, H>(f);
      OPTCC_BLOCK_MARK(1000 + T);
      groups<T + kGroup, H>(n, f);
    } else {
      group_some<T, H>(n, f);
    }
  }
}
template <int T0, int H, class F>
__device__ __forceinline__ void hops(int n, F f) {
  groups<T0, H>(fresh(n), f);
}

// The same with the t-th entry of a pointer table: f(t, rp[t]).  A group's
// entries come with one scalar load, whether or not all of them are used
// (ChainArgs has entries enough behind every chain), issued before the
// previous group's accesses.
struct Ptrs {
  uint64_t p[kGroup];
};
__device__ __forceinline__ Ptrs load_ptrs(PtrTable rp) {
  Ptrs r;
#pragma unroll
  for (int u = 0; u < kGroup; ++u) r.p[u] = rp[u];
  return r;
}
__device__ __forceinline__ void arrived(Ptrs &c) {
  asm volatile(""
               : "+s"(c.p[0]), "+s"(c.p[1]), "+s"(c.p[2]), "+s"(c.p[3]), "+s"(c.p[4]),
                 "+s"(c.p[5]), "+s"(c.p[6]), "+s"(c.p[7]));
}
template <int T, int H, class F>
__device__ __forceinline__ void ptr_groups(int n, PtrTable rp, Ptrs &c, F &f) {
  if constexpr (T < H) {
    Ptrs next;
    if constexpr (T + kGroup < H) next = load_ptrs(rp + T + kGroup);
    auto g = [&](auto t) __attribute__((always_inline)) { f(t, c.p[t - T]); };
    if (T + kGroup <= n) {
      group_all<T, H>(g);
      OPTCC_BLOCK_MARK(1000 + T);
      if constexpr (T + kGroup < H) {
        arrived(next);
        ptr_groups<T + kGroup, H>(n, rp, next, f);
      }
    } else {
      group_some<T, H>(n, g);
    }
  }
}
template <int T0, int H, class F>
__device__ __forceinline__ void ptr_hops(int n, PtrTable rp, F f) {
  rp = fresh(rp);
  Ptrs c = load_ptrs(rp + T0);
  arrived(c);
  ptr_groups<T0, H>(fresh(n), rp, c, f);
}

// Every step of one section's elements for the lanes that are active here.
// rp: the section's ranks R[j], R[j+1], .. (pp entries); sp: the stragglers.
template <class D, int W, int H, ChainPolicy POL>
__device__ __forceinline__ void chain_piece(PtrTable rp, PtrTable sp, int pp, int m, int ord,
                                            int64_t off, uint32_t lane) {
  using V = Held<D, W>;
  constexpr bool kNtL = POL != kResident, kNtM = POL == kStreaming, kNtF = POL != kResident;
  const int nside = m == 0 ? 0 : (ord == 2 ? m : m - 1);
  const int sfirst = ord == 2 ? 0 : 1;
  const bool fin = m >= 1 && ord == 1;
  V x[H];
  V xs;
  x[0] = cload<D, W, kNtL>(rp[0], off, lane);
  ptr_hops<1, H>(pp, rp, [&](auto t, uint64_t b) __attribute__((always_inline)) {
    x[t] = cload<D, W, kNtL>(b, off, lane);
  });
  if (fin) xs = cload<D, W, kNtL>(sp[0], off, lane);
  if (nside > 0) {  // slot 0: the stragglers' raw values into the chain start
    AccV<D, W> acc = widen_held<D, W>(x[0]);
    constexpr int kSide = 16 / V::kWords;  // loads in flight
    for (int i = 0; i < nside; i += kSide) {
      V s[kSide];
#pragma unroll
      for (int u = 0; u < kSide; ++u)
        if (i + u < nside) s[u] = cload<D, W, kNtL>(sp[sfirst + i + u], off, lane);
#pragma unroll
      for (int u = 0; u < kSide; ++u)
        if (i + u < nside) accum_held<D, W>(acc, s[u]);
    }
    x[0] = narrow_held<D, W>(acc);
  }
  V v = x[0];
  hops<1, H>(pp, [&](auto t) __attribute__((always_inline)) {  // slot 1
    v = add_held<D, W>(x[t], v);
    x[t] = v;
  });
  if (fin) v = add_held<D, W>(xs, v);  // slot 2

  rp = fresh(rp);
  if (nside > 0) cstore<D, W, kNtM>(rp[0], off, lane, x[0]);
  OPTCC_STEP_ORDER();
  cstore<D, W, kNtF>(rp[0], off, lane, v);
  // ranks 1 .. pp-2: the hop's partial, then the sum (slot 4); the holder
  // pp-1 the same when a straggler finalises (slot 3), else only the sum,
  // which is its hop's own result
  ptr_hops<1, H>(fin ? pp : pp - 1, rp, [&](auto t, uint64_t b) __attribute__((always_inline)) {
    cstore<D, W, kNtM>(b, off, lane, x[t]);
    OPTCC_STEP_ORDER();
    cstore<D, W, kNtF>(b, off, lane, v);
    OPTCC_STEP_ORDER();
  });
  if (fin) cstore<D, W, kNtF>(sp[0], off, lane, v);        // slot 2
  else cstore<D, W, kNtF>(rp[pp - 1], off, lane, v);
  for (int i = 0; i < nside; ++i) cstore<D, W, kNtF>(sp[sfirst + i], off, lane, v);  // slot 5
}

// One point-to-point chunk's elements: the straggler sums its own value and
// R[0..P'-1] in that order, rounding once, and broadcasts the result.
template <class D, int W, int H, ChainPolicy POL>
__device__ __forceinline__ void p2p_piece(PtrTable rp, PtrTable sp, int pp, int64_t off,
                                          uint32_t lane) {
  using V = Held<D, W>;
  constexpr bool kNtL = POL != kResident, kNtF = POL != kResident;
  V x[H];
  AccV<D, W> acc = widen_held<D, W>(cload<D, W, kNtL>(sp[0], off, lane));
  ptr_hops<0, H>(pp, rp, [&](auto t, uint64_t b) __attribute__((always_inline)) {
    x[t] = cload<D, W, kNtL>(b, off, lane);
  });
  hops<0, H>(pp, [&](auto t) __attribute__((always_inline)) {
    accum_held<D, W, kFixed>(acc, x[t]);
  });
  const V g = narrow_held<D, W>(acc);
  cstore<D, W, kNtF>(sp[0], off, lane, g);
  ptr_hops<0, H>(pp, rp, [&](auto t, uint64_t b) __attribute__((always_inline)) {
    cstore<D, W, kNtF>(b, off, lane, g);
  });
}

typedef const OPTCC_CONST_AS ChainArgs *ChainArgsPtr;

__device__ __forceinline__ uint32_t divide(uint32_t a, const OPTCC_CONST_AS ChainDiv *d) {
  const uint32_t t = __umulhi(a, d->m);
  return (t + ((a - t) >> d->s1)) >> d->s2;
}
// Where a quantum lies: its segment's ordering, its section (-1: the
// point-to-point chunk) and the first quantum past that section or chunk.
// Computed from the plan's few numbers instead of read from a tile table: two
// dependent loads from memory before a wave's first data load cost about a
// third of a short chain's wave time.
struct Place {
  int ord, j;
  uint32_t end;
};
__device__ __forceinline__ Place place_of(ChainArgsPtr a, uint32_t q) {
  uint32_t g, s0, s1;
  if (!a->wide) {
    // segment g starts at quantum floor(g nq / k)
    g = divide((q + 1) * a->k - 1, &a->by_nq);
    s0 = divide(g * a->nq, &a->by_k);
    s1 = divide((g + 1) * a->nq, &a->by_k);
  } else {
    g = (uint32_t)((((uint64_t)q + 1) * a->k - 1) / a->nq);
    s0 = (uint32_t)((uint64_t)g * a->nq / a->k);
    s1 = (uint32_t)(((uint64_t)g + 1) * a->nq / a->k);
  }
  const OPTCC_CONST_AS ChainSeg *sg = &a->seg[s1 - s0 > a->lq ? 1 : 0];
  const uint32_t u = q - s0, ring = s1 - s0 - sg->dq, big = sg->nbig * (sg->qbase + 1);
  Place r;
  r.ord = (a->ord2 >> (g & 3)) & 1 ? 2 : 1;
  if (u >= ring) {
    r.j = -1;
    r.end = s1;
  } else if (u < big) {
    r.j = (int)divide(u, &sg->by_big);
    r.end = s0 + ((uint32_t)r.j + 1) * (sg->qbase + 1);
  } else {
    const uint32_t i = divide(u - big, &sg->by_small);
    r.j = (int)(sg->nbig + i);
    r.end = s0 + big + (i + 1) * sg->qbase;
  }
  return r;
}

// Every step of the lanes' elements, section by section: the wave's quanta
// [q, qe), this lane's first element l * W from element x, in quantum ql.
template <class D, int W, int H, ChainPolicy POL>
__device__ __forceinline__ void chain_span(ChainArgsPtr a, uint32_t q, uint32_t qe, int64_t x,
                                           int l, uint32_t ql, bool whole) {
  constexpr int64_t kEs = sizeof(typename D::S);
  const int pp = a->pp, m = a->m;
  PtrTable rp = a->ptr;
  PtrTable sp = rp + 2 * pp;
  const uint32_t lane = (uint32_t)(l * W * kEs);
  while (q < qe) {
    const Place s = place_of(a, q);
    if (whole && ql >= q && ql < s.end) {
      if (s.j < 0) p2p_piece<D, W, H, POL>(rp, sp, pp, x * kEs, lane);
      else chain_piece<D, W, H, POL>(rp + s.j, sp, pp, m, s.ord, x * kEs, lane);
    }
    q = s.end;
  }
}

// Workgroups of at most this many threads: as many waves as the registers of
// one SIMD hold.
constexpr int chain_threads(int bytes, int h) {
  return bytes * h <= 256 ? 1024 : bytes * h <= 512 ? 512 : 256;
}

template <class D, int W, int H, ChainPolicy POL>
__global__ __launch_bounds__(chain_threads(W * (int)sizeof(typename D::S), H))
void optcc_chain_kernel(ChainArgsOf<chain_ptrs(H)>) {
  ChainArgsPtr a = (ChainArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t i = blockIdx.x;
  const uint32_t b = (i & ((1u << a->runs) - 1)) * (uint32_t)a->per_run + (i >> a->runs);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  const uint32_t nq = a->nq;
  const uint64_t q64 = ((uint64_t)b * a->waves + wave) * W;
  if (q64 >= nq) return;
  const uint32_t q = (uint32_t)q64, qe = nq - q < W ? nq : q + W;
  const int64_t x = (int64_t)q * kQuantum;
  chain_span<D, W, H, POL>(a, q, qe, x, l, q + (uint32_t)(l * W) / kQuantum,
                           x + l * W + W <= a->n);
  if constexpr (W > 1) {  // the rank vectors' last elements, less than a lane's W
    const int rest = (int)(a->n % W);
    if (qe == nq && rest)
      chain_span<D, 1, H, POL>(a, nq - 1, nq, a->n - rest, l, nq - 1, l < rest);
  }
}

}  // namespace kern
}  // namespace optcc
