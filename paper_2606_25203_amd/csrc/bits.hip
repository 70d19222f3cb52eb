// bits.hip -- sweeps of bit-packed populations, for sparse Ising instances
// whose couplings all have one magnitude c (Max-Cut graphs of unit weight,
// +-1 tori and the like).
//
// During a step's sweeps such an instance's spins are held one bit each: the
// 64 replicas of a tile are one 64-bit mask per vertex.  A wavefront reads a
// neighbour's mask with a scalar load and adds it to its lanes' counts with
// one add-with-carry (the mask is the carry-in), so a neighbour costs one
// vector instruction, no vector load and no field array.  The masks live in
// the population buffer that resampling leaves unused between two draws, so
// they take no memory of their own: k_bits_pack fills them from the spin
// words at the start of a step, k_bits_unpack_* write the spin words back and
// recompute the energies at its end.
//
// Measured against the forms they replaced (whole runs, MI355X): 100 x 200
// torus, R = 4096, 120 steps x 10 sweeps 130.6 -> 89.4 ms (a class phase 49.7
// -> 28 us, of which 23 us are its vector instructions; pack 25 us and unpack
// 40 us a step); G(11999, average degree 34), R = 512, 60 steps x 5 sweeps,
// incremental fields before, 63.6 -> 30.6 ms; 48 mixed instances in a batch
// 82.9 -> 46.4 ms; 32 served requests 322 -> 199 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>

#include "bit_rows.hpp"
#include "instance.hpp"
#include "pamc_device.hpp"

namespace pamc {

namespace {

constexpr int kBitWaves = 4;       // waves per work-group
constexpr int kBitQuads = 8;       // vertex quads per wave of the pack kernel
constexpr int kBitTab = 2 * (2 * kBitsMaxDegree + 2);  // threshold entries, staged in LDS
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Lane L of v becomes s.  The intrinsic, not inline asm: the compiler then
// keeps the wait states between a compare that writes s and this read of it.
extern "C" __device__ uint32_t llvm_writelane(uint32_t s, uint32_t lane, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
template <int L>
__device__ __forceinline__ void put_lane(uint32_t& v, uint32_t s) {
  v = llvm_writelane(s, L, v);
}

__device__ __forceinline__ bool lane_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

template <int G>
struct Masks {
  typedef uint64_t type __attribute__((ext_vector_type(G)));
};
template <>
struct Masks<1> {
  typedef uint64_t type;
};

template <int G>
__device__ __forceinline__ uint64_t mask_of(const typename Masks<G>::type& m, int t) {
  if constexpr (G == 1)
    return m;
  else
    return m[t];
}

// Adds N masks (1 or 4) to the lanes' counts, an instruction each with the mask
// as the carry-in; from C the compiler makes one and a half.  It keeps no wait
// states before inline assembly between a vector instruction that writes a
// scalar register (a spilled one read back, a compare) and a vector
// instruction that reads it: the s_nop does, two of them.
#define PAMC_ADDC(a, m) "v_addc_co_u32_e64 %" #a ", vcc, %" #a ", 0, %" #m "\n\t"
template <int G, int N>
__device__ __forceinline__ void count_masks(const typename Masks<G>::type* m, uint32_t (&acc)[G]) {
  static_assert((N == 1 || N == 4) && (G == 1 || G == 2 || G == 4), "");
  auto at = [&](int u, int t) { return mask_of<G>(m[u], t); };
  if constexpr (N == 1 && G == 1) {
    asm("s_nop 1\n\t" PAMC_ADDC(0, 1) : "+v"(acc[0]) : "s"(at(0, 0)) : "vcc");
  } else if constexpr (N == 1 && G == 2) {
    asm("s_nop 1\n\t" PAMC_ADDC(0, 2) PAMC_ADDC(1, 3)
        : "+v"(acc[0]), "+v"(acc[1])
        : "s"(at(0, 0)), "s"(at(0, 1))
        : "vcc");
  } else if constexpr (N == 1) {
    asm("s_nop 1\n\t" PAMC_ADDC(0, 4) PAMC_ADDC(1, 5) PAMC_ADDC(2, 6) PAMC_ADDC(3, 7)
        : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
        : "s"(at(0, 0)), "s"(at(0, 1)), "s"(at(0, 2)), "s"(at(0, 3))
        : "vcc");
  } else if constexpr (G == 1) {
    asm("s_nop 1\n\t" PAMC_ADDC(0, 1) PAMC_ADDC(0, 2) PAMC_ADDC(0, 3) PAMC_ADDC(0, 4)
        : "+v"(acc[0])
        : "s"(at(0, 0)), "s"(at(1, 0)), "s"(at(2, 0)), "s"(at(3, 0))
        : "vcc");
  } else {
#pragma unroll
    for (int t = 0; t < G; t += 2)
      asm("s_nop 1\n\t" PAMC_ADDC(0, 2) PAMC_ADDC(1, 3) PAMC_ADDC(0, 4) PAMC_ADDC(1, 5)
          PAMC_ADDC(0, 6) PAMC_ADDC(1, 7) PAMC_ADDC(0, 8) PAMC_ADDC(1, 9)
          : "+v"(acc[t]), "+v"(acc[t + 1])
          : "s"(at(0, t)), "s"(at(0, t + 1)), "s"(at(1, t)), "s"(at(1, t + 1)), "s"(at(2, t)), "s"(at(2, t + 1)),
            "s"(at(3, t)), "s"(at(3, t + 1))
          : "vcc");
  }
}
#undef PAMC_ADDC

// N byte offsets of masks in a group of one tile (times G in a group of G),
// read at any entry.
template <int N>
using Offsets = int32_t __attribute__((ext_vector_type(N)));
template <int N>
struct OffsetsAt {
  typedef int32_t type __attribute__((ext_vector_type(N), aligned(4)));
};

template <int N>
__device__ __forceinline__ Offsets<N> load_offsets(const PAMC_CONST int32_t* ent) {
  return *reinterpret_cast<const PAMC_CONST typename OffsetsAt<N>::type*>(ent);
}

// Counts of a row's entries e .. e1 - 1, the first N offsets given.  N masks
// are in flight at a time, with the next N offsets behind them, so a chunk
// costs one round trip.  Entries past e1 are read (ent is padded) and not
// counted; with WHOLE, e1 - e is a multiple of 4 and they are told apart by
// blocks of 4.
template <int G, int N, bool WHOLE>
__device__ __forceinline__ void count_row(const PAMC_CONST char* B, const PAMC_CONST int32_t* ent, int e, int e1,
                                          Offsets<N> at, uint32_t (&acc)[G]) {
  using M = typename Masks<G>::type;
  for (;;) {
    M m[N];
#pragma unroll
    for (int u = 0; u < N; ++u) m[u] = *reinterpret_cast<const PAMC_CONST M*>(B + (uint32_t)at[u] * (uint32_t)G);
    const bool more = e + N < e1;
    if (more) at = load_offsets<N>(ent + e + N);
    constexpr int S = WHOLE ? 4 : 1;
#pragma unroll
    for (int u = 0; u < N; u += S)
      if (e + u < e1) count_masks<G, S>(&m[u], acc);
    if (!more) return;
    e += N;
  }
}

// The descriptor and local block of a work-group: of a lone instance (no
// map) from the kernel's own arguments, kLoneOffset bytes into them, which
// spares two dependent reads at the start of every launch.
constexpr int kLoneOffset = 64;
__device__ __forceinline__ const PAMC_CONST BitDesc* bit_desc(const uint64_t* map, const BitDesc* D, int& lb) {
  if (!map) {
    lb = blockIdx.x;
    return (const PAMC_CONST BitDesc*)((const PAMC_CONST char*)__builtin_amdgcn_kernarg_segment_ptr() + kLoneOffset);
  }
  const uint64_t word = cmem(map)[blockIdx.x];
  lb = (int)(uint32_t)word;  // -1: padding block
  return cmem(D) + (int)(word >> 32);
}

// local block -> (tile group, chunk): as in the other sweep kernels, a
// group's blocks stay 8 apart (one XCD) when the group count is a multiple
// of 8.
__device__ __forceinline__ void group_chunk(int G, int lb, int& group, int& chunk) {
  if ((G & 7) == 0) {
    const int xcd = lb & 7, j = lb >> 3, gp = G >> 3;
    group = (j % gp) * 8 + xcd;
    chunk = j / gp;
  } else {
    group = lb % G;
    chunk = lb / G;
  }
}

template <int G, int K>
__device__ __forceinline__ void put_masks(uint32_t& lo, uint32_t& hi, const uint64_t (&m)[G]) {
  put_lane<K * G>(lo, (uint32_t)m[0]);
  put_lane<K * G>(hi, (uint32_t)(m[0] >> 32));
  if constexpr (G > 1) {
    put_lane<K * G + 1>(lo, (uint32_t)m[1]);
    put_lane<K * G + 1>(hi, (uint32_t)(m[1] >> 32));
  }
  if constexpr (G > 2) {
    put_lane<K * G + 2>(lo, (uint32_t)m[2]);
    put_lane<K * G + 2>(hi, (uint32_t)(m[2] >> 32));
    put_lane<K * G + 3>(lo, (uint32_t)m[3]);
    put_lane<K * G + 3>(hi, (uint32_t)(m[3] >> 32));
  }
}

// ---------------------------------------------------------------------------
// One colour class of one sweep (Eqs. 3-4) on the masks, of G tiles; lane =
// replica.  The neighbours' masks hold, per replica, whether the neighbour
// pulls this vertex up (J s_j = +c; with one sign of coupling, whether s_j =
// +1, and the table's halves are exchanged when that sign is negative), so
// with count m of deg neighbours the field is c (2 m - deg).  The threshold
// table in LDS holds T[c (i - X)] and its mirror image, entry i of either
// half at byte 4 i; the spin picks the half, through the start value of the
// count.  The vertices of a class are uncoupled and only they are written, so
// no mask that is read as a neighbour's changes during the launch, and scalar
// loads may read them.
// ---------------------------------------------------------------------------
// Keeps a uniform value in scalar registers from here on.
template <typename T>
__device__ __forceinline__ T pinned(T x) {
  asm volatile("" : "+s"(x));
  return x;
}

// What both forms below read at their start.
template <int G>
struct Phase {
  const PAMC_CONST BitDesc* d;
  int v0, v1, q0, items;  // the class's vertices and quads
  uint32_t gs, plane;     // stream index; bytes of one copy of a group's masks
  int group, chunk, lane, wave;
  char* Bw;
  const PAMC_CONST char* B;
  bool two;
  uint32_t half8;  // start of the count for spins +1: the table's second half, in units of 8 bytes

  // false: nothing to do for this work-group; else tab_s holds the table
  // after the work-group's next barrier
  __device__ __forceinline__ bool open(const uint64_t* map, const BitDesc* D, int sweep_idx, int phase,
                                       uint32_t* tab_s, int quads_per_block) {
    int lb;
    d = bit_desc(map, D, lb);
    if (lb < 0 || phase >= d->ncls || sweep_idx >= d->order_cap) return false;
    const i32x4 rec = cmem(reinterpret_cast<const i32x4*>(d->phases))[sweep_idx * d->ncls + phase];
    for (int i = threadIdx.x; i < 2 * d->tab_half; i += 64 * kBitWaves) tab_s[i] = gmem(d->tab)[i];
    group_chunk(d->T / G, lb, group, chunk);
    v0 = rec.x;
    v1 = rec.y;  // equal: nothing to do in this step
    gs = (uint32_t)rec.z;
    q0 = v0 >> 2;
    items = ((v1 + 3) >> 2) - q0;
    if (v0 >= v1 || chunk * quads_per_block * d->qpw >= items) return false;
    plane = (uint32_t)(d->np + 1) * 8 * G;
    two = d->copies == 2;
    Bw = (char*)(rec.w ? d->S0 : d->S1) + (size_t)group * (two ? 2 * plane : plane);
    B = cmem((const char*)Bw);
    half8 = (uint32_t)d->tab_half >> 1;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return true;
  }

  // Philox words of quad q for the lane's replica of tile t; k0, k1: the
  // stream's key.
  __device__ __forceinline__ u32x4 draw(int q, int t, uint32_t k0, uint32_t k1) const {
    return philox10((uint32_t)q, gs, (uint32_t)((group * G + t) * kLanes + lane), kTagSweep, k0, k1);
  }

  __device__ __forceinline__ typename Masks<G>::type own(int v) const {
    typename Masks<G>::type m = *reinterpret_cast<const PAMC_CONST typename Masks<G>::type*>(B + (uint32_t)(v * 8 * G));
    // this wave overwrites these masks later: they are not to be read again
    asm volatile("" : "+s"(m));
    return m;
  }

  __device__ __forceinline__ void start(const typename Masks<G>::type& own, uint32_t (&acc)[G]) const {
#pragma unroll
    for (int t = 0; t < G; ++t) acc[t] = lane_bit(mask_of<G>(own, t)) ? half8 : 0u;
  }

  // New mask of tile t from its counts and random words; base: the vertex's
  // table offset.
  template <bool METRO>
  __device__ __forceinline__ uint64_t decide(const uint32_t* tab_s, int t, uint32_t acc, int32_t base, uint32_t u,
                                             const typename Masks<G>::type& own, int32_t& nflip) const {
    const uint32_t at = (acc << 3) + (uint32_t)base;  // byte offset in the table
    const uint32_t T = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(tab_s) + at);
    uint64_t flip = __builtin_amdgcn_ballot_w64(u < T);
    if constexpr (METRO)  // x <= 0 always flips: entries le_first .. le_first + le_span (or the others)
      flip |= __builtin_amdgcn_ballot_w64(at - d->le_first <= d->le_span) ^ d->le_xor;
    nflip += __builtin_popcountll(flip);
    return mask_of<G>(own, t) ^ flip;
  }

  // Lane i < COUNT G writes the mask of vertex vb + i / G, tile i % G.
  template <int COUNT>
  __device__ __forceinline__ void store(int vb, uint32_t lo, uint32_t hi) const {
    const int v = vb + lane / G;
    if (lane < COUNT * G && v >= v0 && v < v1) {
      PAMC_GLOBAL char* p = gmem(Bw) + (uint32_t)(v * 8 * G + 8 * (lane % G));
      const uint64_t m = lo | (uint64_t)hi << 32;
      *(PAMC_GLOBAL uint64_t*)p = m;
      if (two) *(PAMC_GLOBAL uint64_t*)(p + plane) = ~m;  // the complement, read along negative couplings
    }
  }

  __device__ __forceinline__ void count_flips(int32_t nflip) const {
    if (d->flip_ctr && lane == 0)
      __hip_atomic_fetch_add((unsigned long long*)&d->flip_ctr[blockIdx.x & 255], (unsigned long long)nflip,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// A quad per work-group, a vertex per wave: wave w draws the random words of
// tile w (waves past the group's tiles none) and passes them on through LDS,
// so the quad's Philox blocks are still computed once, while a launch is as
// long as one vertex's row.
template <int G, bool METRO>
__global__ void __launch_bounds__(64 * kBitWaves) k_sweep_bits_quad(const uint64_t* __restrict__ map,
                                                                    const BitDesc* __restrict__ D, int sweep_idx,
                                                                    int phase, BitDesc) {
  using M = typename Masks<G>::type;
  __shared__ uint32_t tab_s[kBitTab];
  __shared__ uint32_t rnd_s[2][G][4][kLanes];
  Phase<G> ph;
  if (!ph.open(map, D, sweep_idx, phase, tab_s, 1)) return;
  const PAMC_CONST BitDesc& d = *ph.d;
  const PAMC_CONST int32_t* ent = cmem(d.ent);
  const PAMC_CONST i32x2* rows = cmem(reinterpret_cast<const i32x2*>(d.rows));
  const PAMC_CONST int32_t* bases = cmem(d.base);
  const int es = d.row_stride, qpw = d.qpw;
  const uint32_t k0 = d.k0, k1 = d.k1;
  constexpr int N = G == 4 ? 8 : 16;  // masks in flight: up to 64 scalar registers
  int32_t nflip = 0;
  for (int i = 0; i < qpw; ++i) {
    const int it = ph.chunk * qpw + i;
    if (it >= ph.items) break;
    const int v = 4 * (ph.q0 + it) + ph.wave;
    const bool in = v >= ph.v0 && v < ph.v1;
    // rows of one stride are found without the row bounds, whose read then
    // overlaps the entries'
    Offsets<N> at{};
    i32x2 row{};
    int32_t base = 0;
    M own{};
    if (in) {
      if (es) at = load_offsets<N>(ent + v * es);
      row = rows[v];
      base = bases[v];
      own = ph.own(v);
    }
    if (ph.wave < G) {
      // the round keys are summed anew for each quad, not kept over the loop
      const u32x4 w = ph.draw(ph.q0 + it, ph.wave, pinned(k0), pinned(k1));
#pragma unroll
      for (int k = 0; k < 4; ++k) rnd_s[i & 1][ph.wave][k][ph.lane] = pick(w, k);
    }
    uint32_t acc[G];
    if (in) {
      if (!es) at = load_offsets<N>(ent + row.x);
      ph.start(own, acc);
      if (row.x < row.y) count_row<G, N, true>(ph.B, ent, row.x, row.y, at, acc);
    }
    __syncthreads();  // the words are in; the buffer of two quads ago is free again
    if (in) {
      uint32_t lo = 0, hi = 0;
      uint64_t nm[G];
#pragma unroll
      for (int t = 0; t < G; ++t)
        nm[t] = ph.template decide<METRO>(tab_s, t, acc[t], base, rnd_s[i & 1][t][ph.wave][ph.lane], own, nflip);
      put_masks<G, 0>(lo, hi, nm);
      ph.template store<1>(v, lo, hi);
    }
  }
  ph.count_flips(nflip);
}

// Instances whose rows all have at most four entries (grids), where they
// fill the chip: a quad per wave, its entries in one load, each vertex's masks
// on their way while the one before is decided.  Bound by vector issue: per
// visit 10 instructions of Philox, four additions and 7 for the table lookup,
// decision and mask write.
template <int G, bool METRO>
__global__ void __launch_bounds__(64 * kBitWaves) k_sweep_bits_grid(const uint64_t* __restrict__ map,
                                                                    const BitDesc* __restrict__ D, int sweep_idx,
                                                                    int phase, BitDesc) {
  using M = typename Masks<G>::type;
  __shared__ uint32_t tab_s[kBitTab];
  Phase<G> ph;
  if (!ph.open(map, D, sweep_idx, phase, tab_s, kBitWaves)) return;
  const int qpw = ph.d->qpw;
  // held in registers: reading them again would add a round trip per quad
  const PAMC_CONST int32_t* ent = pinned(cmem(ph.d->ent));
  const PAMC_CONST int32_t* bases = pinned(cmem(ph.d->base));
  const uint32_t k0 = pinned(ph.d->k0), k1 = pinned(ph.d->k1);
  int32_t nflip = 0;
  __syncthreads();
  for (int i = 0; i < qpw; ++i) {
    const int it = ph.chunk * (kBitWaves * qpw) + i * kBitWaves + ph.wave;
    if (it >= ph.items) break;
    const int vb = 4 * (ph.q0 + it);
    const Offsets<16> at = load_offsets<16>(ent + 4 * vb);
    const i32x4 base = *reinterpret_cast<const PAMC_CONST i32x4*>(bases + vb);
    uint32_t lo = 0, hi = 0;
    u32x4 rnd[G];
    M m[4], oa, ob;
    uint32_t acc[G];
    auto fetch = [&](int k, M& own) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        m[u] = *reinterpret_cast<const PAMC_CONST M*>(ph.B + (uint32_t)at[4 * k + u] * (uint32_t)G);
      own = ph.own(vb + k);
    };
    auto count = [&](const M& own) {
      ph.start(own, acc);
      count_masks<G, 4>(m, acc);
    };
    auto decide = [&](auto K, const M& own) {
      constexpr int k = decltype(K)::value;
      uint64_t nm[G];
      int32_t flips = 0;
#pragma unroll
      for (int t = 0; t < G; ++t)
        nm[t] = ph.template decide<METRO>(tab_s, t, acc[t], base[k], pick(rnd[t], k), own, flips);
      put_masks<G, k>(lo, hi, nm);
      nflip += vb + k >= ph.v0 && vb + k < ph.v1 ? flips : 0;
    };
    // vertices of the quad outside the class are decided too, and neither
    // counted nor written
    fetch(0, oa);
    const uint32_t a0 = pinned(k0), a1 = pinned(k1);
#pragma unroll
    for (int t = 0; t < G; ++t) rnd[t] = ph.draw(ph.q0 + it, t, a0, a1);
    count(oa);
    fetch(1, ob);
    decide(std::integral_constant<int, 0>(), oa);
    count(ob);
    fetch(2, oa);
    decide(std::integral_constant<int, 1>(), ob);
    count(oa);
    fetch(3, ob);
    decide(std::integral_constant<int, 2>(), oa);
    count(ob);
    decide(std::integral_constant<int, 3>(), ob);
    ph.template store<4>(vb, lo, hi);
  }
  ph.count_flips(nflip);
}

// Lane l of (lo, hi) becomes the mask of the replicas whose vertex l of the
// wave's words has spin +1.
template <size_t... L>
__device__ __forceinline__ void put_signs(uint32_t& lo, uint32_t& hi, const uint32_t (&w)[kBitQuads],
                                          std::index_sequence<L...>) {
  auto put = [&](auto l) {
    constexpr int x = decltype(l)::value;
    const uint64_t m = __builtin_amdgcn_ballot_w64(((w[x / 4] >> (8 * (x % 4) + 7)) & 1u) == 0u);
    put_lane<x>(lo, (uint32_t)m);
    put_lane<x>(hi, (uint32_t)(m >> 32));
  };
  (put(std::integral_constant<int, (int)L>()), ...);
}

// ---------------------------------------------------------------------------
// Spin words -> masks at the start of a step, for one tile per wave and
// kBitQuads quads; energies are cleared for k_bits_unpack's sums, and the
// mask after the last vertex (which padding entries of the rows name) is 0.
// Bound by the read of the spin words (one byte per spin).
// ---------------------------------------------------------------------------
template <int G>
__global__ void __launch_bounds__(64 * kBitWaves) k_bits_pack(const uint64_t* __restrict__ map,
                                                              const BitDesc* __restrict__ D, BitDesc) {
  int lb;
  const PAMC_CONST BitDesc& d = *bit_desc(map, D, lb);
  if (lb < 0) return;
  const PAMC_CONST RunState* st = cmem((const RunState*)d.st);
  if (!st->active || st->nsweeps_now <= 0) return;
  const int cur = st->cur;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int group, chunk;
  group_chunk(d.T / G, lb, group, chunk);
  const uint32_t plane = (uint32_t)(d.np + 1) * 8 * G;
  const bool two = d.copies == 2;
  const PAMC_GLOBAL uint32_t* __restrict__ S = gmem((const uint32_t*)(cur ? d.S1 : d.S0));
  PAMC_GLOBAL char* B = gmem((char*)(cur ? d.S0 : d.S1)) + (size_t)group * (two ? 2 * plane : plane);
  // the work-group's 4 kBitQuads quads of its G tiles: wave w takes quads
  // w kBitQuads ..
  const int qb = (chunk * kBitWaves + wave) * kBitQuads;
#pragma unroll
  for (int t = 0; t < G; ++t) {
    const int tile = group * G + t;
    uint32_t w[kBitQuads];
#pragma unroll
    for (int i = 0; i < kBitQuads; ++i)
      w[i] = qb + i < d.nq ? S[((size_t)tile * d.nq + qb + i) * kLanes + lane] : 0u;
    // lane 4 i + k collects the mask of vertex 4 (qb + i) + k: bit 7 of a
    // spin's byte is its sign
    uint32_t lo = 0, hi = 0;
    put_signs(lo, hi, w, std::make_index_sequence<4 * kBitQuads>());
    const int v = 4 * qb + lane;
    if (lane < 4 * kBitQuads && v < d.np) {
      PAMC_GLOBAL char* p = B + (uint32_t)(v * 8 * G + 8 * t);
      const uint64_t m = lo | (uint64_t)hi << 32;
      *(PAMC_GLOBAL uint64_t*)p = m;
      if (two) *(PAMC_GLOBAL uint64_t*)(p + plane) = ~m;
    }
    if (chunk == 0 && wave == 0) {
      gmem(cur ? d.E1 : d.E0)[tile * kLanes + lane] = 0;
      if (lane < d.copies) *(PAMC_GLOBAL uint64_t*)(B + lane * plane + (uint32_t)(d.np * 8 * G + 8 * t)) = 0;
    }
  }
}

// ---------------------------------------------------------------------------
// Masks -> spin words at the end of a step, and the energies H = -sum_{i<j}
// J s_i s_j: each edge is counted at its end with the lower internal id (the
// rows list their higher neighbours first).  In both forms a work-group takes
// unpack_qpw quads per wave (grids) or per work-group (vertex k of the quad
// to wave k, tile t's spin word to wave t), then adds its sums to the
// energies.  Bound by the write of the spin words where the instance is
// large, by the chain of row reads of one vertex where it is small.
// ---------------------------------------------------------------------------
template <int G>
struct Unpack {
  const PAMC_CONST BitDesc* d;
  int cur, group, chunk, lane, wave;
  const PAMC_CONST char* B;

  __device__ __forceinline__ bool open(const uint64_t* map, const BitDesc* D) {
    int lb;
    d = bit_desc(map, D, lb);
    if (lb < 0) return false;
    const PAMC_CONST RunState* st = cmem((const RunState*)d->st);
    if (!st->active || st->nsweeps_now <= 0) return false;
    cur = st->cur;
    group_chunk(d->T / G, lb, group, chunk);
    B = cmem((const char*)(cur ? d->S0 : d->S1)) +
        (size_t)group * ((uint32_t)(d->np + 1) * 8 * G * (uint32_t)d->copies);
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return true;
  }

  __device__ __forceinline__ void write_word(int q, int t, uint32_t w) const {
    PAMC_GLOBAL uint32_t* S = gmem(cur ? d->S1 : d->S0);
    S[((size_t)(group * G + t) * d->nq + q) * kLanes + lane] = w;
  }

  // byte k of the spin word of vertex 4 q + k, from its mask (padding: 0)
  __device__ __forceinline__ uint32_t byte(int q, int k, uint64_t m) const {
    return 4 * q + k < d->n ? (lane_bit(m) ? 0x01u : 0xFFu) << (8 * k) : 0u;
  }

  // e2: per tile, sum over the wave's vertices and their higher neighbours
  // of J s_i s_j / c
  __device__ __forceinline__ void add_energies(int32_t (*red)[G][kLanes], const int32_t (&e2)[G]) const {
#pragma unroll
    for (int t = 0; t < G; ++t) red[wave][t][lane] = e2[t];
    __syncthreads();
    if (wave < G) {
      int64_t sum = 0;
#pragma unroll
      for (int x = 0; x < kBitWaves; ++x) sum += red[x][wave][lane];
      if (sum != 0)
        __hip_atomic_fetch_add((unsigned long long*)&gmem(cur ? d->E1 : d->E0)[(group * G + wave) * kLanes + lane],
                               (unsigned long long)(-(int64_t)d->coupling * sum), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};

template <int G>
__global__ void __launch_bounds__(64 * kBitWaves) k_bits_unpack_quad(const uint64_t* __restrict__ map,
                                                                     const BitDesc* __restrict__ D, BitDesc) {
  using M = typename Masks<G>::type;
  __shared__ int32_t red[kBitWaves][G][kLanes];
  Unpack<G> u;
  if (!u.open(map, D)) return;
  const PAMC_CONST BitDesc& d = *u.d;
  const PAMC_CONST int32_t* ent = cmem(d.ent);
  const int uq = d.unpack_qpw, es = d.row_stride;
  constexpr int N = G == 4 ? 8 : 16;
  int32_t e2[G];
#pragma unroll
  for (int t = 0; t < G; ++t) e2[t] = 0;
  for (int i = 0; i < uq; ++i) {
    const int q = u.chunk * uq + i;
    if (q >= d.nq) break;
    const int v = 4 * q + u.wave;
    const int first = es ? v * es : cmem(d.rows)[2 * v], up = cmem(d.higher)[v];
    const Offsets<N> at = load_offsets<N>(ent + first);
    const M own = *reinterpret_cast<const PAMC_CONST M*>(u.B + (uint32_t)(v * 8 * G));
    if (u.wave < G) {
      uint32_t w = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        w |= u.byte(q, k, *reinterpret_cast<const PAMC_CONST uint64_t*>(
                             u.B + (uint32_t)((4 * q + k) * 8 * G + 8 * u.wave)));
      u.write_word(q, u.wave, w);
    }
    if (up > 0) {
      uint32_t acc[G];
#pragma unroll
      for (int t = 0; t < G; ++t) acc[t] = 0;
      count_row<G, N, false>(u.B, ent, first, first + up, at, acc);
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const int32_t f = 2 * (int32_t)acc[t] - up;
        e2[t] += lane_bit(mask_of<G>(own, t)) ? f : -f;
      }
    }
  }
  u.add_energies(red, e2);
}

template <int G>
__global__ void __launch_bounds__(64 * kBitWaves) k_bits_unpack_grid(const uint64_t* __restrict__ map,
                                                                     const BitDesc* __restrict__ D, BitDesc) {
  using M = typename Masks<G>::type;
  __shared__ int32_t red[kBitWaves][G][kLanes];
  Unpack<G> u;
  if (!u.open(map, D)) return;
  const PAMC_CONST BitDesc& d = *u.d;
  const int uq = d.unpack_qpw;
  int32_t e2[G];
#pragma unroll
  for (int t = 0; t < G; ++t) e2[t] = 0;
  for (int i = 0; i < uq; ++i) {
    const int q = (u.chunk * uq + i) * kBitWaves + u.wave;
    if (q >= d.nq) break;
    const Offsets<16> at = load_offsets<16>(cmem(d.ent) + 16 * q);
    const i32x4 up = *reinterpret_cast<const PAMC_CONST i32x4*>(cmem(d.higher) + 4 * q);
    M own[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) own[k] = *reinterpret_cast<const PAMC_CONST M*>(u.B + (uint32_t)((4 * q + k) * 8 * G));
#pragma unroll
    for (int t = 0; t < G; ++t) {
      uint32_t w = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) w |= u.byte(q, k, mask_of<G>(own[k], t));
      u.write_word(q, t, w);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (up[k] == 0) continue;
      M m[4];
#pragma unroll
      for (int x = 0; x < 4; ++x)
        m[x] = *reinterpret_cast<const PAMC_CONST M*>(u.B + (uint32_t)at[4 * k + x] * (uint32_t)G);
      uint32_t acc[G];
#pragma unroll
      for (int t = 0; t < G; ++t) acc[t] = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (x < up[k]) count_masks<G, 1>(&m[x], acc);
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const int32_t f = 2 * (int32_t)acc[t] - up[k];
        e2[t] += lane_bit(mask_of<G>(own[k], t)) ? f : -f;
      }
    }
  }
  u.add_energies(red, e2);
}

}  // namespace

int32_t bits_work_groups(int32_t quads, int32_t qpw, bool quad_per_block) {
  const int32_t per = (quad_per_block ? 1 : kBitWaves) * qpw;
  return (quads + per - 1) / per;
}
int32_t bits_pack_chunks(int32_t nq) { return bits_work_groups(nq, kBitQuads, false); }

void launch_bits_sweep(int rule, int form, const BitLaunch& b, int grid, int sweep, int phase, hipStream_t s) {
  using Kernel = void (*)(const uint64_t*, const BitDesc*, int, int, BitDesc);
  static const Kernel k[2][Batch::kBitForms] = {
      {k_sweep_bits_quad<1, false>, k_sweep_bits_quad<2, false>, k_sweep_bits_quad<4, false>,
       k_sweep_bits_grid<1, false>, k_sweep_bits_grid<2, false>, k_sweep_bits_grid<4, false>},
      {k_sweep_bits_quad<1, true>, k_sweep_bits_quad<2, true>, k_sweep_bits_quad<4, true>, k_sweep_bits_grid<1, true>,
       k_sweep_bits_grid<2, true>, k_sweep_bits_grid<4, true>}};
  k[rule][form]<<<grid, 64 * kBitWaves, 0, s>>>(b.map, b.D, sweep, phase, b.lone);
}

void launch_bits_pack(int form, const BitLaunch& b, int grid, bool pack, hipStream_t s) {
  using Kernel = void (*)(const uint64_t*, const BitDesc*, BitDesc);
  static const Kernel k[2][Batch::kBitForms] = {
      {k_bits_unpack_quad<1>, k_bits_unpack_quad<2>, k_bits_unpack_quad<4>, k_bits_unpack_grid<1>,
       k_bits_unpack_grid<2>, k_bits_unpack_grid<4>},
      {k_bits_pack<1>, k_bits_pack<2>, k_bits_pack<4>, k_bits_pack<1>, k_bits_pack<2>, k_bits_pack<4>}};
  k[pack ? 1 : 0][form]<<<grid, 64 * kBitWaves, 0, s>>>(b.map, b.D, b.lone);
}

}  // namespace pamc
