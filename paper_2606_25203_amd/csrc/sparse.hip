// sparse.hip -- gfx950 kernels of the sparse PAMC path and of the
// device-side controller (Algorithm 1), with their batch launchers.
//
// Every kernel works on a batch of instances: it reads the instance's
// descriptor (Desc) and its device-resident run state, and grid kernels map
// blockIdx through a per-batch table to (instance, local block).  A single
// instance is a batch of one, so one code path serves the plain, batched and
// served modes.  One beta step of Algorithm 1 is a fixed launch sequence
// whose behaviour is decided on the device from RunState, so the host never
// waits inside a run:
//   step_begin -> rs_select -> rs_gather -> cl_select -> cl_mis -> cl_apply
//   -> commit -> thresholds -> S x K sweep phases -> step_end
// Kernels with nothing to do for an instance return at once.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "instance.hpp"
#include "pamc_device.hpp"

namespace pamc {

namespace {

constexpr int kSweepWaves = 4;             // waves per sweep workgroup
constexpr int kMaxQuadsPerWave = 4;        // quads per wave per sweep work-group: 1, 2 or 4 (Desc::qpw)
constexpr int kPushWorkGroups = 2048;      // incremental-field sweep work-groups of a lone instance (8 per CU)
constexpr int kPushMinWorkGroups = 512;    // ... and the least per instance of a batch
constexpr int kGatherQuadsPerBlock = 64;
constexpr int kClusterMaxN = 26000;        // LDS: 5 bytes per vertex
constexpr int kRsMaxR = 16384;
constexpr int kThrLds = 2048;              // threshold entries staged in LDS when they fit
constexpr int kThrBlocks = 16;             // threshold work-groups per instance
constexpr int kLongRow = 512;              // entries from which a row's field is summed by four waves
constexpr int kOrderLds = 2048;            // class-order entries shuffled in LDS at a time
constexpr int kInitBlocks = 64;            // spin-init work-groups per instance
constexpr int kApplyChunks = 16;           // cluster-apply work-groups per target
constexpr int kFieldBlocks = 1024;         // max field-init work-groups per instance
constexpr uint32_t kIdle = 0xFFFFFFFFu;    // padding block: returns at once
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));  // at any entry
typedef int i32x8u __attribute__((ext_vector_type(8), aligned(4)));
constexpr int kBufferWord3 = 0x00020000;   // buffer resource word 3: 32-bit raw data

// Map word: instance index in the high half, local block in the low half.
__device__ __forceinline__ bool resolve(const uint64_t* __restrict__ map, int& inst, int& lb) {
  const uint64_t m = map[blockIdx.x];
  inst = (int)(m >> 32);
  lb = (int)(uint32_t)m;
  return (uint32_t)m != kIdle;
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ int32_t spin_at(const uint32_t* S, int nq, int tile, int v, int lane) {
  const uint32_t w = S[((size_t)tile * nq + (v >> 2)) * kLanes + lane];
  return (int32_t)(int8_t)(w >> (8 * (v & 3)));
}

// local block -> (tile group, chunk).  Work-groups are dealt round-robin to
// the eight XCDs in launch order; an instance's blocks start at a multiple of
// 8 in its map, so keeping a group's blocks 8 apart keeps group g on one XCD
// when the group count is a multiple of 8.  Otherwise a plain split.
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

// ---------------------------------------------------------------------------
// Field of Eq. 3 for TPW tiles at once, gathered from the neighbours' spin
// words.  The scalar work (CSR entries, neighbour offsets, coupling masks) is
// shared by the tiles; the spin loads and arithmetic are per tile.
// Neighbours are taken four at a time from a copy of the CSR whose rows are
// padded to multiples of 4 entries (padding: vertex 0, coupling 0), so the
// loop body has no per-entry branches or masks.  Its column entries hold the
// byte offset of the neighbour's spin word within a tile, 256 (v >> 2), plus
// (v & 3) in coupling modes 0 and 1.  Spin words are read with
// buffer loads: the neighbour quad as the scalar offset, tile and lane as the
// vector offset, so address arithmetic stays on the scalar unit.  Coupling modes (JM): 0 full 32-bit products, 1 24-bit
// products (|J| < 2^23), 2 int8 couplings pre-shifted to the neighbour's byte
// of its spin word, so one 4 x int8 dot product adds J s_j.
// ---------------------------------------------------------------------------
template <int JM, int TPW>
__device__ __forceinline__ void gather_fields(const PAMC_CONST int32_t* __restrict__ gcol,
                                              const PAMC_CONST int32_t* __restrict__ gJ, int e0, int e1,
                                              __amdgpu_buffer_rsrc_t Sr, const int (&voff)[TPW],
                                              int32_t (&h)[TPW]) {
#pragma unroll
  for (int t = 0; t < TPW; ++t) h[t] = 0;
  for (int e = e0; e < e1; e += 4) {
    // rows start at multiples of 4 entries: one 16-byte scalar load each
    const i32x4 cj = *reinterpret_cast<const PAMC_CONST i32x4*>(gcol + e);
    const i32x4 cJ = *reinterpret_cast<const PAMC_CONST i32x4*>(gJ + e);
    const int j[4] = {cj.x, cj.y,
                      cj.z, cj.w};
    const int32_t c[4] = {cJ.x, cJ.y,
                          cJ.z, cJ.w};
    uint32_t w[TPW][4];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        w[t][u] = __builtin_amdgcn_raw_buffer_load_b32(Sr, voff[t], JM == 2 ? j[u] : (j[u] & ~3), 0);
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (JM == 2) {
          h[t] = __builtin_amdgcn_sdot4((int)w[t][u], c[u], h[t], false);
        } else {
          const int32_t sv = __builtin_amdgcn_sbfe((int32_t)w[t][u], 8u * (uint32_t)(j[u] & 3), 8u);  // byte of the spin
          h[t] += JM == 1 ? __mul24(c[u], sv) : c[u] * sv;
        }
      }
  }
}

// Hub fields of the current population buffer (null without hubs).
__device__ __forceinline__ int32_t* st_cur_hub(const Desc& d) {
  return d.nhub ? (gmem((const RunState*)d.st)->cur ? d.HF1 : d.HF0) : nullptr;
}

// Work-group totals: energy changes per replica (red[wave * ntiles + t][lane])
// into E, flip counts per wave (fred, filled by lane 0 of each wave) into
// the profiling counters.
__device__ __forceinline__ void reduce_energy_and_flips(int64_t (*red)[kLanes], int32_t* fred, int wave,
                                                        int lane, int ntiles, int tile0,
                                                        PAMC_GLOBAL int64_t* E,
                                                        PAMC_GLOBAL int64_t* flip_ctr) {
  __syncthreads();
  if (wave < ntiles) {
    const int t = wave;
    int64_t sum = 0;
#pragma unroll
    for (int w = 0; w < kSweepWaves; ++w) sum += red[w * ntiles + t][lane];
    if (sum != 0)
      __hip_atomic_fetch_add((unsigned long long*)&E[(tile0 + t) * kLanes + lane], (unsigned long long)sum,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (flip_ctr && threadIdx.x == 0) {
    const int64_t f = (int64_t)fred[0] + fred[1] + fred[2] + fred[3];
    __hip_atomic_fetch_add((unsigned long long*)&flip_ctr[blockIdx.x & 255], (unsigned long long)f,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------
// One colour class of one sweep with fields gathered at visit time (Eqs.
// 3-4).  Work-group = (group of TPW replica tiles, chunk of the class's
// vertex quads); wave = up to 4 quads; lane = replica.  For each vertex:
// x = s*h, u = Philox word (quad, sweep, replica), flip iff u < T[x]
// (Metropolis also for x <= 0).  Vertices of a class are mutually
// uncoupled, so no spin read here as a neighbour is written here.
// The threshold table is read from LDS (THR_LDS) or from global memory.
// With int8 couplings (JM 2) the energy change of a lane over one
// work-group stays below 2^31 (|x| <= X < 2^26, at most 4 kMaxQuadsPerWave
// vertices), so it is summed in 32 bits.
// ---------------------------------------------------------------------------
template <int JM, int TPW, bool THR_LDS, bool HUB>
__device__ __forceinline__ void sweep_pull_body(const PAMC_CONST int32_t* __restrict__ row_ptr,
                                                const PAMC_CONST int32_t* __restrict__ col,
                                                const PAMC_CONST int32_t* __restrict__ Jc,
                                                const PAMC_GLOBAL uint32_t* __restrict__ thr_g,
                                                uint32_t* thr_s, PAMC_GLOBAL uint32_t* __restrict__ S,
                                                PAMC_GLOBAL int64_t* __restrict__ E, const Desc& d,
                                                int group, int chunk, int v0, int v1, uint32_t gs,
                                                int32_t Xt) {
  using acc_t = typename std::conditional<JM == 2, int32_t, int64_t>::type;
  __shared__ int64_t red[kSweepWaves * TPW][kLanes];
  __shared__ int32_t fred[kSweepWaves];
  const int q0 = v0 >> 2;
  const int nqc = ((v1 + 3) >> 2) - q0;
  const bool metropolis = d.rule == 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile0 = group * TPW;
  const uint32_t tstride = (uint32_t)d.nq * kLanes;
  const __amdgpu_buffer_rsrc_t Sr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(S + (size_t)tile0 * tstride), (short)0, (int)(TPW * tstride * 4), kBufferWord3);
  int voff[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) voff[t] = (int)(t * tstride * 4) + lane * 4;
  acc_t dE[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) dE[t] = 0;
  int32_t nflip = 0;
  // hubs (rows too long to gather): their fields come from HF, and each
  // flip's change to them (2 J s_new) is summed per lane in registers, then
  // over the work-group's waves, before one atomic per lane and hub
  const int nhub = HUB ? d.nhub : 0;
  PAMC_GLOBAL int32_t* HF = gmem(HUB ? st_cur_hub(d) : nullptr);
  int32_t hacc[kMaxHubs][TPW];
#pragma unroll
  for (int hk = 0; hk < kMaxHubs; ++hk)
#pragma unroll
    for (int t = 0; t < TPW; ++t) hacc[hk][t] = 0;
  for (int i = 0; i < d.qpw; ++i) {
    const int qi = chunk * (kSweepWaves * d.qpw) + i * kSweepWaves + wave;
    if (qi >= nqc) break;
    const int q = q0 + qi;
    uint32_t sw[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) sw[t] = __builtin_amdgcn_raw_buffer_load_b32(Sr, voff[t], q * (kLanes * 4), 0);
    int32_t h[4][TPW];
    int32_t hj[4][kMaxHubs];  // couplings of the quad's vertices to the hubs (uniform)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = 4 * q + k;
      const bool in = v >= v0 && v < v1;
#pragma unroll
      for (int hk = 0; hk < kMaxHubs; ++hk) hj[k][hk] = (HUB && in) ? cmem(d.hubJ)[v * kMaxHubs + hk] : 0;
      if (HUB && in && (v == d.hub_v0 || v == d.hub_v1)) {
        const int hk = v == d.hub_v0 ? 0 : 1;
#pragma unroll
        for (int t = 0; t < TPW; ++t) h[k][t] = HF[hk * d.R + (tile0 + t) * kLanes + lane];
      } else if (in) {
        gather_fields<JM, TPW>(col, Jc, row_ptr[v], row_ptr[v + 1], Sr, voff, h[k]);
      } else {
#pragma unroll
        for (int t = 0; t < TPW; ++t) h[k][t] = 0;
      }
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const uint32_t r = (uint32_t)((tile0 + t) * kLanes + lane);
      const u32x4 rnd = philox10((uint32_t)q, gs, r, kTagSweep, d.k0, d.k1);
      const uint32_t swt = sw[t];
      uint32_t flipmask = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int v = 4 * q + k;
        if (v < v0 || v >= v1) continue;
        const int32_t s = __builtin_amdgcn_sbfe((int32_t)swt, 8u * k, 8u);
        const int32_t x = __mul24(s, h[k][t]);
        const int32_t xi = min(max(x, -Xt), Xt) + Xt;
        const uint32_t T = THR_LDS ? thr_s[xi] : thr_g[xi];
        const bool flip = (pick(rnd, k) < T) || (metropolis && x <= 0);
        dE[t] += flip ? (acc_t)x : (acc_t)0;
        flipmask |= flip ? (0xFEu << (8 * k)) : 0u;  // +1 (0x01) <-> -1 (0xFF)
        nflip += __popcll(__ballot(flip));
        if constexpr (HUB) {
#pragma unroll
          for (int hk = 0; hk < kMaxHubs; ++hk) hacc[hk][t] += flip ? -2 * s * hj[k][hk] : 0;
        }
      }
      if (flipmask) __builtin_amdgcn_raw_buffer_store_b32(swt ^ flipmask, Sr, voff[t], q * (kLanes * 4), 0);
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) red[wave * TPW + t][lane] = 2 * (int64_t)dE[t];
  if (lane == 0) fred[wave] = nflip;
  reduce_energy_and_flips(red, fred, wave, lane, TPW, tile0, E, gmem(d.flip_ctr));
  if constexpr (HUB) {
    // the energy sums are done with red: it now holds the waves' hub sums
    // (kSweepWaves x kMaxHubs x TPW x 64 int32, the same 2048 TPW bytes)
    int32_t* hred = reinterpret_cast<int32_t*>(&red[0][0]);
    __syncthreads();
#pragma unroll
    for (int hk = 0; hk < kMaxHubs; ++hk)
#pragma unroll
      for (int t = 0; t < TPW; ++t) hred[((wave * kMaxHubs + hk) * TPW + t) * kLanes + lane] = hacc[hk][t];
    __syncthreads();
    if (wave < TPW) {
      const int t = wave;
      for (int hk = 0; hk < nhub; ++hk) {
        int32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kSweepWaves; ++w) sum += hred[((w * kMaxHubs + hk) * TPW + t) * kLanes + lane];
        if (sum != 0)
          __hip_atomic_fetch_add(&HF[hk * d.R + (tile0 + t) * kLanes + lane], sum, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// WIDE: the instance's threshold table (2X + 1 entries) may exceed the LDS
// copy; a step whose table does not fit reads it from global memory.  The
// host picks the variant from X, so instances whose table always fits get
// one loop body.  HUB: the instance keeps the fields of its hub vertices.
template <int JM, int TPW, bool WIDE, bool HUB>
__global__ void __launch_bounds__(256) k_sweep_pull(const Desc* __restrict__ D,
                                                  const uint64_t* __restrict__ map, int sweep_idx,
                                                  int phase) {
  __shared__ uint32_t thr_s[kThrLds];
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  if (!st->active || sweep_idx >= st->nsweeps_now || phase >= d.ncls) return;
  const int cur = st->cur;
  const PAMC_CONST int32_t* __restrict__ order = cmem((const int32_t*)d.order);
  const PAMC_CONST int32_t* __restrict__ class_ptr = cmem(d.class_ptr);
  const int cls = order[sweep_idx * d.ncls + phase];
  const int v0 = class_ptr[cls], v1 = class_ptr[cls + 1];
  const int nqc = ((v1 + 3) >> 2) - (v0 >> 2);
  int group, chunk;
  group_chunk(d.T / TPW, lb, group, chunk);
  if (chunk * (kSweepWaves * d.qpw) >= nqc) return;
  const uint32_t gs = st->gs + (uint32_t)sweep_idx;
  const int32_t Xt = (int32_t)st->table_x;
  const PAMC_GLOBAL uint32_t* __restrict__ thr_g = gmem((const uint32_t*)d.thr);
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0);
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const PAMC_CONST int32_t* __restrict__ Jc = cmem(d.gJ);
  // the step's table (2 Xt + 1 entries) goes to LDS whenever it fits, also
  // for instances whose full range (WIDE: 2X + 1) would not
  if (!WIDE || 2 * Xt + 1 <= kThrLds) {
    for (int i = threadIdx.x; i <= 2 * Xt; i += blockDim.x) thr_s[i] = thr_g[i];
    __syncthreads();
    sweep_pull_body<JM, TPW, true, HUB>(cmem(d.grow), cmem(d.gcol), Jc, thr_g, thr_s, S, E, d, group, chunk, v0,
                                        v1, gs, Xt);
  } else {
    sweep_pull_body<JM, TPW, false, HUB>(cmem(d.grow), cmem(d.gcol), Jc, thr_g, thr_s, S, E, d, group, chunk, v0,
                                         v1, gs, Xt);
  }
}

// ---------------------------------------------------------------------------
// All of a step's sweeps of one replica tile in one work-group, for small
// instances (gathered fields, at most kTileMaxQuads vertex quads): the
// tile's spin words live in LDS for the whole launch, and the work-group
// walks the sweeps and, in each, the colour classes in the sweep's order,
// its four waves sharing a class's quads, with a barrier between classes.
// Replica tiles never interact within a step, so no other synchronisation
// is needed; the decisions are those of k_sweep_pull (same fields, same
// Philox words, same thresholds), so the trajectory is the same, while a
// step is one launch instead of sweeps x classes.
// ---------------------------------------------------------------------------
constexpr int kTileMaxQuads = 512;      // 128 KB of LDS spin words: n <= 2048
constexpr int kTileWaves = 16;          // waves of a tile-resident work-group
constexpr int kTileLdsBytes = 150 * 1024;  // dynamic LDS: spins, table, one class's rows (8 KB static beside)

template <int JM>
__global__ void __launch_bounds__(kTileWaves * 64) k_sweep_tile(const Desc* __restrict__ D,
                                                                const uint64_t* __restrict__ map) {
  // LDS: [nq][64] spin words, the threshold table (kThrLds words), then the
  // current class's gathered rows (columns, then couplings; d.tile_rows
  // entries each at most)
  extern __shared__ uint32_t tl[];
  __shared__ int64_t red[kTileWaves][kLanes];
  __shared__ int32_t fred[kTileWaves];
  int inst, tile;
  if (!resolve(map, inst, tile)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  const int nsw = st->nsweeps_now;
  if (!st->active || nsw <= 0) return;
  const int cur = st->cur;
  const int nq = d.nq;
  const int32_t Xt = (int32_t)st->table_x;
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0) + (size_t)tile * nq * kLanes;
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const PAMC_GLOBAL uint32_t* __restrict__ thr_g = gmem((const uint32_t*)d.thr);
  const PAMC_GLOBAL int32_t* __restrict__ order = gmem((const int32_t*)d.order);
  const PAMC_GLOBAL int32_t* __restrict__ class_ptr = gmem(d.class_ptr);
  const PAMC_GLOBAL int32_t* __restrict__ grow = gmem(d.grow);
  const PAMC_GLOBAL int32_t* __restrict__ gcol = gmem(d.gcol);
  const PAMC_GLOBAL int32_t* __restrict__ gJ = gmem(d.gJ);
  uint32_t* Sl = tl;
  uint32_t* thr_s = tl + (size_t)nq * kLanes;
  int32_t* rc = reinterpret_cast<int32_t*>(thr_s + kThrLds);
  int32_t* rj = rc + d.tile_rows;
  for (int i = threadIdx.x; i < nq * kLanes; i += blockDim.x) Sl[i] = S[i];
  for (int i = threadIdx.x; i <= 2 * Xt; i += blockDim.x) thr_s[i] = thr_g[i];
  const int lane = threadIdx.x & 63;
  const int lane4 = 4 * lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t r = (uint32_t)(tile * kLanes + lane);
  const bool metropolis = d.rule == 1;
  int64_t dE = 0;
  int32_t nflip = 0;
  for (int sw_i = 0; sw_i < nsw; ++sw_i) {
    const uint32_t gs = st->gs + (uint32_t)sw_i;
    for (int p = 0; p < d.ncls; ++p) {
      const int cls = order[sw_i * d.ncls + p];
      const int v0 = class_ptr[cls], v1 = class_ptr[cls + 1];
      const int g0 = grow[v0], ng = grow[v1] - g0;
      __syncthreads();  // the previous class is done with the row buffer (and its spins are in)
      for (int i = threadIdx.x; i < ng; i += blockDim.x) {
        rc[i] = gcol[g0 + i];
        rj[i] = gJ[g0 + i];
      }
      __syncthreads();
      const int q0 = v0 >> 2, nqc = ((v1 + 3) >> 2) - q0;
      for (int qi = wave; qi < nqc; qi += kTileWaves) {
        const int q = q0 + qi;
        uint32_t sw = Sl[q * kLanes + lane];
        int32_t h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int v = 4 * q + k;
          h[k] = 0;
          if (v < v0 || v >= v1) continue;
          const int e1 = grow[v + 1] - g0;
          for (int e = grow[v] - g0; e < e1; e += 4) {
            const i32x4 cj = *reinterpret_cast<const i32x4*>(rc + e);  // uniform: broadcast reads
            const i32x4 cJ = *reinterpret_cast<const i32x4*>(rj + e);
            const int j[4] = {cj.x, cj.y, cj.z, cj.w};
            const int32_t c[4] = {cJ.x, cJ.y, cJ.z, cJ.w};
            // the neighbour's word: j is its byte offset in the tile (plus
            // its byte index in modes 0 and 1), so one add per neighbour
            // addresses it
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              w[u] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(Sl) +
                                                        (JM == 2 ? j[u] : (j[u] & ~3)) + lane4);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (JM == 2) {
                h[k] = __builtin_amdgcn_sdot4((int)w[u], c[u], h[k], false);
              } else {
                const int32_t sv = __builtin_amdgcn_sbfe((int32_t)w[u], 8u * (uint32_t)(j[u] & 3), 8u);
                h[k] += JM == 1 ? __mul24(c[u], sv) : c[u] * sv;
              }
            }
          }
        }
        const u32x4 rnd = philox10((uint32_t)q, gs, r, kTagSweep, d.k0, d.k1);
        uint32_t flipmask = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int v = 4 * q + k;
          if (v < v0 || v >= v1) continue;
          const int32_t s = __builtin_amdgcn_sbfe((int32_t)sw, 8u * k, 8u);
          const int32_t x = __mul24(s, h[k]);
          const int32_t xi = min(max(x, -Xt), Xt) + Xt;
          const bool flip = (pick(rnd, k) < thr_s[xi]) || (metropolis && x <= 0);
          dE += flip ? (int64_t)x : 0;
          flipmask |= flip ? (0xFEu << (8 * k)) : 0u;
          nflip += __popcll(__ballot(flip));
        }
        if (flipmask) Sl[q * kLanes + lane] = sw ^ flipmask;
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nq * kLanes; i += blockDim.x) S[i] = Sl[i];
  red[wave][lane] = 2 * dE;
  if (lane == 0) fred[wave] = nflip;
  __syncthreads();
  if (wave == 0) {  // the work-group owns its tile's replicas: no atomics
    int64_t sum = 0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) sum += red[w][lane];
    E[tile * kLanes + lane] += sum;
    if (d.flip_ctr && lane == 0) {
      int64_t f = 0;
      for (int w = 0; w < kTileWaves; ++w) f += fred[w];
      __hip_atomic_fetch_add((unsigned long long*)&d.flip_ctr[blockIdx.x & 255], (unsigned long long)f,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---------------------------------------------------------------------------
// The tile-resident step with the fields of a colour class computed on the
// matrix cores, for small instances with int8 couplings (at most
// kTmmaMaxN vertices): the class's fields for the tile's 64 replicas are
// h = J[class rows, :] . S, an int8 x int8 -> int32 product (exact: |h| <=
// 127 n), so a dense-ish graph costs one v_mfma_i32_16x16x64_i8 per 16
// rows, 16 replicas and 64 vertices instead of a gather per neighbour.
// The spins sit in LDS replica-major (int8 [64][npk + 16], the B operand);
// J sits in HBM as 16-row x 64-column fragments in the order the A operand
// wants them (1 KB per fragment: lane l holds bytes 16 (l / 16) .. + 15 of
// row l % 16).  Vertices of one class share no edge (J = 0 between them),
// so the product may read the class's spins while they change.  Each wave
// keeps one group of 16 replicas (wave % 4) and takes 16-row tiles of the
// class in turn; the product leaves in each lane the four fields of one
// vertex quad for one replica, exactly the unit of one Philox block, and
// the decisions are those of the other sweep kernels (same fields, words
// and thresholds), so the trajectory is the same.
// ---------------------------------------------------------------------------
constexpr int kComputeUnits = 256;      // MI355X
constexpr int kMfmaGroupTiles = 128;    // tiles up to which a batch takes one work-group per 16-replica group
constexpr int64_t kCuLdsBytes = 160 * 1024;
constexpr int kTmmaMaxN = 1024;  // vertices (padded): 64 x 1040 B of LDS spins
constexpr int kTmmaMaxKs = kTmmaMaxN / 64;

// NW waves per work-group (16, or 8 so that two work-groups share a
// compute unit when a batch has enough of them).
template <int NW>
__global__ void __launch_bounds__(NW * 64) k_sweep_tmma(const Desc* __restrict__ D, const uint64_t* __restrict__ map) {
  extern __shared__ uint32_t tl[];  // int8 spins [64][rowb], then the threshold table
  __shared__ int64_t red[NW][kLanes];
  __shared__ int32_t fred[NW];
  int inst, tile;
  if (!resolve(map, inst, tile)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  const int nsw = st->nsweeps_now;
  if (!st->active || nsw <= 0) return;
  const int cur = st->cur;
  const int nq = d.nq, nks = d.nks;
  const int rowb = 64 * nks + 16;  // bytes per replica row (padded against bank conflicts)
  const int32_t Xt = (int32_t)st->table_x;
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0) + (size_t)tile * nq * kLanes;
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const PAMC_GLOBAL uint32_t* __restrict__ thr_g = gmem((const uint32_t*)d.thr);
  const PAMC_GLOBAL int32_t* __restrict__ order = gmem((const int32_t*)d.order);
  const PAMC_GLOBAL int32_t* __restrict__ class_ptr = gmem(d.class_ptr);
  const PAMC_GLOBAL int8_t* __restrict__ Jt = gmem(d.Jt);
  int8_t* Sb = reinterpret_cast<int8_t*>(tl);
  uint32_t* thr_s = tl + 16 * rowb;  // 64 rowb bytes
  // the tile's spin words into replica-major rows: word (q, l) holds the
  // bytes of vertices 4q .. 4q + 3 of replica l
  for (int i = threadIdx.x; i < nq * kLanes; i += blockDim.x)
    *reinterpret_cast<uint32_t*>(Sb + (i & 63) * rowb + 4 * (i >> 6)) = S[i];
  for (int i = threadIdx.x; i <= 2 * Xt; i += blockDim.x) thr_s[i] = thr_g[i];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave & 3;                 // the wave's 16 replicas
  const int rl = 16 * grp + (lane & 15);    // the lane's replica in the tile
  const uint32_t r = (uint32_t)(tile * kLanes + rl);
  const int kq = lane >> 4;                 // the lane's quad within a 16-row tile
  const int8_t* brow = Sb + rl * rowb + 16 * kq;  // B operand: replica rl, bytes 16 kq ..
  const bool metropolis = d.rule == 1;
  int64_t dE = 0;
  int32_t nflip = 0;
  for (int sw_i = 0; sw_i < nsw; ++sw_i) {
    const uint32_t gs = st->gs + (uint32_t)sw_i;
    for (int p = 0; p < d.ncls; ++p) {
      const int cls = order[sw_i * d.ncls + p];
      const int v0 = class_ptr[cls], v1 = class_ptr[cls + 1];
      const int q0 = v0 >> 2, q1 = (v1 + 3) >> 2;  // the class's quads
      const int t0 = q0 >> 2, t1 = (q1 + 3) >> 2;  // its 16-row tiles
      __syncthreads();  // the previous class's spins are in
      for (int t = t0 + (wave >> 2); t < t1; t += NW / 4) {
        // every A fragment of the row tile first; the lane's random words
        // (they do not depend on the fields) while the fragments arrive;
        // then the products
        const PAMC_GLOBAL int8_t* arow = Jt + ((size_t)t * nks * 64 + lane) * 16;
        i32x4 av[kTmmaMaxKs];
#pragma unroll
        for (int ks = 0; ks < kTmmaMaxKs; ++ks)
          if (ks < nks) av[ks] = *reinterpret_cast<const PAMC_GLOBAL i32x4*>(arow + (size_t)ks * 1024);
        // the lane's quad: vertices 4q .. 4q + 3 of the tile, replica rl
        const int q = 4 * t + kq;
        const u32x4 rnd = philox10((uint32_t)q, gs, r, kTagSweep, d.k0, d.k1);
        __builtin_amdgcn_sched_barrier(0);
        i32x4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < kTmmaMaxKs; ++ks)
          if (ks < nks)
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[ks], *reinterpret_cast<const i32x4*>(brow + 64 * ks),
                                                        acc, 0, 0, 0);
        if (q < q0 || q >= q1) continue;
        uint32_t* wp = reinterpret_cast<uint32_t*>(Sb + rl * rowb + 4 * q);
        const uint32_t sw = *wp;
        uint32_t flipmask = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int v = 4 * q + k;
          if (v < v0 || v >= v1) continue;
          const int32_t s = __builtin_amdgcn_sbfe((int32_t)sw, 8u * k, 8u);
          const int32_t x = __mul24(s, acc[k]);
          const int32_t xi = min(max(x, -Xt), Xt) + Xt;
          const bool flip = (pick(rnd, k) < thr_s[xi]) || (metropolis && x <= 0);
          dE += flip ? (int64_t)x : 0;
          flipmask |= flip ? (0xFEu << (8 * k)) : 0u;
          nflip += flip ? 1 : 0;
        }
        if (flipmask) *wp = sw ^ flipmask;
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nq * kLanes; i += blockDim.x)
    S[i] = *reinterpret_cast<const uint32_t*>(Sb + (i & 63) * rowb + 4 * (i >> 6));
  red[wave][lane] = 2 * dE;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nflip += __shfl_xor(nflip, o, 64);
  if (lane == 0) fred[wave] = nflip;
  __syncthreads();
  if (wave == 0) {  // replica rl = 16 (w % 4) + (l % 16): the waves w and lanes l holding it
    const int g = lane >> 4, c = lane & 15;
    int64_t sum = 0;
#pragma unroll
    for (int w = g; w < NW; w += 4)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) sum += red[w][16 * kk + c];
    E[tile * kLanes + lane] += sum;
    if (d.flip_ctr && lane == 0) {
      int64_t f = 0;
      for (int w = 0; w < NW; ++w) f += fred[w];
      __hip_atomic_fetch_add((unsigned long long*)&d.flip_ctr[blockIdx.x & 255], (unsigned long long)f,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The same step with one work-group per 16-replica group of a tile (four
// per tile): a single instance spreads over four times the compute units,
// each holding a quarter of the tile's spins.  Wave w takes the class's
// 16-row tiles w, w + NW, ...; lane l's replica is 16 g + l % 16 and its
// quad 4 t + l / 16, as above.
//
// The chain from one class's barrier to the next bounds it, and a unit's rate
// of reading J (64 bytes a cycle, every work-group all of J in a sweep).  A wave
// keeps its replicas' spins as B operands in registers and after a barrier
// reads again only the 64-vertex columns that hold the class just visited; the
// roles of the waves rotate by half from class to class, so that while some
// decide a class the others read their couplings, draw their words and
// multiply the columns that are final for the next.  Row tiles start at the
// class's first quad, so a class of 64 vertices is four of them.  G(800,
// 19176), R = 256, 15 classes x 5 sweeps: 84 us, where it took 137 with the
// loads, words and products of a class all behind its barrier; G(300, 2400), R =
// 128, 15 x 3: 21 and 33 us.  A quarter, half, three quarters and all of the
// couplings read by the deciding waves for their next turn: 6.44, 6.28, 6.65 and
// 6.78 ms a run.
template <int NW, int NKP, bool METRO>  // NKP: 64-vertex columns, rounded up to even
__device__ __forceinline__ void sweep_tmma_group(const Desc& d, int lb, uint32_t* tl, int64_t (*red)[kLanes],
                                                 int32_t* fred) {
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  const int nsw = st->nsweeps_now;
  const int tile = lb >> 2, grp = lb & 3;
  const int cur = st->cur;
  const int nq = d.nq, nks = d.nks, ncls = d.ncls;
  constexpr int rowb = 64 * NKP + 16;  // bytes per replica row (padded against bank conflicts)
  const int32_t Xt = (int32_t)st->table_x;
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0) + (size_t)tile * nq * kLanes + 16 * grp;
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const PAMC_GLOBAL uint32_t* __restrict__ thr_g = gmem((const uint32_t*)d.thr);
  const PAMC_CONST int32_t* __restrict__ order = cmem((const int32_t*)d.order);
  const PAMC_CONST int32_t* __restrict__ class_ptr = cmem(d.class_ptr);
  const PAMC_GLOBAL int8_t* __restrict__ Jt = gmem(d.Jt);
  int8_t* Sb = reinterpret_cast<int8_t*>(tl);
  uint32_t* thr_s = tl + 4 * rowb;  // 16 rowb bytes
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15;                  // the lane's replica in the group
  const uint32_t r = (uint32_t)(tile * kLanes + 16 * grp + c);
  const int kq = lane >> 4;                 // the lane's quad within a row tile
  const int8_t* brow = Sb + c * rowb + 16 * kq;  // B operand: replica c, bytes 16 kq ..
  const uint32_t k0 = d.k0, k1 = d.k1;
  const int phases = nsw * ncls;
  int64_t dE = 0;
  int32_t dEs = 0, nflip = 0;  // dEs: of the sweep, |x| < 2^10 and at most n / 4 spins a lane
  // a phase's class (empty past the last)
  struct Class {
    int v0, v1;
    __device__ int tiles() const { return (v1 - (v0 & ~3) + 15) >> 4; }
  };
  auto class_of = [&](int i) -> Class {
    if (i >= phases) return {0, 0};
    const int cls = order[i];
    return {class_ptr[cls], class_ptr[cls + 1]};
  };
  i32x4 av[NKP], bv[NKP];
  // fragments lo .. hi - 1 of row tile u of a class (rows of other classes are
  // left as they are: no result of them is used; an odd last column is followed
  // by other couplings, against spins of 0)
  auto load_a = [&](const Class& x, int u, int lo, int hi) {
    const int row = (x.v0 & ~3) + 16 * u + c;
    const uint32_t at = ((uint32_t)(row >> 4) * nks * 64 + (row & 15) + 16 * kq) * 16;
    if (row < x.v1)
#pragma unroll
      for (int ks = 0; ks < NKP; ++ks)
        if (ks >= lo && ks < hi)
          av[ks] = *reinterpret_cast<const PAMC_GLOBAL i32x4*>(Jt + at + 1024 * ks);
  };
  auto quad_of = [&](const Class& x, int u) { return (x.v0 >> 2) + 4 * u + kq; };
  auto word_at = [&](int q) { return reinterpret_cast<uint32_t*>(Sb + c * rowb + 4 * q); };
  // products over the columns not in the mask
  auto multiply_rest = [&](uint32_t mask) {
    i32x4 a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < NKP; ++ks)
      if (!(mask >> ks & 1u)) {
        if (ks & 1)
          a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[ks], bv[ks], a1, 0, 0, 0);
        else
          a0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[ks], bv[ks], a0, 0, 0, 0);
      }
    return a0 + a1;
  };
  // What a visit of a quad needs beside its fields: its spins (after the barrier
  // of the phase before: they may share a word with, or be, the class visited
  // there), its words, and which of its vertices are of the class.
  struct Quad {
    int q;
    uint32_t sw, in;
    u32x4 rnd;
  };
  auto quad_ready = [&](const Class& x, int u, uint32_t gs) {
    Quad z;
    z.q = quad_of(x, u);
    z.in = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) z.in |= (uint32_t)(4 * z.q + k - x.v0) < (uint32_t)(x.v1 - x.v0) ? 0xFEu << (8 * k) : 0u;
    z.rnd = philox10((uint32_t)z.q, gs, r, kTagSweep, k0, k1);
    return z;
  };
  const uint32_t* thr_mid = thr_s + Xt;
  auto decide = [&](const Quad& z, const i32x4& h) {
    uint32_t flipmask = 0;
    int32_t x[4];
    uint32_t T[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = __mul24(__builtin_amdgcn_sbfe((int32_t)z.sw, 8u * k, 8u), h[k]);
      T[k] = thr_mid[min(max(x[k], -Xt), Xt)];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      bool flip = pick(z.rnd, k) < T[k];
      if constexpr (METRO) flip |= x[k] <= 0;
      const uint32_t m = flip ? z.in & (0xFEu << (8 * k)) : 0u;  // +1 (0x01) <-> -1 (0xFF)
      dEs += m ? x[k] : 0;
      flipmask |= m;
    }
    nflip += __builtin_popcount(flipmask & 0x02020202u);
    if (flipmask) *word_at(z.q) = z.sw ^ flipmask;
  };
  Class x0 = class_of(0), x1 = class_of(1), x2 = class_of(2);
  // the group's spin words (q, 16 grp + c) into replica-major rows, 0 past the last
  for (int i = threadIdx.x; i < 16 * NKP * 16; i += blockDim.x)
    *reinterpret_cast<uint32_t*>(Sb + (i & 15) * rowb + 4 * (i >> 4)) =
        (i >> 4) < nq ? S[(i >> 4) * kLanes + (i & 15)] : 0u;
  for (int i = threadIdx.x; i <= 2 * Xt; i += blockDim.x) thr_s[i] = thr_g[i];
  // wave w's row tile (if the class has that many; then also every NW-th
  // after it) in even and odd phases
  const int j0 = wave, j1 = (wave + NW / 2) % NW;
  if (j0 < x0.tiles()) load_a(x0, j0, 0, NKP);
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < NKP; ++ks) bv[ks] = *reinterpret_cast<const i32x4*>(brow + 64 * ks);
  uint32_t gs = st->gs;
  int left = ncls;  // phases left in the sweep
  i32x4 h = {0, 0, 0, 0};
  Quad z{};
  bool now = j0 < x0.tiles(), early = false;  // early: the next class's first half is on its way
  if (now) {
    z = quad_ready(x0, j0, gs);
    z.sw = *word_at(z.q);
    h = multiply_rest(0u);
  }
  constexpr int kEarly = NKP / 2;
  int i = 0;
  auto phase = [&](int jc, int jn) {  // the wave's row tiles in this phase and the next
    const Class x3 = class_of(i + 3);
    const bool next = jn < x1.tiles();
    if (now) {
      decide(z, h);
      for (int u = jc + NW; u < x0.tiles(); u += NW) {  // further row tiles of a large class
        load_a(x0, u, 0, NKP);
        z = quad_ready(x0, u, gs);
        z.sw = *word_at(z.q);
        decide(z, multiply_rest(0u));
      }
    }
    if (--left == 0) {
      left = ncls;
      ++gs;
      dE += dEs;
      dEs = 0;
    }
    // the columns that hold the class (if it has a vertex)
    const uint32_t mask = x0.v1 > x0.v0 ? (2u << ((x0.v1 - 1) >> 6)) - (1u << (x0.v0 >> 6)) : 0u;
    if (next) {
      if (!early) load_a(x1, jn, 0, kEarly);
      load_a(x1, jn, kEarly, NKP);
      z = quad_ready(x1, jn, gs);
      h = multiply_rest(mask);
    }
    early = !next && jc < x2.tiles();
    if (early) load_a(x2, jc, 0, kEarly);
    lds_barrier();  // the class's spins are in
    if (next) z.sw = *word_at(z.q);
#pragma unroll
    for (int ks = 0; ks < NKP; ++ks)
      if (mask >> ks & 1u) {
        bv[ks] = *reinterpret_cast<const i32x4*>(brow + 64 * ks);
        if (next) h = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[ks], bv[ks], h, 0, 0, 0);
      }
    now = next;
    x0 = x1;
    x1 = x2;
    x2 = x3;
    return ++i < phases;
  };
  if (phases > 0)
    while (phase(j0, j1) && phase(j1, j0)) {
    }
  __syncthreads();
  for (int j = threadIdx.x; j < nq * 16; j += blockDim.x)
    S[(j >> 4) * kLanes + (j & 15)] = *reinterpret_cast<const uint32_t*>(Sb + (j & 15) * rowb + 4 * (j >> 4));
  red[wave][lane] = dE;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nflip += __shfl_xor(nflip, o, 64);
  if (lane == 0) fred[wave] = nflip;
  __syncthreads();
  if (wave == 0 && lane < 16) {  // replica 16 grp + lane: lanes lane, 16 + lane, ... of every wave
    int64_t sum = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) sum += red[w][16 * kk + lane];
    E[tile * kLanes + 16 * grp + lane] += 2 * sum;
    if (d.flip_ctr && lane == 0) {
      int64_t f = 0;
      for (int w = 0; w < NW; ++w) f += fred[w];
      __hip_atomic_fetch_add((unsigned long long*)&d.flip_ctr[blockIdx.x & 255], (unsigned long long)f,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

template <int NW, bool METRO>
__device__ __forceinline__ void sweep_tmma_groups(const Desc& d, int lb, uint32_t* tl, int64_t (*red)[kLanes],
                                                  int32_t* fred) {
  switch ((d.nks + 1) / 2) {
    case 1: sweep_tmma_group<NW, 2, METRO>(d, lb, tl, red, fred); break;
    case 2: sweep_tmma_group<NW, 4, METRO>(d, lb, tl, red, fred); break;
    case 3: sweep_tmma_group<NW, 6, METRO>(d, lb, tl, red, fred); break;
    case 4: sweep_tmma_group<NW, 8, METRO>(d, lb, tl, red, fred); break;
    case 5: sweep_tmma_group<NW, 10, METRO>(d, lb, tl, red, fred); break;
    case 6: sweep_tmma_group<NW, 12, METRO>(d, lb, tl, red, fred); break;
    case 7: sweep_tmma_group<NW, 14, METRO>(d, lb, tl, red, fred); break;
    default: sweep_tmma_group<NW, 16, METRO>(d, lb, tl, red, fred); break;
  }
}

template <int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_sweep_tmma_g(const Desc* __restrict__ D, const uint64_t* __restrict__ map) {
  extern __shared__ uint32_t tl[];  // int8 spins [16][rowb], then the threshold table
  __shared__ int64_t red[NW][kLanes];
  __shared__ int32_t fred[NW];
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  if (!st->active || st->nsweeps_now <= 0) return;
  if (d.rule == 1)
    sweep_tmma_groups<NW, true>(d, lb, tl, red, fred);
  else
    sweep_tmma_groups<NW, false>(d, lb, tl, red, fred);
}

// ---------------------------------------------------------------------------
// The same class phase with incremental fields: x = s*h from the field
// array; on a flip E += 2x and every neighbour field gets 2 J s_new by a
// coalesced no-return atomic.  Used where gathering is dearer (high degree,
// hub vertices).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sweep_push_body(const PAMC_CONST int32_t* __restrict__ row_ptr,
                                                const PAMC_CONST int32_t* __restrict__ col,
                                                const PAMC_CONST int32_t* __restrict__ Jc,
                                                const PAMC_CONST int32_t* __restrict__ class_ptr,
                                                const PAMC_CONST int32_t* __restrict__ order,
                                                const PAMC_GLOBAL uint32_t* __restrict__ thr_g, const Desc& d,
                                                int lb, int sweep_idx, int phase) {
  __shared__ int64_t red[kSweepWaves][kLanes];
  __shared__ int32_t fred[kSweepWaves];
  __shared__ uint32_t thr_s[kThrLds];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  const int cur = st->cur;
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0);
  PAMC_GLOBAL int32_t* H = gmem(cur ? d.H1 : d.H0);
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const int cls = order[sweep_idx * d.ncls + phase];
  const int v0 = class_ptr[cls], v1 = class_ptr[cls + 1];
  const int q0 = v0 >> 2;
  const int nqc = ((v1 + 3) >> 2) - q0;
  int tile, chunk0;
  group_chunk(d.T, lb, tile, chunk0);
  // a class whose quads fit one pass of the tile's work-groups at one quad
  // per wave takes one (a shorter chain per wave); larger ones the
  // instance's quads per wave
  const int qpw = (nqc + kSweepWaves - 1) / kSweepWaves <= d.sweep_stride ? 1 : d.qpw;
  if (chunk0 * (kSweepWaves * qpw) >= nqc) return;
  const uint32_t gs = st->gs + (uint32_t)sweep_idx;
  const int rule = d.rule;
  const int32_t Xt = (int32_t)st->table_x;
  const bool thr_lds = 2 * Xt + 1 <= kThrLds;
  if (thr_lds)
    for (int i = threadIdx.x; i <= 2 * Xt; i += blockDim.x) thr_s[i] = thr_g[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t r = (uint32_t)(tile * kLanes + lane);
  const size_t hbase = (size_t)tile * d.np;
  int64_t dE = 0;
  int32_t nflip = 0;
  // the work-group's chunks of the class: chunk0, chunk0 + stride, ... (the
  // tile stays the same, so the energy sums stay per tile)
  for (int chunk = chunk0; chunk * (kSweepWaves * qpw) < nqc; chunk += d.sweep_stride) {
    // the spin words and fields of all of the wave's quads up front: the
    // vertices of one class are not neighbours, so no flip of this phase
    // changes them (v < np always)
    constexpr int kMaxQpw = 4;
    uint32_t swq[kMaxQpw];
    int32_t hqq[kMaxQpw][4];
#pragma unroll
    for (int i = 0; i < kMaxQpw; ++i) {
      const int qi = chunk * (kSweepWaves * qpw) + i * kSweepWaves + wave;
      if (i < qpw && qi < nqc) {
        const int q = q0 + qi;
        swq[i] = S[((size_t)tile * d.nq + q) * kLanes + lane];
#pragma unroll
        for (int k = 0; k < 4; ++k) hqq[i][k] = H[(hbase + 4 * q + k) * kLanes + lane];
      }
    }
#pragma unroll
    for (int i = 0; i < kMaxQpw; ++i) {
      if (i >= qpw) break;
      const int qi = chunk * (kSweepWaves * qpw) + i * kSweepWaves + wave;
      if (qi >= nqc) break;
      const int q = q0 + qi;
      const size_t sidx = ((size_t)tile * d.nq + q) * kLanes + lane;
      uint32_t sw = swq[i];
      const u32x4 rnd = philox10((uint32_t)q, gs, r, kTagSweep, d.k0, d.k1);
      const int32_t (&hq)[4] = hqq[i];
      uint32_t flips = 0;  // bit k: vertex k of the quad
      int32_t x[4];
      uint32_t T[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (int32_t)(int8_t)(sw >> (8 * k)) * hq[k];
      // The four thresholds together, of vertices outside the class too: a
      // choice of table for each with its wait cost 0.7 us a launch (Max-3-Cut
      // embedding of G(7000, 21000), R = 2,048, at beta 2 and 4: 15.4 and 14.2 us;
      // 14.7 and 13.4 so).
      if (thr_lds) {
#pragma unroll
        for (int k = 0; k < 4; ++k) T[k] = thr_s[min(max(x[k], -Xt), Xt) + Xt];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) T[k] = thr_g[min(max(x[k], -Xt), Xt) + Xt];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int v = 4 * q + k;
        if (v < v0 || v >= v1) continue;
        const bool flip = (rule == 1 && x[k] <= 0) || (pick(rnd, k) < T[k]);
        if (flip) {
          dE += 2 * (int64_t)x[k];
          sw ^= (0xFEu << (8 * k));
          flips |= 1u << k;
          ++nflip;
        }
      }
      // the flipped vertices' rows
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool flip = flips >> k & 1u;
        if (!__ballot(flip)) continue;
        const int v = 4 * q + k;
        const int e0 = row_ptr[v], e1 = row_ptr[v + 1];
        const int32_t dd = 2 * (int32_t)(int8_t)(sw >> (8 * k));  // twice the new spin
        // eight entries at a time (the arrays have room past the last): the
        // reads of them, not the additions, are waited for
        for (int e = e0; e < e1; e += 8) {
          const i32x8u j = *reinterpret_cast<const PAMC_CONST i32x8u*>(col + e);
          const i32x8u c = *reinterpret_cast<const PAMC_CONST i32x8u*>(Jc + e);
          if (flip) {
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (e + u < e1)
                __hip_atomic_fetch_add(&H[(hbase + j[u]) * kLanes + lane], c[u] * dd, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
      if (flips) S[sidx] = sw;
    }
  }
  red[wave][lane] = dE;
  if (d.flip_ctr) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nflip += __shfl_xor(nflip, o, 64);
    if (lane == 0) fred[wave] = nflip;
  }
  reduce_energy_and_flips(red, fred, wave, lane, 1, tile, E, gmem(d.flip_ctr));
}

__global__ void __launch_bounds__(256) k_sweep_push(const Desc* __restrict__ D,
                                                  const uint64_t* __restrict__ map, int sweep_idx,
                                                  int phase) {
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  if (!st->active || sweep_idx >= st->nsweeps_now || phase >= d.ncls) return;
  sweep_push_body(cmem(d.row_ptr), cmem(d.col), cmem(d.J), cmem(d.class_ptr), cmem((const int32_t*)d.order),
                  gmem((const uint32_t*)d.thr), d, lb, sweep_idx, phase);
}

// ---------------------------------------------------------------------------
// Potts labels (Sec. "Max-3-Cut"; Eqs. 6-9; the cascaded K = 3 sampler of the
// Supplement).  A label word holds the labels (bytes 0..K-1) of the four
// vertices of a quad, like a spin word.  Visiting vertex v of replica r:
// the K-label field syn_k = sum_j J_vj [s_j = k] over the CSR row (Eq. 7),
// omega_k = e^{beta (syn_k - max syn)} from the step's table, then the
// comparisons of the paper's formulas multiplied through by their positive
// denominators (no division):
//   softmax: the k with the largest omega_k - (gamma u_k 2^-32) S, S = sum
//     omega (Eqs. 8-9: P_k - gamma U_k times S; lowest k on ties);
//   cascade: label 0 iff w0 - s12 > eta_1 (w0 + s12), s12 = w1 + w2 (the
//     p-bit tanh(Delta_1) > eta_1), else label 1 iff w1 - w2 > eta_2 s12,
//     else 2; eta = u 2^-31 - 1;
// u: the visit's words of its quad's Philox blocks (below).  Every operation
// is a correctly rounded binary64 operation in a fixed order (no
// contraction), so the choice is the same wherever it is computed.  The
// energy (Eq. 6) changes by -2 (syn_new - syn_old).
// ---------------------------------------------------------------------------
template <int K>
__device__ __forceinline__ int32_t syn_of(const int32_t (&syn)[K], int k) {
  int32_t x = 0;  // every entry is read, none indexed by k (see the uniform words in k_sweep_potts)
#pragma unroll
  for (int i = 0; i < K; ++i) x |= syn[i] & -(int32_t)(k == i);
  return x;
}

template <int K>
__device__ __forceinline__ int potts_choose(const int32_t (&syn)[K], const uint32_t (&u)[K],
                                            const double* __restrict__ tab, int32_t last, int rule, double gamma) {
  int32_t m = syn[0];
#pragma unroll
  for (int k = 1; k < K; ++k) m = max(m, syn[k]);
  double om[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int32_t dd = m - syn[k];
    om[k] = dd <= last ? tab[dd] : 0.0;
  }
  if constexpr (K == 3) {
    if (rule == 1) {
      const double s12 = om[1] + om[2];
      const double eta1 = (double)u[0] * (1.0 / 2147483648.0) - 1.0;
      if (om[0] - s12 > eta1 * (om[0] + s12)) return 0;
      const double eta2 = (double)u[1] * (1.0 / 2147483648.0) - 1.0;
      return om[1] - om[2] > eta2 * s12 ? 1 : 2;
    }
  }
  double S = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) S += om[k];
  int best = 0;
  double bs = om[0] - (gamma * ((double)u[0] * (1.0 / 4294967296.0))) * S;
#pragma unroll
  for (int k = 1; k < K; ++k) {
    const double sc = om[k] - (gamma * ((double)u[k] * (1.0 / 4294967296.0))) * S;
    if (sc > bs) {
      bs = sc;
      best = k;
    }
  }
  return best;
}

constexpr int kPottsTabLds = 1024;  // doubles of the weight table kept in LDS (8 KB: occupancy)

// K-label fields of the vertices of a quad from the gathered CSR (rows padded
// to multiples of 4 entries with coupling 0; columns as the byte offset of the
// neighbour's label word in a tile plus its byte index).  The four rows lie
// one after another (vertex k's from entry row[k] to row[k + 1]; empty outside
// the class), so the walk takes kAhead groups of four entries together
// wherever the rows meet, with all their label words in flight, and notes the
// running sum at each row's end.
//
// PACKED, when every |syn_k| fits W = 32 / K bits less one (X < 2^(W-1)): the
// K sums are kept as W-bit fields of one 32-bit integer, sum_j J_vj 2^(W
// label_j), so a neighbour costs a shift and an add instead of K
// compare-select-adds; the fields are taken apart at the end, each as the
// sign-extended low W bits of what remains (exact: a row's integer is sum_k
// syn_k 2^(W k) with every |syn_k| < 2^(W-1), which fits 32 bits, and
// differences of the running sums hold modulo 2^32).
//
// A wave's chain of reads bounds it (one quad per wave: n = 7,000, degree 6,
// R = 2,048 is 13 waves a SIMD).  With one row after another, through vector
// loads of its entries, a phase took 38 us; the four rows together with the
// entries from scalar loads, and no array in LDS (see the uniform words
// below), take 22.
template <int K, bool PACKED>
__device__ __forceinline__ void gather_labels(const PAMC_CONST int32_t* __restrict__ gcol,
                                              const PAMC_CONST int32_t* __restrict__ gJ, const int (&row)[5],
                                              __amdgpu_buffer_rsrc_t Sr, int voff, int32_t (&syn)[4][K]) {
  constexpr int kAhead = 4, W = 32 / K, N = PACKED ? 1 : K;
  uint32_t run[N], at_end[4][N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    run[n] = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) at_end[k][n] = 0;
  }
  for (int e = row[0]; e < row[4]; e += 4 * kAhead) {
    int j[kAhead][4];
    uint32_t c[kAhead][4], w[kAhead][4];
#pragma unroll
    for (int g = 0; g < kAhead; ++g) {
      const int at = min(e + 4 * g, row[4] - 4);  // past the last row: its last group again, not counted
      const i32x4 cj = *reinterpret_cast<const PAMC_CONST i32x4*>(gcol + at);
      const i32x4 cJ = *reinterpret_cast<const PAMC_CONST i32x4*>(gJ + at);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        j[g][u] = cj[u];
        c[g][u] = (uint32_t)cJ[u];
      }
    }
#pragma unroll
    for (int g = 0; g < kAhead; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u) w[g][u] = __builtin_amdgcn_raw_buffer_load_b32(Sr, voff, j[g][u] & ~3, 0);
#pragma unroll
    for (int g = 0; g < kAhead; ++g) {
      const int p = e + 4 * g + 4;
      if (p > row[4]) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t lab = __builtin_amdgcn_ubfe(w[g][u], 8u * (uint32_t)(j[g][u] & 3), 8u);
        if constexpr (PACKED) {
          run[0] += c[g][u] << (W * lab);
        } else {
#pragma unroll
          for (int n = 0; n < K; ++n) run[n] += lab == (uint32_t)n ? c[g][u] : 0u;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (p == row[k + 1])
#pragma unroll
          for (int n = 0; n < N; ++n) at_end[k][n] = run[n];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (PACKED) {
      int32_t rest = (int32_t)(at_end[k][0] - (k ? at_end[k - 1][0] : 0u));
#pragma unroll
      for (int n = 0; n < K - 1; ++n) {
        const int32_t f = (int32_t)((uint32_t)rest << (32 - W)) >> (32 - W);
        syn[k][n] = f;
        rest = (rest - f) >> W;
      }
      syn[k][K - 1] = rest;
    } else {
#pragma unroll
      for (int n = 0; n < K; ++n) syn[k][n] = (int32_t)(at_end[k][n] - (k ? at_end[k - 1][n] : 0u));
    }
  }
}

template <int K>
__global__ void __launch_bounds__(256) k_sweep_potts(const Desc* __restrict__ D,
                                                   const uint64_t* __restrict__ map, int sweep_idx,
                                                   int phase) {
  __shared__ int64_t red[kSweepWaves][kLanes];
  __shared__ int32_t fred[kSweepWaves];
  __shared__ double tab_s[kPottsTabLds];
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const PAMC_GLOBAL RunState* __restrict__ st = gmem((const RunState*)d.st);
  if (!st->active || sweep_idx >= st->nsweeps_now || phase >= d.ncls) return;
  const PAMC_CONST int32_t* __restrict__ grow = cmem(d.grow);
  const PAMC_CONST int32_t* __restrict__ gcol = cmem(d.gcol);
  const PAMC_CONST int32_t* __restrict__ gJ = cmem(d.gJ);
  const PAMC_GLOBAL int32_t* __restrict__ class_ptr = gmem(d.class_ptr);
  const int cur = st->cur;
  PAMC_GLOBAL uint32_t* __restrict__ S = gmem(cur ? d.S1 : d.S0);
  PAMC_GLOBAL int64_t* __restrict__ E = gmem(cur ? d.E1 : d.E0);
  const int cls = gmem((const int32_t*)d.order)[sweep_idx * d.ncls + phase];
  const int v0 = class_ptr[cls], v1 = class_ptr[cls + 1];
  const int q0 = v0 >> 2;
  const int nqc = ((v1 + 3) >> 2) - q0;
  int tile, chunk;
  group_chunk(d.T, lb, tile, chunk);
  if (chunk * (kSweepWaves * d.qpw) >= nqc) return;
  const uint32_t gs = st->gs + (uint32_t)sweep_idx;
  const int32_t last = (int32_t)st->table_x;
  const bool lds = last < kPottsTabLds;
  if (lds)
    for (int i = threadIdx.x; i <= last; i += blockDim.x) tab_s[i] = d.ptab[i];
  __syncthreads();
  const double* __restrict__ tab = lds ? tab_s : (const double*)d.ptab;
  const int rule = d.potts_rule;
  const double gamma = d.potts_gamma;
  const bool packed = d.X < (1 << (32 / K - 1));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t r = (uint32_t)(tile * kLanes + lane);
  const uint32_t tstride = (uint32_t)d.nq * kLanes;
  const __amdgpu_buffer_rsrc_t Sr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(S + (size_t)tile * tstride), (short)0, (int)(tstride * 4), kBufferWord3);
  const int voff = lane * 4;
  int64_t dE = 0;
  int32_t nflip = 0;
  for (int i = 0; i < d.qpw; ++i) {
    const int qi = chunk * (kSweepWaves * d.qpw) + i * kSweepWaves + wave;
    if (qi >= nqc) break;
    const int q = q0 + qi;
    uint32_t sw = __builtin_amdgcn_raw_buffer_load_b32(Sr, voff, q * (kLanes * 4), 0);
    const uint32_t sw0 = sw;
    // the four fields first (the class's vertices do not see each other)
    int32_t synq[4][K];
    int row[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) row[k] = grow[min(max(4 * q + k, v0), v1)];
    if (packed)
      gather_labels<K, true>(gcol, gJ, row, Sr, voff, synq);
    else
      gather_labels<K, false>(gcol, gJ, row, Sr, voff, synq);
    // uniform words: W per visit (K, or 2 for the cascade); the quad's
    // visits share W Philox blocks (quad, sweep, replica, POTTS | b << 8),
    // read as one sequence, vertex k of the quad taking words k W .. k W + W-1
    // (both sequences' words are read before the choice between them: an
    // array indexed by the rule would be moved to LDS, with every work-group
    // reading its shape from the dispatch packet in host memory, 7 to 12 us)
    uint32_t uw[4 * K];
    const bool cascade = K == 3 && rule == 1;
#pragma unroll
    for (int b = 0; b < K; ++b) {
      u32x4 w = {0, 0, 0, 0};
      if (b < 2 || !cascade) w = philox10((uint32_t)q, gs, r, kTagPotts | ((uint32_t)b << 8), d.k0, d.k1);
      uw[4 * b] = w.a;
      uw[4 * b + 1] = w.b;
      uw[4 * b + 2] = w.c;
      uw[4 * b + 3] = w.d;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = 4 * q + k;
      if (v >= v0 && v < v1) {
        int32_t syn[K];
#pragma unroll
        for (int c = 0; c < K; ++c) syn[c] = synq[k][c];
        uint32_t u[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
          const uint32_t own = uw[K * k + c], two = c < 2 ? uw[2 * k + c] : 0u;
          u[c] = cascade ? two : own;
        }
        const int old = (int)((sw >> (8 * k)) & 0xFFu);
        const int nw = potts_choose<K>(syn, u, tab, last, rule, gamma);
        if (nw != old) {
          dE += -2 * (int64_t)(syn_of<K>(syn, nw) - syn_of<K>(syn, old));
          sw = (sw & ~(0xFFu << (8 * k))) | ((uint32_t)nw << (8 * k));
          ++nflip;
        }
      }
    }
    if (sw != sw0) __builtin_amdgcn_raw_buffer_store_b32(sw, Sr, voff, q * (kLanes * 4), 0);
  }
  red[wave][lane] = dE;
  if (d.flip_ctr) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nflip += __shfl_xor(nflip, o, 64);
    if (lane == 0) fred[wave] = nflip;
  }
  reduce_energy_and_flips(red, fred, wave, lane, 1, tile, E, gmem(d.flip_ctr));
}

// ---------------------------------------------------------------------------
// Population initialisation (Algorithm 1, initialization): spins uniform from
// Philox(quad, 0, replica, INIT) (spin +1 iff the word < 2^31); then local
// fields by Eq. 3 and energies H = -1/2 sum s h.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_init_spins(const Desc* __restrict__ D,
                                                    const uint64_t* __restrict__ map) {
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const size_t total = (size_t)d.T * d.nq * kLanes;
  for (size_t i = (size_t)lb * blockDim.x + threadIdx.x; i < total; i += (size_t)kInitBlocks * blockDim.x) {
    const int lane = (int)(i & 63);
    const size_t tq = i >> 6;
    const int q = (int)(tq % d.nq);
    const int tile = (int)(tq / d.nq);
    const uint32_t r = (uint32_t)(tile * kLanes + lane);
    const u32x4 w = philox10((uint32_t)q, 0u, r, kTagInit, d.k0, d.k1);
    uint32_t sw = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = 4 * q + k;
      int8_t s = 0;
      if (d.potts_K)  // label floor(u K / 2^32)
        s = v < d.n ? (int8_t)(((uint64_t)pick(w, k) * (uint64_t)d.potts_K) >> 32) : (int8_t)0;
      else if (v < d.n)
        s = pick(w, k) < 0x80000000u ? (int8_t)1 : (int8_t)-1;
      sw |= (uint32_t)(uint8_t)s << (8 * k);
    }
    d.S0[i] = sw;
    if (q == 0) d.F0[r] = (int32_t)r;
  }
}

// h = J s per (tile, vertex) row of buffer `buf` (-1: the current one);
// writes H (Hout if given, else the instance's field array if it has one)
// and, if asked, accumulates sum s h into E.  Work item = (64-vertex chunk,
// tile), dealt to the instance's min(items, kFieldBlocks) work-groups.
__global__ void __launch_bounds__(256) k_init_fields(const Desc* __restrict__ D,
                                                     const uint64_t* __restrict__ map, int32_t buf,
                                                     int32_t* Hout, int32_t accumulate_energy) {
  __shared__ int64_t red[4][kLanes];
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const int b = buf < 0 ? d.st->cur : buf;
  const PAMC_GLOBAL uint32_t* S = gmem((const uint32_t*)(b ? d.S1 : d.S0));
  PAMC_GLOBAL int32_t* H = gmem(Hout ? Hout : (b ? d.H1 : d.H0));
  PAMC_GLOBAL int32_t* HF = gmem(!Hout && d.nhub ? (b ? d.HF1 : d.HF0) : nullptr);  // the kept hub fields
  const int nq = d.nq, np = d.np, n = d.n, T = d.T, hub0 = d.hub_v0, hub1 = d.hub_v1, R = d.R;
  const bool potts = d.potts_K != 0;
  auto spin = [&](int tile, int v, int lane) {
    return (int32_t)(int8_t)(S[((size_t)tile * nq + (v >> 2)) * kLanes + lane] >> (8 * (v & 3)));
  };
  int64_t* E = accumulate_energy ? (b ? d.E1 : d.E0) : nullptr;
  const PAMC_CONST int32_t* __restrict__ row_ptr = cmem(d.row_ptr);
  const PAMC_CONST int32_t* __restrict__ col = cmem(d.col);
  const PAMC_CONST int32_t* __restrict__ J = cmem(d.J);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t items = (int64_t)T * ((n + 63) / 64);
  const int64_t nblocks = items < kFieldBlocks ? items : kFieldBlocks;
  for (int64_t it = lb; it < items; it += nblocks) {
    const int tile = (int)(it % T);
    const int vchunk = (int)(it / T);
    const int v_end = min(n, (vchunk + 1) * 64);
    int64_t acc = 0;
    // sum of J s over the entries e0 .. e1 - 1: eight spin reads in flight, the
    // entries four to a scalar load (one costs a compute unit 8 cycles)
    auto four = [&](int e, int64_t(&hp)[4]) {
      const i32x4u c = *reinterpret_cast<const PAMC_CONST i32x4u*>(col + e);
      const i32x4u w = *reinterpret_cast<const PAMC_CONST i32x4u*>(J + e);
#pragma unroll
      for (int u = 0; u < 4; ++u) hp[u] += (int64_t)w[u] * spin(tile, c[u], lane);
    };
    auto row_field = [&](int e0, int e1) {
      int64_t hp[4] = {0, 0, 0, 0};
      int e = e0;
      for (; e + 8 <= e1; e += 8) {
        four(e, hp);
        four(e + 4, hp);
      }
      if (e + 4 <= e1) {
        four(e, hp);
        e += 4;
      }
      for (; e < e1; ++e) hp[0] += (int64_t)J[e] * spin(tile, col[e], lane);
      return (hp[0] + hp[1]) + (hp[2] + hp[3]);
    };
    auto keep = [&](int v, int64_t h) {
      if (H) H[((size_t)tile * np + v) * kLanes + lane] = (int32_t)h;
      if (HF && (v == hub0 || v == hub1)) HF[(v == hub0 ? 0 : 1) * R + tile * kLanes + lane] = (int32_t)h;
      acc += h * spin(tile, v, lane);
    };
    for (int v = vchunk * 64 + wave; v < v_end; v += 4) {
      const int e0 = row_ptr[v], e1 = row_ptr[v + 1];
      if (potts) {
        // Potts labels (Eq. 6): sum_j J_vj (2 delta(s_v, s_j) - 1); no fields
        const int32_t lv = spin(tile, v, lane);
        for (int e = e0; e < e1; ++e) acc += spin(tile, col[e], lane) == lv ? J[e] : -J[e];
        if (H) H[((size_t)tile * np + v) * kLanes + lane] = 0;
      } else if (e1 - e0 < kLongRow) {
        keep(v, row_field(e0, e1));
      }
    }
    // long (hub) rows: a quarter to each wave.  With a row of 21,000 entries the
    // launch takes 0.64 ms; walked by one wave, its entries through vector loads,
    // it took 2.1 (G(800, 19176), R = 256: 0.054 and 0.086).
    for (int v = vchunk * 64; v < v_end && !potts; ++v) {
      const int e0 = row_ptr[v], e1 = row_ptr[v + 1], len = e1 - e0;
      if (len < kLongRow) continue;
      const int from = e0 + (int)((int64_t)len * wave / 4), to = e0 + (int)((int64_t)len * (wave + 1) / 4);
      __syncthreads();
      red[wave][lane] = row_field(from, to);
      __syncthreads();
      if (wave == 0) keep(v, (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]));
    }
    __syncthreads();
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && E) {
      const int64_t t = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
      if (t != 0)
        __hip_atomic_fetch_add((unsigned long long*)&E[tile * kLanes + lane], (unsigned long long)t,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// E currently holds sum_v s_v h_v (= 2 sum_{i<j} J s s; Potts labels: 2
// sum_{i<j} J (2 delta - 1)); H = -that / 2.  The best configuration starts
// with cut 0: all spins +1, or all labels 0.  One work-group per instance.
__global__ void __launch_bounds__(256) k_init_finish(const Desc* __restrict__ D) {
  const Desc& d = D[blockIdx.x];
  for (int i = threadIdx.x; i < d.R; i += blockDim.x) d.E0[i] = -(d.E0[i] / 2);
  for (int v = threadIdx.x; v < d.np; v += blockDim.x) d.best[v] = d.potts_K ? 0 : 1;
  if (threadIdx.x == 0) {
    RunState* st = d.st;
    st->mstar = 0;
    st->cur = 0;
    st->gs = st->g_rs = st->g_cl = 0;
    st->stopped = 0;
    st->active = 0;
    st->steps_run = 0;
  }
}

// Population loaded by the host into buffer 0: E holds sum_v s_v h_v (Potts
// labels: 2 sum_{i<j} J (2 delta - 1)); H = -that / 2, and buffer 0 becomes
// the current one.  One work-group per instance.
__global__ void __launch_bounds__(256) k_load_finish(const Desc* __restrict__ D) {
  const Desc& d = D[blockIdx.x];
  for (int i = threadIdx.x; i < d.R; i += blockDim.x) d.E0[i] = -(d.E0[i] / 2);
  if (threadIdx.x == 0) d.st->cur = 0;
}

// ---------------------------------------------------------------------------
// Controller kernels (one thread per instance): Algorithm 1's decisions.
// ---------------------------------------------------------------------------
__global__ void k_anneal_setup(const Desc* __restrict__ D, const Schedule* __restrict__ sched,
                               const int32_t* __restrict__ idx, int32_t count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  RunState* st = D[idx ? idx[i] : i].st;
  const Schedule s = sched[i];
  st->beta0 = s.beta0;
  st->dbeta = s.dbeta;
  st->reheat = s.reheat;
  st->target = s.target;
  st->steps = s.steps;
  st->sweeps = s.sweeps;
  st->z_rst = s.z_rst;
  st->augmented = s.augmented;
  st->resample = s.resample;
  st->win_short = s.win_short;
  st->win_long = s.win_long;
  st->max_ds = s.max_ds;
  st->max_dl = s.max_dl;
  st->tau = s.tau;
  st->n_top = s.n_top;
  st->mis_trials = s.mis_trials;
  st->stop_at_target = s.stop_at_target;
  st->literal_break = s.literal_break;
  st->stopped = 0;
  st->active = 0;
  st->dh_every = s.dh_every;
  st->dh_sum = 0;
  st->t_start = wall_clock64();
  st->t_last = st->t_start;
  if (s.resume) {  // the run goes on from the controller it holds
    st->t_reached = st->step_reached >= 0 ? st->t_start : 0;
    return;
  }
  st->z = 1;
  st->cycle = 0;
  st->beta = s.beta0;
  st->delta = s.dbeta;
  st->enable = 0;
  st->cooldown = 0;
  st->hist_len = 0;
  st->step_reached = -1;
  st->steps_run = 0;
  st->sum_lnq = 0.0;
  st->last_lnq = 0.0;
  st->n_cluster_moves = st->n_reheats = st->n_reversals = st->n_restarts = 0;
  st->t_reached = 0;
}

// Decisions of a run's beta step (Algorithm 1), by one thread per instance.
__device__ __forceinline__ void begin_step(const Desc& d) {
  RunState* st = d.st;
  if (st->stopped || st->steps_run >= st->steps || (st->stop_at_target && st->mstar >= st->target)) {
    st->stopped = 1;
    st->active = 0;
    return;
  }
  st->active = 1;
  st->step = st->steps_run;
  st->do_resample = (st->z > 1 && st->resample) ? 1 : 0;
  // cluster moves are defined for Ising spins only
  st->do_cluster = (st->do_resample && st->augmented && st->enable && st->cooldown == 0 && !d.potts_K) ? 1 : 0;
  st->rs_delta = st->delta;
  st->sweep_beta = st->beta;
  st->nsweeps_now = st->sweeps;
  st->cl_n_top = st->n_top;
  st->cl_trials = st->mis_trials;
  st->table_x = d.potts_K ? potts_table_last(st->beta, d.X) : table_halfwidth(st->beta, d.X);
  st->last_lnq = 0.0;
}

__global__ void k_step_begin(const Desc* __restrict__ D, int32_t ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ninst) begin_step(D[i]);
}

// Primitive calls: one data-parallel action outside a run.
__global__ void k_prim_set(const Desc* __restrict__ D, int32_t ninst, int32_t kind, double value,
                           int32_t n_top, int32_t trials, int32_t nsweeps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  RunState* st = D[i].st;
  st->active = 1;
  st->do_resample = kind == 1;
  st->do_cluster = kind == 2;
  st->rs_delta = value;
  st->sweep_beta = value;
  st->nsweeps_now = nsweeps;
  st->cl_n_top = n_top;
  st->cl_trials = trials;
  st->table_x = D[i].potts_K ? potts_table_last(value, D[i].X) : table_halfwidth(value, D[i].X);
  st->last_lnq = 0.0;
}

// After resampling / cluster move: switch population buffers and advance the
// stream counters; in a run also apply Algorithm 1's "enable <- false;
// cooldown <- tau" after a cluster move.
__device__ __forceinline__ void commit_step(const Desc& d, int32_t in_run) {
  RunState* st = d.st;
  if (!st->active) return;
  if (st->do_resample) {
    st->cur ^= 1;
    st->g_rs += 1;
    if (in_run) {
      st->sum_lnq += st->last_lnq;
      if (st->step < d.tr_cap) d.tr_lnq[st->step] = st->last_lnq;
    }
  } else if (in_run && st->step < d.tr_cap) {
    d.tr_lnq[st->step] = 0.0;
  }
  if (st->do_cluster) {
    st->g_cl += 1;
    if (in_run) {
      st->enable = 0;
      st->cooldown = st->tau;
      st->n_cluster_moves += 1;
    }
  }
}

__global__ void k_commit(const Desc* __restrict__ D, int32_t ninst, int32_t in_run) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ninst) commit_step(D[i], in_run);
}

// Threshold table for the step's beta (entries x = -Xt..Xt) and the class
// order of each of the step's sweeps: a Fisher-Yates shuffle driven by
// Philox(i, sweep, 0, ORDER), j = floor(u (i+1) / 2^32).  With commit >= 0
// the instance's first block also commits the step's resampling / cluster
// move (commit = in_run); no field read here is changed by that.
__global__ void __launch_bounds__(256) k_thresholds(const Desc* __restrict__ D,
                                                    const uint64_t* __restrict__ map, int32_t commit,
                                                    int32_t bit_sweeps) {
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  const RunState* st = d.st;
  const bool bits = d.bits && bit_sweeps > 0;
  const int bsw = bits ? min(bit_sweeps, d.order_cap) : 0;  // sweeps whose phases will be launched
  if (!st->active) {
    // an instance at rest: its bit-packed phases are empty
    if (lb == 0)
      for (int i = threadIdx.x; i < bsw * d.ncls; i += blockDim.x)
        reinterpret_cast<int4*>(d.bphases)[i] = make_int4(0, 0, 0, 0);
    return;
  }
  if (commit >= 0 && lb == 0) {
    if (threadIdx.x == 0) commit_step(d, commit);
    __syncthreads();  // the phase records below name the buffer it makes current
  }
  if (d.not_monotone && lb == 0 && threadIdx.x == 0) *d.not_monotone = 0;
  const int64_t Xt = st->table_x;
  const double beta = st->sweep_beta;
  if (d.potts_K) {  // e^{beta (syn_k - max syn)} for max syn - syn_k = i
    for (int64_t i = (int64_t)lb * blockDim.x + threadIdx.x; i <= Xt; i += (int64_t)kThrBlocks * blockDim.x)
      d.ptab[i] = exp_cw(beta * (double)(-i));
  } else if (bits) {
    // bit-packed sweeps: entry i of one half is T[c (i - X)], of the other
    // T[-c (i - X)] (X the longest row, c the coupling's magnitude)
    const int32_t half = 2 * d.bmaxdeg + 2;
    for (int32_t i = lb * blockDim.x + threadIdx.x; i < 2 * half; i += kThrBlocks * blockDim.x) {
      const int32_t k = i % half;
      int64_t x = (int64_t)(k - d.bmaxdeg) * d.bcoup;
      if (i < half) x = -x;
      d.btab[i] = k > 2 * d.bmaxdeg ? 0u : flip_threshold(beta, d.rule, x < -Xt ? -Xt : (x > Xt ? Xt : x));
    }
  } else {
    for (int64_t i = (int64_t)lb * blockDim.x + threadIdx.x; i <= 2 * Xt; i += (int64_t)kThrBlocks * blockDim.x)
      d.thr[i] = flip_threshold(beta, d.rule, i - Xt);
  }
  if (lb == 0 && d.ncls > 0) {
    const int nsw = min(st->nsweeps_now, d.order_cap), ncls = d.ncls;
    if (ncls <= kOrderLds) {
      // as many sweeps at a time as LDS holds: their draws and results by all
      // threads, each sweep's exchanges by one (a chain of reads and writes
      // that took a microsecond a class in memory)
      __shared__ int32_t perm[kOrderLds], with[kOrderLds];
      const int per = kOrderLds / ncls;
      for (int s0 = 0; s0 < nsw; s0 += per) {
        const int ns = min(per, nsw - s0);
        for (int i = threadIdx.x; i < ns * ncls; i += blockDim.x) {
          const int k = i % ncls;
          perm[i] = k;
          if (d.shuffle) {
            const u32x4 w = philox10((uint32_t)k, st->gs + (uint32_t)(s0 + i / ncls), 0u, kTagOrder, d.k0, d.k1);
            with[i] = (int)(((uint64_t)w.a * (uint64_t)(k + 1)) >> 32);
          }
        }
        __syncthreads();
        if (d.shuffle)
          for (int s = threadIdx.x; s < ns; s += blockDim.x) {
            int32_t* o = perm + s * ncls;
            for (int i = ncls - 1; i >= 1; --i) {
              const int j = with[s * ncls + i];
              const int32_t t = o[i];
              o[i] = o[j];
              o[j] = t;
            }
          }
        __syncthreads();
        for (int i = threadIdx.x; i < ns * ncls; i += blockDim.x) {
          const int32_t c = perm[i];
          d.order[s0 * ncls + i] = c;
          if (bits)  // the phases in visiting order
            reinterpret_cast<int4*>(d.bphases)[s0 * ncls + i] =
                make_int4(d.class_ptr[c], d.class_ptr[c + 1], (int32_t)(st->gs + (uint32_t)(s0 + i / ncls)), st->cur);
        }
        __syncthreads();
      }
    } else {
      for (int s = threadIdx.x; s < nsw; s += blockDim.x) {
        int32_t* o = d.order + (size_t)s * ncls;
        for (int k = 0; k < ncls; ++k) o[k] = k;
        const uint32_t gs = st->gs + (uint32_t)s;
        for (int i = d.shuffle ? ncls - 1 : 0; i >= 1; --i) {
          const u32x4 w = philox10((uint32_t)i, gs, 0u, kTagOrder, d.k0, d.k1);
          const int j = (int)(((uint64_t)w.a * (uint64_t)(i + 1)) >> 32);
          const int32_t t = o[i];
          o[i] = o[j];
          o[j] = t;
        }
        if (bits)
          for (int k = 0; k < ncls; ++k)
            reinterpret_cast<int4*>(d.bphases)[(size_t)s * ncls + k] =
                make_int4(d.class_ptr[o[k]], d.class_ptr[o[k] + 1], (int32_t)gs, st->cur);
      }
    }
    if (bits)  // sweeps that other instances of a batch still make
      for (int i = nsw * d.ncls + threadIdx.x; i < bsw * d.ncls; i += blockDim.x)
        reinterpret_cast<int4*>(d.bphases)[i] = make_int4(0, 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Block-wide helpers for the 1024-thread per-instance kernels: shuffles
// within each wave, then the 16 wave results through LDS.
// ---------------------------------------------------------------------------
template <typename V>
__device__ __forceinline__ V block_excl_scan(V x, V* part16) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  V inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) part16[wv] = inc;
  __syncthreads();
  V off = 0;
  for (int i = 0; i < wv; ++i) off += part16[i];
  __syncthreads();
  return off + inc - x;
}

// Stagnation classes of the recent-progress history (Sec. "Augmented PAMC"),
// from the distinct M* values in its short (ds) and long (dl) tails: few
// distinct values in both tails is a strong stall, in the short tail only a
// mild one, otherwise the search still progresses.
enum : int { kStagNone = 0, kStagProgress = 1, kStagMild = 2, kStagStrong = 3 };
__device__ __forceinline__ int stagnation_class(int ds, int dl, int max_ds, int max_dl) {
  if (ds > max_ds) return kStagProgress;
  return dl <= max_dl ? kStagStrong : kStagMild;
}

// ---------------------------------------------------------------------------
// Best cut (Algorithm 1: M* <- max(M*, max Cut(P)), lowest slot on ties),
// then, in a run, the recent-progress history, the adaptive temperature rule
// and the schedule advance.  One work-group per instance; the distinct
// counts over the two history windows are taken by one thread per entry.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_step_end(const Desc* __restrict__ D, int32_t in_run) {
  __shared__ int64_t bc[16];
  __shared__ int32_t bs[16];
  __shared__ int64_t hs[kHistCap];
  const Desc& a = D[blockIdx.x];
  RunState* st = a.st;
  if (!st->active) return;
  // every thread reads the state it needs before the first barrier; thread
  // 0 writes it only after the last one
  const int cur = st->cur;
  const int64_t mstar_old = st->mstar;
  const int L0 = st->hist_len, wl = st->win_long, ws = st->win_short;
  const bool eval_ok = st->augmented && st->cooldown == 0;
  const int64_t* E = cur ? a.E1 : a.E0;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int64_t c = INT64_MIN;
  int32_t cs = 0x7FFFFFFF;
  for (int r = tid; r < a.R; r += blockDim.x) {
    const int64_t cut = (a.W - E[r]) / 2;
    if (cut > c) { c = cut; cs = r; }  // r increases: ties keep the lower slot
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t c2 = __shfl_xor(c, o, 64);
    const int32_t s2 = __shfl_xor(cs, o, 64);
    if (c2 > c || (c2 == c && s2 < cs)) { c = c2; cs = s2; }
  }
  if (lane == 0) { bc[wv] = c; bs[wv] = cs; }
  __syncthreads();
  int64_t m = bc[0];
  int32_t slot = bs[0];
  for (int i = 1; i < 16; ++i)
    if (bc[i] > m || (bc[i] == m && bs[i] < slot)) { m = bc[i]; slot = bs[i]; }
  const bool improved = m > mstar_old;
  if (improved) {
    if (a.dense) {
      const int8_t* Dsp = (cur ? a.D1 : a.D0) + (size_t)slot * a.np;
      for (int v = tid; v < a.np; v += blockDim.x) a.best[v] = Dsp[v];
    } else {
      // one spin word (4 spins) per thread and step
      const uint32_t* S = cur ? a.S1 : a.S0;
      const int tile = slot >> 6, sl = slot & 63;
      for (int q = tid; q < a.nq; q += blockDim.x)
        reinterpret_cast<uint32_t*>(a.best)[q] = S[((size_t)tile * a.nq + q) * kLanes + sl];
    }
  }
  if (!in_run) {
    if (tid == 0 && improved) {
      st->mstar = m;
      st->best_slot = slot;
    }
    return;
  }
  const int64_t ms = improved ? m : mstar_old;
  // recent-progress history: the oldest value leaves once win_long are
  // held, then M* is appended
  const int drop = L0 >= wl ? 1 : 0;
  const int L = L0 - drop + 1;
  if (tid < L - 1) hs[tid] = st->hist[tid + drop];
  if (tid == L - 1) hs[tid] = ms;
  __syncthreads();
  if (tid < L) st->hist[tid] = hs[tid];
  int ds = 0, dl = 0;
  if (eval_ok && L >= wl) {  // uniform
    // entry tid counts for a window when no earlier entry of that window
    // holds the same value
    bool first_s = tid >= L - ws && tid < L, first_l = tid >= L - wl && tid < L;
    if (first_l) {
      const int64_t v = hs[tid];
      for (int j = L - wl; j < tid; ++j)
        if (hs[j] == v) {
          first_l = false;
          if (j >= L - ws) first_s = false;
        }
    }
    ds = __syncthreads_count(first_s);
    dl = __syncthreads_count(first_l);
  }
  if (tid != 0) return;
  if (improved) {
    st->mstar = m;
    st->best_slot = slot;
  }
  st->hist_len = L;
  int32_t ev = (st->do_resample ? 1 : 0) | (st->do_cluster ? 2 : 0);
  const uint64_t now = wall_clock64();
  if (st->step_reached < 0 && ms >= st->target) {
    st->step_reached = st->step;
    st->t_reached = now;
  }
  // the history's stagnation class picks the temperature action (see
  // stagnation_class), then the schedule moves on
  switch (eval_ok && L >= wl ? stagnation_class(ds, dl, st->max_ds, st->max_dl) : kStagNone) {
    case kStagStrong:  // reheat and arm the cluster move
      st->beta = st->reheat * st->beta;
      st->delta = st->dbeta;
      st->enable = 1;
      ev |= 4;
      st->n_reheats += 1;
      break;
    case kStagMild:  // run the schedule backwards while above beta0
      if (st->beta > st->beta0) {
        st->delta = -st->dbeta;
        ev |= 8;
        st->n_reversals += 1;
      } else if (st->literal_break) {
        st->stopped = 1;
      } else {
        st->delta = st->dbeta;
      }
      break;
    case kStagProgress:
      st->delta = st->dbeta;
      break;
    default:
      break;
  }
  const bool restart = st->z_rst > 0 && st->z >= st->z_rst;
  if (restart) {  // schedule, arming, cooldown and history start over
    st->cycle += 1;
    st->z = 1;
    st->beta = st->beta0;
    st->delta = st->dbeta;
    st->enable = 0;
    st->cooldown = 0;
    st->hist_len = 0;
    ev |= 16;
    st->n_restarts += 1;
  } else {
    st->z += 1;
    st->beta = st->beta + st->delta;
    if (st->cooldown > 0) st->cooldown -= 1;
  }
  st->gs += (uint32_t)st->sweeps;
  st->steps_run = st->step + 1;
  st->t_last = now;
  if (st->step < a.tr_cap) {
    a.tr_mstar[st->step] = ms;
    a.tr_beta[st->step] = st->sweep_beta;
    a.tr_events[st->step] = ev;
    a.tr_time[st->step] = now;
  }
  if (st->stop_at_target && ms >= st->target) st->stopped = 1;
  if (st->steps_run >= st->steps) st->stopped = 1;
}

__global__ void k_advance_sweeps(const Desc* __restrict__ D, int32_t ninst, int32_t nsweeps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  D[i].st->gs += (uint32_t)nsweeps;
  D[i].st->active = 0;
}

__global__ void k_deactivate(const Desc* __restrict__ D, int32_t ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ninst) D[i].st->active = 0;
}

// Per-instance status words for the host: bit 0 stopped, bits 1.. steps run.
__global__ void k_status(const Desc* __restrict__ D, int32_t ninst, int32_t* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ninst) out[i] = (D[i].st->steps_run << 1) | (D[i].st->stopped ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Targets of the non-local cluster move: the n_top slots with the lowest
// (E, slot), by a radix select on E - min E; they are listed in slot order
// (each target's move depends on its slot only).
// ---------------------------------------------------------------------------
// LDS of the target selection (declared by the calling kernel).
struct SelectLds {
  uint32_t hist[256];
  uint64_t part_u[16];
  int32_t part_i[16];
  uint64_t pick_prefix;
  int32_t pick_want;
};

// Energy of slot r of the population the cluster move acts on: E[r], or,
// right after the resampling draw, the energy of r's parent.
__device__ __forceinline__ int64_t target_energy(const int64_t* E, const int32_t* parent, int r) {
  return E[parent ? parent[r] : r];
}

// Called by all 1024 threads of the work-group.
__device__ __forceinline__ void select_cluster_targets(const Desc& d, const RunState* st, const int64_t* E,
                                       const int32_t* parent, SelectLds& L) {
  uint32_t* hist = L.hist;
  uint64_t* part_u = L.part_u;
  int32_t* part_i = L.part_i;
  const int R = d.R;
  // no targets without scratch (a move with no trials flips nothing)
  const int n_top = (d.cl_targets && st->cl_trials > 0) ? min(st->cl_n_top, R) : 0;
  if (n_top <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // a contiguous chunk of slots per thread, keys E - min E as unsigned
  constexpr int kPer = kRsMaxR / 1024;
  const int per = (R + 1023) >> 10;
  const int r0 = min(R, tid * per), r1 = min(R, r0 + per);
  int64_t e[kPer];
  int64_t emin = INT64_MAX;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    e[i] = r0 + i < r1 ? target_energy(E, parent, r0 + i) : INT64_MAX;
    emin = e[i] < emin ? e[i] : emin;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t y = __shfl_xor(emin, o, 64);
    emin = y < emin ? y : emin;
  }
  if (lane == 0) part_u[wv] = (uint64_t)emin;
  __syncthreads();
  emin = (int64_t)part_u[0];
  for (int i = 1; i < 16; ++i) emin = (int64_t)part_u[i] < emin ? (int64_t)part_u[i] : emin;
  __syncthreads();
  uint64_t key[kPer], kmax = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    key[i] = (uint64_t)e[i] - (uint64_t)emin;
    if (r0 + i < r1 && key[i] > kmax) kmax = key[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t y = __shfl_xor(kmax, o, 64);
    kmax = y > kmax ? y : kmax;
  }
  if (lane == 0) part_u[wv] = kmax;
  __syncthreads();
  kmax = part_u[0];
  for (int i = 1; i < 16; ++i) kmax = part_u[i] > kmax ? part_u[i] : kmax;
  // radix select, 8 bits a pass from the highest used bit: t = the key of
  // the n_top-th smallest (E, slot); want = how many slots with key t are
  // taken (the lowest ones)
  const int nbits = kmax ? 64 - __clzll((long long)kmax) : 0;
  uint64_t t = 0;
  int want = n_top;
  for (int s = ((nbits + 7) / 8) * 8 - 8; s >= 0; s -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (r0 + i < r1 && (s + 8 >= 64 || ((key[i] ^ t) >> (s + 8)) == 0))
        atomicAdd(&hist[(key[i] >> s) & 255u], 1u);
    __syncthreads();
    if (wv == 0) {
      uint32_t h[4], tot = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) { h[j] = hist[4 * lane + j]; tot += h[j]; }
      uint32_t inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
      }
      uint32_t cum = inc - tot;
      if (cum < (uint32_t)want && (uint32_t)want <= inc) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (cum + h[j] >= (uint32_t)want) {
            L.pick_prefix = t | ((uint64_t)(4 * lane + j) << s);
            L.pick_want = want - (int)cum;
            break;
          }
          cum += h[j];
        }
      }
    }
    __syncthreads();
    t = L.pick_prefix;
    want = L.pick_want;
  }
  // selected: key < t, or key == t among the first `want` such slots
  int neq = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) neq += (r0 + i < r1 && key[i] == t) ? 1 : 0;
  int eq_before = block_excl_scan<int32_t>(neq, part_i);
  bool sel[kPer];
  int nsel = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    sel[i] = false;
    if (r0 + i < r1) {
      if (key[i] < t) sel[i] = true;
      else if (key[i] == t) sel[i] = eq_before++ < want;
    }
    nsel += sel[i] ? 1 : 0;
  }
  int pos = block_excl_scan<int32_t>(nsel, part_i);
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (sel[i]) d.cl_targets[pos++] = r0 + i;
}

// ---------------------------------------------------------------------------
// Resampling (Eqs. 1-2), one work-group per instance.  Weights relative to
// the extreme energy, w_r = e^{-Delta (E_r - E_ref)} in binary64; ln Q =
// -Delta E_ref + ln sum w - ln R.  Selection is exact integer arithmetic:
// q_r = floor(w_r 2^48), inclusive prefix P, child k draws a 64-bit Philox
// word u, y = floor(u Q / 2^64), parent = least j with P_j > y; children are
// then laid out by parent (counting sort).
// ---------------------------------------------------------------------------
// In a run (fused = 1) the kernel first takes the step's decisions and,
// when the step makes a cluster move, ends by selecting its targets from the
// children's energies.
__global__ void __launch_bounds__(1024) k_rs_select(const Desc* __restrict__ D, int32_t fused) {
  // the prefix P in LDS for the children's searches, then the same space
  // holds the number of children of each slot
  extern __shared__ uint64_t P[];
  __shared__ int64_t part_m[16];
  __shared__ uint64_t part_u[16];
  __shared__ double part_d[16];
  __shared__ int32_t part_i[16];
  __shared__ SelectLds L;
  const Desc& a = D[blockIdx.x];
  RunState* st = a.st;
  if (fused) {
    if (threadIdx.x == 0) begin_step(a);
    __syncthreads();
  }
  if (!st->active || !st->do_resample) return;
  const int64_t* E = st->cur ? a.E1 : a.E0;
  // Potts labels: the update of Eq. 8 at beta leaves e^{-(beta/2) E}
  // invariant for the Eq. 6 energy, so the weights use Delta/2
  const double delta = a.potts_K ? 0.5 * st->rs_delta : st->rs_delta;
  const bool lowest = delta >= 0;  // reference energy: min for delta >= 0, max otherwise
  const int R = a.R;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int64_t m = E[0];
  for (int r = tid; r < R; r += 1024) {
    const int64_t e = E[r];
    if (lowest ? e < m : e > m) m = e;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t y = __shfl_xor(m, o, 64);
    if (lowest ? y < m : y > m) m = y;
  }
  if (lane == 0) part_m[wv] = m;
  __syncthreads();
  int64_t eref = part_m[0];
  for (int i = 1; i < 16; ++i)
    if (lowest ? part_m[i] < eref : part_m[i] > eref) eref = part_m[i];
  // weights and their integer prefix, a contiguous chunk of slots per thread
  const int per = (R + 1023) >> 10;
  const int r0 = min(R, tid * per), r1 = min(R, r0 + per);
  double wsum = 0.0;
  uint64_t run = 0;
  for (int r = r0; r < r1; ++r) {
    const double w = exp_cw(-(delta * (double)(E[r] - eref)));
    wsum += w;
    run += (uint64_t)floor(w * 281474976710656.0);
    P[r] = run;  // local inclusive prefix
  }
  const uint64_t off = block_excl_scan<uint64_t>(run, part_u);
  for (int r = r0; r < r1; ++r) P[r] += off;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) wsum += __shfl_xor(wsum, o, 64);
  if (lane == 0) part_d[wv] = wsum;
  __syncthreads();
  double wtot = 0.0;
  for (int i = 0; i < 16; ++i) wtot += part_d[i];
  const uint64_t Q = P[R - 1];
  const uint32_t g = st->g_rs;
  // searches with a fixed number of steps (no divergence; the LDS reads of a
  // thread's searches overlap): least j with P[j] > y, as the count of
  // entries <= y; P[R-1] = Q > y
  const int top = 1 << (31 - __clz(R));  // largest power of two <= R
  int par[kRsMaxR / 1024];
#pragma unroll
  for (int i0 = 0; i0 < kRsMaxR / 1024; i0 += 4) {  // four searches at a time
    uint64_t yv[4];
#pragma unroll
    for (int i = i0; i < i0 + 4; ++i) {
      const int k = tid + 1024 * i;
      par[i] = -1;
      yv[i - i0] = 0;
      if (k < R) {
        const u32x4 w = philox10((uint32_t)(k >> 1), g, 0u, kTagResample, a.k0, a.k1);
        const uint64_t u = (k & 1) ? ((uint64_t)w.c | ((uint64_t)w.d << 32))
                                   : ((uint64_t)w.a | ((uint64_t)w.b << 32));
        yv[i - i0] = __umul64hi(u, Q);
        par[i] = 0;
      }
    }
    if (tid + 1024 * i0 >= R) continue;
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        const int nx = par[i] + step;  // candidate count: P[nx - 1] <= y
        if (par[i] >= 0 && nx <= R && P[nx - 1] <= yv[i - i0]) par[i] = nx;
      }
    }
  }
  __syncthreads();
  int32_t* cnt = reinterpret_cast<int32_t*>(P);
  for (int r = tid; r < R; r += 1024) cnt[r] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRsMaxR / 1024; ++i)
    if (par[i] >= 0) atomicAdd(&cnt[par[i]], 1);
  __syncthreads();
  // children ordered by parent: cnt becomes the inclusive prefix C, and
  // child j's parent is the least r with C_r > j
  int local = 0;
  for (int r = r0; r < r1; ++r) {
    local += cnt[r];
    cnt[r] = local;
  }
  const int coff = block_excl_scan<int32_t>(local, part_i);
  for (int r = r0; r < r1; ++r) cnt[r] += coff;
  __syncthreads();
#pragma unroll
  for (int i0 = 0; i0 < kRsMaxR / 1024; i0 += 4) {
    if (tid + 1024 * i0 >= R) break;
    int pj[4] = {0, 0, 0, 0};
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = tid + 1024 * (i0 + i), nx = pj[i] + step;
        if (j < R && nx <= R && cnt[nx - 1] <= j) pj[i] = nx;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (tid + 1024 * (i0 + i) < R) a.rs_parent[tid + 1024 * (i0 + i)] = pj[i];
  }
  if (tid == 0) st->last_lnq = -delta * (double)eref + log(wtot) - log((double)R);
  if (fused && st->do_cluster) {
    __syncthreads();
    select_cluster_targets(a, st, E, a.rs_parent, L);
  }
}

// Copies every child's spins, fields, energy and lineage from its parent into
// the other population buffer.  Local block = (tile, quad chunk).
__global__ void __launch_bounds__(256) k_rs_gather(const Desc* __restrict__ D,
                                                   const uint64_t* __restrict__ map) {
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& a = D[inst];
  RunState* st = a.st;
  if (!st->active || !st->do_resample) return;
  const int cur = st->cur;
  const PAMC_GLOBAL uint32_t* __restrict__ Ss = gmem((const uint32_t*)(cur ? a.S1 : a.S0));
  PAMC_GLOBAL uint32_t* __restrict__ Sd = gmem(cur ? a.S0 : a.S1);
  const PAMC_GLOBAL int32_t* __restrict__ Hs = gmem((const int32_t*)(cur ? a.H1 : a.H0));
  PAMC_GLOBAL int32_t* __restrict__ Hd = gmem(cur ? a.H0 : a.H1);
  int tile, chunk;
  group_chunk(a.T, lb, tile, chunk);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = tile * kLanes + lane;
  const int p = gmem(a.rs_parent)[c];
  const int pt = p >> 6, pl = p & 63;
  if (chunk == 0 && wave == 0) {
    (cur ? a.E0 : a.E1)[c] = (cur ? a.E1 : a.E0)[p];
    (cur ? a.F0 : a.F1)[c] = (cur ? a.F1 : a.F0)[p];
    for (int hk = 0; hk < a.nhub; ++hk) (cur ? a.HF0 : a.HF1)[hk * a.R + c] = (cur ? a.HF1 : a.HF0)[hk * a.R + p];
  }
  const int qb = chunk * kGatherQuadsPerBlock;
  // the wave's spin words: every read issued before the first write, so
  // that they are in flight together
  constexpr int kPer = kGatherQuadsPerBlock / 4;
  uint32_t w[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int q = qb + wave + 4 * i;
    if (q < a.nq) w[i] = Ss[((size_t)pt * a.nq + q) * kLanes + pl];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int q = qb + wave + 4 * i;
    if (q < a.nq) Sd[((size_t)tile * a.nq + q) * kLanes + lane] = w[i];
  }
  if (!Hs) return;
  // the fields (incremental mode), four quads (16 words) in flight at a time
  for (int i0 = 0; i0 < kPer; i0 += 4) {
    int32_t hv[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = qb + wave + 4 * (i0 + i);
      if (q < a.nq) {
#pragma unroll
        for (int k = 0; k < 4; ++k) hv[i][k] = Hs[((size_t)pt * a.np + 4 * q + k) * kLanes + pl];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = qb + wave + 4 * (i0 + i);
      if (q < a.nq) {
#pragma unroll
        for (int k = 0; k < 4; ++k) Hd[((size_t)tile * a.np + 4 * q + k) * kLanes + lane] = hv[i][k];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Non-local cluster move (Algorithm 1; Sec. "Augmented PAMC").
// cl_select: the targets (see select_cluster_targets; in a run this is done
//   at the end of the resampling selection).
// cl_mis: per (target, trial), the greedy independent set of iso-sites
//   (h = 0) in the order of Philox keys (v, g_cl, r, CL | t<<8), ties by id.
//   The sequential greedy is computed with parallel rounds: an undecided
//   vertex joins once no undecided neighbour precedes it, and leaves once a
//   neighbour has joined; this selects exactly the sequential greedy set.
// cl_apply: flips the largest set (earliest trial on ties); fields of the
//   neighbours change, the energy does not (every flipped spin has h = 0 and
//   no two are coupled).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_cl_select(const Desc* __restrict__ D) {
  __shared__ SelectLds L;
  const Desc& d = D[blockIdx.x];
  RunState* st = d.st;
  if (!st->active || !st->do_cluster) return;
  const int buf = st->cur ^ st->do_resample;
  select_cluster_targets(d, st, buf ? d.E1 : d.E0, nullptr, L);
}

enum : uint8_t { kOut = 0, kUnd = 1, kCand = 2, kIn = 3 };

// Local block = target * trials + trial.
__global__ void __launch_bounds__(1024) k_cl_mis(const Desc* __restrict__ D, const uint64_t* __restrict__ map) {
  extern __shared__ uint8_t lds[];
  __shared__ int32_t cnt_s;
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& a = D[inst];
  RunState* st = a.st;
  if (!st->active || !st->do_cluster) return;
  const int trials = st->cl_trials;
  if (trials <= 0) return;
  const int i = lb / trials, t = lb % trials;
  if (i >= min(st->cl_n_top, a.R)) return;
  const int buf = st->cur ^ st->do_resample;
  const int32_t* H = buf ? a.H1 : a.H0;
  const uint32_t* S = buf ? a.S1 : a.S0;
  uint32_t* key = (uint32_t*)lds;
  uint8_t* state = lds + sizeof(uint32_t) * (size_t)a.np;
  const int r = a.cl_targets[i];
  const int tile = r >> 6, lane = r & 63;
  const uint32_t g = st->g_cl;
  for (int v = threadIdx.x; v < a.np; v += blockDim.x) {
    uint8_t s = kOut;
    int32_t h = 1;
    if (v < a.n) {
      if (H) {
        h = H[((size_t)tile * a.np + v) * kLanes + lane];
      } else if (a.nhub && (v == a.hub_v0 || v == a.hub_v1)) {
        h = (buf ? a.HF1 : a.HF0)[(v == a.hub_v0 ? 0 : 1) * a.R + r];
      } else {
        h = 0;
        for (int e = a.row_ptr[v]; e < a.row_ptr[v + 1]; ++e) h += a.J[e] * spin_at(S, a.nq, tile, a.col[e], lane);
      }
    }
    if (v < a.n && h == 0) {
      s = kUnd;
      key[v] = philox10((uint32_t)v, g, (uint32_t)r, kTagCluster | ((uint32_t)t << 8), a.k0, a.k1).a;
    }
    state[v] = s;
  }
  __syncthreads();
  while (true) {
    for (int v = threadIdx.x; v < a.n; v += blockDim.x) {
      if (state[v] != kUnd) continue;
      const uint32_t kv = key[v];
      bool root = true;
      for (int e = a.row_ptr[v]; e < a.row_ptr[v + 1]; ++e) {
        const int u = a.col[e];
        const uint8_t su = state[u];
        if ((su == kUnd || su == kCand) && (key[u] < kv || (key[u] == kv && u < v))) {
          root = false;
          break;
        }
      }
      if (root) state[v] = kCand;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < a.n; v += blockDim.x)
      if (state[v] == kCand) state[v] = kIn;
    __syncthreads();
    int und = 0;
    for (int v = threadIdx.x; v < a.n; v += blockDim.x) {
      if (state[v] != kUnd) continue;
      bool out = false;
      for (int e = a.row_ptr[v]; e < a.row_ptr[v + 1]; ++e)
        if (state[a.col[e]] == kIn) { out = true; break; }
      if (out) state[v] = kOut; else und = 1;
    }
    if (!__syncthreads_or(und)) break;
  }
  if (threadIdx.x == 0) cnt_s = 0;
  __syncthreads();
  int mine = 0;
  uint8_t* out = a.cl_sel + (size_t)lb * a.np;
  for (int v = threadIdx.x; v < a.np; v += blockDim.x) {
    const uint8_t in = state[v] == kIn;
    out[v] = in;
    mine += in;
  }
  atomicAdd(&cnt_s, mine);
  __syncthreads();
  if (threadIdx.x == 0) a.cl_sizes[lb] = cnt_s;
}

// Local block = target * kApplyChunks + chunk.
__global__ void __launch_bounds__(256) k_cl_apply(const Desc* __restrict__ D, const uint64_t* __restrict__ map) {
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& a = D[inst];
  RunState* st = a.st;
  if (!st->active || !st->do_cluster) return;
  const int i = lb / kApplyChunks, chunk = lb % kApplyChunks;
  if (i >= min(st->cl_n_top, a.R)) return;
  const int trials = st->cl_trials;
  if (trials <= 0) return;
  const int buf = st->cur ^ st->do_resample;
  uint32_t* S = buf ? a.S1 : a.S0;
  int32_t* H = buf ? a.H1 : a.H0;
  int tb = 0, best = -1;
  for (int t = 0; t < trials; ++t) {
    const int s = a.cl_sizes[i * trials + t];
    if (s > best) { best = s; tb = t; }
  }
  const uint8_t* sel = a.cl_sel + (size_t)(i * trials + tb) * a.np;
  const int r = a.cl_targets[i];
  const int tile = r >> 6, lane = r & 63;
  int mine = 0;
  for (int v = chunk * blockDim.x + threadIdx.x; v < a.n; v += kApplyChunks * blockDim.x) {
    if (!sel[v]) continue;
    int8_t* sb = (int8_t*)&S[((size_t)tile * a.nq + (v >> 2)) * kLanes + lane] + (v & 3);
    const int32_t snew = -(int32_t)*sb;
    *sb = (int8_t)snew;
    if (H)
      for (int e = a.row_ptr[v]; e < a.row_ptr[v + 1]; ++e)
        __hip_atomic_fetch_add(&H[((size_t)tile * a.np + a.col[e]) * kLanes + lane], 2 * a.J[e] * snew,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      for (int hk = 0; hk < a.nhub; ++hk) {  // gathered fields: only the kept hub fields change
        const int32_t hj = a.hubJ[v * kMaxHubs + hk];
        if (hj)
          __hip_atomic_fetch_add(&(buf ? a.HF1 : a.HF0)[hk * a.R + r], 2 * hj * snew, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      }
    ++mine;
  }
  // one counter update per work-group
  __shared__ int32_t part[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mine;
  __syncthreads();
  const int total = part[0] + part[1] + part[2] + part[3];
  if (threadIdx.x == 0 && total)
    __hip_atomic_fetch_add((unsigned long long*)a.cl_flipped, (unsigned long long)total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Max-3-Cut decode (see pamc.h) and the pairwise Hamming diagnostic.
// ---------------------------------------------------------------------------
__global__ void k_m3_decode(const int8_t* spins_internal, const int32_t* to_internal_emb, int32_t n3,
                            int32_t* labels) {
  const int anc = to_internal_emb[3 * n3];
  const int g = spins_internal[anc] < 0 ? -1 : 1;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n3; i += gridDim.x * blockDim.x) {
    int lab = 0;
    for (int aa = 2; aa >= 0; --aa)
      if (g * spins_internal[to_internal_emb[3 * i + aa]] > 0) lab = aa;
    labels[i] = lab;
  }
}

__global__ void k_m3_cut(const int32_t* labels, int32_t n3, const int32_t* row_ptr, const int32_t* col,
                         const int32_t* w, int64_t* cut) {
  int64_t c = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n3; i += gridDim.x * blockDim.x)
    for (int e = row_ptr[i]; e < row_ptr[i + 1]; ++e) {
      const int j = col[e];
      if (j > i && labels[i] != labels[j]) c += w[e];
    }
  c = wave_sum_i64(c);
  if ((threadIdx.x & 63) == 0 && c)
    __hip_atomic_fetch_add((unsigned long long*)cut, (unsigned long long)c, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Distances of all replica pairs.  d(a, b) = (n - s_a . s_b) / 2, so the pairs
// of two 64-replica tiles are a matrix product of the spin bytes, exact in
// int32.  One work-group per pair of tiles ta <= tb; its 16 waves share the
// spins, 32 of them (8 quads) at a time, and meet by additions in LDS.  A lane
// supplies, for replica l % 32 of a 32 x 32 product, the four words of quads 4
// (l / 32) .. + 3: rows of the population as stored, no data moves between
// lanes.  Bound by the caches: each tile is read by every work-group that it
// takes part in.  n = 20,000, R = 1,024 (136 work-groups, 348 MB of reads):
// 63 us, where a thread that compared two replicas word by word took 5.7 ms.
constexpr int kPairThreads = 1024;
typedef int i32x16 __attribute__((ext_vector_type(16)));

// Products s_a . s_b of tile pair p into dot[64][64]; sets ta, tb.
__device__ __forceinline__ void pair_products(const uint32_t* __restrict__ S, int32_t n, int32_t nq, int32_t T, int p,
                                              int& ta, int& tb, int32_t* dot) {
  ta = 0;
  while (p >= T - ta) p -= T - ta++;
  tb = ta + p;
  const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < 64 * 64; i += kPairThreads) dot[i] = 0;
  const uint32_t* at = S + (size_t)ta * nq * kLanes + c;
  const uint32_t* bt = S + (size_t)tb * nq * kLanes + c;
  i32x16 acc[2][2] = {};
  i32x4 x[2][2][2];  // [slot][side][half of the tile's replicas]
  auto load = [&](i32x4(&v)[2][2], int step) {
    const size_t row = (size_t)(8 * step + 4 * g) * kLanes;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[0][h][i] = (int32_t)at[row + i * kLanes + 32 * h];
        v[1][h][i] = (int32_t)bt[row + i * kLanes + 32 * h];
      }
  };
  auto multiply = [&](const i32x4(&v)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(v[0][i], v[1][j], acc[i][j], 0, 0, 0);
  };
  constexpr int kWaves = kPairThreads / 64;
  const int steps = n / 32;  // of whole quads
  int st = wave;
  if (st < steps) load(x[0], st);
  for (; st < steps; st += 2 * kWaves) {
    load(x[1], min(st + kWaves, steps - 1));
    multiply(x[0]);
    load(x[0], min(st + 2 * kWaves, steps - 1));
    if (st + kWaves < steps) multiply(x[1]);
  }
  if (32 * steps < n && wave == steps % kWaves) {  // the last spins; bytes beyond n do not count
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 8 * steps + 4 * g + i, left = n - 4 * q;
        const uint32_t mask = left >= 4 ? 0xFFFFFFFFu : (left > 0 ? (1u << (8 * left)) - 1u : 0u);
        const size_t row = (size_t)min(q, nq - 1) * kLanes + 32 * h;
        x[0][0][h][i] = (int32_t)(at[row] & mask);
        x[0][1][h][i] = (int32_t)(bt[row] & mask);
      }
    multiply(x[0]);
  }
  __syncthreads();
  // (waves without a step add nothing)
  if (wave < steps || (32 * steps < n && wave == steps % kWaves))
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        atomicAdd(&dot[(32 * i + 8 * (e >> 2) + 4 * g + (e & 3)) * 64 + 32 * j + c], acc[i][j][e]);
  __syncthreads();
}

// The thread's pairs a < b of the tile pair: f(min(d, n - d)).
template <typename F>
__device__ __forceinline__ void for_pair_distances(const int32_t* dot, int32_t n, int ta, int tb, F&& f) {
#pragma unroll
  for (int i = threadIdx.x; i < 64 * 64; i += kPairThreads) {
    const int32_t d = (n - dot[i]) / 2;
    if (ta != tb || (i >> 6) < (i & 63)) f(min(d, n - d));
  }
}

// Adds a value of every thread to *sum, by way of LDS: an addition per
// work-group (one per wave, all to one address, took n = 400, R = 16,384 6.5 ms).
__device__ __forceinline__ void add_to_total(int64_t acc, unsigned long long* total, int64_t* sum) {
  acc = wave_sum_i64(acc);
  if ((threadIdx.x & 63) == 0) atomicAdd(total, (unsigned long long)acc);
  __syncthreads();
  if (threadIdx.x == 0 && *total)
    __hip_atomic_fetch_add((unsigned long long*)sum, *total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the distances, and (nbins > 0) their histogram, in LDS first.
__global__ void __launch_bounds__(kPairThreads) k_pair_hist(const uint32_t* S0, const uint32_t* S1, const RunState* st,
                                                            int32_t n, int32_t nq, int32_t T, int32_t nbins,
                                                            int64_t* hist, int64_t* sum) {
  __shared__ int32_t dot[64 * 64];
  __shared__ unsigned long long total;
  extern __shared__ int32_t hl[];
  for (int i = threadIdx.x; i < nbins; i += blockDim.x) hl[i] = 0;
  if (threadIdx.x == 0) total = 0;  // (barriers in the products)
  int ta, tb;
  pair_products(st->cur ? S1 : S0, n, nq, T, blockIdx.x, ta, tb, dot);
  int64_t acc = 0;
  for_pair_distances(dot, n, ta, tb, [&](int32_t dh) {
    acc += dh;
    if (nbins) atomicAdd(&hl[(int)min((int64_t)nbins - 1, (2 * (int64_t)nbins * dh) / n)], 1);
  });
  add_to_total(acc, &total, sum);
  for (int i = threadIdx.x; i < nbins; i += blockDim.x)
    if (hl[i])
      __hip_atomic_fetch_add((unsigned long long*)&hist[i], (unsigned long long)hl[i], __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

__host__ __device__ static inline int32_t pair_tiles(int32_t T) { return T * (T + 1) / 2; }  // tile pairs ta <= tb
// Work-groups of a sample: a tile pair each, in turns where there are more pairs
// than replicas (a batch's map has no more entries than that).
__host__ __device__ static inline int32_t pair_blocks(int32_t T) { return min(pair_tiles(T), T * kLanes); }

// In a run with a diversity trace: local block lb of an instance sums
// min(d, n - d) over its tile pairs of the population just swept, on the
// steps the trace samples.
__global__ void __launch_bounds__(kPairThreads) k_step_dh(const Desc* __restrict__ D,
                                                          const uint64_t* __restrict__ map) {
  __shared__ int32_t dot[64 * 64];
  __shared__ unsigned long long total;
  int inst, lb;
  if (!resolve(map, inst, lb)) return;
  const Desc& d = D[inst];
  RunState* st = d.st;
  if (!st->active || st->dh_every <= 0 || st->step % st->dh_every != 0) return;
  if (threadIdx.x == 0) total = 0;  // (barriers in the products)
  const int pairs = pair_tiles(d.T), blocks = pair_blocks(d.T);
  int64_t acc = 0;
  for (int p = lb; p < pairs; p += blocks) {
    int ta, tb;
    if (p != lb) __syncthreads();  // the products before are read
    pair_products(st->cur ? d.S1 : d.S0, d.n, d.nq, d.T, p, ta, tb, dot);
    for_pair_distances(dot, d.n, ta, tb, [&](int32_t dh) { acc += dh; });
  }
  add_to_total(acc, &total, &st->dh_sum);
}

// The sampled step's mean d_H into the trace (-1 on steps not sampled).
__global__ void k_step_dh_finish(const Desc* __restrict__ D, int32_t ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  const Desc& d = D[i];
  RunState* st = d.st;
  if (!st->active || st->dh_every <= 0) return;
  const int step = st->step;
  if (step < d.tr_cap && d.tr_dh) {
    const double pairs = 0.5 * (double)d.R * (double)(d.R - 1);
    d.tr_dh[step] = (step % st->dh_every == 0 && d.R > 1) ? (double)st->dh_sum / ((double)d.n * pairs) : -1.0;
  }
  st->dh_sum = 0;
}

}  // namespace

// ===========================================================================
// Batches and their launchers
// ===========================================================================
int32_t cluster_max_n() { return kClusterMaxN; }
int32_t sweep_waves() { return kSweepWaves; }
int32_t tile_max_quads() { return kTileMaxQuads; }
int64_t tile_lds_bytes(int32_t nq, int32_t rows) { return (int64_t)nq * kLanes * 4 + kThrLds * 4 + 8 * (int64_t)rows; }
int64_t tile_lds_limit() { return kTileLdsBytes; }
int32_t tmma_max_n() { return kTmmaMaxN; }
// (16-row work-groups take an even number of 64-vertex columns)
int64_t tmma_lds_bytes(int32_t nks, int32_t rows) {
  return rows * (64 * (int64_t)(rows == 16 ? (nks + 1) / 2 * 2 : nks) + 16) + kThrLds * 4;
}

// Kernels whose dynamic LDS may exceed the default limit.
hipError_t prepare_kernel_lds() {
  hipError_t e = hipFuncSetAttribute((const void*)k_cl_mis, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     kClusterMaxN * 5 + 64);
  if (e != hipSuccess) return e;
  for (const void* k : {(const void*)k_sweep_tile<0>, (const void*)k_sweep_tile<1>, (const void*)k_sweep_tile<2>,
                        (const void*)k_sweep_tmma<16>, (const void*)k_sweep_tmma<8>, (const void*)k_sweep_tmma_g<8>})
    if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kTileLdsBytes)) != hipSuccess)
      return e;
  return hipFuncSetAttribute((const void*)k_rs_select, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)sizeof(uint64_t) * kRsMaxR);
}

static int64_t sweep_chunks(const pamc_instance* I) {
  const int qpb = kSweepWaves * I->qpw;
  return (I->max_class_quads + qpb - 1) / qpb;
}

// Work-groups per replica tile of a sweep launch.  Incremental-field sweeps
// keep about `budget` per instance that loop over the class's chunks (a
// launch sized for the largest class then costs a small class little: its
// idle work-groups are few), the others one per chunk (capping those was
// measured too: C2's gathered-field phase took 50.1 us with 4,096
// work-groups and 60.2 with 1,024 against 49.4 uncapped; C4's Potts sweep
// 28.0 us with 2,048 against 28.3).
static int64_t sweep_slots(const pamc_instance* I, int64_t budget) {
  const int64_t chunks = sweep_chunks(I);
  if (I->pull || I->potts_K) return chunks;
  return std::min<int64_t>(chunks, std::max<int64_t>(1, budget / I->T));
}

// The budget: kPushWorkGroups for a lone instance, shared by the batch's
// incremental-field instances down to kPushMinWorkGroups each (C4: 2,048
// work-groups alone 3.21e11 attempts/s against 3.04e11 with 1,024 and
// 3.11e11 with 4,096; 16 instances 5.14e11 with 512 each against 4.83e11
// with 2,048).  PAMC_PUSH_WGS overrides.
static int64_t push_budget(const std::vector<pamc_instance*>& insts) {
  if (const char* e = getenv("PAMC_PUSH_WGS")) return std::max(1, atoi(e));
  int64_t n_push = 0;
  for (const pamc_instance* I : insts)
    if (!I->dense && !I->potts_K && !I->pull && !I->tile) ++n_push;
  return std::max<int64_t>(kPushMinWorkGroups, kPushWorkGroups / std::max<int64_t>(1, n_push));
}

Desc make_desc(const pamc_instance* I) {
  Desc d;
  memset(&d, 0, sizeof d);
  d.row_ptr = I->g.row_ptr;
  d.col = I->g.col;
  d.J = I->g.J;
  d.grow = I->g.grow;
  d.gcol = I->g.gcol;
  d.gJ = I->g.gJ;
  d.class_ptr = I->g.class_ptr;
  d.hubJ = I->g.hubJ;
  d.HF0 = I->pop.HF[0];
  d.HF1 = I->pop.HF[1];
  d.nhub = I->nhub;
  d.hub_v0 = I->hub_v[0];
  d.hub_v1 = I->hub_v[1];
  d.order = I->order;
  d.thr = I->thr;
  d.S0 = I->pop.S[0];
  d.S1 = I->pop.S[1];
  // incremental fields only in push mode (an instance keeping both forms
  // has them allocated in pull mode too, stale there)
  d.H0 = I->pull ? nullptr : I->pop.H[0];
  d.H1 = I->pull ? nullptr : I->pop.H[1];
  d.E0 = I->pop.E[0];
  d.E1 = I->pop.E[1];
  d.F0 = I->pop.fam[0];
  d.F1 = I->pop.fam[1];
  d.best = I->best;
  d.st = I->st;
  d.rs_parent = I->rs_parent;
  d.cl_targets = I->cl_targets;
  d.cl_sel = I->cl_sel;
  d.cl_sizes = I->cl_sizes;
  d.cl_flipped = I->flip_ctr ? I->flip_ctr + 256 : nullptr;
  d.tr_mstar = I->tr_mstar;
  d.tr_beta = I->tr_beta;
  d.tr_lnq = I->tr_lnq;
  d.tr_events = I->tr_events;
  d.tr_time = I->tr_time;
  d.tr_dh = I->tr_dh;
  d.flip_ctr = I->prof ? I->flip_ctr : nullptr;
  d.D0 = I->Sd;
  d.D1 = I->Sd2;
  d.W = I->W;
  d.X = I->X;
  d.n = I->n;
  d.np = I->np;
  d.nq = I->nq;
  d.R = I->R;
  d.T = I->T;
  d.ncls = I->ncls;
  d.rule = I->rule;
  d.pull = I->pull;
  d.dense = I->dense;
  d.ptab = I->ptab;
  d.potts_gamma = I->potts_gamma;
  d.potts_K = I->potts_K;
  d.potts_rule = I->potts_rule;
  d.shuffle = (I->flags & 1u) ? 0 : 1;
  d.tr_cap = I->tr_cap;
  d.qpw = I->qpw;
  d.sweep_stride = (int32_t)sweep_slots(I, kPushWorkGroups);  // batch_build sets the batch's
  d.tile_rows = I->tile_rows;
  d.Jt = I->g.Jt;
  d.nks = I->nks;
  d.order_cap = I->order_cap;
  d.k0 = (uint32_t)I->seed;
  d.k1 = (uint32_t)(I->seed >> 32);
  d.btab = I->btab;
  d.bphases = I->bphases;
  d.bcoup = I->bcoup;
  d.bmaxdeg = I->bmaxdeg;
  d.not_monotone = I->dense ? reinterpret_cast<int32_t*>(I->flip_ctr + kMonotoneSlot) : nullptr;
  return d;
}

static BitDesc make_bit_desc(const pamc_instance* I, const Desc& d, int32_t qpw, int32_t unpack_qpw) {
  BitDesc b;
  memset(&b, 0, sizeof b);
  b.rows = I->g.brows;
  b.base = I->g.brows + 2 * (size_t)I->np;
  b.higher = I->g.brows + 3 * (size_t)I->np;
  b.ent = I->g.bent;
  b.phases = d.bphases;
  b.tab = I->btab;
  b.st = I->st;
  b.S0 = d.S0;
  b.S1 = d.S1;
  b.E0 = d.E0;
  b.E1 = d.E1;
  b.flip_ctr = d.flip_ctr;
  const uint32_t X4 = 4u * (uint32_t)I->bmaxdeg;  // byte offset of x = 0 in a half
  b.tab_half = 2 * I->bmaxdeg + 2;
  if (I->bcoup > 0) {  // x <= 0: the first half's upper part, the second half's lower part
    b.le_first = X4;
    b.le_span = 4u * (uint32_t)b.tab_half;
  } else {  // the halves are exchanged: everything but x > 0
    b.le_first = X4 + 4;
    b.le_span = 4u * (uint32_t)b.tab_half - 8;
    b.le_xor = ~0ull;
  }
  b.n = I->n;
  b.np = I->np;
  b.nq = I->nq;
  b.T = I->T;
  b.ncls = I->ncls;
  b.order_cap = d.order_cap;
  b.copies = I->bcopies;
  b.coupling = I->bcoup;
  b.qpw = qpw;
  b.unpack_qpw = unpack_qpw;
  b.row_stride = I->bstride;
  b.k0 = d.k0;
  b.k1 = d.k1;
  return b;
}

int Batch::group_of(const pamc_instance* I) {
  if (I->potts_K) return 37 + (I->potts_K - 2);
  if (!I->pull) return 0;
  const int ti = I->tpw == 4 ? 2 : (I->tpw == 2 ? 1 : 0);
  const int wide = 2 * I->X + 1 > kThrLds ? 1 : 0;
  return 1 + 18 * (I->nhub ? 1 : 0) + 9 * wide + 3 * I->jmode + ti;
}

static void batch_free(Batch& b, void* p) {
  // pieces of an arena or of the batch's block are not freed by themselves
  if (!p || b.arena || (b.block && (char*)p >= b.block && (char*)p < b.block + b.block_cap)) return;
  if (b.al)
    b.al->free(b.al->ctx, p, (void*)b.stream);
  else
    hipFree(p);
}

void Batch::free_device() {
  auto release = [&](void* p) { batch_free(*this, p); };
  release(d_desc);
  d_desc = nullptr;
  block_used = 0;
  Launch* all[] = {&init_spins, &init_fields, &thr, &thr_dense, &gather, &cl_mis, &cl_apply, &dh};
  for (Launch* l : all) {
    release(l->map);
    l->map = nullptr;
    l->grid = 0;
  }
  for (Launch& l : sweep) {
    release(l.map);
    l.map = nullptr;
    l.grid = 0;
  }
  for (Launch& l : tile) {
    release(l.map);
    l.map = nullptr;
    l.grid = 0;
  }
  for (int64_t& x : tile_lds) x = 0;
  for (int f = 0; f < kBitForms; ++f) {
    for (int r = 0; r < 2; ++r) {
      release(bit_sweep[r][f].map);
      bit_sweep[r][f] = Launch();
      bit_grid[r][f].clear();
    }
    release(bit_pack[f].map);
    release(bit_unpack[f].map);
    bit_pack[f] = bit_unpack[f] = Launch();
  }
  release(d_bits);
  d_bits = nullptr;
  tmma_waves = 16;
  arena_used = 0;
  if (step_graph) hipGraphExecDestroy(step_graph);
  step_graph = nullptr;
  graph_key = -1;
}

hipError_t batch_alloc(Batch& b, void** p, size_t bytes) {
  if (!b.arena && b.al) {
    *p = b.al->alloc(b.al->ctx, bytes, (void*)b.stream);
    return *p ? hipSuccess : hipErrorOutOfMemory;
  }
  if (!b.arena) {
    const size_t at = (b.block_used + 255) & ~(size_t)255;
    if (at > b.block_cap || bytes > b.block_cap - at) return hipMalloc(p, bytes);
    *p = b.block + at;
    b.block_used = at + bytes;
    return hipSuccess;
  }
  const size_t at = (b.arena_used + 255) & ~(size_t)255;
  b.arena_need = at + bytes;
  if (bytes > b.arena_cap || at > b.arena_cap - bytes) return hipErrorOutOfMemory;
  *p = b.arena + at;
  b.arena_used = at + bytes;
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Fixed device scratch for callers that cannot allocate device memory
// (pamc_anneal_batch_noalloc).  Every GPU the library runs on holds its own
// copy of this array until the process ends.  Host code never uses the
// array's name as an address: the device address comes from
// hipGetSymbolAddress, looked up once per device with that device current.
// ---------------------------------------------------------------------------
constexpr size_t kFixedScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kFixedScratchBytes];

hipError_t fixed_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex m;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(m);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = kFixedScratchBytes;
  return hipSuccess;
}


// Appends an instance's local blocks to a map.  With align8 the instance's
// first block is placed at a multiple of 8 (idle blocks fill the gap), so
// that its XCD placement does not depend on the instances before it.
static void add_blocks(std::vector<uint64_t>& map, int inst, int64_t count, bool align8) {
  if (count <= 0) return;
  const uint64_t hi = (uint64_t)(uint32_t)inst << 32;
  if (align8)
    while (map.size() % 8) map.push_back(hi | kIdle);
  for (int64_t b = 0; b < count; ++b) map.push_back(hi | (uint64_t)b);
}

static int64_t field_blocks(const pamc_instance* I) {
  return std::min<int64_t>((int64_t)I->T * ((I->n + 63) / 64), kFieldBlocks);
}

// A step pays for packing the spins and for unpacking them with their
// energies (11 us for small instances, about two sweeps' gain for large ones),
// each sweep of it gains.  Times of 20 steps without and with bit-packed
// sweeps, one instance:
// - against the gathered per-class launches (each phase gains with the length
//   of the rows): G(5000, degree 5), R = 1024, 1, 2, 3, 5 sweeps a step: 1.75 and
//   2.02, 2.35 and 2.42, 2.91 and 2.86, 4.10 and 3.79 ms; G(20000, degree 9), R =
//   1024: 3.53 and 3.97, 5.51 and 5.27, 7.46 and 6.57, 11.3 and 9.2; G(2000, degree
//   30), R = 256, 1 and 5: 3.64 and 2.63, 13.0 and 7.3 ms;
// - against a work-group per tile for the whole step, whose sweep takes about n
//   (0.02 + 0.0023 degree) + classes us where a bit-packed one takes 4.3 us a
//   class: G(300, degree 7), R = 256, 1 and 5: 1.36 and 1.59, 2.49 and 3.04 ms;
//   G(600, degree 7): 1.53 and 1.65, 3.43 and 3.15; G(1200, degree 7): 1.94 and
//   1.55, 5.24 and 2.84 ms.
int32_t bits_min_sweeps(const std::vector<pamc_instance*>& insts) {
  constexpr int32_t kNever = INT32_MAX;
  bool tiles = true;  // every one could sweep in tiles
  double tile_us = 0, degree = 0;
  int64_t all_tiles = 0;
  int32_t ncls = 0, count = 0;
  for (const pamc_instance* I : insts) {
    if (I->dense || !I->bits_ok || I->bits_from) continue;
    const double deg = I->n > 0 ? (double)I->nnz / I->n : 0.0;
    tiles = tiles && I->tile == 1;
    tile_us = std::max(tile_us, I->n * (0.02 + 0.0023 * deg) + I->ncls);
    degree = std::max(degree, deg);
    ncls = std::max(ncls, I->ncls);
    all_tiles += I->T;
    ++count;
  }
  if (!count) return kNever;
  if (tiles) {
    const double gain = tile_us * (double)((all_tiles + kComputeUnits - 1) / kComputeUnits) - 4.3 * ncls;
    return gain > 0.05 ? (int32_t)std::ceil(11.0 / gain) : kNever;
  }
  return degree >= 20.0 ? 1 : (degree >= 8.0 ? 2 : 3);
}

// The form of an instance's bit-packed launches (Batch::kBitForms), quads: quads
// x tiles of a phase over its batch.
//
// Rows of at most four entries: a quad per wave, else a quad per
// work-group.  A scalar load costs a compute unit about 8 cycles whatever its
// width, so wide tile groups pay once there are enough quads to go round.
// Runs timed with groups of 1, 2 and 4 tiles, a quad per wave: torus 60 x 60,
// R = 512 (3,600 quads x tiles a phase): 1.95, 2.13 and 2.35 ms; R = 4096
// (28,800): 4.68, 3.95 and 3.71; 100 x 200, R = 4096 (160,000): 200, 107 and 89.
// A quad per work-group: G(2000, degree 7), R = 256 (500): 2.65, 2.86 and
// 3.16 ms; G(11999, degree 34), R = 512 (2,000): 37.6, 30.6 and 31.7; G(5000,
// degree 5), R = 1024 (4,000): 5.78, 4.25 and 3.79.
static int bit_form(const pamc_instance* I, int64_t quads) {
  int f = I->bstride == 4 ? (quads < 8192 ? 3 : 5) : (quads < 1000 ? 0 : (quads < 2500 ? 1 : 2));
  if (const char* e = getenv("PAMC_BITS_FORM")) f = std::min(5, std::max(0, atoi(e)));
  if (f >= 3 && I->bstride != 4) f -= 3;
  while (f % 3 > 0 && I->T % (f % 3 == 2 ? 4 : 2) != 0) --f;
  return f;
}

void bits_info(const pamc_instance* I, int32_t* sweeps, int32_t* tiles) {
  *sweeps = *tiles = 0;
  if (I->dense || !I->bits_ok) return;
  const int32_t from = I->bits_from ? I->bits_from : bits_min_sweeps({const_cast<pamc_instance*>(I)});
  if (from == INT32_MAX) return;
  const int f = bit_form(I, (int64_t)I->T * I->max_class_quads);
  *sweeps = from;
  *tiles = f >= 3 ? 1 << (f - 3) : -(1 << f);
}

static hipError_t build_batch(Batch& b, const std::vector<pamc_instance*>& insts, const std::vector<Schedule>* scheds,
                              bool allow_bits) {
  // the old maps may still be read by queued kernels
  if (b.stream && b.n > 0) {
    const hipError_t e = hipStreamSynchronize(b.stream);
    if (e != hipSuccess) return e;
  }
  b.free_device();
  b.I = insts;
  b.n = (int32_t)insts.size();
  if (b.n == 0) return hipSuccess;
  b.stream = insts[0]->stream;
  std::vector<Desc> desc(b.n);
  const int64_t push_wgs = push_budget(insts);
  // An instance's own batch is called with any number of sweeps a step, so it
  // holds the launches of both forms; a batch of runs knows its schedules'.
  const bool own = b.n == 1 && !scheds;
  int32_t most_sweeps = 1;
  if (scheds)
    for (const Schedule& s : *scheds) most_sweeps = std::max(most_sweeps, s.sweeps);
  const int32_t least = bits_min_sweeps(insts);
  auto bits_from = [&](int i) { return insts[i]->bits_from ? insts[i]->bits_from : least; };
  b.bits_from = own ? bits_from(0) : 1;
  auto sweeps_bits = [&](int i) {
    const pamc_instance* I = insts[i];
    return allow_bits && !I->dense && I->bits_ok && (own ? bits_from(i) != INT32_MAX : most_sweeps >= bits_from(i));
  };
  auto sweeps_other = [&](int i) { return !sweeps_bits(i) || b.bits_from > 1; };
  bool any_bits = false;
  for (int i = 0; i < b.n; ++i) {
    desc[i] = make_desc(insts[i]);
    desc[i].sweep_stride = (int32_t)sweep_slots(insts[i], push_wgs);
    desc[i].bits = sweeps_bits(i);
    any_bits = any_bits || desc[i].bits;
  }
  b.has_bits = any_bits;
  // arena mode: per-run scratch sized for each instance's schedule
  std::vector<int32_t> cl_top(b.n), cl_trials(b.n);
  for (int i = 0; i < b.n; ++i) {
    cl_top[i] = std::min(insts[i]->cl_cap_top, insts[i]->R);
    cl_trials[i] = insts[i]->cl_cap_trials;
  }
  if (b.arena) {
    if (!scheds) return hipErrorInvalidValue;
    for (int i = 0; i < b.n; ++i) {
      const pamc_instance* I = insts[i];
      const Schedule& s = (*scheds)[i];
      Desc& d = desc[i];
      d.flip_ctr = nullptr;
      d.tr_cap = 0;
      d.order_cap = std::max(s.sweeps, 1);
      hipError_t e = batch_alloc(b, (void**)&d.order, sizeof(int32_t) * (size_t)d.order_cap * std::max(I->ncls, 1));
      if (e == hipSuccess && d.bits && d.order_cap > I->order_cap)  // else the instance's own
        e = batch_alloc(b, (void**)&d.bphases, 4 * sizeof(int32_t) * (size_t)d.order_cap * std::max(I->ncls, 1));
      if (e != hipSuccess) return e;
      const bool cl = s.augmented && s.resample && s.n_top > 0 && s.mis_trials > 0 && !I->potts_K && !I->dense;
      cl_top[i] = cl ? std::min(s.n_top, I->R) : 0;
      cl_trials[i] = cl ? s.mis_trials : 0;
      d.cl_targets = nullptr;
      d.cl_sel = nullptr;
      d.cl_sizes = nullptr;
      if (cl) {
        if ((e = batch_alloc(b, (void**)&d.cl_targets, sizeof(int32_t) * cl_top[i])) != hipSuccess) return e;
        if ((e = batch_alloc(b, (void**)&d.cl_sizes, sizeof(int32_t) * (size_t)cl_top[i] * cl_trials[i])) != hipSuccess)
          return e;
        if ((e = batch_alloc(b, (void**)&d.cl_sel, (size_t)cl_top[i] * cl_trials[i] * I->np)) != hipSuccess) return e;
      }
    }
  }
  std::vector<uint64_t> m_init, m_fields, m_thr, m_gather, m_mis, m_apply, m_dh;
  std::vector<std::vector<uint64_t>> m_sweep(Batch::kGroups), m_tile(4);
  b.max_ncls = 0;
  for (int g = 0; g < Batch::kGroups; ++g) b.group_ncls[g] = 0;
  b.max_sweeps = 1;
  b.any_cluster = 0;
  b.max_lds = 0;
  b.max_R = 0;
  // Matrix-core tiles: while the batch has at most 128 of them, one
  // work-group per 16-replica group spreads them over four times the
  // compute units (a single instance's step is 1.4x faster); beyond, one
  // work-group per tile shares each coupling block between its four groups
  // in the unit's L1 (1.7x the throughput of group work-groups with 1,024
  // tiles).  PAMC_TMMA_GROUPS = 0 or 1 forces one.
  {
    int64_t mt = 0;
    for (int i = 0; i < b.n; ++i)
      if (!insts[i]->dense && insts[i]->tile == 2 && sweeps_other(i)) mt += insts[i]->T;
    b.tmma_groups = mt <= kMfmaGroupTiles;
    if (const char* g = getenv("PAMC_TMMA_GROUPS")) b.tmma_groups = atoi(g) != 0;
  }
  std::vector<int> bit_insts;
  for (int i = 0; i < b.n; ++i) {
    pamc_instance* I = insts[i];
    b.max_R = std::max(b.max_R, I->R);
    if (I->dense) continue;
    add_blocks(m_init, i, kInitBlocks, false);
    add_blocks(m_fields, i, field_blocks(I), false);
    add_blocks(m_thr, i, kThrBlocks, false);
    add_blocks(m_gather, i, (int64_t)I->T * ((I->nq + kGatherQuadsPerBlock - 1) / kGatherQuadsPerBlock), true);
    if (sweeps_bits(i)) bit_insts.push_back(i);
    if (!sweeps_other(i)) {
      // bit-packed only
    } else if (I->tile == 2) {  // the same with matrix-core fields
      add_blocks(m_tile[3], i, (int64_t)I->T * (b.tmma_groups ? 4 : 1), false);
      b.tile_lds[3] = std::max<int64_t>(b.tile_lds[3], tmma_lds_bytes(I->nks, b.tmma_groups ? 16 : 64));
    } else if (I->tile) {  // one work-group per replica tile walks the whole step
      add_blocks(m_tile[I->jmode], i, I->T, false);
      b.tile_lds[I->jmode] = std::max<int64_t>(b.tile_lds[I->jmode], tile_lds_bytes(I->nq, I->tile_rows));
    } else {
      const int grp = Batch::group_of(I);
      add_blocks(m_sweep[grp], i, (int64_t)(I->T / (I->pull ? I->tpw : 1)) * sweep_slots(I, push_wgs), true);
      b.max_ncls = std::max(b.max_ncls, I->ncls);
      b.group_ncls[grp] = std::max(b.group_ncls[grp], I->ncls);
    }
    const int nt = cl_top[i];
    if (nt > 0 && cl_trials[i] > 0) {
      add_blocks(m_mis, i, (int64_t)nt * cl_trials[i], false);
      add_blocks(m_apply, i, (int64_t)nt * kApplyChunks, false);
      b.max_lds = std::max<int64_t>(b.max_lds, (int64_t)I->np * 5);
    }
  }
  // bit-packed sweeps
  std::vector<std::vector<uint64_t>> m_bits(2 * Batch::kBitForms), m_bpack(Batch::kBitForms),
      m_bunpack(Batch::kBitForms);
  std::vector<BitDesc> bdesc;
  if (!bit_insts.empty()) {
    bdesc.resize(b.n);
    std::stable_sort(bit_insts.begin(), bit_insts.end(),
                     [&](int x, int y) { return insts[x]->ncls > insts[y]->ncls; });
    int64_t quads = 0;  // quads x tiles of a phase, over the batch
    for (int i : bit_insts) quads += (int64_t)insts[i]->T * insts[i]->max_class_quads;
    // Quads per wave or work-group, 1 and 2: G(5000, degree 5), R = 1024 (4,000
    // quads x tiles a phase) 3.79 and 4.04 ms; G(20000, degree 5), R = 1024 (16,000)
    // 8.15 and 7.77; torus 100 x 200, R = 4096 (160,000) 90.6 and 89.2 (3: 88.5, 4:
    // 91.1).
    int qpw = 0, uq = 0;
    if (const char* e = getenv("PAMC_BITS_QPW")) qpw = std::max(1, atoi(e));
    if (const char* e = getenv("PAMC_BITS_UQ")) uq = std::max(1, atoi(e));
    for (int i : bit_insts) {
      const pamc_instance* I = insts[i];
      const int f = bit_form(I, quads);
      int qw = qpw, u = uq;
      if (!qw) qw = quads >= (I->bstride == 4 ? 65536 : 12000) ? 2 : 1;
      if (!u) u = I->nq >= 4096 ? 8 : 4;  // G(20000, degree 9), R = 64: 2.24 and 2.03 ms; n = 5,000: 2.05 and 2.11
      const int G = 1 << (f % 3);
      std::vector<uint64_t>& m = m_bits[I->rule * Batch::kBitForms + f];
      std::vector<int32_t>& grid = b.bit_grid[I->rule][f];
      add_blocks(m, i, (int64_t)(I->T / G) * bits_work_groups(I->max_class_quads, qw, f < 3), true);
      if ((int)grid.size() < I->ncls) grid.resize(I->ncls);
      for (int p = 0; p < I->ncls; ++p) grid[p] = (int32_t)m.size();
      add_blocks(m_bpack[f], i, (int64_t)(I->T / G) * bits_pack_chunks(I->nq), true);
      add_blocks(m_bunpack[f], i, (int64_t)(I->T / G) * bits_work_groups(I->nq, u, f < 3), true);
      bdesc[i] = make_bit_desc(I, desc[i], qw, u);
    }
  }
  // diversity samples: pair_blocks work-groups.  A batch without
  // schedules (an instance's own) keeps the map; its runs switch it on.
  b.any_dh = 0;
  for (int i = 0; i < b.n; ++i) {
    if (scheds) {
      const Schedule& s = (*scheds)[i];
      b.max_sweeps = std::max(b.max_sweeps, s.sweeps);
      if (s.augmented && s.resample && s.n_top > 0 && s.mis_trials > 0) b.any_cluster = 1;
      if (s.dh_every <= 0) continue;
    }
    if (insts[i]->dense || insts[i]->potts_K) continue;
    add_blocks(m_dh, i, pair_blocks(insts[i]->T), false);
    if (scheds) b.any_dh = 1;
  }
  if (!b.arena && !b.al) {
    // One block for the descriptors and the dozen maps, of their size: an
    // allocation and a release cost 20 us, at each rebuild of a small instance
    // 0.25 ms in all.  (Without room for it they are allocated one by one.)
    size_t need = sizeof(Desc) * b.n;
    auto take = [&](size_t bytes) { need = ((need + 255) & ~(size_t)255) + bytes; };
    for (const auto* m : {&m_init, &m_fields, &m_thr, &m_gather, &m_mis, &m_apply, &m_dh}) take(8 * m->size());
    for (const auto& m : m_sweep) take(8 * m.size());
    for (const auto& m : m_tile) take(8 * m.size());
    if (b.n > 1) {  // a lone instance's bit-packed launches need none
      for (const auto* v : {&m_bits, &m_bpack, &m_bunpack})
        for (const auto& m : *v) take(8 * m.size());
      take(sizeof(BitDesc) * bdesc.size());
    }
    if (need > b.block_cap) {
      if (b.block) hipFree(b.block);
      b.block = nullptr;
      const size_t unit = b.n > 1 ? 65536 : 4096;
      b.block_cap = (need + unit - 1) / unit * unit;
      if (hipMalloc((void**)&b.block, b.block_cap) != hipSuccess) {
        (void)hipGetLastError();
        b.block = nullptr;
        b.block_cap = 0;
      }
    }
  }
  hipError_t e = batch_alloc(b, (void**)&b.d_desc, sizeof(Desc) * b.n);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(b.d_desc, desc.data(), sizeof(Desc) * b.n, hipMemcpyHostToDevice, b.stream);
  if (e != hipSuccess) return e;
  auto up = [&](std::vector<uint64_t>& m, Batch::Launch& l) -> hipError_t {
    if (m.size() > (size_t)INT32_MAX) return hipErrorInvalidValue;
    l.grid = (int32_t)m.size();
    if (m.empty()) return hipSuccess;
    hipError_t err = batch_alloc(b, (void**)&l.map, sizeof(uint64_t) * m.size());
    if (err != hipSuccess) return err;
    return hipMemcpyAsync(l.map, m.data(), sizeof(uint64_t) * m.size(), hipMemcpyHostToDevice, b.stream);
  };
  if ((e = up(m_init, b.init_spins)) != hipSuccess) return e;
  if ((e = up(m_fields, b.init_fields)) != hipSuccess) return e;
  if ((e = up(m_thr, b.thr)) != hipSuccess) return e;
  if ((e = up(m_gather, b.gather)) != hipSuccess) return e;
  if ((e = up(m_mis, b.cl_mis)) != hipSuccess) return e;
  if ((e = up(m_apply, b.cl_apply)) != hipSuccess) return e;
  if ((e = up(m_dh, b.dh)) != hipSuccess) return e;
  // (a lone instance's launches need no maps)
  auto up_bits = [&](std::vector<uint64_t>& m, Batch::Launch& l) -> hipError_t {
    if (b.n > 1) return up(m, l);
    l.grid = (int32_t)m.size();
    return hipSuccess;
  };
  for (int f = 0; f < Batch::kBitForms; ++f) {
    for (int r = 0; r < 2; ++r)
      if ((e = up_bits(m_bits[r * Batch::kBitForms + f], b.bit_sweep[r][f])) != hipSuccess) return e;
    if ((e = up_bits(m_bpack[f], b.bit_pack[f])) != hipSuccess) return e;
    if ((e = up_bits(m_bunpack[f], b.bit_unpack[f])) != hipSuccess) return e;
  }
  if (!bdesc.empty()) b.lone_bits = bdesc[0];
  if (!bdesc.empty() && b.n > 1) {
    if ((e = batch_alloc(b, (void**)&b.d_bits, sizeof(BitDesc) * b.n)) != hipSuccess) return e;
    e = hipMemcpyAsync(b.d_bits, bdesc.data(), sizeof(BitDesc) * b.n, hipMemcpyHostToDevice, b.stream);
    if (e != hipSuccess) return e;
  }
  for (int g = 0; g < Batch::kGroups; ++g)
    if ((e = up(m_sweep[g], b.sweep[g])) != hipSuccess) return e;
  for (int g = 0; g < 4; ++g)
    if ((e = up(m_tile[g], b.tile[g])) != hipSuccess) return e;
  // matrix-core tiles: 8-wave work-groups, two per compute unit, once the
  // launch has at least two per unit and two fit the unit's LDS
  // (PAMC_TMMA_WAVES = 8 or 16 forces a size)
  b.tmma_waves = ((int64_t)m_tile[3].size() >= 2 * kComputeUnits &&
                  2 * (b.tile_lds[3] + (int64_t)sizeof(int64_t) * 8 * kLanes + 64) <= kCuLdsBytes)
                     ? 8
                     : 16;
  if (const char* w = getenv("PAMC_TMMA_WAVES")) b.tmma_waves = atoi(w) == 8 ? 8 : 16;
  // the staging vectors are local: wait for the copies before they go
  return hipStreamSynchronize(b.stream);
}

hipError_t batch_build(Batch& b, const std::vector<pamc_instance*>& insts, const std::vector<Schedule>* scheds,
                       size_t later) {
  const hipError_t e = build_batch(b, insts, scheds, true);
  if (!b.arena || !b.has_bits) return e;
  const bool fits = e == hipSuccess && ((b.arena_used + 255) & ~(size_t)255) + later <= b.arena_cap;
  if (fits || (e != hipSuccess && e != hipErrorOutOfMemory)) return e;
  // the fixed scratch holds the batch without the bit-packed launches' maps:
  // the other sweep kernels give the same results
  b.arena_used = 0;
  return build_batch(b, insts, scheds, false);
}

using SweepKernel = void (*)(const Desc*, const uint64_t*, int, int);
using SweepTileKernel = void (*)(const Desc*, const uint64_t*);

template <bool WIDE, bool HUB>
static SweepKernel pull_kernel(int jm, int ti) {
  static const SweepKernel k[3][3] = {
      {k_sweep_pull<0, 1, WIDE, HUB>, k_sweep_pull<0, 2, WIDE, HUB>, k_sweep_pull<0, 4, WIDE, HUB>},
      {k_sweep_pull<1, 1, WIDE, HUB>, k_sweep_pull<1, 2, WIDE, HUB>, k_sweep_pull<1, 4, WIDE, HUB>},
      {k_sweep_pull<2, 1, WIDE, HUB>, k_sweep_pull<2, 2, WIDE, HUB>, k_sweep_pull<2, 4, WIDE, HUB>}};
  return k[jm][ti];
}

static SweepKernel sweep_kernel_of_group(int g) {
  // group = 0 (incremental fields), 1 + 18 * hubs + 9 * wide table + 3 * coupling mode +
  // tiles-per-wave index (gathered fields), 37 + K - 2 (Potts labels)
  if (g == 0) return k_sweep_push;
  if (g >= 37) return g == 37 ? k_sweep_potts<2> : (g == 38 ? k_sweep_potts<3> : k_sweep_potts<4>);
  int x = g - 1;
  const bool hub = x >= 18;
  x %= 18;
  const bool wide = x >= 9;
  x %= 9;
  if (hub) return wide ? pull_kernel<true, true>(x / 3, x % 3) : pull_kernel<false, true>(x / 3, x % 3);
  return wide ? pull_kernel<true, false>(x / 3, x % 3) : pull_kernel<false, false>(x / 3, x % 3);
}

static hipEvent_t next_event(pamc_instance* I) {
  if (I->ev_used == I->ev_pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    I->ev_pool.push_back(e);
  }
  return I->ev_pool[I->ev_used++];
}

static inline int tgrid(int n) { return (n + 63) / 64; }

// thresholds + class orders (and, with commit >= 0, the step's commit), then
// nsweeps x max_ncls phase launches.  When
// profiling, one event pair brackets the step's back-to-back sweep launches
// (nothing else runs between them), so the mean launch time includes the
// launch boundaries and the events cost two markers per step, not two per
// launch.
static hipError_t batch_sweeps(Batch& b, int32_t nsweeps, int32_t commit = -1) {
  pamc_instance* P = b.I[0];
  const bool prof = P->prof && !b.arena;
  const bool bits = b.has_bits && nsweeps >= b.bits_from;
  const bool other = !bits || b.bits_from <= 1;  // also: the other instances' of a batch
  if (b.thr.grid)
    k_thresholds<<<b.thr.grid, 256, 0, b.stream>>>(b.d_desc, b.thr.map, commit, bits ? nsweeps : 0);
  int64_t launches = 0;
  if (prof) hipEventRecord(next_event(P), b.stream);
  static const SweepTileKernel tile_kernels[3] = {k_sweep_tile<0>, k_sweep_tile<1>, k_sweep_tile<2>};
  for (int g = 0; g < 3; ++g)
    if (other && b.tile[g].grid) {  // every sweep of the step, in one launch
      tile_kernels[g]<<<b.tile[g].grid, kTileWaves * 64, b.tile_lds[g], b.stream>>>(b.d_desc, b.tile[g].map);
      ++launches;
    }
  if (other && b.tile[3].grid) {
    if (b.tmma_groups)
      k_sweep_tmma_g<8><<<b.tile[3].grid, 8 * 64, b.tile_lds[3], b.stream>>>(b.d_desc, b.tile[3].map);
    else if (b.tmma_waves == 8)
      k_sweep_tmma<8><<<b.tile[3].grid, 8 * 64, b.tile_lds[3], b.stream>>>(b.d_desc, b.tile[3].map);
    else
      k_sweep_tmma<16><<<b.tile[3].grid, 16 * 64, b.tile_lds[3], b.stream>>>(b.d_desc, b.tile[3].map);
    ++launches;
  }
  int max_ncls = other ? b.max_ncls : 0;
  BitLaunch bl;
  bl.D = b.d_bits;
  if (b.n == 1) bl.lone = b.lone_bits;
  auto bits_map = [&](const Batch::Launch& l) -> const BitLaunch& {
    bl.map = b.n == 1 ? nullptr : l.map;
    return bl;
  };
  for (int f = 0; f < Batch::kBitForms; ++f)
    if (bits && b.bit_pack[f].grid) {
      launch_bits_pack(f, bits_map(b.bit_pack[f]), b.bit_pack[f].grid, true, b.stream);
      for (int r = 0; r < 2; ++r) max_ncls = std::max(max_ncls, (int)b.bit_grid[r][f].size());
    }
  for (int s = 0; s < nsweeps; ++s) {
    for (int p = 0; p < max_ncls; ++p) {
      for (int r = 0; r < 2; ++r)
        for (int f = 0; f < Batch::kBitForms; ++f) {
          if (!bits || p >= (int)b.bit_grid[r][f].size()) continue;
          launch_bits_sweep(r, f, bits_map(b.bit_sweep[r][f]), b.bit_grid[r][f][p], s, p, b.stream);
          ++launches;
        }
      for (int g = 0; g < Batch::kGroups; ++g) {
        if (!other || !b.sweep[g].grid || p >= b.group_ncls[g]) continue;  // no instance of the group has class p
        sweep_kernel_of_group(g)<<<b.sweep[g].grid, 256, 0, b.stream>>>(b.d_desc, b.sweep[g].map, s, p);
        ++launches;
      }
    }
  }
  for (int f = 0; f < Batch::kBitForms; ++f)
    if (bits && b.bit_unpack[f].grid) launch_bits_pack(f, bits_map(b.bit_unpack[f]), b.bit_unpack[f].grid, false, b.stream);
  if (prof) {
    hipEventRecord(next_event(P), b.stream);
    P->prof_launches += launches;
    for (pamc_instance* I : b.I) P->prof_attempts += (int64_t)nsweeps * I->n * I->R;
  }
  return hipGetLastError();
}

hipError_t batch_init(Batch& b) {
  if (b.init_spins.grid) k_init_spins<<<b.init_spins.grid, 256, 0, b.stream>>>(b.d_desc, b.init_spins.map);
  for (pamc_instance* I : b.I) hipMemsetAsync(I->pop.E[0], 0, sizeof(int64_t) * I->R, b.stream);
  if (b.init_fields.grid)
    k_init_fields<<<b.init_fields.grid, 256, 0, b.stream>>>(b.d_desc, b.init_fields.map, 0, nullptr, 1);
  k_init_finish<<<b.n, 256, 0, b.stream>>>(b.d_desc);
  return hipGetLastError();
}

hipError_t batch_anneal_setup(Batch& b, const Schedule* d_sched, const int32_t* d_idx, int32_t count) {
  if (count <= 0) return hipSuccess;
  k_anneal_setup<<<tgrid(count), 64, 0, b.stream>>>(b.d_desc, d_sched, d_idx, count);
  return hipGetLastError();
}

// fused: the run step's decisions before, the cluster targets after the draw
static hipError_t batch_resample(Batch& b, int32_t fused) {
  k_rs_select<<<b.n, 1024, sizeof(uint64_t) * b.max_R, b.stream>>>(b.d_desc, fused);
  if (b.gather.grid) k_rs_gather<<<b.gather.grid, 256, 0, b.stream>>>(b.d_desc, b.gather.map);
  return hipGetLastError();
}

// select: false when the targets were chosen with the resampling draw
static hipError_t batch_cluster(Batch& b, bool select) {
  if (select) k_cl_select<<<b.n, 1024, 0, b.stream>>>(b.d_desc);
  if (b.cl_mis.grid) k_cl_mis<<<b.cl_mis.grid, 1024, b.max_lds, b.stream>>>(b.d_desc, b.cl_mis.map);
  if (b.cl_apply.grid) k_cl_apply<<<b.cl_apply.grid, 256, 0, b.stream>>>(b.d_desc, b.cl_apply.map);
  return hipGetLastError();
}

hipError_t batch_step(Batch& b) {
  // step decisions + resampling draw (+ cluster targets), gather, cluster
  // move, thresholds + commit, sweeps, step end
  batch_resample(b, 1);
  if (b.any_cluster) batch_cluster(b, false);
  hipError_t e = batch_sweeps(b, b.max_sweeps, 1);
  if (e != hipSuccess) return e;
  if (b.any_dh && b.dh.grid) {  // diversity of the swept population, on sampled steps
    k_step_dh<<<b.dh.grid, kPairThreads, 0, b.stream>>>(b.d_desc, b.dh.map);
    k_step_dh_finish<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  }
  k_step_end<<<b.n, 1024, 0, b.stream>>>(b.d_desc, 1);
  return hipGetLastError();
}

// k beta steps.  Without profiling, one step is captured once as a HIP graph
// (kernels only: the launch sequence of a step is fixed and every decision
// is read from device state) and replayed; if the stream cannot be captured
// the steps are launched one by one.  PAMC_NO_GRAPH=1 forces the latter.
hipError_t batch_run_steps(Batch& b, int32_t k) {
  const char* ng = getenv("PAMC_NO_GRAPH");
  const bool no_graph = ng && atoi(ng) != 0;
  const int64_t key = ((int64_t)b.max_sweeps << 2) | (b.any_dh ? 2 : 0) | (b.any_cluster ? 1 : 0);
  bool use_graph = !no_graph && !b.arena && !b.I[0]->prof && !b.graph_failed && k > 1;
  if (use_graph && (!b.step_graph || b.graph_key != key)) {
    if (b.step_graph) hipGraphExecDestroy(b.step_graph);
    b.step_graph = nullptr;
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamBeginCapture(b.stream, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      const hipError_t es = batch_step(b);
      e = hipStreamEndCapture(b.stream, &g);
      if (es != hipSuccess) e = es;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&b.step_graph, g, nullptr, nullptr, 0);
    if (g) hipGraphDestroy(g);
    if (e != hipSuccess) {
      (void)hipGetLastError();  // clear the capture error; launch eagerly from now on
      b.step_graph = nullptr;
      b.graph_failed = true;
      use_graph = false;
    } else {
      b.graph_key = key;
    }
  }
  for (int32_t i = 0; i < k; ++i) {
    const hipError_t e = use_graph ? hipGraphLaunch(b.step_graph, b.stream) : batch_step(b);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t batch_status(Batch& b, int32_t* d_out) {
  k_status<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, d_out);
  return hipGetLastError();
}

hipError_t prim_sweep(Batch& b, double beta, int32_t nsweeps) {
  pamc_instance* I = b.I[0];
  int done = 0;
  while (done < nsweeps) {
    const int chunk = std::min(nsweeps - done, I->order_cap);
    k_prim_set<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 0, beta, 0, 0, chunk);
    hipError_t e = batch_sweeps(b, chunk);
    if (e != hipSuccess) return e;
    k_advance_sweeps<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, chunk);
    done += chunk;
  }
  return hipGetLastError();
}

hipError_t prim_resample(Batch& b, double delta) {
  k_prim_set<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 1, delta, 0, 0, 0);
  batch_resample(b, 0);
  k_commit<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 0);
  k_deactivate<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  return hipGetLastError();
}

hipError_t prim_cluster(Batch& b, int32_t n_top, int32_t trials) {
  k_prim_set<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 2, 0.0, n_top, trials, 0);
  batch_cluster(b, true);
  k_commit<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 0);
  k_deactivate<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  return hipGetLastError();
}

hipError_t prim_update_best(Batch& b) {
  k_prim_set<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, 0, 0.0, 0, 0, 0);
  k_step_end<<<b.n, 1024, 0, b.stream>>>(b.d_desc, 0);
  k_deactivate<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  return hipGetLastError();
}

hipError_t launch_fields(Batch& b, int32_t buf, int32_t* H) {
  k_init_fields<<<b.init_fields.grid, 256, 0, b.stream>>>(b.d_desc, b.init_fields.map, buf, H, 0);
  return hipGetLastError();
}

hipError_t launch_load_population(Batch& b) {
  for (pamc_instance* I : b.I) hipMemsetAsync(I->pop.E[0], 0, sizeof(int64_t) * I->R, b.stream);
  if (b.init_fields.grid)
    k_init_fields<<<b.init_fields.grid, 256, 0, b.stream>>>(b.d_desc, b.init_fields.map, 0, nullptr, 1);
  k_load_finish<<<b.n, 256, 0, b.stream>>>(b.d_desc);
  return hipGetLastError();
}

hipError_t launch_m3_decode(pamc_instance* I, const int8_t* spins_internal_dev) {
  hipMemsetAsync(I->m3_cut, 0, sizeof(int64_t), I->stream);
  const int grid = (I->m3_n + 255) / 256;
  k_m3_decode<<<grid, 256, 0, I->stream>>>(spins_internal_dev, I->to_internal_dev, I->m3_n, I->m3_labels);
  k_m3_cut<<<grid, 256, 0, I->stream>>>(I->m3_labels, I->m3_n, I->m3_row_ptr, I->m3_col, I->m3_w,
                                        I->m3_cut);
  return hipGetLastError();
}

// The fields the instance's current form keeps, recomputed from the current
// population (no energy change): the incremental fields in push mode, the
// kept hub fields.
hipError_t launch_refresh_fields(Batch& b) {
  if (b.init_fields.grid)
    k_init_fields<<<b.init_fields.grid, 256, 0, b.stream>>>(b.d_desc, b.init_fields.map, -1, nullptr, 0);
  return hipGetLastError();
}

hipError_t launch_pair_hist(pamc_instance* I, int32_t nbins, int64_t* out_dev) {
  hipMemsetAsync(out_dev, 0, sizeof(int64_t) * (nbins + 1), I->stream);
  k_pair_hist<<<pair_tiles(I->T), kPairThreads, sizeof(int32_t) * nbins, I->stream>>>(
      I->pop.S[0], I->pop.S[1], I->st, I->n, I->nq, I->T, nbins, out_dev, out_dev + nbins);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Controller pieces used by the dense path (single instance via its batch).
// ---------------------------------------------------------------------------
hipError_t ctl_step_begin(Batch& b) {
  k_step_begin<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  return hipGetLastError();
}
hipError_t ctl_resample_select(Batch& b) {
  k_rs_select<<<b.n, 1024, sizeof(uint64_t) * b.max_R, b.stream>>>(b.d_desc, 0);
  return hipGetLastError();
}
hipError_t ctl_commit(Batch& b, int32_t in_run) {
  k_commit<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, in_run);
  return hipGetLastError();
}
hipError_t ctl_thresholds(Batch& b) {
  // dense instances have no classes: only the table is computed
  if (!b.thr_dense.grid) {
    std::vector<uint64_t> m;
    for (int i = 0; i < b.n; ++i) add_blocks(m, i, kThrBlocks, false);
    b.thr_dense.grid = (int32_t)m.size();
    hipError_t e = batch_alloc(b, (void**)&b.thr_dense.map, sizeof(uint64_t) * m.size());
    if (e != hipSuccess) return e;
    e = hipMemcpy(b.thr_dense.map, m.data(), sizeof(uint64_t) * m.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
  }
  k_thresholds<<<b.thr_dense.grid, 256, 0, b.stream>>>(b.d_desc, b.thr_dense.map, -1, 0);
  return hipGetLastError();
}
hipError_t ctl_step_end(Batch& b, int32_t in_run) {
  k_step_end<<<b.n, 1024, 0, b.stream>>>(b.d_desc, in_run);
  return hipGetLastError();
}
hipError_t ctl_prim_set(Batch& b, int32_t kind, double value, int32_t nsweeps) {
  k_prim_set<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, kind, value, 0, 0, nsweeps);
  return hipGetLastError();
}
hipError_t ctl_advance(Batch& b, int32_t nsweeps) {
  k_advance_sweeps<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n, nsweeps);
  return hipGetLastError();
}
hipError_t ctl_deactivate(Batch& b) {
  k_deactivate<<<tgrid(b.n), 64, 0, b.stream>>>(b.d_desc, b.n);
  return hipGetLastError();
}
hipEvent_t ctl_event(pamc_instance* I) { return next_event(I); }

}  // namespace pamc
