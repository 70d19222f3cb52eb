// dense.hip -- fully connected instances (Sec. "Scalability on a Large-Scale
// Ising Problem"): int8 couplings J[n][n] in HBM, spins visited in the fixed
// order 0..n-1.
//
// J is stored as matrix-core A fragments of 16 rows x 64 columns, 1 KB each
// (lane l's 16 bytes: row l % 16, columns 16 (l / 16) .. + 15), a row block's
// fragments one after another: the field product reads it as contiguous
// streams straight into registers.
//
// A sweep runs over super-blocks of kSB = 1024 consecutive spins.  For each,
// one matrix-core launch computes the local fields of Eq. 3 of all its rows
// against the spins as they stand, G = J[sb, :] . S (int8 x int8 -> int32,
// exact since |h| <= 127 n < 2^31; split over the K dimension and summed
// atomically).  A sequential pass (one work-group per 16 replicas) then
// walks the super-block in blocks of kDB = 64 spins: the couplings to spins
// already flipped in earlier blocks of the super-block are added with small
// matrix-core products over the recorded changes dS, and the block's spins
// are decided in order with h_k = G_k + C_k + sum_{k' < k in block} J_kk' d_k'
// (d = 2 s_new for flipped spins), by the same threshold test as the sparse
// path in the form x < c (each visit's critical field c, computed for the
// whole sweep beforehand).  The pass and the next super-block's product share
// one launch.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/pamc.h"
#include "instance.hpp"
#include "pamc_device.hpp"

namespace pamc {

namespace {

constexpr int kDB = 64;          // spins per sequential block
constexpr int kSB = 1024;        // rows per super-block: one field product, one sequential launch
constexpr int kDenseThreads = 512;             // threads of the field-product and step work-groups
constexpr int kGM = 128;                       // rows of a field-product tile
constexpr int kStage = 128;                    // its columns per stage: two matrix-core steps of 64
constexpr int kLdsRow = kStage + 16;           // bytes per staged row (padded)
constexpr int kCritThreads = 1024;             // threads of a critical-field work-group
constexpr int kCritLds = 32768;                // its threshold entries in LDS
constexpr int32_t kCritInf = 1 << 30;  // critical field of a visit that flips (or not) at every x
typedef int v4i __attribute__((ext_vector_type(4)));

// Byte offset of J[row][col] in the fragment layout.
__host__ __device__ __forceinline__ size_t frag_at(int32_t np, int32_t row, int32_t col) {
  return (((size_t)(row >> 4) * (np >> 6) + (col >> 6)) * 64 + (row & 15) + 16 * ((col & 63) >> 4)) * 16 + (col & 15);
}

// J_ij = J_ji = +-1 from the low bit of Philox(key = seed; (i, j, 0, DENSE))
// word 0 for i < j; zero diagonal and zero padding.  Also accumulates
// W = sum_{i<j} (-J_ij).  A thread makes a lane's 16 bytes of a fragment.
__global__ void __launch_bounds__(256) k_dense_generate(v4i* J, int32_t n, int32_t np, uint32_t k0, uint32_t k1,
                                                        int64_t* W) {
  const int64_t total = (int64_t)np * np / 16;
  const int nst = np >> 6;
  int64_t wsum = 0;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int lane = (int)(idx & 63);
    const int64_t f = idx >> 6;
    const int i = 16 * (int)(f / nst) + (lane & 15), j0 = 64 * (int)(f % nst) + 16 * (lane >> 4);
    v4i out;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      uint32_t word = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int j = j0 + 4 * w + b;
        int32_t v = 0;
        if (i < n && j < n && i != j) {
          const int lo = i < j ? i : j, hi = i < j ? j : i;
          v = (philox10((uint32_t)lo, (uint32_t)hi, 0u, kTagDense, k0, k1).a & 1u) ? 1 : -1;
          if (i < j) wsum -= v;
        }
        word |= (uint32_t)(uint8_t)(int8_t)v << (8 * b);
      }
      out[w] = (int32_t)word;
    }
    J[idx] = out;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) wsum += __shfl_xor(wsum, o, 64);
  if ((threadIdx.x & 63) == 0 && wsum)
    __hip_atomic_fetch_add((unsigned long long*)W, (unsigned long long)wsum, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Spins: +1 iff word (v & 3) of Philox(v >> 2, 0, r, INIT) < 2^31 (the same
// stream as sparse instances); padding columns are 0.
__global__ void __launch_bounds__(256) k_dense_init_spins(int8_t* S, int32_t* fam, int32_t n,
                                                          int32_t np, int32_t R, uint32_t k0,
                                                          uint32_t k1) {
  const int64_t total = (int64_t)R * (np / 4);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(i / (np / 4));
    const int q = (int)(i % (np / 4));
    const u32x4 w = philox10((uint32_t)q, 0u, (uint32_t)r, kTagInit, k0, k1);
    uint32_t word = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = 4 * q + k;
      const int8_t s = v < n ? (pick(w, k) < 0x80000000u ? (int8_t)1 : (int8_t)-1) : (int8_t)0;
      word |= (uint32_t)(uint8_t)s << (8 * k);
    }
    reinterpret_cast<uint32_t*>(S)[i] = word;
    if (q == 0) fam[r] = r;
  }
}

// G[m][r] += sum_{k in slice p} J[row0 + m][k] S[r][k] for the super-block's
// rows m < rows and every replica r (the K slices meet by atomic addition in
// G, which its reader clears).  Work-group = (128-row tile, NT-replica tile, K
// slice), eight waves, v_mfma_i32_16x16x64_i8 tiles.  The couplings go from
// memory to registers, three stages of two 64-column steps ahead; the spins,
// which all of the tile's rows share, through LDS (three buffers, rows padded
// by 16 bytes against bank conflicts).  Operand fragments: lane l
// supplies 16 consecutive K bytes at 16*(l/16) of row (A) / replica (B) l %
// 16; the result holds rows 4*(l/16)..+3 of column l % 16.
// The product runs over the columns 0 .. kcount + xlen with the xlen columns
// from x0 left out (x0, xlen and kcount multiples of 64): compacted column k
// maps to k, plus xlen once k >= x0.
struct GemmArgs {
  const int8_t* J;
  const int8_t* S0;
  const int8_t* S1;
  int32_t* G;
  const RunState* st;
  int32_t row0, rows, np, R, use_state, kslice;
  int32_t kcount, x0, xlen;
};

//
// Reading J (102 MB a super-block at n = 100,000, 22 us at a copy's rate),
// the fragments' way through LDS (64 KB per CU for 576 cycles of products)
// and the atomic additions bound it: with R = 256, 24 slices of 4,224 columns
// take 50 us, 39 of them without the additions; 61 with two buffers and the
// compiler's own order.
template <int NT>
struct GemmLds {
  __attribute__((aligned(16))) int8_t Bs[3][NT * kLdsRow];
};

template <int NT>
__device__ __forceinline__ void gemm_body(const GemmArgs& g, int bid, GemmLds<NT>& L) {
  int8_t* Bs = L.Bs[0];
  int32_t* __restrict__ G = g.G;
  const int32_t row0 = g.row0, rows = g.rows, np = g.np, R = g.R;
  if (g.use_state == 1 && !g.st->active) return;
  const int8_t* __restrict__ S = (g.use_state ? g.st->cur : 0) ? g.S1 : g.S0;
  // XCD-aware order: work-groups are dealt to the 8 XCDs round-robin, so
  // every output tile of K slice p lands on XCD p % 8 and the slice's
  // spins are fetched into that XCD's L2 once, not once per row tile
  const int MT = (rows + kGM - 1) / kGM, NTs = (R + NT - 1) / NT;
  const int xcd = bid & 7, q = bid >> 3;
  const int tile = q % (MT * NTs);
  const int p = (q / (MT * NTs)) * 8 + xcd;
  const int mt = tile % MT, ntile = tile / MT;
  const int k_beg = p * g.kslice, k_end = min(g.kcount, k_beg + g.kslice);
  if (k_beg >= k_end) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // waves: 4 x 2 over the tile (32 rows x NT / 2 replicas each), or 8 x 1
  constexpr int WN = NT >= 128 ? 2 : 1, WM = 8 / WN;
  constexpr int FM = kGM / WM / 16, FN = NT / WN / 16;  // 16 x 16 tiles per wave
  const int wm = wave % WM, wn = wave / WM;
  const int steps = (k_end - k_beg) / 64, nst = (steps + 1) / 2;
  auto column = [&](int step) {  // of a step of the slice, clamped to its last
    const int kc = k_beg + 64 * min(step, steps - 1);
    return kc + (kc >= g.x0 ? g.xlen : 0);
  };
  // A: the wave's row blocks (past the super-block: the last one again, its
  // results are dropped below)
  const int8_t* ag[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int rb = min((row0 >> 4) + mt * (kGM / 16) + wm * FM + i, ((row0 + rows) >> 4) - 1);
    ag[i] = g.J + (size_t)rb * (np >> 6) * 1024 + lane * 16;
  }
  // B: chunks of 16 bytes, chunk c = (replica c / 8, bytes 16 (c % 8) ..)
  constexpr int PB = NT * 8 / kDenseThreads;
  const int8_t* bg[PB];
  int lb[PB];
  const int half = (t & 7) >> 2;  // the step of the stage that the thread's chunks belong to
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int row = (t >> 3) + (kDenseThreads / 8) * i;
    bg[i] = S + (size_t)min(ntile * NT + row, R - 1) * np + 16 * (t & 3);
    lb[i] = row * kLdsRow + 16 * (t & 7);
  }
  constexpr int DA = 4;  // A register slots
  static_assert(2 * FM <= FN && 2 * PB <= FN, "a half-stage issues these loads between its FN column tiles");
  v4i ra[DA][2][FM], rb[2][PB], bf[2][FN], acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = v4i{0, 0, 0, 0};
  auto a_at = [&](int step) { return (size_t)(column(step) >> 6) * 1024; };
  auto b_at = [&](int stage) {
    const int k0 = column(2 * stage), k1 = column(2 * stage + 1);
    return half ? k1 : k0;
  };
  auto load_a = [&](int slot, int h, int i, size_t at) { ra[slot][h][i] = *reinterpret_cast<const v4i*>(ag[i] + at); };
  auto load_b = [&](int slot, int i, int at) { rb[slot][i] = *reinterpret_cast<const v4i*>(bg[i] + at); };
  auto write_b = [&](int slot, int buf, int i) { *reinterpret_cast<v4i*>(Bs + buf + lb[i]) = rb[slot][i]; };
  const int frag = (wn * FN * 16 + (lane & 15)) * kLdsRow + 16 * (lane >> 4);
  auto read_b = [&](int h, int buf, int j) {
    bf[h][j] = *reinterpret_cast<const v4i*>(Bs + buf + frag + j * 16 * kLdsRow + 64 * h);
  };
  constexpr int kBuf = NT * kLdsRow;
  // every load is unconditional (past the last step it reads the last one
  // again), so the compiler waits for exactly the stage it uses
#pragma unroll
  for (int d = 0; d < DA - 1; ++d)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < FM; ++i) load_a(d, h, i, a_at(2 * d + h));
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma unroll
    for (int i = 0; i < PB; ++i) load_b(d & 1, i, b_at(d));
    if (d < 2)
#pragma unroll
      for (int i = 0; i < PB; ++i) write_b(d & 1, d * kBuf, i);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < FN; ++j) read_b(0, 0, j);
  // Stage st multiplies from A slot st % 4 and the fragments read from LDS
  // half a stage before; between its matrix-core instructions it reads the
  // next half's fragments, loads A of stage st + 3 and B of stage st + 3 and
  // writes B of stage st + 2 to the third buffer, whose last reads ended
  // before the previous barrier.  The scheduling barriers keep that order.
  int st = 0, b0 = 0, b1 = kBuf, b2 = 2 * kBuf;
  auto stage = [&](auto J) {
    constexpr int sl = decltype(J)::value, nx = (sl + DA - 1) % DA, bs = sl & 1;
    const size_t at[2] = {a_at(2 * (st + DA - 1)), a_at(2 * (st + DA - 1) + 1)};
    const int kb = b_at(st + 3);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      read_b(1, b0, j);
#pragma unroll
      for (int i = 0; i < FM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra[sl][0][i], bf[0][j], acc[i][j], 0, 0, 0);
      if (j < 2 * FM) load_a(nx, j / FM, j % FM, at[j / FM]);
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool two = 2 * st + 1 < steps;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      read_b(0, b1, j);
      if (two) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra[sl][1][i], bf[1][j], acc[i][j], 0, 0, 0);
      }
      if (j < PB) write_b(bs, b2, j);
      else if (j < 2 * PB) load_b(bs ^ 1, j - PB, kb);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int free = b0;
    b0 = b1;
    b1 = b2;
    b2 = free;
    __syncthreads();
    return ++st < nst;
  };
  while (stage(std::integral_constant<int, 0>()) && stage(std::integral_constant<int, 1>()) &&
         stage(std::integral_constant<int, 2>()) && stage(std::integral_constant<int, 3>())) {
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = mt * kGM + (wm * FM + i) * 16 + 4 * (lane >> 4) + e;
        const int n = ntile * NT + (wn * FN + j) * 16 + (lane & 15);
        const int32_t v = acc[i][j][e];
        if (v != 0 && m < rows && n < R)
          __hip_atomic_fetch_add(&G[(size_t)m * R + n], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
}

template <int NT>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) k_dense_gemm(GemmArgs g) {
  __shared__ GemmLds<NT> L;
  gemm_body<NT>(g, blockIdx.x, L);
}

// Sequential visit of one super-block's spins for one group of 16 replicas.
struct SeqArgs {
  const int8_t* J;
  int8_t* S0;
  int8_t* S1;
  int64_t* E0;
  int64_t* E1;
  int32_t* G;   // [kSB][R] fields of the super-block rows against its starting spins
  const uint32_t* thr;
  const v4i* C;  // [n_pad / 4][R] negated critical fields of the sweep (k_dense_crit)
  const int32_t* not_monotone;  // nonzero: the thresholds rise somewhere, so critical fields do not exist
  RunState* st;
  int32_t n, np, R;
  uint32_t k0, k1;
  int64_t* flip_ctr;
};

// Critical fields of one sweep's visits.  The thresholds T[x + Xt] (|x| <=
// Xt) do not increase with x, so the test u < T[x + Xt] holds exactly for
// x < c - Xt, c = the number of leading entries of T above u.  The stored
// value is -(c - Xt), with c = 0 stored as +2^30 (no field flips) and c =
// 2Xt + 1 as -2^30, so that a field beyond the table (|x| > Xt, where the
// table is saturated) meets the decision of the clamped lookup (|x| < 2^30 -
// 2^12); Metropolis raises c - Xt to 1 (x <= 0 always flips), and padding
// vertices never flip.  C[q][r] holds the four spins of quad q for replica r,
// from the same Philox words (q, sweep, r, SWEEP) as the visits.  The search
// is a fixed-step binary lifting: over every 2^shift-th entry, held in LDS,
// then over the entries between two of them, read through the caches (at
// most three steps while the table has fewer than 2^18 entries).  Should the
// table rise anywhere (a negative beta), *not_monotone is set.
template <int RULE>
__global__ void __launch_bounds__(kCritThreads) k_dense_crit(const uint32_t* __restrict__ thr, const RunState* st,
                                                             v4i* C, int32_t* not_monotone, int32_t sweep_idx,
                                                             int32_t n, int32_t nq, int32_t R, uint32_t k0,
                                                             uint32_t k1) {
  extern __shared__ uint32_t thr_s[];
  if (!st->active) return;
  const int32_t Xt = (int32_t)st->table_x, L = 2 * Xt + 1;
  const uint32_t gs = st->gs + (uint32_t)sweep_idx;
  int shift = 0;
  while ((L >> shift) > kCritLds) ++shift;
  const int32_t coarse = L >> shift;  // entries (m << shift) - 1, m = 1 .. coarse
  for (int i = threadIdx.x; i < coarse; i += blockDim.x) thr_s[i] = thr[((i + 1) << shift) - 1];
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  bool rises = false;
  for (int64_t i = first; i + 1 < L; i += stride) rises = rises || thr[i] < thr[i + 1];
  if (rises) *not_monotone = 1;
  int top = 1;
  while (2 * top <= coarse) top *= 2;
  __syncthreads();
  const int64_t total = (int64_t)nq * R;
  int32_t q = (int32_t)(first / R), r = (int32_t)(first % R);
  const int32_t dq = (int32_t)(stride / R), dr = (int32_t)(stride % R);
  for (int64_t it = first; it < total; it += stride) {
    const u32x4 w = philox10((uint32_t)q, gs, (uint32_t)r, kTagSweep, k0, k1);
    int32_t pos[4] = {0, 0, 0, 0};
    for (int step = top; step > 0; step >>= 1)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int32_t p = pos[kk] + step;
        const uint32_t tv = thr_s[min(p, coarse) - 1];
        pos[kk] = (p <= coarse && tv > pick(w, kk)) ? p : pos[kk];
      }
    if (shift) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) pos[kk] <<= shift;
      for (int step = 1 << (shift - 1); step > 0; step >>= 1)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int32_t p = pos[kk] + step;
          const uint32_t tv = thr[min(p, L) - 1];
          pos[kk] = (p <= L && tv > pick(w, kk)) ? p : pos[kk];
        }
    }
    v4i c;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      int32_t v = pos[kk] == 0 ? -kCritInf : pos[kk] == L ? kCritInf : pos[kk] - Xt;
      if (RULE == 1) v = max(v, 1);
      c[kk] = 4 * q + kk < n ? -v : kCritInf;
    }
    C[it] = c;
    q += dq;
    r += dr;
    if (r >= R) {
      r -= R;
      q += 1;
    }
  }
}

// LDS of the sequential pass; buffers are taken in turn by the block's
// number.  Fragments are those of v_mfma_i32_16x16x64_i8, [strip of 16
// rows][lane].
struct SeqLds {
  v4i field[2][4][64];  // fields of the block from everything but the block before it and itself
  v4i h0[2][4][64];     // fields at the block's start
  v4i ain[4][4][64];    // J of the block against itself, columns permuted (see seq_body)
  v4i anx[3][4][64];    // J of the block against the block before it, columns permuted
  v4i crit[3][4][64];   // negated critical fields
  v4i sw[4][64];        // spin words, one per strip
  v4i jin[3][4][4][2];  // [strip][lane / 16]: twice J within a lane's four spins, pairs 10, 20, 21, 30, 31, 32
  __attribute__((aligned(16))) int8_t dsl[16][kSB + 16];  // spin changes d, [replica][row - row0]
  __attribute__((aligned(16))) int8_t spl[16][kSB + 16];  // the super-block before's spins, final
};

// One work-group per 16 replicas walks the super-block's 64-spin blocks in
// order.  Wave 0 decides block b from registers while the others prepare
// block b + 1 and finish block b - 1; one LDS barrier per block.
//
// The deciding wave.  Its lane l = 16 g + c keeps, for replica c, the fields
// of spins 16 s + 4 g + j (strip s, j < 4) where the matrix cores leave them:
// element j of accumulator s.  Groups of four spins are decided in order (s,
// then g): every lane decides its four spins, one after another, with the
// couplings inside the four (dot4), and the lanes whose turn it is keep the
// result, one word d (bytes 0, 2 or -2).  A product J . d then brings the
// change to the fields of the spins to come.  The order of its K dimension is
// free: lane group g supplies K bytes 16 g .. 16 g + 15, and as byte 4 s + j
// of them it supplies spin 16 s + 4 g + j, so its operand is the four words
// it decided itself and no data moves between lanes; the couplings are stored
// with their columns in that order (ain, anx).
//
// Decision: with m = 0 or -1 for s = +1 or -1, s h < c is (h ^ m) < c + m (h ^
// -1 = -h - 1), i.e. the sign of t = (h ^ m) - (c + m).  Inside the four, a
// flip of j' (f = t >> 31 = -1) adds f times 2 s_j s_j' J_jj' to t_j, products
// taken beforehand, so the chain per spin is one multiply-add and one shift
// (a dot4 instead costs three wait states more).  That chain bounds a block:
// 16 groups of four, each eight dependent operations and a matrix-core
// product whose result the next group waits for, 1.8 us a block and 29 us a
// super-block of 1,024 spins.  One work-group per 64 replicas with the
// couplings applied by dot products took 5.6 us a block, and 24 where the
// threshold table outgrew LDS.
//
// Energy: flips change it by -d.h, summed over the block as -d.(h0 + J d /
// 2) by another wave, from the fields h0 at the block's start.
template <int RULE, bool EXACT>
__device__ __forceinline__ void seq_body(const SeqArgs& a, int group, int32_t sweep_idx, int32_t row0, int32_t rows,
                                         SeqLds& L) {
  RunState* st = a.st;
  if (!st->active) return;
  const int cur = st->cur;
  int8_t* S = cur ? a.S1 : a.S0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int r = group * 16 + c;
  const int nb = min(rows, a.n - row0 + kDB - 1) / kDB;  // blocks holding real spins
  const v4i zero = {0, 0, 0, 0};
  if (nb <= 0) return;
  // fragment (row block, step) of the super-block's rows and any columns
  auto frag = [&](int row, int col) {
    return a.J + ((size_t)((row0 + row) >> 4) * (a.np >> 6) + (col >> 6)) * 1024;
  };
  auto word = [&](const int8_t* p) { return *reinterpret_cast<const int32_t*>(p); };
  // The passes over blocks -1, 0, 1, .. between barriers: what block b + 1
  // needs last (its fields) is made while block b is decided, everything else
  // one block earlier.
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);
    const uint32_t gs = st->gs + (uint32_t)sweep_idx;
    const int32_t Xt = (int32_t)st->table_x;
    struct Inputs {
      v4i ain[4], anx[4], ncc[4], jin[4][2], sw;
    };
    auto fetch = [&](int b, Inputs& x) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        x.ain[s] = L.ain[b & 3][s][lane];
        x.ncc[s] = L.crit[b % 3][s][lane];
        x.jin[s][0] = L.jin[b % 3][s][g][0];
        x.jin[s][1] = L.jin[b % 3][s][g][1];
        if (b > 0) x.anx[s] = L.anx[b % 3][s][lane];
      }
      x.sw = L.sw[b & 3][lane];
    };
    v4i dprev = zero;
    auto decide = [&](int b, const Inputs& x) {
      v4i acc[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s] = L.field[b & 1][s][lane];
      if (b > 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x.anx[s], dprev, acc[s], 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) L.h0[b & 1][s][lane] = acc[s];
      v4i dw = zero;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t w = (uint32_t)x.sw[s];
        u32x4 rnd;
        if constexpr (EXACT)
          rnd = philox10((uint32_t)((row0 + b * kDB + 16 * s + 4 * g) >> 2), gs, (uint32_t)r, kTagSweep, a.k0, a.k1);
        int32_t m[4], nt[4], pr[6];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          m[j] = __builtin_amdgcn_sbfe((int32_t)w, 8u * j + 7u, 1u);
          nt[j] = EXACT ? -m[j] : x.ncc[s][j] - m[j];
        }
#pragma unroll
        for (int j = 1, k = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < j; ++i, ++k) pr[k] = __mul24((m[j] ^ m[i]) | 1, x.jin[s][k >> 2][k & 3]);
        // the change of a flip, -2 s: 0xFE for s = +1 (0x01), 0x02 for s = -1 (0xFF)
        const uint32_t bw = 0xFEFEFEFEu ^ (((w >> 7) & 0x01010101u) * 0xFCu);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t dg = 0;
          int32_t f[4];  // all ones: flip
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            int32_t t = (acc[s][j] ^ m[j]) + nt[j];  // EXACT: x = s h
#pragma unroll
            for (int i = 0; i < j; ++i) t = __mul24(f[i], pr[j * (j - 1) / 2 + i]) + t;
            if constexpr (EXACT) {
              const uint32_t T = a.thr[min(max(t, -Xt), Xt) + Xt];
              bool fl = pick(rnd, j) < T;
              if (RULE == 1) fl = fl || t <= 0;
              f[j] = fl && row0 + b * kDB + 16 * s + 4 * g + j < a.n ? -1 : 0;
            } else {
              f[j] = t >> 31;
            }
            dg |= (uint32_t)f[j] & (bw & (0xFFu << (8 * j)));
          }
          const int32_t mine = g == q ? (int32_t)dg : 0;
          dw[s] |= mine;
          if (q < 3) {
            v4i bv = zero;
            bv[s] = mine;
            acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x.ain[s], bv, acc[s], 0, 0, 0);
          }
        }
        v4i bv = zero;
        bv[s] = dw[s];
#pragma unroll
        for (int s2 = s + 1; s2 < 4; ++s2)
          acc[s2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x.ain[s2], bv, acc[s2], 0, 0, 0);
        *reinterpret_cast<int32_t*>(&L.dsl[c][b * kDB + 16 * s + 4 * g]) = dw[s];
      }
      dprev = dw;
    };
    Inputs xa, xb;
    lds_barrier();
    fetch(0, xa);
    lds_barrier();
    for (int b = 0; b < nb; b += 2) {
      if (b + 1 < nb) fetch(b + 1, xb);
      decide(b, xa);
      lds_barrier();
      if (b + 1 < nb) {
        if (b + 2 < nb) fetch(b + 2, xa);
        decide(b + 1, xb);
        lds_barrier();
      }
    }
    lds_barrier();
  } else if (wave <= 4) {
    // strip sr of block x: its fields from the field product (cleared behind
    // for the next super-block's), from the super-block before (whose
    // columns that product left out) and from the flips of blocks 0 .. x - 2;
    // read two blocks ahead (the super-block before's couplings one), multiplied
    // one ahead
    const int sr = wave - 1;
    constexpr int kMaxSteps = kSB / kDB - 2, kPrev = kSB / kDB;
    const int prev = row0 > 0 ? row0 - kSB : -1;  // first column of the super-block before
    v4i av[2][kMaxSteps], pv[kPrev];
    int32_t gv[2][4];
    auto load_prev = [&](int x) {
      if (x >= nb || prev < 0) return;
      const int8_t* p = frag(x * kDB + 16 * sr, prev) + lane * 16;
#pragma unroll
      for (int k = 0; k < kPrev; ++k) pv[k] = *reinterpret_cast<const v4i*>(p + 1024 * k);
    };
    auto load = [&](int x, v4i(&v)[kMaxSteps], int32_t(&f)[4]) {
      if (x >= nb) return;
      int32_t* gp = a.G + (size_t)(x * kDB + 16 * sr + 4 * g) * a.R + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = gp[(size_t)j * a.R];
      const int8_t* p = frag(x * kDB + 16 * sr, row0) + lane * 16;
#pragma unroll
      for (int k = 0; k < kMaxSteps; ++k)
        if (k < x - 1) v[k] = *reinterpret_cast<const v4i*>(p + 1024 * k);
    };
    auto prepare = [&](int x, const v4i(&v)[kMaxSteps], const int32_t(&f)[4]) {
      if (x >= nb) return;
      v4i s0 = {f[0], f[1], f[2], f[3]}, s1 = zero;
      if (prev >= 0) {
#pragma unroll
        for (int k = 0; k < kPrev; k += 2) {
          s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(
              pv[k], *reinterpret_cast<const v4i*>(&L.spl[c][64 * k + 16 * g]), s0, 0, 0, 0);
          s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(
              pv[k + 1], *reinterpret_cast<const v4i*>(&L.spl[c][64 * (k + 1) + 16 * g]), s1, 0, 0, 0);
        }
      }
      load_prev(x + 1);
#pragma unroll
      for (int k = 0; k < kMaxSteps; ++k)
        if (k < x - 1) {
          const v4i bv = *reinterpret_cast<const v4i*>(&L.dsl[c][64 * k + 16 * g]);
          if (k & 1)
            s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(v[k], bv, s1, 0, 0, 0);
          else
            s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(v[k], bv, s0, 0, 0, 0);
        }
      L.field[x & 1][sr][lane] = s0 + s1;
      int32_t* gp = a.G + (size_t)(x * kDB + 16 * sr + 4 * g) * a.R + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) gp[(size_t)j * a.R] = 0;
    };
    load(0, av[0], gv[0]);
    load_prev(0);
    load(1, av[1], gv[1]);
    lds_barrier();  // the spins of the super-block before are in
    prepare(0, av[0], gv[0]);
    lds_barrier();
    for (int b = 0; b < nb; b += 2) {
      // while block b is decided: block b + 1; then b + 2 while b + 1 is
      load(b + 2, av[0], gv[0]);
      prepare(b + 1, av[1], gv[1]);
      lds_barrier();
      if (b + 1 < nb) {
        load(b + 3, av[1], gv[1]);
        prepare(b + 2, av[0], gv[0]);
        lds_barrier();
      }
    }
    lds_barrier();
  } else if (wave <= 6) {
    // wave 5: the couplings of block x to itself, those inside a lane's four
    // spins, its critical fields and spin words; wave 6: its couplings to the
    // block before it
    const bool self = wave == 5;
    v4i fa[4], cr[4], ji[2], sw;
    auto load = [&](int x) {
      if (x >= nb) return;
      if (self || x > 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int8_t* f = frag(x * kDB + 16 * s, row0 + (self ? x : x - 1) * kDB) + 16 * c + 4 * g;
#pragma unroll
          for (int e = 0; e < 4; ++e) fa[s][e] = word(f + 256 * e);
        }
      }
      if (!self) return;
      const int rb0 = row0 + x * kDB;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        cr[s] = a.C[(size_t)((rb0 >> 2) + 4 * s + g) * a.R + r];
        sw[s] = word(S + (size_t)r * a.np + rb0 + 16 * s + 4 * g);
      }
      // lane = (strip c / 4, group c % 4): its four rows against its four columns
      const int8_t* f = frag(x * kDB + 16 * (c >> 2), rb0) + 256 * (c >> 2) + 4 * (c & 3);
#pragma unroll
      for (int j = 1, k = 0; j < 4; ++j) {
        const int32_t w = word(f + 16 * (4 * (c & 3) + j));
#pragma unroll
        for (int i = 0; i < j; ++i, ++k) ji[k >> 2][k & 3] = 2 * __builtin_amdgcn_sbfe(w, 8u * i, 8u);
      }
    };
    auto put = [&](int x) {
      if (x >= nb) return;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (self) {
          L.ain[x & 3][s][lane] = fa[s];
          L.crit[x % 3][s][lane] = cr[s];
        } else if (x > 0) {
          L.anx[x % 3][s][lane] = fa[s];
        }
      }
      if (!self) return;
      L.sw[x & 3][lane] = sw;
      if (lane < 16) {
        L.jin[x % 3][lane >> 2][lane & 3][0] = ji[0];
        L.jin[x % 3][lane >> 2][lane & 3][1] = ji[1];
      }
    };
    load(0);
    put(0);
    load(1);
    lds_barrier();
    put(1);
    load(2);
    lds_barrier();
    for (int b = 0; b < nb; ++b) {
      put(b + 2);
      load(b + 3);
      lds_barrier();
    }
    lds_barrier();
  } else {
    // wave 7: first the spins of the super-block before; then the energy
    // change and the new spin words of block x
    if (row0 > 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        *reinterpret_cast<v4i*>(&L.spl[i][16 * lane]) =
            *reinterpret_cast<const v4i*>(S + (size_t)(group * 16 + i) * a.np + row0 - kSB + 16 * lane);
    }
    int64_t dE = 0;
    int32_t nflip = 0;
    auto finish = [&](int x) {
      v4i d, sw = L.sw[x & 3][lane];
      int32_t e = 0;
#pragma unroll
      for (int s = 0; s < 4; ++s) d[s] = *reinterpret_cast<const int32_t*>(&L.dsl[c][x * kDB + 16 * s + 4 * g]);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        v4i p = L.h0[x & 1][s][lane];
        p = __builtin_amdgcn_mfma_i32_16x16x64_i8(L.ain[x & 3][s][lane], d, p + p, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) e += __builtin_amdgcn_sbfe(d[s], 8u * j + 1u, 7u) * p[j];  // d / 2
        // a flip turns 0x01 <-> 0xFF, i.e. xor 0xFE
        const uint32_t f = (uint32_t)d[s] & 0x02020202u;
        *reinterpret_cast<uint32_t*>(S + (size_t)r * a.np + row0 + x * kDB + 16 * s + 4 * g) = (uint32_t)sw[s] ^ (f * 0x7Fu);
        nflip += __builtin_popcount(f);
      }
      dE -= e;  // |e| < 2^31: |p| <= 2 X + 2^14, X < 2^25, 16 spins per lane
    };
    lds_barrier();
    lds_barrier();
    for (int b = 0; b < nb; ++b) {
      if (b > 0) finish(b - 1);
      lds_barrier();
    }
    finish(nb - 1);
    lds_barrier();
    // the four lanes of a replica
    dE += __shfl_xor(dE, 16, 64);
    dE += __shfl_xor(dE, 32, 64);
    if (g == 0 && dE != 0)
      __hip_atomic_fetch_add((unsigned long long*)&(cur ? a.E1 : a.E0)[r], (unsigned long long)dE, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    if (a.flip_ctr) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) nflip += __shfl_xor(nflip, o, 64);
      if (lane == 0)
        __hip_atomic_fetch_add((unsigned long long*)&a.flip_ctr[group & 255], (unsigned long long)nflip,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// One super-block step: work-groups 0 .. NG-1 run the sequential pass of this
// super-block (one per 16 replicas); with gemm_on the others compute the
// field product of the next super-block over every column except this
// super-block's own (which the pass is changing; the next pass adds them),
// into the other field buffer.  The two parts share no data, so the product
// runs on the compute units the pass leaves idle: 61 us a
// super-block at n = 100,000, R = 256, where the product is the longer part (90
// with the former layout and pass), and 32 us at n = 2,047, R = 64, where the
// pass is (757).
template <int RULE, int NT>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_dense_step(SeqArgs a, GemmArgs g, int32_t sweep_idx, int32_t row0, int32_t rows, int32_t NG, int32_t gemm_on) {
  __shared__ union {
    SeqLds seq;
    GemmLds<NT> gemm;
  } L;
  if ((int)blockIdx.x < NG) {
    if (*a.not_monotone)
      seq_body<RULE, true>(a, blockIdx.x, sweep_idx, row0, rows, L.seq);
    else
      seq_body<RULE, false>(a, blockIdx.x, sweep_idx, row0, rows, L.seq);
  } else if (gemm_on) {
    gemm_body<NT>(g, blockIdx.x - NG, L.gemm);
  }
}

// Energy of the population from super-block fields: E_r += sum_k s_rk G_kr
// (the caller negates and halves at the end); clears G.  Work-group =
// (tile, kEnergyRows-row block), lanes = replicas.
constexpr int kEnergyRows = 8;
__global__ void __launch_bounds__(64) k_dense_energy_sb(const int8_t* S, int32_t* G, int64_t* E, int32_t row0,
                                                        int32_t rows, int32_t n, int32_t np, int32_t R) {
  const int T = R / 64;
  const int tile = blockIdx.x % T, rb = blockIdx.x / T;
  const int r = tile * 64 + threadIdx.x;
  int64_t acc = 0;
#pragma unroll
  for (int k = kEnergyRows * rb; k < kEnergyRows * (rb + 1); ++k) {
    if (row0 + k >= n) break;
    int32_t* gp = G + (size_t)k * R + r;
    acc += (int64_t)*gp * S[(size_t)r * np + row0 + k];
    *gp = 0;
  }
  if (acc)
    __hip_atomic_fetch_add((unsigned long long*)&E[r], (unsigned long long)acc, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_dense_init_finish(int64_t* E, int32_t R, RunState* st, int8_t* best, int32_t np) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < R) E[i] = -(E[i] / 2);
  for (int v = i; v < np; v += gridDim.x * blockDim.x) best[v] = 1;
  if (i == 0) {
    st->mstar = 0;
    st->cur = 0;
    st->gs = st->g_rs = st->g_cl = 0;
    st->stopped = 0;
    st->active = 0;
    st->steps_run = 0;
  }
}

// Energies of a population the host loaded into buffer 0: E = -E / 2 and
// buffer 0 becomes the current one.
__global__ void k_dense_load_finish(int64_t* E, int32_t R, RunState* st) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < R) E[i] = -(E[i] / 2);
  if (i == 0) st->cur = 0;
}

// Resampling gather for the replica-major layout.
__global__ void __launch_bounds__(256) k_dense_gather(const RunState* st, int8_t* S0, int8_t* S1,
                                                      int64_t* E0, int64_t* E1, int32_t* F0, int32_t* F1,
                                                      const int32_t* parent, int32_t np, int32_t R) {
  if (!st->active || !st->do_resample) return;
  const int cur = st->cur;
  const uint32_t* Ss = reinterpret_cast<const uint32_t*>(cur ? S1 : S0);
  uint32_t* Sd = reinterpret_cast<uint32_t*>(cur ? S0 : S1);
  const int c = blockIdx.y;
  const int p = parent[c];
  const int words = np / 4;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x)
    Sd[(size_t)c * words + i] = Ss[(size_t)p * words + i];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    (cur ? E0 : E1)[c] = (cur ? E1 : E0)[p];
    (cur ? F0 : F1)[c] = (cur ? F1 : F0)[p];
  }
}



// H[r][row0 + k] = G[k][r] for the super-block's rows (snapshots); clears G.
__global__ void __launch_bounds__(256) k_dense_collect_sb(int32_t* G, int32_t* H, int32_t row0, int32_t rows,
                                                          int32_t n, int32_t np, int32_t R) {
  const int64_t total = (int64_t)rows * R;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(i / R), r = (int)(i % R);
    if (row0 + k < n) H[(size_t)r * np + row0 + k] = G[i];
    G[i] = 0;
  }
}

}  // namespace


// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline uint32_t key0(const pamc_instance* I) { return (uint32_t)I->seed; }
static inline uint32_t key1(const pamc_instance* I) { return (uint32_t)(I->seed >> 32); }
// Set by k_dense_crit where the thresholds rise; cleared with each table.
static inline int32_t* dense_monotone_flag(const pamc_instance* I) {
  return reinterpret_cast<int32_t*>(I->flip_ctr + kMonotoneSlot);
}

// Kernels whose dynamic LDS may exceed the default limit.
hipError_t prepare_dense_lds() {
  for (const void* k : {(const void*)k_dense_crit<0>, (const void*)k_dense_crit<1>}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (kCritLds + 1));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_dense_generate(pamc_instance* I, uint64_t graph_seed) {
  int64_t* W = I->flip_ctr + 400;
  hipMemsetAsync(W, 0, sizeof(int64_t), I->stream);
  const int64_t total = (int64_t)I->dn_pad * I->dn_pad / 16;
  const int grid = (int)std::min<int64_t>((total + 255) / 256, 1 << 16);
  k_dense_generate<<<grid, 256, 0, I->stream>>>(reinterpret_cast<v4i*>(I->Jd), I->n, I->dn_pad, (uint32_t)graph_seed,
                                                (uint32_t)(graph_seed >> 32), W);
  return hipGetLastError();
}

void dense_fragments(int32_t np, const int8_t* rows, int8_t* out) {
  for (int32_t i = 0; i < 16; ++i)
    for (int32_t j = 0; j < np; j += 16) memcpy(out + frag_at(np, i, j), rows + (size_t)i * np + j, 16);
}

// rows of the super-block starting at row0 (a multiple of 64)
static inline int sb_rows(const pamc_instance* I, int row0) { return std::min(kSB, I->dn_pad - row0); }

// Replicas per tile of the field product: all of them up to 256, so that the
// couplings are read once.
static inline int gemm_nt(const pamc_instance* I) { return I->R <= 64 ? 64 : (I->R <= 128 ? 128 : 256); }

// K slices of the field product, each a multiple of the 64-column stage.
struct GemmShape {
  int grid, kslice;
};
// About kGemmWorkGroups working work-groups: the K range is cut into P
// slices of whole stages; the grid covers the slices in groups of 8 (one per
// XCD; work-groups of slices past the end return at once).  P above 8 is a
// multiple of 8, or some XCDs would get a slice more than others and, beside
// the pass's work-groups, more work-groups than CUs: n = 100,000, R = 256
// takes 82 ms a run of 12 sweeps with 128 + 64 of them, 99 with 128 (16
// slices) and 124 with 224 (28 slices).
constexpr int kGemmWorkGroups = 192;
static inline GemmShape gemm_shape(const pamc_instance* I, int rows, int kcount) {
  const int nt = gemm_nt(I);
  const int tiles = ((rows + kGM - 1) / kGM) * ((I->R + nt - 1) / nt);
  const int stages = std::max(1, (kcount + kStage - 1) / kStage);
  int P = std::max(1, std::min(stages / 2, kGemmWorkGroups / tiles));  // at least two stages per work-group
  if (P > 8) P -= P % 8;
  const int kslice = ((stages + P - 1) / P) * kStage;
  const int slices = (kcount + kslice - 1) / kslice;
  return {tiles * ((slices + 7) / 8) * 8, kslice};
}

// Field product G = J[row0 .. row0 + rows) . S over the K domain (kcount, x0,
// xlen; see GemmArgs), and its grid.
struct GemmLaunch {
  GemmArgs g;
  int grid;
};
static GemmLaunch gemm_launch(const pamc_instance* I, int32_t row0, int32_t rows, int32_t use_state, int32_t* G,
                              int32_t kcount, int32_t x0, int32_t xlen) {
  const GemmShape gsh = gemm_shape(I, rows, kcount);
  GemmArgs g;
  g.J = I->Jd;
  g.S0 = I->Sd;
  g.S1 = I->Sd2;
  g.G = G;
  g.st = I->st;
  g.row0 = row0;
  g.rows = rows;
  g.np = I->dn_pad;
  g.R = I->R;
  g.use_state = use_state;
  g.kslice = gsh.kslice;
  g.kcount = kcount;
  g.x0 = x0;
  g.xlen = xlen;
  return {g, gsh.grid};
}
static void launch_gemm(const pamc_instance* I, const GemmLaunch& gl) {
  switch (gemm_nt(I)) {
    case 64: k_dense_gemm<64><<<gl.grid, kDenseThreads, 0, I->stream>>>(gl.g); break;
    case 128: k_dense_gemm<128><<<gl.grid, kDenseThreads, 0, I->stream>>>(gl.g); break;
    default: k_dense_gemm<256><<<gl.grid, kDenseThreads, 0, I->stream>>>(gl.g); break;
  }
}
static GemmLaunch gemm_full(const pamc_instance* I, int32_t row0, int32_t rows, int32_t use_state, int32_t* G) {
  return gemm_launch(I, row0, rows, use_state, G, I->dn_pad, I->dn_pad, 0);
}

static hipError_t dense_full_energy(pamc_instance* I, int buf) {
  const int T = I->R / 64;
  hipMemsetAsync(I->pop.E[buf], 0, sizeof(int64_t) * I->R, I->stream);
  for (int row0 = 0; row0 < I->n; row0 += kSB) {
    const int rows = sb_rows(I, row0);
    const GemmLaunch gl = gemm_full(I, row0, rows, 0, I->Gd);
    launch_gemm(I, gl);
    k_dense_energy_sb<<<T * (rows / kEnergyRows), 64, 0, I->stream>>>(buf ? I->Sd2 : I->Sd, I->Gd, I->pop.E[buf], row0,
                                                             rows, I->n, I->dn_pad, I->R);
  }
  return hipGetLastError();
}

hipError_t launch_init_dense(pamc_instance* I) {
  const int64_t total = (int64_t)I->R * (I->dn_pad / 4);
  const int grid = (int)std::min<int64_t>((total + 255) / 256, 65535);
  k_dense_init_spins<<<grid, 256, 0, I->stream>>>(I->Sd, I->pop.fam[0], I->n, I->dn_pad, I->R, key0(I),
                                                  key1(I));
  dense_full_energy(I, 0);
  k_dense_init_finish<<<(std::max(I->R, I->dn_pad) + 255) / 256, 256, 0, I->stream>>>(
      I->pop.E[0], I->R, I->st, I->best, I->dn_pad);
  return hipGetLastError();
}

hipError_t launch_dense_load(pamc_instance* I) {
  dense_full_energy(I, 0);
  k_dense_load_finish<<<(I->R + 255) / 256, 256, 0, I->stream>>>(I->pop.E[0], I->R, I->st);
  return hipGetLastError();
}

// Sweeps of the dense path, super-block by super-block (rows row0_i ..).
// The field buffer alternates between two halves of Gd.  Each sweep starts
// with its critical fields (every visit's, one launch); super-block 0 of a
// sweep gets its full product first; then, for each super-block i, the
// launch that runs its sequential pass also computes the product of i+1
// over every column except i's, which (final by then) the pass of i+1 adds
// itself.  With profiling, one event pair brackets each super-block step (the
// pass with the overlapped product).
static hipError_t dense_sweeps(Batch& b, int32_t nsweeps) {
  pamc_instance* I = b.I[0];
  const int NG = I->R / 16;
  using StepKernel = void (*)(SeqArgs, GemmArgs, int32_t, int32_t, int32_t, int32_t, int32_t);
  static const StepKernel step_kernels[2][3] = {{k_dense_step<0, 64>, k_dense_step<0, 128>, k_dense_step<0, 256>},
                                                {k_dense_step<1, 64>, k_dense_step<1, 128>, k_dense_step<1, 256>}};
  const int nt = gemm_nt(I);
  const StepKernel step = step_kernels[I->rule == 1][nt == 64 ? 0 : (nt == 128 ? 1 : 2)];
  int32_t* const not_monotone = dense_monotone_flag(I);
  SeqArgs a;
  a.J = I->Jd;
  a.S0 = I->Sd;
  a.S1 = I->Sd2;
  a.E0 = I->pop.E[0];
  a.E1 = I->pop.E[1];
  a.thr = I->thr;
  a.C = reinterpret_cast<const v4i*>(I->Cd);
  a.not_monotone = not_monotone;
  a.st = I->st;
  a.n = I->n;
  a.np = I->dn_pad;
  a.R = I->R;
  a.k0 = key0(I);
  a.k1 = key1(I);
  a.flip_ctr = I->prof ? I->flip_ctr : nullptr;
  auto gbuf = [&](int i) { return I->Gd + (size_t)(i & 1) * kSB * I->R; };
  const int nsb = (I->n + kSB - 1) / kSB;
  ctl_thresholds(b);
  for (int s = 0; s < nsweeps; ++s) {
    for (int i = 0; i < nsb; ++i) {
      const int row0 = i * kSB, rows = sb_rows(I, row0);
      hipEvent_t e0 = nullptr;
      if (I->prof) {
        e0 = ctl_event(I);
        hipEventRecord(e0, I->stream);
      }
      if (i == 0) {
        // the sweep's critical fields, then super-block 0's full product
        const int64_t items = (int64_t)(I->dn_pad / 4) * I->R;
        const int cgrid = (int)std::min<int64_t>((items + kCritThreads - 1) / kCritThreads, 256);
        // LDS for the table at its widest, 2 X + 1 entries
        const size_t lds = sizeof(uint32_t) * (size_t)std::min<int64_t>(2 * I->X + 1, kCritLds + 1);
        v4i* C = reinterpret_cast<v4i*>(I->Cd);
        if (I->rule == 1)
          k_dense_crit<1><<<cgrid, kCritThreads, lds, I->stream>>>(I->thr, I->st, C, not_monotone, s, I->n,
                                                                   I->dn_pad / 4, I->R, a.k0, a.k1);
        else
          k_dense_crit<0><<<cgrid, kCritThreads, lds, I->stream>>>(I->thr, I->st, C, not_monotone, s, I->n,
                                                                   I->dn_pad / 4, I->R, a.k0, a.k1);
        launch_gemm(I, gemm_full(I, row0, rows, 1, gbuf(0)));
      }
      a.G = gbuf(i);
      const bool next = i + 1 < nsb;
      GemmLaunch nx{};
      if (next) {
        const int n0 = row0 + kSB;
        nx = gemm_launch(I, n0, sb_rows(I, n0), 1, gbuf(i + 1), I->dn_pad - rows, row0, rows);
      }
      step<<<NG + (next ? nx.grid : 0), kDenseThreads, 0, I->stream>>>(a, nx.g, s, row0, rows, NG, next ? 1 : 0);
      if (I->prof) {
        hipEvent_t e1 = ctl_event(I);
        hipEventRecord(e1, I->stream);
        I->prof_launches += 1;
      }
    }
    if (I->prof) I->prof_attempts += (int64_t)I->n * I->R;
  }
  return hipGetLastError();
}

static void dense_gather(pamc_instance* I) {
  k_dense_gather<<<dim3(std::max(1, std::min(64, I->dn_pad / 1024)), I->R), 256, 0, I->stream>>>(
      I->st, I->Sd, I->Sd2, I->pop.E[0], I->pop.E[1], I->pop.fam[0], I->pop.fam[1], I->rs_parent,
      I->dn_pad, I->R);
}

hipError_t launch_dense_step(Batch& b, int32_t sweeps, int32_t resample) {
  pamc_instance* I = b.I[0];
  ctl_step_begin(b);
  if (resample) {
    ctl_resample_select(b);
    dense_gather(I);
  }
  ctl_commit(b, 1);
  hipError_t e = dense_sweeps(b, sweeps);
  if (e != hipSuccess) return e;
  ctl_step_end(b, 1);
  return hipGetLastError();
}

hipError_t launch_dense_prim_sweep(Batch& b, double beta, int32_t nsweeps) {
  ctl_prim_set(b, 0, beta, nsweeps);
  hipError_t e = dense_sweeps(b, nsweeps);
  if (e != hipSuccess) return e;
  ctl_advance(b, nsweeps);
  return hipGetLastError();
}

hipError_t launch_dense_prim_resample(Batch& b, double delta) {
  ctl_prim_set(b, 1, delta, 0);
  ctl_resample_select(b);
  dense_gather(b.I[0]);
  ctl_commit(b, 0);
  ctl_deactivate(b);
  return hipGetLastError();
}

hipError_t launch_dense_prim_update_best(Batch& b) {
  ctl_prim_set(b, 0, 0.0, 0);
  ctl_step_end(b, 0);
  ctl_deactivate(b);
  return hipGetLastError();
}

hipError_t launch_dense_fields(pamc_instance* I, int32_t* H_rmajor) {
  // fields H[r][v] (replica-major) of the current population, for snapshots
  for (int row0 = 0; row0 < I->n; row0 += kSB) {
    const int rows = sb_rows(I, row0);
    const GemmLaunch gl = gemm_full(I, row0, rows, 2, I->Gd);
    launch_gemm(I, gl);
    k_dense_collect_sb<<<std::min(1024, (rows * I->R + 255) / 256), 256, 0, I->stream>>>(
        I->Gd, H_rmajor, row0, rows, I->n, I->dn_pad, I->R);
  }
  return hipGetLastError();
}

int32_t dense_superblock_rows() { return kSB; }
int32_t dense_field_buffers() { return 2; }

}  // namespace pamc
