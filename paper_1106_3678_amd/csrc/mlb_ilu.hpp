// ILU(0) right preconditioning for Algorithm 7.1 (Section 7), the
// preconditioner of the paper's experiments (Section 5).
//
// M = L U with L unit lower and U upper triangular (3x3 blocks for BSR3: L with
// identity diagonal blocks, U with full ones), both on A's pattern, and
// (L U)_ij = a_ij wherever A is stored.  The factors live in one matrix with
// A's pattern, each row sorted by column: the entries left of the diagonal are
// L, the rest U.  The factorisation eliminates row by row: for every stored
// k < i of row i, in increasing k, l_ik = a_ik u_kk^{-1}, then a_ij -= l_ik u_kj
// for every stored j > k of row i that row k also stores.  A row only reads
// rows k < i of its own pattern, so all the rows of one level (rows whose
// longest chain of such dependencies has the same length) are factored
// together, one launch per level.  The triangular solves of M^{-1} v = U^{-1}
// (L^{-1} v) are one launch each (k_ilu_solve_block or k_ilu_solve_sweep), and M^{-H} v = L^{-H}
// (U^{-H} v) runs on the conjugate transpose of the factor matrix, whose lower
// part is U^H and whose upper part is L^H.
//
// The engine iterates on A M^{-1} y = b: every product with A is preceded by
// M^{-1} applied to its input, F = M^{-H} A^H Q(:, 1:n-1), y_0 = M x_0 and
// x = M^{-1} y at the end.
#pragma once

#include <hip/hip_runtime.h>

#include "mlb_precond.hpp"
#include "mlb_types.hpp"

namespace mlb {

// Position of the diagonal entry of every (block) row of a row-sorted matrix,
// and a check of its pattern.  bad |= 1: no stored diagonal; bad |= 4: a column
// stored twice in one row.
__global__ void k_ilu_diag_pos(const int* __restrict__ rp, const int* __restrict__ ci, int nbrows,
                               int* __restrict__ dpos, int* __restrict__ bad) {
  for (int row = blockIdx.x * blockDim.x + threadIdx.x; row < nbrows; row += gridDim.x * blockDim.x) {
    int qd = -1;
    for (int q = rp[row]; q < rp[row + 1]; ++q) {
      if (q > rp[row] && ci[q] == ci[q - 1]) atomicOr(bad, 4);
      if (ci[q] == row) qd = q;
    }
    if (qd < 0) atomicOr(bad, 1);
    dpos[row] = qd < 0 ? rp[row] : qd;
  }
}

// o = a b for 3x3 row-major blocks (BS = 3) or scalars (BS = 1).
template <class V, int BS>
__device__ inline void blk_mul(const V* a, const V* b, V* o) {
#pragma unroll
  for (int r = 0; r < BS; ++r)
#pragma unroll
    for (int c = 0; c < BS; ++c) {
      V acc = zero<V>();
#pragma unroll
      for (int k = 0; k < BS; ++k) acc = axpy(acc, a[BS * r + k], b[BS * k + c]);
      o[BS * r + c] = acc;
    }
}

// Factor the rows of one level in place (val holds A's values on entry, the
// factors on exit) and store the inverse of each row's diagonal (block) in
// dinv.  bad |= 2: a zero or singular pivot.
template <class V, int BS>
__global__ void k_ilu_factor_level(const int* __restrict__ rp, const int* __restrict__ ci, V* __restrict__ val,
                                   const int* __restrict__ dpos, V* __restrict__ dinv, const int* __restrict__ rows,
                                   int count, int* __restrict__ bad) {
  constexpr int B2 = BS * BS;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < count; t += gridDim.x * blockDim.x) {
    const int i = rows[t];
    const int beg = rp[i], end = rp[i + 1], qd = dpos[i];
    for (int q = beg; q < qd; ++q) {   // stored k < i, increasing
      const int k = ci[q];
      V l[B2];
      if constexpr (BS == 1) {
        l[0] = val[q] / val[dpos[k]];   // l_ik = a_ik / u_kk
      } else {
        blk_mul<V, 3>(val + (size_t)B2 * q, dinv + (size_t)B2 * k, l);   // l_ik = a_ik u_kk^{-1}
      }
#pragma unroll
      for (int e = 0; e < B2; ++e) val[(size_t)B2 * q + e] = l[e];
      // a_ij -= l_ik u_kj for stored j > k of row i that row k stores (both rows sorted)
      int p = dpos[k] + 1;
      const int pend = rp[k + 1];
      for (int q2 = q + 1; q2 < end && p < pend; ++q2) {
        const int j = ci[q2];
        while (p < pend && ci[p] < j) ++p;
        if (p < pend && ci[p] == j) {
          V prod[B2];
          blk_mul<V, BS>(l, val + (size_t)B2 * p, prod);
#pragma unroll
          for (int e = 0; e < B2; ++e) val[(size_t)B2 * q2 + e] = val[(size_t)B2 * q2 + e] - prod[e];
        }
      }
    }
    const V* d = val + (size_t)B2 * qd;
    V* di = dinv + (size_t)B2 * i;
    if constexpr (BS == 1) {
      if (is_zero(d[0]) || !finite(d[0])) {
        atomicOr(bad, 2);
        di[0] = from_real<V>(1.0);
      } else {
        di[0] = from_real<V>(1.0) / d[0];
      }
    } else {
      if (!inv3(d, di)) {
        atomicOr(bad, 2);
        for (int e = 0; e < 9; ++e) di[e] = from_real<V>((e % 4) == 0 ? 1.0 : 0.0);
      }
    }
  }
}

// Inverse of every diagonal (block) of a matrix (for the conjugate-transposed
// factor, whose diagonal blocks are U_ii^H).
template <class V, int BS>
__global__ void k_ilu_inv_diag(const V* __restrict__ val, const int* __restrict__ dpos, int nbrows,
                               V* __restrict__ dinv, int* __restrict__ bad) {
  constexpr int B2 = BS * BS;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nbrows; i += gridDim.x * blockDim.x) {
    const V* d = val + (size_t)B2 * dpos[i];
    V* di = dinv + (size_t)B2 * i;
    if constexpr (BS == 1) {
      if (is_zero(d[0]) || !finite(d[0])) { atomicOr(bad, 2); di[0] = from_real<V>(1.0); }
      else di[0] = from_real<V>(1.0) / d[0];
    } else {
      if (!inv3(d, di)) {
        atomicOr(bad, 2);
        for (int e = 0; e < 9; ++e) di[e] = from_real<V>((e % 4) == 0 ? 1.0 : 0.0);
      }
    }
  }
}

// ---- one launch per triangular solve, blocks of rows ------------------------
//
// The rows are cut into blocks of consecutive rows, one workgroup each, claimed
// from a counter in the order of the solve: every block that a claimed one reads
// is claimed too, by a workgroup that is running.  A workgroup takes its rows by
// level, in chunks of at most 64 rows of one level, a wave each.  A solved value is
// its own completion flag: where it will stand, in memory and in LDS, is first
// filled with a pending mark, and its 64-bit words are stored and read with relaxed
// atomics (in memory at agent scope, which keeps them coherent across the XCDs' L2
// caches without a release of a whole cache).
//
// What bounds it is the chain of dependent rows: on an m^3 7-point grid 3m - 2
// rows long.  So the work of a row is split over the waves of the workgroup:
//  * loader waves read what is known beforehand (the row's entries and right-hand
//    side), wait for the values of other blocks, subtract their part and lay the
//    rest of the row out in a slot in LDS;
//  * compute waves wait for the values of their own block, which stand in a ring in
//    LDS, finish the row and store it, in the ring and in memory.  They read no
//    memory, so nothing but the LDS is in the chain.
// Rows that were handed out in level order over all CUs, each link of the chain a
// store to and a load from memory, took about 1.45 us a level.
//
// A slot is free again once the chunk that used it is done.  The loader of chunk x
// waits until all chunks up to x - ns (ns slots) are; then it marks the ring's places
// of chunk x + ns pending.  A value is read from the ring by rows up to `safe` positions
// behind it and from memory by later ones; the ring has safe + 128 ns places or more, so
// whoever reads a place that is marked again is done, and whoever reads the new value
// finds the mark or the value.

// The pending mark: a signalling-NaN bit pattern.  Arithmetic never returns
// one (it quiets NaNs); a value that would be stored with this pattern (only a
// row copied through without arithmetic, from an input that holds it) is
// stored as the canonical quiet NaN instead.
constexpr unsigned long long ILU_PENDING = 0x7FF00000000000A5ull;
constexpr unsigned long long ILU_QNAN = 0x7FF8000000000000ull;
// Wall-clock ticks (s_memrealtime, 100 MHz) one wait may take before it counts as
// lost, far beyond any legitimate wait (a whole solve takes a few ms): err is then set
// and the workgroup leaves, and every wave still waiting does within 256 further
// tries, so the launch always ends.
constexpr long long ILU_WAIT_TICKS = 200000000;

__device__ inline unsigned long long ilu_ld(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned ilu_ld32(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void ilu_st(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v == ILU_PENDING ? ILU_QNAN : v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Marks nw 64-bit words of a solve's output pending and resets the two claim
// counters (ctl[0] and ctl[1]) of the solves that follow.
__global__ void k_ilu_pending(unsigned long long* __restrict__ w, long long nw, unsigned* __restrict__ ctl,
                              const int* done) {
  if (done && *(volatile const int*)done) return;
  if (blockIdx.x == 0 && threadIdx.x < 2) ctl[threadIdx.x] = 0;
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < nw; k += (long long)gridDim.x * blockDim.x)
    w[k] = ILU_PENDING;
}

// Entries of a row that are packed in solve order (coalesced): the first ILU_W, those of
// the ring first; further ones come from the factor matrix.
constexpr int ILU_W = 4;
// Threads of a block's workgroup, and its compute waves; the other waves load.
template <int BS>
constexpr int ilu_threads() { return BS == 1 ? 1024 : 512; }
template <int BS>
constexpr int ilu_compute() { return BS == 1 ? 4 : 2; }
constexpr int ILU_MAX_SLOTS = 32;
constexpr int ILU_LOOK = 10;   // chunks ahead of the last one done whose loaders look in memory (3: 46, 6: 32.3, 10: 30.8 ms a 96^3 solve)

// The rows of one solve in solve order.  lv: {i, q0, q1, mask}, [q0, q1) the entries left
// (lower solve) or right of the diagonal of row i; bit k of mask: entry q0 + k is packed
// (all of them, and mask 0, where there are at most w).  pc, pv: the packed entries, entry
// u (element e) of position t at pc[u m + t], pv[(u B2 + e) m + t]; pc: -1 none, >= 0 the
// position of its value, read from memory, else -2 - its position, read from the ring.
// pd (solves with a diagonal): its value, or the inverse block, element e at pd[e m + t].
// Chunk c takes positions cstart[c] .. cstart[c + 1], block b chunks bchunk[b] .. bchunk[b + 1].
// src: where the right-hand side of a position stands in the solve's input; pos: the position
// of every row.
template <class V>
struct IluRows {
  int4* lv = nullptr;
  int* src = nullptr;
  int* pos = nullptr;
  int* pc = nullptr;
  V* pv = nullptr;
  V* pd = nullptr;
  int* cstart = nullptr;
  int* bchunk = nullptr;
  int w = 0;
};

// How a block's workgroup uses its LDS.
struct IluLds {
  int ring = 0;    // places of the ring, a power of two
  int slots = 0;
  int safe = 0;    // largest distance of a value read from the ring
  size_t bytes = 0;
  int room = 0;    // bytes that a workgroup may have
};
// 64-bit words of a slot for entries of b2 values of `words` words: the row's partial
// sums, its w entries, its diagonal (scalars: and the reciprocal), then w + 2 ints a lane.
__host__ __device__ constexpr int ilu_slot_words(int bs, int words, int w) {
  return WAVE * words * (bs + w * bs * bs + (bs == 1 ? 2 : bs * bs)) + WAVE / 2 * (w + 2);
}

// The position of every row, and src: the rows themselves (before null) or their positions
// in the solve before, whose output is this one's input.
__global__ void k_ilu_positions(const int4* __restrict__ lv, int m, int* __restrict__ pos, const int* before,
                                int* __restrict__ src) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < m; t += gridDim.x * blockDim.x) {
    const int i = lv[t].x;
    pos[i] = t;
    src[t] = before ? before[i] : i;
  }
}

template <class V, int BS>
__global__ void k_ilu_pack(const int* __restrict__ ci, const V* __restrict__ val, const V* __restrict__ dinv,
                           IluRows<V> p, int m, int block, int safe, bool lower) {
  constexpr int B2 = BS * BS;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < m; t += gridDim.x * blockDim.x) {
    const int4 rw = p.lv[t];
    int u = 0;
    unsigned mask = 0;
    for (int near = 1; near >= 0; --near)
      for (int q = rw.y; q < rw.z && u < p.w; ++q) {
        const int tj = p.pos[ci[q]];
        const bool ring = tj / block == t / block && t - tj <= safe;
        if (ring != (near == 1) || (rw.z - rw.y > p.w && q - rw.y > 30)) continue;
        p.pc[(size_t)u * m + t] = ring ? -2 - tj : tj;
        for (int e = 0; e < B2; ++e) p.pv[((size_t)u * B2 + e) * m + t] = val[(size_t)B2 * q + e];
        if (q - rw.y <= 30) mask |= 1u << (q - rw.y);
        ++u;
      }
    for (; u < p.w; ++u) {
      p.pc[(size_t)u * m + t] = -1;
      for (int e = 0; e < B2; ++e) p.pv[((size_t)u * B2 + e) * m + t] = zero<V>();
    }
    p.lv[t].w = rw.z - rw.y > p.w ? (int)mask : 0;
    if (p.pd)
      for (int e = 0; e < B2; ++e)
        p.pd[(size_t)e * m + t] = BS == 1 ? val[lower ? rw.z : rw.y - 1] : dinv[(size_t)B2 * rw.x + e];
  }
}

// s / d where 1 / d was computed beforehand: the product and one correction, which
// rounds as the division does; where that leaves the range, the division itself.  It
// takes the division's chain (some 250 cycles) out of the chain of dependent rows.
__device__ inline double ilu_div(double s, double d, double rd) {
  double q = s * rd;
  q = fma(fma(-d, q, s), rd, q);
  if (!finite(q) || !(fabs(d) > 1e-290 && fabs(d) < 1e290)) q = s / d;
  return q;
}
__device__ inline cplx<double> ilu_div(cplx<double> s, cplx<double> d, cplx<double> rd) {
  cplx<double> q = s * rd;
  q = axpy(q, axpy(s, -d, q), rd);
  const double m = fmax(fabs(d.re), fabs(d.im));
  if (!finite(q) || !(m > 1e-140 && m < 1e140)) q = s / d;
  return q;
}

// One triangular solve with a factor matrix: LOWER: y_i = x_i - sum_{stored j < i}
// a_ij y_j, else with the stored j > i; UNIT: that value is y_i, else y_i = a_ii^{-1}
// (value) (a division for scalars, the stored inverse block for 3x3 blocks).  The entries
// read from memory are subtracted first, then those of the ring, each in entry order.
// Workgroup k of the claim order takes block k: positions k block, .. of `rows`.
// xch: y in solve order, which the workgroups exchange; it must hold the pending mark
// (k_ilu_pending).  In solve order the rows of a chunk, and those that they read, stand next
// to each other (on a grid): in row order each of a chunk's stores and far loads touched 64
// lines, which bounded the rows a workgroup could take.  in: x, at rows.src.  out: y in row
// order, or null.  next: the xch of the solve that follows, marked pending here, or null.
// tick: this solve's claim counter, 0 at launch; err: set to 1 when a
// wait ran past its bound; max_tries: tries of one wait before it counts as lost regardless
// of time (~0u: no such limit; a small value forces that path in tests).  done: the
// solve's done flag (the launch returns at once when it is set), or null.
template <class V, int BS, bool LOWER, bool UNIT>
__global__ __launch_bounds__((ilu_threads<BS>())) void k_ilu_solve_block(
    const int* __restrict__ ci, const V* __restrict__ val, IluRows<V> rows, int m, int block, IluLds lds,
    const V* __restrict__ in, V* xch, V* out, V* next, unsigned* tick, unsigned* err, unsigned max_tries, const int* done) {
  constexpr int B2 = BS * BS;
  constexpr int W = sizeof(V) / 8;   // 64-bit words per value (1 real, 2 complex)
  constexpr int CW = ilu_compute<BS>(), NL = ilu_threads<BS>() / WAVE - CW;
  using U = unsigned long long;
  static_assert(sizeof(V) == 8 * W, "fp64 values only");
  static_assert(NL <= WAVE, "a lane looks at a chunk each");
  extern __shared__ U sm[];          // the ring, then the slots
  __shared__ int ready[ILU_MAX_SLOTS], finished[ILU_MAX_SLOTS];   // chunk + 1 (of the block) a slot holds / held
  __shared__ int claimed, dead, front;   // front: a chunk done lately, at most CW before the last
  if (done && *(volatile const int*)done) return;
  if (threadIdx.x == 0) {
    claimed = (int)atomicAdd(tick, 1u);
    dead = 0;
    front = -1;
  }
  if (threadIdx.x < ILU_MAX_SLOTS) ready[threadIdx.x] = finished[threadIdx.x] = 0;
  const int ring_words = lds.ring * BS * W;
  for (int w = threadIdx.x; w < ring_words; w += ilu_threads<BS>()) sm[w] = ILU_PENDING;
  __syncthreads();
  const int k = claimed;
  const int b0 = k * block;          // < m: the grid has as many workgroups as blocks
  const int lane = threadIdx.x & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int c0 = rows.bchunk[k], nc = rows.bchunk[k + 1] - c0;
  const int ns = lds.slots, w_ = rows.w, mask_ring = lds.ring - 1;
  const int slot_words = ilu_slot_words(BS, W, w_);
  // fields of a slot: word f of lane l at f 64 + l
  const int f_a = BS * W, f_d = f_a + w_ * B2 * W, f_i = f_d + (BS == 1 ? 2 : B2) * W;
  U* ow = reinterpret_cast<U*>(xch);
  // The LDS runs a wave's accesses in the order they are issued, so flags order the words
  // around them as long as the compiler keeps that order too.  (Acquire and release at
  // workgroup scope would also wait for the stores to memory, about 1 us a chunk.)
  auto order = [] { asm volatile("" ::: "memory"); };
  auto ld = [](const auto* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto put = [&](U* f, const auto& v) {   // a value's words into fields of a slot
    U t[sizeof(v) / 8];
    __builtin_memcpy(t, &v, sizeof(v));
#pragma unroll
    for (int e = 0; e < (int)(sizeof(v) / 8); ++e) f[e * WAVE + lane] = t[e];
  };
  auto get = [&](const U* f, auto& v) {
    U t[sizeof(v) / 8];
#pragma unroll
    for (int e = 0; e < (int)(sizeof(v) / 8); ++e) t[e] = f[e * WAVE + lane];
    __builtin_memcpy(&v, t, sizeof(v));
  };
  // Bounded waits: called once a try by the whole wave, true when the wave should leave:
  // after ILU_WAIT_TICKS, once another wave has (looked at every 256 tries), or after
  // max_tries tries.
  struct Wait {
    unsigned tries = 0;
    long long t0 = 0;
  };
  auto give_up = [&](Wait& wt) {
    ++wt.tries;
    if (wt.tries < max_tries) {
      if ((wt.tries & 15u) == 0 && ld(&dead)) return true;
      if (wt.tries & 255u) return false;
      const long long now = wall_clock64();
      if (wt.tries == 256) wt.t0 = now;
      if (now - wt.t0 <= ILU_WAIT_TICKS && ilu_ld32(err) == 0) return false;
    }
    if (lane == 0) {
      atomicOr(err, 1u);
      __hip_atomic_store(&dead, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return true;
  };

  if (wave < CW) {
    // ---- compute
    __builtin_amdgcn_s_setprio(2);
    // no load is outstanding in the loop below, so nothing in it waits for its stores
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    // What a chunk's slot holds; 3x3 entries are read where they are used.
    struct Row {
      int i, t, at[ILU_W];       // i: -1 no row; t: its position in the block
      V s[BS], a[BS == 1 ? ILU_W : 1], dg, rd;
    };
    auto read_slot = [&](int x, Row& r) {
      const U* f = sm + ring_words + (size_t)(x % ns) * slot_words;
      const int* fi = reinterpret_cast<const int*>(f + f_i * WAVE);
#pragma unroll
      for (int e = 0; e < BS; ++e) get(f + e * W * WAVE, r.s[e]);
      r.i = fi[w_ * WAVE + lane];
      r.t = fi[(w_ + 1) * WAVE + lane];
#pragma unroll
      for (int u = 0; u < ILU_W; ++u) {
        r.at[u] = u < w_ ? fi[u * WAVE + lane] : -1;
        if constexpr (BS == 1) {
          r.a[u] = zero<V>();
          if (u < w_) get(f + (f_a + u * W) * WAVE, r.a[u]);
        }
      }
      if constexpr (BS == 1 && !UNIT) {
        get(f + f_d * WAVE, r.dg);
        get(f + (f_d + W) * WAVE, r.rd);
      }
    };
    for (int x = wave; x < nc; x += CW) {
      const int sl = x % ns;
      Wait wt;
      while (ld(&ready[sl]) != x + 1)
        if (give_up(wt)) return;
      order();
      Row row;
      read_slot(x, row);
      const U* f = sm + ring_words + (size_t)sl * slot_words;
      // the values of this block; 0 where there is no entry
      V xv[ILU_W][BS] = {};
      wt = Wait{};
      for (;;) {
        U xw[ILU_W][BS * W];
#pragma unroll
        for (int u = 0; u < ILU_W; ++u)
#pragma unroll
          for (int e = 0; e < BS * W; ++e) xw[u][e] = u < w_ ? ld(sm + max(row.at[u], 0) + e) : 0ull;
        bool pend = false;
#pragma unroll
        for (int u = 0; u < ILU_W; ++u)
#pragma unroll
          for (int e = 0; e < BS * W; ++e) {
            pend |= row.at[u] >= 0 && xw[u][e] == ILU_PENDING;
            xw[u][e] = row.at[u] >= 0 ? xw[u][e] : 0ull;
          }
        if (!__any(pend)) {
#pragma unroll
          for (int u = 0; u < ILU_W; ++u) __builtin_memcpy(xv[u], xw[u], sizeof(xv[u]));
          break;
        }
        if (give_up(wt)) return;
      }
      V s[BS];
#pragma unroll
      for (int e = 0; e < BS; ++e) s[e] = row.s[e];
      if constexpr (BS == 1) {
#pragma unroll
        for (int u = 0; u < ILU_W; ++u) s[0] = s[0] - axpy(zero<V>(), row.a[u], xv[u][0]);   // a 0 without an entry
      } else {
#pragma unroll
        for (int u = 0; u < ILU_W; ++u)
          if (row.at[u] >= 0) {
            V a[B2];
#pragma unroll
            for (int e = 0; e < B2; ++e) get(f + (f_a + (u * B2 + e) * W) * WAVE, a[e]);
#pragma unroll
            for (int r = 0; r < BS; ++r) {
              V acc = zero<V>();
#pragma unroll
              for (int e = 0; e < BS; ++e) acc = axpy(acc, a[BS * r + e], xv[u][e]);
              s[r] = s[r] - acc;
            }
          }
      }
      V o[BS];
      if constexpr (UNIT) {
#pragma unroll
        for (int e = 0; e < BS; ++e) o[e] = s[e];
      } else if constexpr (BS == 1) {
        o[0] = ilu_div(s[0], row.dg, row.rd);
      } else {
#pragma unroll
        for (int r = 0; r < BS; ++r) {
          V acc = zero<V>();
#pragma unroll
          for (int e = 0; e < BS; ++e) {
            V d;
            get(f + (f_d + (BS * r + e) * W) * WAVE, d);
            acc = axpy(acc, d, s[e]);
          }
          o[r] = acc;
        }
      }
      U ww[BS * W];
      __builtin_memcpy(ww, o, sizeof(o));
      if (row.i >= 0) {
        U* r = sm + (size_t)(row.t & mask_ring) * (BS * W);
#pragma unroll
        for (int e = 0; e < BS * W; ++e)
          __hip_atomic_store(r + e, ww[e] == ILU_PENDING ? ILU_QNAN : ww[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const size_t t = (size_t)BS * (b0 + row.t);
#pragma unroll
        for (int e = 0; e < BS * W; ++e) ilu_st(ow + W * t + e, ww[e]);
        if (out) {
#pragma unroll
          for (int e = 0; e < BS; ++e) out[(size_t)BS * row.i + e] = o[e];
        }
      }
      order();
      if (lane == 0) {
        __hip_atomic_store(&finished[sl], x + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&front, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    return;
  }

  // ---- load
  // A chunk's records, loaded one chunk of this wave ahead.
  struct Rec {
    int t0, n, p0, pn;   // its positions, and those of the chunk whose places are marked again
    int4 rw;
    int src, c[ILU_W];
    V a[ILU_W][B2];
    V dg[UNIT ? 1 : B2];
  };
  auto load_rec = [&](int x, Rec& r) {
    r.t0 = rows.cstart[c0 + x];
    r.n = rows.cstart[c0 + x + 1] - r.t0;
    r.p0 = x + ns < nc ? rows.cstart[c0 + x + ns] : 0;
    r.pn = x + ns < nc ? rows.cstart[c0 + x + ns + 1] - r.p0 : 0;
    const bool on = lane < r.n;
    const int t = r.t0 + (on ? lane : 0);
    r.rw = rows.lv[t];
    r.src = rows.src[t];
#pragma unroll
    for (int u = 0; u < ILU_W; ++u) {
      r.c[u] = -1;
      if (u < w_) {
        r.c[u] = on ? rows.pc[(size_t)u * m + t] : -1;
#pragma unroll
        for (int e = 0; e < B2; ++e) r.a[u][e] = rows.pv[((size_t)u * B2 + e) * m + t];
      }
    }
    if constexpr (!UNIT) {
#pragma unroll
      for (int e = 0; e < B2; ++e) r.dg[e] = rows.pd[(size_t)e * m + t];
    }
  };
  Rec rec, ahead;
  if (wave - CW < nc) load_rec(wave - CW, rec);
  for (int x = wave - CW; x < nc; x += NL, rec = ahead) {
    if (x + NL < nc) load_rec(x + NL, ahead);
    const int n = rec.n, p0 = rec.p0, pn = rec.pn;
    const bool on = lane < n;
    const int t = rec.t0 + (on ? lane : 0);
    const int4 rw = rec.rw;
    auto& c = rec.c;
    auto& a = rec.a;
    auto& dg = rec.dg;
    V s[BS];
#pragma unroll
    for (int e = 0; e < BS; ++e) s[e] = in[(size_t)BS * rec.src + e];
    if (on && next) {
      U* nw = reinterpret_cast<U*>(next) + (size_t)BS * W * t;
#pragma unroll
      for (int e = 0; e < BS * W; ++e) nw[e] = ILU_PENDING;
    }
    // the slot, once all chunks up to x - ns are done: all but the row's partial sums
    Wait wt;
    for (;;) {
      const int y = x - ns - lane;
      const bool wait = lane < NL && y >= 0 &&
                        ld(&finished[y >= 0 ? y % ns : 0]) < y + 1;
      if (!__any(wait)) break;
      if (give_up(wt)) return;
      __builtin_amdgcn_s_sleep(1);
    }
    order();
    if (lane < pn) {
      U* r = sm + (size_t)((p0 + lane - b0) & mask_ring) * (BS * W);
#pragma unroll
      for (int e = 0; e < BS * W; ++e) r[e] = ILU_PENDING;
    }
    const int sl = x % ns;
    U* f = sm + ring_words + (size_t)sl * slot_words;
    int* fi = reinterpret_cast<int*>(f + f_i * WAVE);
#pragma unroll
    for (int u = 0; u < ILU_W; ++u)
      if (u < w_) {
#pragma unroll
        for (int e = 0; e < B2; ++e)   // one subtracted here is not in the row's rest (an infinite one times 0 would be)
          put(f + (f_a + (u * B2 + e) * W) * WAVE, BS == 1 && c[u] >= 0 ? zero<V>() : a[u][e]);
        fi[u * WAVE + lane] = c[u] < -1 ? ((-2 - c[u] - b0) & mask_ring) * (BS * W) : -1;
      }
    if constexpr (!UNIT) {
#pragma unroll
      for (int e = 0; e < B2; ++e) put(f + (f_d + e * W) * WAVE, dg[e]);
      if constexpr (BS == 1) put(f + (f_d + W) * WAVE, from_real<V>(1.0) / dg[0]);
    }
    fi[w_ * WAVE + lane] = on ? rw.x : -1;
    fi[(w_ + 1) * WAVE + lane] = t - b0;
    // the values read from memory (of other blocks, or solved long ago); true once come
    auto fetch = [&](int at, V (&v)[BS]) {
      U xw[BS * W];
#pragma unroll
      for (int e = 0; e < BS * W; ++e) xw[e] = ilu_ld(ow + (size_t)BS * W * at + e);
      bool ok = true;
#pragma unroll
      for (int e = 0; e < BS * W; ++e) ok &= xw[e] != ILU_PENDING;
      __builtin_memcpy(v, xw, sizeof(xw));
      return ok;
    };
    auto subtract = [&](const V* au, const V (&v)[BS]) {
#pragma unroll
      for (int r = 0; r < BS; ++r) {
        V acc = zero<V>();
#pragma unroll
        for (int e = 0; e < BS; ++e) acc = axpy(acc, au[BS * r + e], v[e]);
        s[r] = s[r] - acc;
      }
    };
    wt = Wait{};
    // Waits until the value at position `at` (-1: no need) has come in every lane that needs it.  Only the
    // loaders of the next ILU_LOOK chunks look in memory: with all of them looking, the lines
    // that the waiting waves move hold up the stores they wait for.
    auto arrive = [&](int at, V (&v)[BS]) {
      bool miss = at >= 0;
      for (;;) {
        if (miss && fetch(at, v)) miss = false;
        if (!__any(miss)) return true;
        do {
          if (give_up(wt)) return false;
          __builtin_amdgcn_s_sleep(1);
        } while (x > ld(&front) + ILU_LOOK);
      }
    };
#pragma unroll
    for (int u = 0; u < ILU_W; ++u)
      if (u < w_ && __any(c[u] >= 0)) {
        V v[BS];
        if (!arrive(c[u], v)) return;
        if (c[u] >= 0) subtract(a[u], v);
      }
    // entries that are not packed
    const bool more = on && rw.w != 0;
    if (__any(more)) {
      const int len = more ? rw.z - rw.y : 0;
      for (int q = 0; __any(q < len); ++q) {
        const bool take = q < len && !(q <= 30 && ((unsigned)rw.w >> q & 1u));
        V v[BS];
        if (!__any(take)) continue;
        if (!arrive(take ? rows.pos[ci[rw.y + q]] : -1, v)) return;
        if (take) subtract(val + (size_t)B2 * (rw.y + q), v);
      }
    }
#pragma unroll
    for (int e = 0; e < BS; ++e) put(f + e * W * WAVE, s[e]);
    order();
    if (lane == 0) __hip_atomic_store(&ready[sl], x + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// ---- one launch per triangular solve, rows dealt out one level after the other -----
//
// For patterns that blocks of consecutive rows do not suit: entries that mostly lead
// into other blocks, or rows longer than what is packed, whose values would all come
// through memory to one workgroup.  Here the rows of the whole solve go through one
// launch in level order: each wave claims the next 64 positions from a counter, so
// every position below a claimed one is claimed too, by a wave that is running, and
// every link of the chain is a store to and a load from memory, 1.5 to 2.1 us.  The
// lowest position still waiting reads only finished rows, so the solve always moves on;
// a wave whose lanes wait on each other (a level boundary inside its 64 positions)
// retries its pending lanes together, so a finished lane stores before the others test
// again.

// One group of (at most) 4 entries of a row: loads the solved values they
// reference (entries at u >= cnt repeat the last one, unused) and, when none
// is pending, subtracts a_u x_u from s in entry order.  Returns false, leaving
// s as it was, while one is pending; *waitw then holds the address of a
// pending word.
template <class V, int BS>
__device__ inline bool ilu_group(const V (&a)[4][BS * BS], const int (&c)[4], int cnt, unsigned long long* ow,
                                 V (&s)[BS], unsigned long long** waitw) {
  constexpr int W = sizeof(V) / 8;
  using U = unsigned long long;
  U xw[4][BS * W];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int k = 0; k < BS * W; ++k) xw[u][k] = ilu_ld(ow + (size_t)BS * W * c[u] + k);
  bool ready = true;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int k = 0; k < BS * W; ++k)
      if (xw[u][k] == ILU_PENDING) {
        ready = false;
        *waitw = ow + (size_t)BS * W * c[u] + k;
      }
  if (!ready) return false;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < cnt) {
      V xv[BS];
#pragma unroll
      for (int e = 0; e < BS; ++e) __builtin_memcpy(&xv[e], &xw[u][W * e], sizeof(V));
#pragma unroll
      for (int r = 0; r < BS; ++r) {
        V acc = zero<V>();
#pragma unroll
        for (int k = 0; k < BS; ++k) acc = axpy(acc, a[u][BS * r + k], xv[k]);
        s[r] = s[r] - acc;
      }
    }
  return true;
}

// One triangular solve with a factor matrix, the same arithmetic as one
// launch per level (the same entries in the same order): LOWER: out_i = in_i -
// sum_{stored j < i} a_ij out_j, else with the stored j > i; UNIT: that value is
// out_i, else out_i = a_ii^{-1} (value) (a division for scalars, the stored
// inverse block dinv for 3x3 blocks).  lv: all m rows in level order, {i, q0,
// q1, 0} with [q0, q1) the entries left (LOWER) or right of the diagonal.  out
// must hold the pending mark (k_ilu_pending) and may not overlap in.  next: the
// output of the solve that follows, or null: row i of it is marked pending
// once in_i is read (so next may be in).  tick: this solve's claim counter, 0
// at launch; err: set to 1 when a wait ran past its bound; max_tries: tries of
// one row before it gives up regardless of time (~0u: no such limit; a small
// value forces the give-up path in tests).  done: the solve's done flag (the
// launch returns at once when it is set), or null.
template <class V, int BS, bool LOWER, bool UNIT>
__global__ __launch_bounds__(WAVE) void k_ilu_solve_sweep(const int* __restrict__ ci, const V* __restrict__ val,
                                                          const V* __restrict__ dinv, const int4* __restrict__ lv,
                                                          int m, const V* in, V* out, V* next, unsigned* tick,
                                                          unsigned* err, unsigned max_tries, const int* done) {
  constexpr int B2 = BS * BS;
  constexpr int W = sizeof(V) / 8;   // 64-bit words per value (1 real, 2 complex)
  using U = unsigned long long;
  static_assert(sizeof(V) == 8 * W, "fp64 values only");
  if (done && *(volatile const int*)done) return;
  const int lane = threadIdx.x & (WAVE - 1);
  U* ow = reinterpret_cast<U*>(out);
  for (;;) {
    unsigned base = 0;
    if (lane == 0) base = atomicAdd(tick, (unsigned)WAVE);
    base = __shfl(base, 0, WAVE);
    if (base >= (unsigned)m) return;
    const int t = (int)base + lane;
    bool pending = t < m;
    int4 rw = make_int4(0, 0, 0, 0);
    if (pending) rw = lv[t];
    const int i = rw.x, q0 = rw.y, q1 = rw.z;
    V s0[BS];
#pragma unroll
    for (int e = 0; e < BS; ++e) s0[e] = pending ? in[(size_t)BS * i + e] : zero<V>();
    if (pending && next) {
      U* nw = reinterpret_cast<U*>(next) + (size_t)BS * W * i;
#pragma unroll
      for (int k = 0; k < BS * W; ++k) nw[k] = ILU_PENDING;
    }
    // the first (at most) 4 entries, held in registers across the tries: most rows
    // have no more, and a try then reloads only the solved values they reference
    int c0[4];
    V a0[4][B2];
    const bool has0 = pending && q0 < q1;
    if (has0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + u < q1 ? q0 + u : q1 - 1;
        c0[u] = ci[q];
#pragma unroll
        for (int e = 0; e < B2; ++e) a0[u][e] = val[(size_t)B2 * q + e];
      }
    }
    // the diagonal (block) inverse's operand, off the waiting path
    V dg[UNIT ? 1 : (BS == 1 ? 1 : B2)];
    if constexpr (!UNIT) {
      if (pending) {
        if constexpr (BS == 1) {
          dg[0] = val[LOWER ? q1 : q0 - 1];
        } else {
#pragma unroll
          for (int e = 0; e < B2; ++e) dg[e] = dinv[(size_t)B2 * i + e];
        }
      }
    }
    const long long t_start = wall_clock64();
    unsigned tries = 0;
    U* waitw = nullptr;   // a word the last try found pending: polled alone first
    while (__any(pending)) {
      if (pending) {
        V s[BS];
#pragma unroll
        for (int e = 0; e < BS; ++e) s[e] = s0[e];
        bool ready = !waitw || ilu_ld(waitw) != ILU_PENDING;
        if (ready) waitw = nullptr;
        if (ready && has0) ready = ilu_group<V, BS>(a0, c0, q1 - q0, ow, s, &waitw);
        // further entries in groups of 4, loaded again on every try
        for (int q4 = q0 + 4; q4 < q1 && ready; q4 += 4) {
          int c[4];
          V a[4][B2];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int q = q4 + u < q1 ? q4 + u : q1 - 1;
            c[u] = ci[q];
#pragma unroll
            for (int e = 0; e < B2; ++e) a[u][e] = val[(size_t)B2 * q + e];
          }
          ready = ilu_group<V, BS>(a, c, q1 - q4, ow, s, &waitw);
        }
        // give up on this row after ILU_WAIT_TICKS, or once another row has (err), both
        // read every 256 tries, or after max_tries tries
        bool lost = false;
        if (!ready) {
          ++tries;
          lost = tries >= max_tries ||
                 ((tries & 255u) == 0 && (wall_clock64() - t_start > ILU_WAIT_TICKS ||
                                          __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0));
          if (lost) atomicOr(err, 1u);
        }
        if (ready || lost) {
          U ww[BS * W];
          if (lost) {
#pragma unroll
            for (int k = 0; k < BS * W; ++k) ww[k] = ILU_QNAN;
          } else {
            V o[BS];
            if constexpr (UNIT) {
#pragma unroll
              for (int e = 0; e < BS; ++e) o[e] = s[e];
            } else if constexpr (BS == 1) {
              o[0] = s[0] / dg[0];
            } else {
#pragma unroll
              for (int r = 0; r < BS; ++r) {
                V acc = zero<V>();
#pragma unroll
                for (int k = 0; k < BS; ++k) acc = axpy(acc, dg[BS * r + k], s[k]);
                o[r] = acc;
              }
            }
            __builtin_memcpy(ww, o, sizeof(o));
          }
#pragma unroll
          for (int k = 0; k < BS * W; ++k) ilu_st(ow + (size_t)BS * W * i + k, ww[k]);
          pending = false;
        }
      }
      if (__any(pending)) __builtin_amdgcn_s_sleep(8);
    }
  }
}

// y = U x (the diagonal (block) and right of it) or y = L x (unit diagonal and
// left of it) of the factor matrix, every (block) row independently: the
// forward map y_0 = M x_0 = L (U x_0).
template <class V, int BS, bool LOWER>
__global__ void k_ilu_tri_matvec(const int* __restrict__ rp, const int* __restrict__ ci, const V* __restrict__ val,
                                 const int* __restrict__ dpos, int nbrows, const V* __restrict__ x,
                                 V* __restrict__ y) {
  constexpr int B2 = BS * BS;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nbrows; i += gridDim.x * blockDim.x) {
    const int qd = dpos[i];
    const int q0 = LOWER ? rp[i] : qd;
    const int q1 = LOWER ? qd : rp[i + 1];
    V s[BS];
#pragma unroll
    for (int e = 0; e < BS; ++e) s[e] = LOWER ? x[(size_t)BS * i + e] : zero<V>();
    for (int q = q0; q < q1; ++q) {
      const V* a = val + (size_t)B2 * q;
      const V* xc = x + (size_t)BS * ci[q];
#pragma unroll
      for (int r = 0; r < BS; ++r)
#pragma unroll
        for (int k = 0; k < BS; ++k) s[r] = axpy(s[r], a[BS * r + k], xc[k]);
    }
#pragma unroll
    for (int e = 0; e < BS; ++e) y[(size_t)BS * i + e] = s[e];
  }
}

}  // namespace mlb
