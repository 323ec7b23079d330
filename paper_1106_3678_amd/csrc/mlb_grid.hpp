// Whole solves in one launch, a group of workgroups per system.
//
// A system of up to a few hundred thousand rows is bound by launch latency on
// the multi-launch path: an inner step is seven dependent launches of 3-5 us
// each, whatever N is.  Here a group of P workgroups runs the whole of
// Algorithm 7.1 (M = I, or A M^{-1} formed beforehand) for one system: the same
// passes, coefficient recurrences and exits as the multi-launch path.  Each
// workgroup owns a contiguous slice of rows and keeps it for the whole solve,
// so every vector pass reads and writes its own slice only (ordinary cached
// accesses).  Two things cross workgroups:
//  * inner products: every workgroup stores its partial sums into a slot, reads
//    the slots of all P (each wave one sum) and runs the coefficient recurrence
//    on its own copy of the scalar state in LDS.  All copies see the same sums,
//    added in the same order, so they stay equal and every workgroup takes the
//    same exits.
//  * the vector a product with A gathers from: the rows of the own slice come
//    from LDS, the others from an exchange buffer.
// Both use the scheme of the one-launch triangular solves: every 64-bit (fp32:
// 32-bit) word is first marked pending with a signalling-NaN pattern that no
// arithmetic returns, stored and read with agent-scope relaxed atomics (which
// are coherent across the XCDs' L2 caches), and is its own completion flag: no
// cache is written back or invalidated, and one store and one load are all the
// latency of a reduction or an exchange.
// Words are marked pending again once everybody has read them:
//  * slots: phase q uses ring position q mod 4.  A workgroup all of whose waves
//    have read their sums of phase q + 1 knows that everybody has finished
//    reading phase q (they published q + 1 afterwards) and marks its words of
//    phase q; it waits for its outstanding stores before it publishes phase
//    q + 2, so a reader that has passed q + 3 finds them pending, or the new
//    ones of q + 4.
//  * exchange buffers alternate: the rows of exchange e are marked once the
//    reduction after its product has been read, and used again by e + 2.
// The workgroups of a group must all be running.  Logical workgroup numbers are
// claimed from a counter, so those of the lowest unfinished group are; a gate at
// the start counts the group's arrivals, and if they are not complete within
// entry_ticks the group leaves without having written anything but marks
// (the host starts it again).  Every later wait is bounded by GRID_WAIT_TICKS:
// then the group's err word is set, everybody in it leaves, and the host
// reports an error.
#pragma once

#include "mlb_kernels.hpp"
#include "mlb_spmv.hpp"

namespace mlb {

constexpr int GB = 512;                 // threads of a workgroup (8 waves)
constexpr int GRID_RING = 4;            // slot sets in use by consecutive reductions
constexpr int GRID_MAX_P = 256;         // workgroups of one system, at most
// Wall-clock ticks (s_memrealtime, 100 MHz)
constexpr long long GRID_ENTRY_TICKS = 20000000;    // 0.2 s for the group to be complete
constexpr long long GRID_WAIT_TICKS = 200000000;    // 2 s for any word, far beyond a legitimate wait
// Rows of a workgroup's slice, at most: two LDS copies of a slice (64 KB of the CU's 160)
template <class V>
constexpr int grid_max_rows() { return sizeof(V) > 8 ? 2048 : 4096; }

// words of the state's ctl
enum { GRID_ARRIVED = 0, GRID_GATE = 1, GRID_ERR = 2 };
enum { GATE_CLOSED = 0, GATE_OPEN = 1, GATE_LEFT = 2 };

// What the host reads after a solve.
struct GridOut {
  int status;         // 0: the group left at its gate, 1: done, 2: a wait was lost
  int lost;           // a workgroup lost a wait: after the last sums were out, too, when the first has its result
  int flag;
  long long iter;
  double err;
  double rr, bb;      // ||b - A x||^2 and ||b||^2, if asked for
  long long setup_ticks;
};

template <class V, class Sc>
struct GridJob {
  int N = 0, n = 0;
  int P = 1, R = 0;           // workgroups and rows per workgroup: P = ceil(N / R)
  const int* rp = nullptr;    // A (CSR, or BSR3 block rows)
  const int* ci = nullptr;
  const V* val = nullptr;
  const int* rpT = nullptr;   // A^H
  const int* ciT = nullptr;
  const V* valT = nullptr;
  const V* b = nullptr;
  V* x = nullptr;
  const V* Q = nullptr;
  long long ldq = 0;
  V *G = nullptr, *W = nullptr, *F = nullptr;   // N x n, N x n, N x (n-1); ld = N
  V* r = nullptr;
  V* xb = nullptr;            // two exchange buffers of N values each
  V* xb1 = nullptr;
  Sc* slots = nullptr;        // partial sums: GRID_RING x copies x P x grid_slot words
  State<Sc>* st = nullptr;    // receives the final state; holds the group's ctl words
  GridOut* out = nullptr;
  V* xrec = nullptr;          // iterate record: x_k in column k-1, k <= K (or null)
  long long K = 0;
  double tol = 0, kappa = 0;
  long long maxit = 0;
  long long stag_window = 0;
  int tf = 0;                 // transpose-free inner steps (rpT, ciT, valT and F unused)
  long long entry_ticks = GRID_ENTRY_TICKS;
  unsigned max_tries = ~0u;   // tries of one wait before it counts as lost whatever the time (for tests)
  int resid = 0;              // also ||b - A x||^2 and ||b||^2 into the state's aux
};

template <class R> struct grid_word;
template <> struct grid_word<double> {
  using U = unsigned long long;
  static constexpr U pending = 0x7FF00000000000A5ull, qnan = 0x7FF8000000000000ull;
};
template <> struct grid_word<float> {
  using U = unsigned;
  static constexpr U pending = 0x7F8000A5u, qnan = 0x7FC00000u;
};

// Marks the exchange buffers and slots of every job pending and clears its ctl
// words, before k_grid.  use_one: the only job is `one`, stored in jobs[0].
template <class V, class Sc>
__global__ __launch_bounds__(BLOCK) void k_grid_init(GridJob<V, Sc>* jobs, GridJob<V, Sc> one, int use_one,
                                                     int slot_words, unsigned* tick) {
  using Wd = grid_word<typename traits<V>::real>;
  using U = typename Wd::U;
  const GridJob<V, Sc> J = use_one ? one : jobs[blockIdx.y];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (use_one) jobs[0] = one;
    for (int k = 0; k < 3; ++k) J.st->ctl[k] = 0;
    J.out->status = 0;
    J.out->lost = 0;
    if (blockIdx.y == 0) *tick = 0;
  }
  if (J.P == 1) return;
  const int stride = gridDim.x * BLOCK, t0 = blockIdx.x * BLOCK + threadIdx.x;
  U* a = reinterpret_cast<U*>(J.xb);
  U* b = reinterpret_cast<U*>(J.xb1);
  const long long nw = (long long)J.N * (long long)(sizeof(V) / sizeof(U));
  for (long long k = t0; k < nw; k += stride) {
    a[k] = Wd::pending;
    b[k] = Wd::pending;
  }
  unsigned long long* s = reinterpret_cast<unsigned long long*>(J.slots);
  const long long ns = (long long)slot_words * J.P;
  for (long long k = t0; k < ns; k += stride) s[k] = grid_word<double>::pending;
}

template <class U>
__device__ inline U grid_ld(const U* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class U>
__device__ inline void grid_st(U* p, U v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until this wave's stores have reached memory.
__device__ inline void grid_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A DPP move (VALU only): lanes without a source get 0.
template <int CTRL>
__device__ inline float dpp0_(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline double dpp0_(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL, class R>
__device__ inline cplx<R> dpp0_(cplx<R> v) {
  return {dpp0_<CTRL>(v.re), dpp0_<CTRL>(v.im)};
}
// Sums of four values over the 64 lanes: lane k (and every lane equal to it mod 4) of
// the upper half of each row of 16 ends with the sum of v[k % 4].  Halving: two exchange
// steps leave each lane one of the four, so 7 steps of moves and adds do for 24.
__device__ inline void swap16_(double v, double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  a = __hiloint2double((int)hi[0], (int)lo[0]);
  b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ inline void swap32_(double v, double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  a = __hiloint2double((int)hi[0], (int)lo[0]);
  b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ inline void swap16_(float v, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
  a = __int_as_float((int)r[0]);
  b = __int_as_float((int)r[1]);
}
__device__ inline void swap32_(float v, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  a = __int_as_float((int)r[0]);
  b = __int_as_float((int)r[1]);
}
template <class T>
__device__ inline T wave_sums4(T v0, T v1, T v2, T v3, int lane) {
  const bool o1 = lane & 1, o2 = lane & 2;
  T p = (o1 ? v1 : v0) + dpp0_<DPP_XOR1>(o1 ? v0 : v1);
  T q = (o1 ? v3 : v2) + dpp0_<DPP_XOR1>(o1 ? v2 : v3);
  T s = (o2 ? q : p) + dpp0_<DPP_XOR2>(o2 ? p : q);
  s += dpp0_<0x114>(s);   // row_shr:4
  s += dpp0_<0x118>(s);   // row_shr:8: lanes 12..15 of a row hold its sums
  T a, b;
  swap16_(s, a, b);       // the other row of a pair
  s = a + b;
  swap32_(s, a, b);       // the other half
  return a + b;
}
template <class R>
__device__ inline cplx<R> wave_sums4(cplx<R> v0, cplx<R> v1, cplx<R> v2, cplx<R> v3, int lane) {
  return {wave_sums4(v0.re, v1.re, v2.re, v3.re, lane), wave_sums4(v0.im, v1.im, v2.im, v3.im, lane)};
}

// Bounded waits: true once the caller should give up (checked every 256 tries).
struct GridWait {
  unsigned tries = 0;
  long long t0 = 0;
  __device__ inline bool give_up(unsigned* err, unsigned max_tries) {
    ++tries;
    if (tries < max_tries) {
      if (tries & 255u) return false;
      const long long now = wall_clock64();
      if (tries == 256) t0 = now;
      if (now - t0 <= GRID_WAIT_TICKS && grid_ld(err) == 0) return false;
    }
    grid_st(err, 1u);
    return true;
  }
};

// A job as the kernel reads it: in the constant address space, so that its many
// pointers are scalar loads where they are used and not registers held throughout.
template <class V, class Sc>
using grid_job_ref = const GridJob<V, Sc> __attribute__((address_space(4)))&;

// Slots of a reduction: every workgroup's words, padded to whole 64-byte requests, in
// so many copies (as many as the partial-sum buffer of the multi-launch path holds).
constexpr int grid_copies(int nb) { return nb <= 4 ? 8 : nb <= 8 ? 4 : nb <= 16 ? 2 : 1; }
template <class Sc>
constexpr int grid_slot(int nb) { return ((nb + 1) * (int)(sizeof(Sc) / 8) + 7) / 8 * 8; }
template <class Sc>
constexpr bool grid_slots_fit(int nb) {
  return (size_t)GRID_RING * grid_copies(nb) * grid_slot<Sc>(nb) * GRID_MAX_P * 8 <=
         (size_t)MAX_PARTIAL_ROWS * (NMAX + 1) * sizeof(Sc);
}
static_assert(grid_slots_fit<double>(4) && grid_slots_fit<double>(8) && grid_slots_fit<double>(16) &&
              grid_slots_fit<double>(32) && grid_slots_fit<cplx<double>>(4) && grid_slots_fit<cplx<double>>(8) &&
              grid_slots_fit<cplx<double>>(16) && grid_slots_fit<cplx<double>>(32));

// -a b, a / b (Smith's method) and |a|^2 with every fma written out: where the compiler chooses
// which product of a complex expression it fuses, it chooses otherwise from variant to variant of
// the kernel, and a system's result would depend on the largest n of its batch.
__device__ inline double neg_mul(double a, double b) { return -(a * b); }
__device__ inline cplx<double> neg_mul(cplx<double> a, cplx<double> b) {
  return {fma(a.im, b.im, -(a.re * b.re)), fma(-a.re, b.im, -(a.im * b.re))};
}
__device__ inline double grid_div(double a, double b) { return a / b; }
__device__ inline cplx<double> grid_div(cplx<double> a, cplx<double> b) {
  if (fabs(b.re) >= fabs(b.im)) {
    const double t = b.im / b.re, den = fma(b.im, t, b.re);
    return {fma(a.im, t, a.re) / den, fma(-a.re, t, a.im) / den};
  }
  const double t = b.re / b.im, den = fma(b.re, t, b.im);
  return {fma(a.re, t, a.im) / den, fma(a.im, t, -a.re) / den};
}
__device__ inline double grid_abs2(double a) { return a * a; }
__device__ inline double grid_abs2(cplx<double> a) { return fma(a.re, a.re, a.im * a.im); }

// The recurrences of a step (scalar_program's) as the
// whole-solve kernel runs them: what they read of the state is loaded before the wait for
// the sums, and the scalars (wave 0) and the triangular recurrence (wave 1) of a phase run
// side by side.
template <class Sc, int NB>
struct GridPre {
  static constexpr bool ROW = NB * sizeof(Sc) <= 128;   // a row of S fits in registers
  double bnrm2, tol;
  long long iter, maxit;
  Sc e, omega;
  Sc cinv, row[ROW ? NB : 1];
  __device__ inline void load(const State<Sc>& st, int wid, int phase, int i, int n) {
    if (wid == 0) {
      bnrm2 = st.bnrm2;
      tol = st.tol;
      iter = st.iter;
      maxit = st.maxit;
      e = st.e;
      return;
    }
    if (!ROW) return;
    const int lo = phase == PH_INNER ? i : 0, hi = phase == PH_COMBINE ? i : n;
    const int s = lo + (int)(threadIdx.x % WAVE);
    const bool mine = s < hi;
    omega = st.omega;
    cinv = mine ? st.cinv[s] : zero<Sc>();
#pragma unroll
    for (int u = 0; u < (ROW ? NB : 1); ++u) row[u] = mine && s > lo + u ? st.S[s * NMAX + lo + u] : zero<Sc>();
  }
  __device__ inline void recurrence(State<Sc>& st, const Sc* sums, int phase, int i, int j, int n) const {
    const bool tilde = (phase == PH_INNER && j >= 1) || phase == PH_OMEGA_UPD;
    if (!tilde && phase != PH_COMBINE) return;
    const int lo = phase == PH_INNER ? i : 0, hi = phase == PH_COMBINE ? i : n;
    const Sc* d = tilde ? sums + 1 : sums;
    const int lane = threadIdx.x % WAVE, s = lo + lane;
    const bool mine = s < hi;
    Sc acc = mine ? d[lane] : zero<Sc>();
    Sc xs = zero<Sc>();
    auto column = [&](int u, Sc ci, Sc su) {   // column lo + u of the triangle
      const Sc xu = bcast_(neg_mul(acc, ci), u);
      if (lane == u) xs = xu;
      if (mine && lane > u) acc = axpy(acc, xu, su);
    };
    if constexpr (ROW) {   // the row preloaded
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (lo + u < hi) column(u, cinv, row[u]);
    } else {
      for (int u = 0; lo + u < hi; ++u) column(u, st.cinv[lo + u], mine ? st.S[s * NMAX + lo + u] : zero<Sc>());
    }
    if (!mine) return;
    if (tilde) {
      st.t[s] = xs;
      st.tg[s] = zero<Sc>() - grid_div(xs, ROW ? omega : st.omega);
    } else {
      st.beta[s] = xs;
    }
  }
  // Every lane computes, lane 0 stores.
  __device__ inline void scalars(State<Sc>& st, const Sc* sums, int phase, int i, int n) const {
    const int l = threadIdx.x % WAVE;
    const bool w0 = l == 0;
    switch (phase) {
      case PH_INNER:
      case PH_OMEGA_UPD: {
        const long long k = iter + 1;
        const double err = sqrt(re(sums[0])) / bnrm2;
        if (w0) {
          st.iter = k;
          st.err = err;
          st.e = sums[1];
        }
        if (!finite(err)) finish(&st, -1);
        else if (err < tol) finish(&st, 0);
        else if (k >= maxit) finish(&st, 1);
        else if (stagnated(&st, err, k)) finish(&st, 2);
        break;
      }
      case PH_SPMV_STEP: {
        if (i + l < n) st.S[(i + l) * NMAX + i] = sums[l];
        const Sc ci = sums[0];
        if (is_zero(ci) || !finite(ci)) {
          finish(&st, -1);
        } else if (w0) {
          st.c[i] = ci;
          st.cinv[i] = grid_div(from_real<Sc>(1.0), ci);
          st.alpha = grid_div(e, ci);
        }
        break;
      }
      case PH_HALF: {   // and the minimisation step: ||u||^2, z^H z, z^H u
        const double uu = re(sums[0]), zz = re(sums[1]);
        const double err = sqrt(uu) / bnrm2;
        if (w0) {
          st.uu = uu;
          st.err = err;
        }
        if (!finite(err)) {
          finish(&st, -1);
          break;
        }
        if (err < tol) {
          if (w0) st.iter = iter + 1;
          finish(&st, 0);
          break;
        }
        if (zz == 0.0 || !finite(zz)) {
          finish(&st, -1);
          break;
        }
        const Sc rho = sums[2];
        Sc om = rho / zz;
        if (st.kappa > 0) {
          const Sc rn = rho / (sqrt(zz) * sqrt(uu));
          const double a = sqrt(grid_abs2(rn));
          if (a < st.kappa && a != 0.0) om = (st.kappa / a) * om;
        }
        if (is_zero(om) || !finite(om)) {
          finish(&st, -1);
          break;
        }
        if (w0) st.omega = om;
        break;
      }
      case PH_COMBINE: break;
      default: scalar_program(&st, sums, phase, i, 0, n);   // set-up and the residual's sums
    }
  }
};

// The iteration of one system by the calling workgroup, rank `rank` of its group
// (state in ss; gl and zl: LDS copies of the own slice of the product's input and
// of z).  FMT: 0 CSR, 1 BSR3 (a lane takes one scalar row).  KR: a slice of at most GB
// rows, whose rows of x, r, G, W, F and Q each thread keeps in registers for the whole
// solve: a pass then reads no memory at all.  (Columns are selected by tests on uniform
// values, so that every array index is a constant.)
template <class V, class Sc, int NB, int FMT, bool KR>
__device__ __forceinline__ void grid_solve(grid_job_ref<V, Sc> J, const int rank, State<Sc>& ss, double* sums, V* gl,
                                           V* zl, int* lost, long long* setup_end) {
  constexpr int NA = NB + 1, NW = GB / WAVE;
  using real = typename traits<V>::real;
  using Wd = grid_word<real>;
  using U = typename Wd::U;
  using U64 = unsigned long long;
  constexpr int W = sizeof(V) / sizeof(U);       // words of an exchanged value
  constexpr int WS = sizeof(Sc) / 8;             // 64-bit words of a sum
  constexpr int COPIES = grid_copies(NB), NS = grid_slot<Sc>(NB);
  constexpr U64 pending64 = grid_word<double>::pending;
  int tid = threadIdx.x;
  const int N = J.N, n = J.n, P = J.P;
  const int lo = rank * J.R, hi = min(lo + J.R, N);
  const long long ldq = J.ldq;
  unsigned* err = &J.st->ctl[GRID_ERR];
  int q_ring = 0;       // ring position of the next reduction
  int xcur = 0;         // exchange buffer of the next product
  __shared__ Sc red[NW][NA];
  __shared__ double tot[GB];
  V acc[NA];
  auto clear = [&] {
#pragma unroll
    for (int d = 0; d < NA; ++d) acc[d] = zero<V>();
  };

  // Sums over the group, in a fixed order (a thread's rows in V, from there on in Sc: the
  // partial sums of fp32 values are fp64 beyond a thread's at most 8 rows; a tree over each
  // wave, the waves of a workgroup in order, then the workgroups: every thread some of them, a tree over the lanes of a
  // wave that hold the same sum, the waves in order), and the recurrence of `phase` on
  // them: the scalars on wave 0, a triangular recurrence on wave 1.  The k-th sum is that
  // of acc[k] for k < base, of acc[k + shift] from base on.
  // A workgroup's sums stand next to each other in GRID_COPIES slots, each read by its
  // part of the group: one store instruction, and fewer readers of a line (with the sums
  // of a group side by side in one slot, a reduction over 64 workgroups took 2.3 us and
  // one over 203 4.5 us, where two workgroups take 0.95 us).
  auto reduce = [&](int nsum, int base, int shift, int phase, int pi, int pj) {
    const int lane = tid % WAVE, wid = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int need0 = base > 0 ? 0 : shift, need1 = nsum + (nsum > base ? shift : 0);
#pragma unroll
    for (int d4 = 0; d4 < NA; d4 += 4)
      if (d4 + 4 > need0 && d4 < need1) {
        auto of = [&](int d) { return d < NA ? convert<Sc>(acc[d < NA ? d : 0]) : zero<Sc>(); };
        const Sc v = wave_sums4(of(d4), of(d4 + 1), of(d4 + 2), of(d4 + 3), lane);
        if (lane >= WAVE - 4 && d4 + (lane & 3) < NA) red[wid][d4 + (lane & 3)] = v;
      }
    if (P > 1) grid_stores_done();
    __syncthreads();
    const int nw = nsum * WS;   // words of the sums
    // word k of the workgroup's own sums
    auto own = [&](int k) {
      const int d = k / WS, src = d < base ? d : d + shift;
      Sc s = red[0][src];
#pragma unroll
      for (int w = 1; w < NW; ++w) add_(s, red[w][src]);
      double t[WS];
      __builtin_memcpy(t, &s, sizeof(Sc));
      return WS == 2 && (k & 1) ? t[WS - 1] : t[0];
    };
    GridPre<Sc, NB> pre;
    if (wid < 2) pre.load(ss, wid, phase, pi, n);
    if (P > 1) {
      const int kl = nw <= 8 ? 3 : nw <= 16 ? 4 : nw <= 32 ? 5 : nw <= 64 ? 6 : 7, KS = 1 << kl;
      U64* slots = reinterpret_cast<U64*>(J.slots) + (size_t)q_ring * COPIES * NS * P;
      {
        const int c = tid >> kl, k = tid & (KS - 1);
        if (c < COPIES && k < nw) {
          const double v = own(k);
          const U64 u = (U64)__double_as_longlong(v);
          grid_st(slots + ((size_t)c * P + rank) * NS + k, u == pending64 ? grid_word<double>::qnan : u);
        }
      }
      const int k = tid & (KS - 1), p0 = tid >> kl, pstep = GB >> kl;
      const U64* rd = slots + (size_t)(rank % COPIES) * P * NS + k;
      double t = 0.0;
      constexpr int PB = 4;   // words of a thread in flight
      GridWait wt;
      for (int pb = 0; pb < P; pb += PB * pstep) {
        U64 v[PB];
        for (int first = 1;; first = 0) {
          bool pend = false;
#pragma unroll
          for (int q = 0; q < PB; ++q) {
            const int p = pb + p0 + q * pstep;
            if (first || v[q] == pending64) v[q] = k < nw && p < P ? grid_ld(rd + (size_t)p * NS) : 0ull;
          }
#pragma unroll
          for (int q = 0; q < PB; ++q) pend |= v[q] == pending64;
          if (!__any(pend)) break;
          if (wt.give_up(err, J.max_tries)) {
            *lost = 1;
            break;
          }
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) t += __longlong_as_double((long long)v[q]);   // 0 past P
      }
      double ta, tb;
      if (kl <= 3) t += dpp0_<0x118>(t);   // row_shr:8: lanes 8..15 of a row
      if (kl <= 4) {
        swap16_(t, ta, tb);
        t = ta + tb;
      }
      if (kl <= 5) {
        swap32_(t, ta, tb);
        t = ta + tb;
      }
      if (kl >= 6) tot[tid] = t;
      else if (lane >= WAVE - KS) tot[wid * KS + k] = t;
      __syncthreads();
      // This workgroup has seen the words of all P (each wave those of some of them, so only
      // after the barrier): everybody has read the previous reduction's.
      U64* prev = reinterpret_cast<U64*>(J.slots) + (size_t)((q_ring + GRID_RING - 1) % GRID_RING) * COPIES * NS * P;
      for (int w = tid - 2 * WAVE; w >= 0 && w < COPIES * NA * WS; w += GB - 2 * WAVE)   // not the waves at work below
        grid_st(prev + ((size_t)(w / (NA * WS)) * P + rank) * NS + w % (NA * WS), (U64)pending64);
      q_ring = (q_ring + 1) % GRID_RING;
      if (wid < 2) {
        const int rows = kl >= 7 ? GB >> kl : NW;
        for (int w = lane; w < nw; w += WAVE) {
          double s = tot[w];
          for (int r = 1; r < rows; ++r) s += tot[(r << kl) + w];
          sums[wid * (NA * WS) + w] = s;
        }
      }
    } else if (wid < 2) {
      for (int w = lane; w < nw; w += WAVE) sums[wid * (NA * WS) + w] = own(w);
    }
    if (wid < 2) {
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const Sc* sm = reinterpret_cast<const Sc*>(sums + wid * (NA * WS));
      if (wid == 0) pre.scalars(ss, sm, phase, pi, n);
      else pre.recurrence(ss, sm, phase, pi, pj, n);
    }
    __syncthreads();
  };
  // row `row` of the next product's input (every own row, before product()).  A value that
  // holds the pending pattern (only from an x_0 that does) is a quiet NaN in both places.
  auto put = [&](int row, V v) {
    U u[W];
    __builtin_memcpy(u, &v, sizeof(V));
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (u[w] == Wd::pending) u[w] = Wd::qnan;
    __builtin_memcpy(&v, u, sizeof(V));
    gl[row - lo] = v;
    if (P > 1) {
      U* d = reinterpret_cast<U*>(xcur ? J.xb1 : J.xb) + (size_t)row * W;
#pragma unroll
      for (int w = 0; w < W; ++w) grid_st(d + w, u[w]);
    }
  };
  // after the reduction that follows a product: its exchange buffer is free again
  auto recycle = [&] {
    if (P > 1) {
      U* d = reinterpret_cast<U*>(xcur ? J.xb1 : J.xb);
      for (int k = lo * W + tid; k < hi * W; k += GB) grid_st(d + k, (U)Wd::pending);
      xcur ^= 1;
    }
  };

  // Every pass takes one row per thread at a time and issues all loads of the row
  // together, before any is used: a load under a per-column test, or one behind a store
  // that it might alias, would wait for the one before it, and the loads' latency is what
  // a pass over a slice costs.  Columns past the last repeat it (cache hits); their sums
  // are not read.  CG: columns loaded together.
  constexpr int CG = NB * (int)sizeof(V) <= 128 ? NB : 128 / (int)sizeof(V);

  // y = A xin, one scalar row per lane, with the epilogue of `mode`.  xin: a vector
  // of global memory that nobody writes meanwhile (xg), or the vector put() before.
  // The first RB entries of the thread's first row of A stay in registers (held).
  constexpr int C = FMT == 0 ? 1 : 3;                                                        // columns of an entry
  constexpr int RT = FMT == 0 ? 8 : (sizeof(V) > 8 ? 2 : 4);                               // entries of a tree
  constexpr int RB = FMT == 0 && sizeof(V) * NB > 256 ? RT / 2 : RT;                       // entries in flight
  auto entries = [&](const int* ci, const V* val, int beg, int end, int sub, int (&c)[RB], V (&v)[RB][C]) {
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int q = beg + k;
      const bool on = q < end;
      c[k] = on ? C * ci[q] : -1;
#pragma unroll
      for (int e = 0; e < C; ++e) v[k][e] = on ? val[FMT == 0 ? (size_t)q : (size_t)9 * q + sub + e] : zero<V>();
    }
  };
  int hbeg, hend, hc[RB];
  V hv[RB][C];
  {
    const int row = lo + tid, br = FMT == 0 ? row : row / 3;
    hbeg = row < hi ? J.rp[br] : 0;
    hend = row < hi ? J.rp[br + 1] : 0;
    entries(J.ci, J.val, hbeg, hend, FMT == 0 ? 0 : 3 * (row - 3 * br), hc, hv);
  }
  // the thread's row (KR); rows past the slice hold zeros, which add nothing to any sum
  constexpr int NK = KR ? NB : 1;
  V kx = zero<V>(), kr = zero<V>(), kg = zero<V>(), kz = zero<V>();   // x, r, the put vector, z
  V kQ[NK], kG[NK], kW[NK], kF[NK];
  const bool mine = lo + tid < hi;
  if constexpr (KR) {
    if (mine) kx = J.x[lo + tid];
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      kQ[s] = mine && s < n ? J.Q[lo + tid + (long long)s * ldq] : zero<V>();
      kG[s] = kW[s] = kF[s] = zero<V>();
    }
  }

  auto product = [&](bool held, const int* rp, const int* ci, const V* val, const V* xg, V* out1, V* out2, int mode,
                     int d0, int nd, int col) {
    const unsigned nloc = (unsigned)(hi - lo);
    const U* xe = reinterpret_cast<const U*>(xcur ? J.xb1 : J.xb);
    __syncthreads();   // gl is complete
    for (int r0 = lo + tid; r0 < hi; r0 += GB) {
      const int row = r0;
      const int br = FMT == 0 ? row : row / 3;
      const int sub = FMT == 0 ? 0 : 3 * (row - 3 * br);
      const bool h = held && r0 < lo + GB;
      int beg, end;
      if (h) {
        beg = hbeg;
        end = hend;
      } else {
        beg = rp[br];
        end = rp[br + 1];
      }
      V y = zero<V>(), part = zero<V>();
      int e0 = beg;
      do {
        int c[RB];
        V v[RB][C];
        if (h && e0 == beg) {
#pragma unroll
          for (int k = 0; k < RB; ++k) {
            c[k] = hc[k];
#pragma unroll
            for (int e = 0; e < C; ++e) v[k][e] = hv[k][e];
          }
        } else {
          entries(ci, val, e0, end, sub, c, v);
        }
        V xs[RB][C];
        if (xg) {
#pragma unroll
          for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int e = 0; e < C; ++e) xs[k][e] = xg[c[k] < 0 ? 0 : c[k] + e];
        } else {
          GridWait wt;
          for (;;) {
            bool pend = false;
#pragma unroll
            for (int k = 0; k < RB; ++k)
#pragma unroll
              for (int e = 0; e < C; ++e) {
                const int cc = c[k] + e;
                U w[W];
                if ((unsigned)(cc - lo) < nloc || c[k] < 0) {
                  const V t = gl[c[k] < 0 ? 0 : cc - lo];
                  __builtin_memcpy(w, &t, sizeof(V));
                } else {
#pragma unroll
                  for (int t = 0; t < W; ++t) w[t] = grid_ld(xe + (size_t)cc * W + t);
                }
                __builtin_memcpy(&xs[k][e], w, sizeof(V));
              }
#pragma unroll
            for (int k = 0; k < RB; ++k)
#pragma unroll
              for (int e = 0; e < C; ++e) {
                U w[W];
                __builtin_memcpy(w, &xs[k][e], sizeof(V));
#pragma unroll
                for (int t = 0; t < W; ++t) pend |= w[t] == Wd::pending;
              }
            if (!pend) break;
            if (wt.give_up(err, J.max_tries)) {
              *lost = 1;
              break;
            }
          }
        }
        // the entries' products, then a tree over them, as the lanes of a row add them in the
        // multi-launch products
        V t[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) {
          t[k] = zero<V>();
          if (c[k] >= 0) {
#pragma unroll
            for (int e = 0; e < C; ++e) t[k] = axpy(t[k], v[k][e], xs[k][e]);
          }
        }
#pragma unroll
        for (int m = 1; m < RB; m *= 2)
#pragma unroll
          for (int k = 0; k < RB; k += 2 * m) add_(t[k], t[k + m]);
        // a tree spans RT entries in every variant, so a row's sum does not depend on NB
        if constexpr (RB < RT) {
          if ((e0 - beg) % RT == 0 && e0 + RB < end) {
            part = t[0];
            e0 += RB;
            continue;
          }
          if ((e0 - beg) % RT) {
            add_(part, t[0]);
            t[0] = part;
          }
        }
        add_(y, t[0]);
        e0 += RB;
      } while (e0 < end);
      if constexpr (KR) {
        if (mode == SM_RESID) {
          const V bv = J.b[row], rv = bv - y;
          if (out1) kr = rv;
          cdot_acc(acc[0], rv, rv);
          cdot_acc(acc[1], bv, bv);
          cdot_acc(acc[2], kQ[0], rv);
        } else if (mode == SM_STEP) {   // col: the column of W (tf: of v = A g)
#pragma unroll
          for (int s = 0; s < NK; ++s) {
            if (s == col) kW[s] = y;
            cdot_acc(acc[s], kQ[s], y);
          }
          if (out2) kG[0] = kg;
        } else if (mode == SM_OMEGA) {
          kz = y;
          cdot_acc(acc[1], y, y);
          cdot_acc(acc[2], y, kg);
        } else {
#pragma unroll
          for (int s = 0; s < NK; ++s)
            if (s == col) kF[s] = y;
        }
      } else if (mode == SM_RESID) {
        const V bv = J.b[row];
        const V q0 = J.Q[row];
        const V rv = bv - y;
        if (out1) out1[row] = rv;
        cdot_acc(acc[0], rv, rv);
        cdot_acc(acc[1], bv, bv);
        cdot_acc(acc[2], q0, rv);
      } else if (mode == SM_STEP) {
        const V own = gl[row - lo];
#pragma unroll
        for (int g = 0; g < NB; g += CG)
          if (g < nd) {
            V qv[CG];
#pragma unroll
            for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)(d0 + min(g + d, nd - 1)) * ldq];
#pragma unroll
            for (int d = 0; d < CG; ++d) cdot_acc(acc[g + d], qv[d], y);
          }
        out1[row] = y;
        if (out2) out2[row] = own;
      } else if (mode == SM_OMEGA) {
        zl[row - lo] = y;
        cdot_acc(acc[1], y, y);
        cdot_acc(acc[2], y, gl[row - lo]);
      } else {
        out1[row] = y;
      }
    }
  };
  // KR: x_k into the iterate record
  auto record = [&] {
    const long long k = ss.iter + 1;
    if (J.xrec && k <= J.K && mine) J.xrec[(k - 1) * (long long)N + lo + tid] = kx;
  };
  // x += alpha g_prev ; r -= alpha w_prev ; ||r||^2, q_s^H r (s in [d0, d0+nd)).
  // half: the half step that ends a cycle; the new r = u is the next product's input.
  auto alpha = [&](int iprev, int d0, int nd, bool half) {
    const V al = convert<V>(ss.alpha), mal = convert<V>(zero<Sc>() - ss.alpha);
    if constexpr (KR) {
      V gv = zero<V>(), wv = zero<V>();
#pragma unroll
      for (int s = 0; s < NK; ++s)
        if (s == iprev) {
          gv = kG[s];
          wv = kW[s];
        }
      kx = axpy(kx, al, gv);
      kr = axpy(kr, mal, wv);
      cdot_acc(acc[0], kr, kr);
      if (nd > 0) {
#pragma unroll
        for (int s = 0; s < NK; ++s) cdot_acc(acc[1 + s], kQ[s], kr);
      }
      record();
      if (half) {
        kg = kr;
        if (mine) put(lo + tid, kr);
      }
      return;
    }
    const V* gh = J.G + (size_t)iprev * N;
    const V* w = J.W + (size_t)iprev * N;
    const long long k = ss.iter + 1;
    V* rec = (J.xrec && k <= J.K) ? J.xrec + (k - 1) * (long long)N : nullptr;
    for (int row = lo + tid; row < hi; row += GB) {
      const V x0 = J.x[row], gv = gh[row], r0 = J.r[row], wv = w[row];
      V qv[CG];
      if (nd > 0) {
#pragma unroll
        for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)(d0 + min(d, nd - 1)) * ldq];
      }
      const V xn = axpy(x0, al, gv);
      const V rn = axpy(r0, mal, wv);
      cdot_acc(acc[0], rn, rn);
      if (nd > 0) {
#pragma unroll
        for (int d = 0; d < CG; ++d) cdot_acc(acc[1 + d], qv[d], rn);
#pragma unroll
        for (int g = CG; g < NB; g += CG)
          if (g < nd) {
#pragma unroll
            for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)(d0 + min(g + d, nd - 1)) * ldq];
#pragma unroll
            for (int d = 0; d < CG; ++d) cdot_acc(acc[1 + g + d], qv[d], rn);
          }
      }
      J.x[row] = xn;
      if (rec) rec[row] = xn;
      J.r[row] = rn;
      if (half) put(row, rn);
    }
  };
  // g = r + sum_{s in [t0, t1)} (t_s W_s + tg_s G_s) ; f_s^H g (s < nf).  g stays in gl
  // for recombine(), or (last) is the next product's input.
  auto combine = [&](int t0, int t1, int nf, bool last) {
    if constexpr (KR) {
      V g = kr;
#pragma unroll
      for (int s = 0; s < NK; ++s)
        if (s >= t0 && s < t1) {
          g = axpy(g, convert<V>(ss.t[s]), kW[s]);
          g = axpy(g, convert<V>(ss.tg[s]), kG[s]);
        }
      if (nf > 0) {
#pragma unroll
        for (int s = 0; s < NK; ++s) cdot_acc(acc[s], kF[s], g);
      }
      kg = g;
      if (last && mine) put(lo + tid, g);
      return;
    }
    constexpr int CC = CG > 1 && CG * (int)sizeof(V) > 64 ? CG / 2 : CG;
    for (int row = lo + tid; row < hi; row += GB) {
      V g = J.r[row];
      V fv[CG];
      if (nf > 0) {
#pragma unroll
        for (int d = 0; d < CG; ++d) fv[d] = J.F[row + (size_t)min(d, nf - 1) * N];
      }
#pragma unroll
      for (int s0 = 0; s0 < NB; s0 += CC)
        if (t0 + s0 < t1) {
          V wv[CC], gv[CC];
#pragma unroll
          for (int u = 0; u < CC; ++u) {
            const size_t col = (size_t)min(t0 + s0 + u, t1 - 1) * N;
            wv[u] = J.W[row + col];
            gv[u] = J.G[row + col];
          }
#pragma unroll
          for (int u = 0; u < CC; ++u) {
            const int s = t0 + s0 + u;
            if (s < t1) {
              g = axpy(g, convert<V>(ss.t[s]), wv[u]);
              g = axpy(g, convert<V>(ss.tg[s]), gv[u]);
            }
          }
        }
      if (nf > 0) {
#pragma unroll
        for (int d = 0; d < CG; ++d) cdot_acc(acc[d], fv[d], g);
#pragma unroll
        for (int f = CG; f < NB; f += CG)
          if (f < nf) {
#pragma unroll
            for (int d = 0; d < CG; ++d) fv[d] = J.F[row + (size_t)min(f + d, nf - 1) * N];
#pragma unroll
            for (int d = 0; d < CG; ++d) cdot_acc(acc[f + d], fv[d], g);
          }
      }
      if (last) put(row, g);
      else gl[row - lo] = g;
    }
  };
  // G_i = g + sum_{s<i} beta_s G_s (g in gl), the next product's input.  Transpose-free
  // (wi): v = A g was stored in W_i; W_i = v + sum_{s<i} beta_s W_s with its S column
  // instead of a product.
  auto recombine = [&](int i, bool wi) {
    if constexpr (KR) {
      V v = kg, wv = zero<V>();
#pragma unroll
      for (int s = 0; s < NK; ++s)
        if (s == i) wv = kW[s];
#pragma unroll
      for (int s = 0; s < NK; ++s)
        if (s < i) {
          const V bs = convert<V>(ss.beta[s]);
          v = axpy(v, bs, kG[s]);
          if (wi) wv = axpy(wv, bs, kW[s]);
        }
#pragma unroll
      for (int s = 0; s < NK; ++s)
        if (s == i) {
          kG[s] = v;
          kW[s] = wv;   // not wi: unchanged, the product writes it
        }
      if (wi) {
#pragma unroll
        for (int s = 0; s < NK; ++s) cdot_acc(acc[s], kQ[s], wv);
      } else {
        kg = v;
        if (mine) put(lo + tid, v);
      }
      return;
    }
    constexpr int CC = CG > 1 && CG * (int)sizeof(V) > 64 ? CG / 2 : CG;
    for (int row = lo + tid; row < hi; row += GB) {
      V v = gl[row - lo];
      V wv = wi ? J.W[row + (size_t)i * N] : zero<V>();
#pragma unroll
      for (int s0 = 0; s0 < NB; s0 += CC)
        if (s0 < i) {
          V gv[CC], wa[CC];
#pragma unroll
          for (int u = 0; u < CC; ++u) gv[u] = J.G[row + (size_t)min(s0 + u, i - 1) * N];
          if (wi) {
#pragma unroll
            for (int u = 0; u < CC; ++u) wa[u] = J.W[row + (size_t)min(s0 + u, i - 1) * N];
#pragma unroll
            for (int u = 0; u < CC; ++u)
              if (s0 + u < i) wv = axpy(wv, convert<V>(ss.beta[s0 + u]), wa[u]);
          }
#pragma unroll
          for (int u = 0; u < CC; ++u)
            if (s0 + u < i) v = axpy(v, convert<V>(ss.beta[s0 + u]), gv[u]);
        }
      if (wi) {
        const int nd = n - i;
#pragma unroll
        for (int g = 0; g < NB; g += CG)
          if (g < nd) {
            V qv[CG];
#pragma unroll
            for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)(i + min(g + d, nd - 1)) * ldq];
#pragma unroll
            for (int d = 0; d < CG; ++d) cdot_acc(acc[g + d], qv[d], wv);
          }
        J.W[row + (size_t)i * N] = wv;
      } else {
        put(row, v);
      }
      J.G[row + (size_t)i * N] = v;
    }
  };
  // x += omega u ; r = u - omega z (u held in r, z in zl) ; ||r||^2, q_s^H r, s < n
  auto omega = [&] {
    const V om = convert<V>(ss.omega), mom = convert<V>(zero<Sc>() - ss.omega);
    if constexpr (KR) {
      kx = axpy(kx, om, kr);
      kr = axpy(kr, mom, kz);
      cdot_acc(acc[0], kr, kr);
#pragma unroll
      for (int s = 0; s < NK; ++s) cdot_acc(acc[1 + s], kQ[s], kr);
      record();
      return;
    }
    const long long k = ss.iter + 1;
    V* rec = (J.xrec && k <= J.K) ? J.xrec + (k - 1) * (long long)N : nullptr;
    for (int row = lo + tid; row < hi; row += GB) {
      const V uv = J.r[row], x0 = J.x[row], zv = zl[row - lo];
      V qv[CG];
#pragma unroll
      for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)min(d, n - 1) * ldq];
      const V xn = axpy(x0, om, uv);
      const V rn = axpy(uv, mom, zv);
      cdot_acc(acc[0], rn, rn);
#pragma unroll
      for (int d = 0; d < CG; ++d) cdot_acc(acc[1 + d], qv[d], rn);
#pragma unroll
      for (int g = CG; g < NB; g += CG)
        if (g < n) {
#pragma unroll
          for (int d = 0; d < CG; ++d) qv[d] = J.Q[row + (long long)min(g + d, n - 1) * ldq];
#pragma unroll
          for (int d = 0; d < CG; ++d) cdot_acc(acc[1 + g + d], qv[d], rn);
        }
      J.x[row] = xn;
      if (rec) rec[row] = xn;
      J.r[row] = rn;
    }
  };

  // The solve as a sequence of stages: a vector pass, then a product with A or A^H, then
  // a reduction with its recurrence, each of them or none.  One loop over them keeps one
  // copy of every pass in the code (written out in the order of the algorithm, the copies
  // of product() and the recurrence took 256 registers and spilled).
  enum { S_SETUP, S_F, S_CLOSE, S_ALPHA, S_COMBINE, S_RECOMBINE, S_HALF, S_OMEGA, S_RESID };
  int stage = S_SETUP;
  int i = 0, j = 0, fcol = 0;          // step, 0 in the first cycle, column of F
  bool first = true;                   // S_CLOSE before the first cycle: g_0 = r_0
  const long long max_cycles = J.maxit / n + 2;
  long long cycles = 0;
  for (;;) {
    const int *rp = J.rp, *ci = J.ci;  // the product's matrix
    const V* val = J.val;
    const V* xg = nullptr;             // its input, when not the vector put
    V *out1 = nullptr, *out2 = nullptr;
    int mode = -1, d0 = 0, nd = 0;     // no product
    int nsum = 0, phase = PH_NONE, pi = i, pj = j;
    int base = 0, shift = 0;           // KR: where the sums stand in acc, see reduce()
    int col = 0;                       // KR: the product's column
    asm volatile("" : "+v"(tid));   // no row address is computed before the loop and kept
    clear();
    switch (stage) {
      case S_SETUP:   // r_0 = b - A x_0, ||b||, e_0
        xg = J.x; out1 = J.r; mode = SM_RESID;
        nsum = 3; phase = PH_SETUP;
        break;
      case S_F:       // f_s = A^H q_s
        rp = J.rpT; ci = J.ciT; val = J.valT;
        xg = J.Q + (size_t)fcol * ldq; out1 = J.F + (size_t)fcol * N; mode = SM_PLAIN; col = fcol;
        break;
      case S_CLOSE:   // g_{jn+n} (or g_0 = r_0), w, S column 0, c, alpha
        combine(0, first ? 0 : n, 0, true);
        out1 = J.W; out2 = J.G; mode = SM_STEP; nd = n;
        nsum = n; phase = PH_SPMV_STEP; pi = 0;
        break;
      case S_ALPHA:
        nd = j >= 1 ? n - i : 1;
        alpha(i - 1, i, nd, false);
        nsum = nd + 1; phase = PH_INNER; base = 1; shift = i;
        break;
      case S_COMBINE: // transpose-free: also v = A g -> W_i with q_s^H v (s < i)
        combine(i, j >= 1 ? n : i, J.tf ? 0 : i, J.tf != 0);
        if (J.tf) { out1 = J.W + (size_t)i * N; mode = SM_STEP; nd = i; col = i; }
        nsum = i; phase = PH_COMBINE;
        break;
      case S_RECOMBINE:
        recombine(i, J.tf != 0);
        if (!J.tf) { out1 = J.W + (size_t)i * N; mode = SM_STEP; d0 = i; nd = n - i; col = i; }
        nsum = n - i; phase = PH_SPMV_STEP; shift = i;
        break;
      case S_HALF:    // half step to u, z = A u: one reduction for both
        alpha(n - 1, 0, 0, true);
        mode = SM_OMEGA;
        nsum = 3; phase = PH_HALF; pi = n;
        break;
      case S_OMEGA:
        omega();
        nsum = n + 1; phase = PH_OMEGA_UPD; pi = 0; pj = 1;
        break;
      default:        // S_RESID
        for (int row = lo + tid; row < hi; row += GB) put(row, KR ? kx : J.x[row]);
        mode = SM_RESID;
        nsum = 2;
    }
    if (mode >= 0) product(stage != S_F, rp, ci, val, xg, out1, out2, mode, d0, nd, col);
    if (nsum > 0) {
      reduce(nsum, KR ? base : 0, KR ? shift : 0, phase, pi, pj);
      if (mode >= 0 && !xg) recycle();
      if (*lost || stage == S_RESID) return;
      if (ss.done) {
        if (KR && mine) J.x[lo + tid] = kx;
        if (!J.resid) return;
        stage = S_RESID;
        continue;
      }
    }
    switch (stage) {
      case S_SETUP: stage = J.tf || n == 1 ? S_CLOSE : S_F; break;
      case S_F: if (++fcol + 1 >= n) stage = S_CLOSE; break;
      case S_CLOSE:
        if (first && tid == 0) *setup_end = wall_clock64();
        if (!first) j = 1;
        first = false;
        if (cycles++ > max_cycles) {   // the recurrence ends a solve at maxit before this
          if (KR && mine) J.x[lo + tid] = kx;
          return;
        }
        i = 1;
        stage = i < n ? S_ALPHA : S_HALF;
        break;
      case S_ALPHA: stage = S_COMBINE; break;
      case S_COMBINE: stage = S_RECOMBINE; break;
      case S_RECOMBINE: stage = ++i < n ? S_ALPHA : S_HALF; break;
      case S_HALF: stage = S_OMEGA; break;
      default: stage = S_CLOSE;
    }
  }
}

// jobs / map: the systems and {job, rank} of every logical workgroup; without a map
// one system, logical workgroup = rank.  tick: claim counter, 0 at launch.
template <class V, class Sc, int NB, int FMT, bool KR>
__global__ __launch_bounds__(GB) void k_grid(const GridJob<V, Sc>* __restrict__ jobs, const int2* __restrict__ map,
                                             unsigned* tick) {
  static_assert(sizeof(State<Sc>) % 8 == 0, "state is copied in 8-byte words");
  __shared__ State<Sc> ss;
  __shared__ double sums[2 * (NB + 1) * (sizeof(Sc) / 8)];   // a copy each for waves 0 and 1
  constexpr int ROWS = KR ? GB : grid_max_rows<V>();
  __shared__ V gl[ROWS], zl[ROWS];
  __shared__ int lost, ticket, gate;
  __shared__ long long setup_end;
  const long long start = wall_clock64();
  const int tid = threadIdx.x;
  if (tid == 0) {
    lost = 0;
    setup_end = start;
    ticket = (int)atomicAdd(tick, 1u);
  }
  __syncthreads();
  const int t = __builtin_amdgcn_readfirstlane(ticket);
  const int rank = __builtin_amdgcn_readfirstlane(map ? map[t].y : t);
  const int job = __builtin_amdgcn_readfirstlane(map ? map[t].x : 0);
  grid_job_ref<V, Sc> J = *(const GridJob<V, Sc> __attribute__((address_space(4)))*)(jobs + job);
  if (J.P > 1) {
    if (tid == 0) {
      unsigned* ctl = J.st->ctl;
      if (atomicAdd(&ctl[GRID_ARRIVED], 1u) == (unsigned)J.P - 1) atomicCAS(&ctl[GRID_GATE], GATE_CLOSED, GATE_OPEN);
      const long long t0 = wall_clock64();
      unsigned g;
      while ((g = grid_ld(&ctl[GRID_GATE])) == GATE_CLOSED)
        if (wall_clock64() - t0 > J.entry_ticks) atomicCAS(&ctl[GRID_GATE], GATE_CLOSED, GATE_LEFT);
      gate = (int)g;
    }
    __syncthreads();
    if (gate != GATE_OPEN) return;
  }
  // the state a solve starts from
  {
    unsigned long long* lw = reinterpret_cast<unsigned long long*>(&ss);
    for (int w = tid; w < (int)(sizeof(State<Sc>) / 8); w += GB) lw[w] = 0ull;
    __syncthreads();
    if (tid == 0) {
      ss.flag = 1;
      ss.maxit = J.maxit;
      ss.tol = J.tol;
      ss.kappa = J.kappa;
      ss.bnrm2 = 1.0;
      ss.omega = from_real<Sc>(1.0);
      ss.stag_window = J.stag_window;
    }
    __syncthreads();
  }
  grid_solve<V, Sc, NB, FMT, KR>(J, rank, ss, sums, gl, zl, &lost, &setup_end);
  __syncthreads();
  if (tid == 0 && lost) J.out->lost = 1;   // its rows of x may be missing, whatever the others have
  if (rank != 0) return;
  // the final state, without the ctl words and the Gram matrix
  unsigned long long* gw = reinterpret_cast<unsigned long long*>(J.st);
  const unsigned long long* lw = reinterpret_cast<const unsigned long long*>(&ss);
  for (int w = tid; w < (int)(offsetof(State<Sc>, ctl) / 8); w += GB) gw[w] = lw[w];
  if (tid == 0) {
    // a lost wait is flagged before its workgroup publishes anything further
    GridOut* o = J.out;
    o->status = lost || (J.P > 1 && grid_ld(&J.st->ctl[GRID_ERR])) ? 2 : 1;
    o->flag = ss.done ? ss.flag : 1;
    o->iter = ss.iter;
    o->err = ss.err;
    o->rr = re(ss.aux[0]);
    o->bb = re(ss.aux[1]);
    o->setup_ticks = setup_end - start;
  }
}

// Whether the kernel for V and bucket NB has a variant that keeps rows in registers (KR):
// 4 NB + 2 values a thread, beside up to 8 entries of its row of A, within 256 registers.
template <class V, int NB>
constexpr bool grid_keeps_rows() { return NB * sizeof(V) <= 64; }
template <class V>
constexpr bool grid_keeps_rows(int nb) { return nb * sizeof(V) <= 64; }

// Host launches (mlb_grid.hip).
// Marks everything pending and runs the systems: njobs systems of `jobs` with `wgs`
// logical workgroups in all, or (one, no map) that one alone, with room for it in
// jobs[0].  nb: bucket of the largest n.  kr: every slice has at most GB rows, and
// grid_keeps_rows.
template <class V>
int grid_launch(GridJob<V, typename traits<V>::wide>* jobs, const int2* map,
                const GridJob<V, typename traits<V>::wide>* one, int njobs, int wgs, int nb, int fmt, bool kr,
                unsigned* tick, hipStream_t s);
// Workgroups of the kernel the current device holds at once.
template <class V>
int grid_capacity(int nb, int fmt, bool kr);

}  // namespace mlb
