// Launches of the whole-solve kernel (mlb_grid.hpp), in a source file of their own,
// compiled once per value type: MLB_GRID_TYPE.
#include <atomic>

#include "mlb_grid.hpp"

namespace mlb {

namespace {

// A kernel's capacity on a device does not change, so it is asked for once (each solver and
// each change of n needs it: 0.2 ms a time); 0 in `known` = not yet.
template <class V, int NB, int FMT, bool KR>
int capacity_t() {
  using Sc = typename traits<V>::wide;
  static std::atomic<int> known[16];
  int per_cu = 0, dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (dev < 16)
    if (const int c = known[dev].load(std::memory_order_relaxed)) return c;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_grid<V, Sc, NB, FMT, KR>, GB, 0) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (dev < 16) known[dev].store(per_cu * cus, std::memory_order_relaxed);
  return per_cu * cus;
}

template <class V, int NB, int FMT, bool KR>
int launch_t(GridJob<V, typename traits<V>::wide>* jobs, const int2* map,
             const GridJob<V, typename traits<V>::wide>* one, int njobs, int wgs, unsigned* tick, hipStream_t s) {
  using Sc = typename traits<V>::wide;
  const int slot_words = GRID_RING * grid_copies(NB) * grid_slot<Sc>(NB);
  k_grid_init<V, Sc><<<dim3(one ? 64 : 8, njobs), BLOCK, 0, s>>>(jobs, one ? *one : GridJob<V, Sc>{}, one != nullptr,
                                                                 slot_words, tick);
  k_grid<V, Sc, NB, FMT, KR><<<wgs, GB, 0, s>>>(jobs, map, tick);
  return 0;
}

}  // namespace

// F<V, NB, FMT, KR>(args) for the run-time nb, fmt and kr
#define MLB_GRID_NB(F, B, ...)                                                          \
  if constexpr (grid_keeps_rows<V, B>())                                                \
    if (kr) return fmt ? F<V, B, 1, true>(__VA_ARGS__) : F<V, B, 0, true>(__VA_ARGS__); \
  return fmt ? F<V, B, 1, false>(__VA_ARGS__) : F<V, B, 0, false>(__VA_ARGS__)
#define MLB_GRID(F, ...)                      \
  switch (nb) {                               \
    case 4: MLB_GRID_NB(F, 4, __VA_ARGS__);   \
    case 8: MLB_GRID_NB(F, 8, __VA_ARGS__);   \
    case 16: MLB_GRID_NB(F, 16, __VA_ARGS__); \
    default: MLB_GRID_NB(F, 32, __VA_ARGS__); \
  }

template <class V>
int grid_capacity(int nb, int fmt, bool kr) {
  MLB_GRID(capacity_t)
}

template <class V>
int grid_launch(GridJob<V, typename traits<V>::wide>* jobs, const int2* map,
                const GridJob<V, typename traits<V>::wide>* one, int njobs, int wgs, int nb, int fmt, bool kr,
                unsigned* tick, hipStream_t s) {
  MLB_GRID(launch_t, jobs, map, one, njobs, wgs, tick, s)
}

using T = MLB_GRID_TYPE;
template int grid_capacity<T>(int, int, bool);
template int grid_launch<T>(GridJob<T, traits<T>::wide>*, const int2*, const GridJob<T, traits<T>::wide>*, int, int,
                            int, int, bool, unsigned*, hipStream_t);

}  // namespace mlb
