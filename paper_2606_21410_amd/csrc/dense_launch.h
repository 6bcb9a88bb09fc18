// Instantiation and dispatch of the matrix-core axis pass.
#pragma once

#include "dense_pass.h"
#include "internal.h"
#include "line_wave.h"

namespace cheb {

// Persistent launch: at most as many workgroups as the device holds at once
// (CUs and resident workgroups per CU, queried once per kernel and device), at
// most one per tile.  A two-axis launch gives each axis half of them, a multiple of 8 (the
// kernel's segment bit is bit 3 of the workgroup index).
template <typename T, int MT, int MODE, bool FIRST, bool CG>
static int launch_line_inst(const LineArgs<T>& a, hipStream_t s) {
  constexpr int lds = line_lds_bytes<T>(MT);
  static_assert(lds <= 64 * 1024, "matrix-core tile exceeds the default LDS limit");
  constexpr bool ALLP = MODE == LINE_FULL || MODE == LINE_DERIV || MODE == LINE_DMUL;
  static DeviceCache cache;
  int dev = 0;
  if (int rc = current_device(&dev)) return rc;
  int resident = cache.v[dev].load(std::memory_order_relaxed);
  if (resident == 0) {
    int cus = 0, per_cu = 0;
    int rc = hip_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "CU count");
    if (!rc)
      rc = hip_check(hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         &per_cu, (const void*)k_line_pass<T, MT, MODE, FIRST, CG>, 64 * MT, lds),
                     "occupancy query");
    if (rc) return rc;
    resident = (cus > 0 ? cus : 1) << 8 | (per_cu > 0 ? (per_cu < 255 ? per_cu : 255) : 1);
    cache.v[dev].store(resident, std::memory_order_relaxed);
  }
  auto tiles_of = [&](int axis) {
    const int o = ALLP ? 0 : 2;
    const int ta = axis == 0 ? a.n[1] : a.n[0], tb = axis == 2 ? a.n[1] : a.n[2];
    return ((ta - o) * (tb - o) + 15) / 16 * (a.sys ? a.nact : 1);
  };
  // Workgroups per CU where several fit (five and six row blocks in FP32, and
  // derivatives; an FP64 product holds one): the fewest rounds of tiles, weighted by
  // what a round takes, about 2 + W for W workgroups that share the CU.  Against as
  // many as fit: apply 161x161x65 FP32 31.3 us and 35.9, 130^3 47.7 and 50.1,
  // 145x145x257 93 and 101; nowhere slower over 16 grids from 65 to 257 nodes.
  auto per_cu_of = [&](int tiles) {
    const int cus = resident >> 8, occ = resident & 255;
    int best = 1, cost = 1 << 30;
    for (int w = 1; w <= occ; ++w) {
      const int c = (tiles + w * cus - 1) / (w * cus) * (2 + w);
      if (c < cost) cost = c, best = w;
    }
    return best * cus;
  };
  int grid;
  if (a.nseg == 2) {
    const int t0 = tiles_of(a.ax[0].axis), t1 = tiles_of(a.ax[1].axis);
    const int need = ((t0 > t1 ? t0 : t1) + 7) / 8 * 8;
    int half = per_cu_of(t0 + t1) / 2 / 8 * 8;
    if (need < half) half = need;
    if (half < 8) half = 8;
    grid = 2 * half;
  } else {
    const int tiles = tiles_of(a.ax[0].axis), full = per_cu_of(tiles);
    grid = tiles < full ? (tiles > 0 ? tiles : 1) : full;
  }
  hipLaunchKernelGGL((k_line_pass<T, MT, MODE, FIRST, CG>), dim3(grid), dim3(64 * MT), lds, s, a);
  return hip_check(hipGetLastError(), "matrix-core pass launch");
}

template <typename T, int MT, int MODE>
static int launch_line_g(const LineArgs<T>& a, int first, hipStream_t s) {
  const bool cg = a.ax[0].axis == 2;
  if constexpr (MODE == LINE_DERIV || MODE == LINE_DMUL) {
    return cg ? launch_line_inst<T, MT, MODE, true, true>(a, s) : launch_line_inst<T, MT, MODE, true, false>(a, s);
  } else {
    if (first)
      return cg ? launch_line_inst<T, MT, MODE, true, true>(a, s) : launch_line_inst<T, MT, MODE, true, false>(a, s);
    return cg ? launch_line_inst<T, MT, MODE, false, true>(a, s) : launch_line_inst<T, MT, MODE, false, false>(a, s);
  }
}

// k_line_wave: persistent over the XCDs' task ranges, a grid of whole XCD
// rounds.  Few tasks are spread over the CUs before a workgroup takes more than one
// wave's worth (a wave more than that everywhere: 129^3 FP64 51 us, 56 with half as
// many), and it takes a wave more where the rounding to whole XCD rounds would
// otherwise give some CUs a second workgroup: 121x81x61, 731 tasks, three waves in
// 304 workgroups 33.6 us FP64 and 21.5 FP32, four in 224 25.9 and 17.5.
template <typename T, int MT, int MODE, bool FIRST, bool CG, int NW>
static int launch_wave_inst(LineArgs<T>& a, hipStream_t s) {
  constexpr int lds = wave_lds_bytes<T>(MT, NW, CG);
  static_assert(lds <= 160 * 1024, "fragment table exceeds LDS");
  constexpr bool ALLP = MODE == LINE_FULL || MODE == LINE_DERIV || MODE == LINE_DMUL;
  static DeviceCache cache;
  int dev = 0;
  if (int rc = current_device(&dev)) return rc;
  int resident = cache.v[dev].load(std::memory_order_relaxed);
  if (resident == 0) {
    int cus = 0, per_cu = 0, rc = CHEB_OK;
    if (lds > 64 * 1024)
      rc = hip_check(hipFuncSetAttribute((const void*)k_line_wave<T, MT, MODE, FIRST, CG, NW>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, lds),
                     "matrix-core pass LDS attribute");
    if (!rc) rc = hip_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "CU count");
    if (!rc)
      rc = hip_check(hipOccupancyMaxActiveBlocksPerMultiprocessor(
                         &per_cu, (const void*)k_line_wave<T, MT, MODE, FIRST, CG, NW>, 64 * NW, lds),
                     "occupancy query");
    if (rc) return rc;
    resident = (cus > 0 ? cus : 1) << 8 | (per_cu > 0 ? (per_cu < 255 ? per_cu : 255) : 1);
    cache.v[dev].store(resident, std::memory_order_relaxed);
  }
  const int cus = resident >> 8, occ = resident & 255;
  auto tasks_of = [&](int axis) {
    const int o = ALLP ? 0 : 2;
    const int ta = axis == 0 ? a.n[1] : a.n[0], tb = axis == 2 ? a.n[1] : a.n[2];
    return ((ta - o) * (tb - o) + 15) / 16 * (a.sys ? a.nact : 1);
  };
  const int t0 = tasks_of(a.ax[0].axis), t1 = a.nseg == 2 ? tasks_of(a.ax[1].axis) : 0;
  // workgroups per XCD and segment with w tasks each at a time
  const int most = t0 > t1 ? t0 : t1;
  auto groups = [&](int w) { return ((most + 7) / 8 + w - 1) / w; };
  int w = (t0 + t1 + cus - 1) / cus;
  if (w < 1) w = 1;
  while (w < NW && 8 * groups(w) * a.nseg > cus) ++w;
  a.wpw = w < NW ? w : NW;
  int g = groups(a.wpw);
  const int cap = cus * occ / 8 / a.nseg;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  hipLaunchKernelGGL((k_line_wave<T, MT, MODE, FIRST, CG, NW>), dim3(8 * g * a.nseg), dim3(64 * NW), lds, s, a);
  return hip_check(hipGetLastError(), "matrix-core pass launch");
}

template <typename T, int MT, int MODE, int NW>
static int launch_wave_g(LineArgs<T>& a, int first, hipStream_t s) {
  const bool cg = a.ax[0].axis == 2;
  if constexpr (MODE == LINE_DERIV || MODE == LINE_DMUL) {
    return cg ? launch_wave_inst<T, MT, MODE, true, true, NW>(a, s) : launch_wave_inst<T, MT, MODE, true, false, NW>(a, s);
  } else {
    if (first)
      return cg ? launch_wave_inst<T, MT, MODE, true, true, NW>(a, s)
                : launch_wave_inst<T, MT, MODE, true, false, NW>(a, s);
    return cg ? launch_wave_inst<T, MT, MODE, false, true, NW>(a, s)
              : launch_wave_inst<T, MT, MODE, false, false, NW>(a, s);
  }
}

// shape 0: 8-wave workgroups for the reduced operator and its transpose (one
// table copy serves eight tasks), shape 1: 4-wave workgroups
template <typename T, int MT, int NW>
static int launch_wave_nw(LineArgs<T>& a, int mode, int first, hipStream_t s) {
  switch (mode) {
    case LINE_REDUCED: return launch_wave_g<T, MT, LINE_REDUCED, NW>(a, first, s);
    case LINE_TRANSP: return launch_wave_g<T, MT, LINE_TRANSP, NW>(a, first, s);
    case LINE_FULL: return launch_wave_g<T, MT, LINE_FULL, 4>(a, first, s);
    case LINE_DERIV: return launch_wave_g<T, MT, LINE_DERIV, 4>(a, first, s);
    case LINE_JAC:
      if constexpr (sizeof(T) == sizeof(double)) return launch_wave_g<T, MT, LINE_JAC, 4>(a, first, s);
      break;
    case LINE_DMUL:
      if constexpr (sizeof(T) == sizeof(double)) return launch_wave_g<T, MT, LINE_DMUL, 4>(a, first, s);
      break;
  }
  set_error("matrix-core pass: bad mode");
  return CHEB_ERR_INVALID_ARG;
}

template <typename T, int MT>
static int launch_pass_modes(LineArgs<T>& a, int mode, int first, hipStream_t s) {
  switch (mode) {
    case LINE_REDUCED: return launch_line_g<T, MT, LINE_REDUCED>(a, first, s);
    case LINE_TRANSP: return launch_line_g<T, MT, LINE_TRANSP>(a, first, s);
    case LINE_FULL: return launch_line_g<T, MT, LINE_FULL>(a, first, s);
    case LINE_DERIV: return launch_line_g<T, MT, LINE_DERIV>(a, first, s);
    case LINE_JAC:
      if constexpr (sizeof(T) == sizeof(double)) return launch_line_g<T, MT, LINE_JAC>(a, first, s);
      break;
    case LINE_DMUL:
      if constexpr (sizeof(T) == sizeof(double)) return launch_line_g<T, MT, LINE_DMUL>(a, first, s);
      break;
  }
  set_error("matrix-core pass: bad mode");
  return CHEB_ERR_INVALID_ARG;
}

// Three and four row blocks with at most one task per CU (a.tasks: of the pass, or
// of both axes that can share a launch, so that the choice is the same whether they
// do) go to k_line_pass: its four waves share a task's products, where k_line_wave
// would leave three of a CU's four SIMDs idle.  FP64, one launch of 4 to 250 tasks,
// N = 128: 8.7-13 us against 14.4-16; N = 96: 7.6-9.8 against 9.8-11.6; from about
// 400 tasks on k_line_wave is faster, and with two row blocks it always is.  Batches
// keep k_line_wave: their task count changes as systems finish, and the two differ
// in the rounding of a lone middle row.
template <typename T>
static int launch_few(const LineArgs<T>& a, bool* few) {
  static DeviceCache cache;
  int dev = 0;
  *few = false;
  if (a.sys) return CHEB_OK;
  if (int rc = current_device(&dev)) return rc;
  int cus = cache.v[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (int rc = hip_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "CU count")) return rc;
    cache.v[dev].store(cus, std::memory_order_relaxed);
  }
  *few = a.tasks <= cus;
  return CHEB_OK;
}

template <typename T, int MT>
int launch_line_mt(LineArgs<T>& a, int mode, int first, int shape, hipStream_t s) {
  if constexpr (MT <= kWaveMaxMT) {
    if constexpr (MT >= 3) {
      bool few = false;
      if (int rc = launch_few<T>(a, &few)) return rc;
      if (few) return launch_pass_modes<T, MT>(a, mode, first, s);
    }
    return shape == 0 ? launch_wave_nw<T, MT, 8>(a, mode, first, s) : launch_wave_nw<T, MT, 4>(a, mode, first, s);
  } else {
    return launch_pass_modes<T, MT>(a, mode, first, s);
  }
}

// the row-block counts are instantiated in files of their own (dense_f64_*.hip,
// dense_f32_*.hip) so that they compile in parallel
#define LINE_EXTERN(T, MT) extern template int launch_line_mt<T, MT>(LineArgs<T>&, int, int, int, hipStream_t)
#define LINE_INSTANCE(T, MT) template int launch_line_mt<T, MT>(LineArgs<T>&, int, int, int, hipStream_t)

}  // namespace cheb
