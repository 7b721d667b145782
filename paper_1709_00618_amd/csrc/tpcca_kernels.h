// Host-side launchers of the gfx950 kernels (GPU library internal).
#pragma once
#include <hip/hip_runtime.h>

#include "tpcca_internal.h"

namespace tpcca {

// Static description of a run as the host knows it (grid sizing).
struct RunHost {
  int32_t u0, u1, c0, c1, cl0, cl1;
  int64_t bin0, bin1;
  int32_t trk0, trk_cap;
  int32_t tile0, tile1;
  int32_t rows;  // how full the pad rows of the run's units are: a RowClass
  int32_t lds_unit;  // the run's units have at most this many hits (0: more), see unit_class
  int32_t many;      // the run has kManyUnits units or more (a captured launch's u1 is a capacity)
  int32_t lists;     // the cleaning lists the chain starts (the chains do not go by units)
};

// By mean hits in a pad row: which kernels sort the rows and search the
// neighbours.  The lines lie where the two kernels on their sides meet on time
// frames of few events (45 hits in a row per event; us):
//   neighbours, wave per tile / block per tile: 21 / 24 at 90 hits, 46 / 39 at
//     180, 161 / 132 at 720 (a wave takes the 64-hit lots of its tile one after
//     the other);
//   row sort, wave per row / block of 256: 18 / 30 at 270 hits, 55 / 34 at 360
//     (rows above 512 hits leave the wave form);
//   row sort, block of 256 / staged in LDS: at 1024 hits a row begins to fill
//     the staging block.
enum RowClass { kRowsSparse, kRowsShort, kRowsLong, kRowsDense };
inline int row_class(int64_t units, int64_t hits, int R) {
  const int64_t rows = units * (R + 1);
  return hits < rows * 96 ? kRowsSparse : hits < rows * 300 ? kRowsShort : hits < rows * 1024 ? kRowsLong : kRowsDense;
}

// Units of up to kLdsUnit hits (133 of a CU's 160 KB) have their chains built in
// LDS, one block per unit (kLdsUnitSmall: several blocks share a CU).  The second
// kernel sums the tracklet counts of all units before its own, which bounds the
// units.  From kManyUnits on (a block for every CU) the units up to kLdsUnitSmall
// have a launch of their own, as one of the larger blocks fills a CU, and the
// assignment is written per unit as well.
constexpr int kLdsUnitSmall = 8192, kLdsUnit = 40960, kLdsUnits = 4096;
constexpr int kManyUnits = 256;
inline int unit_class(int64_t units, int64_t largest) {
  return units > kLdsUnits ? 0 : largest <= kLdsUnitSmall ? kLdsUnitSmall : largest <= kLdsUnit ? kLdsUnit : 0;
}

// The fit's order is by unit and start hit: what the chains by units give.
inline bool plain_order(const ParamsDev &P) { return P.kf_split <= 0 && P.kf_bands <= 0 && P.kf_rows <= 0; }

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s);
hipError_t launch_write_run(const Bufs &B, int run, const RunDev &d, hipStream_t s);
hipError_t launch_grid(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
hipError_t launch_links(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
hipError_t launch_clean(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
hipError_t launch_chains(const Bufs &B, const ParamsDev &P, int run, const RunHost &h,
                         hipStream_t s);
hipError_t launch_kf(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
// Row-synchronous fit (tpcca_fit_rows.hip): its processing order and chunks
// (called by launch_chains), the fit itself (called by launch_kf).
hipError_t launch_kf_order_rows(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
hipError_t launch_kf_rows(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
// Exclusive scan of n int64 values in place (one block); sums[n] = total.
hipError_t launch_scan_tiles(int64_t *sums, int64_t n, hipStream_t s);
hipError_t launch_select(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s);
hipError_t launch_links_by_id(const Bufs &B, const int32_t *up, const int32_t *dn, int32_t *out_up,
                              int32_t *out_dn, int32_t cl_begin, int32_t n, hipStream_t s);
hipError_t launch_to_ids(const Bufs &B, const int32_t *in, int32_t *out, int64_t n, hipStream_t s);

}  // namespace tpcca
