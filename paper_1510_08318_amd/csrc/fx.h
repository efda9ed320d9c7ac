// Visibility-route (FX) image on the device: launch arguments of fx.hip (its
// host tables are built by fx_tables.cpp, declared in fx_tables.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fx_tables.h"

namespace moff {

// Visibility-route (FX) image of one integration, for cross-checks of the MOFF
// image on the device (fx.hip).  NL = 2L - 1 lags per axis, NTP = n_types^2
// ordered pairs of table types.
struct FxArgs {
  const void* E;
  const float2* gains;         // [n_chan][n_ant] or null (unit gains)
  int n_ant, n_chan, n_types;  // n_chan: channels of E, gains and out
  int c0, n_launch;            // this launch's channels c0 .. c0 + n_launch - 1 (workspace holds n_launch)
  int64_t n_time;
  int N, L, NL, xs;            // xs: side of each pair-response table
  const int* order;            // [n_ant] antennas in the order of the visibilities (FxTables)
  const int* place;            // [n_ant] each antenna's position in it
  const int* rows;             // [n_rows] lag rows that are summed, (p * n_types + q) * NL + dy
  const int* row_ptr;          // [n_rows + 1] their entries
  const uint32_t* pair_ab;     // [entries] upper-triangle index of V, kFxConjBit: read conjugated
  const uint16_t* pair_dx;     // [entries] column
  int n_rows;
  int longest;                 // entries of the longest row
  int copies;                  // of a lag row's sums per wave of the binning (set by launch_fx)
  int real_tables;             // every table entry is real
  const double* Pp;            // [N][N] power pattern (one type)
  const int* ktype_k;          // [n_types]
  const float2* xcorr;         // [NTP][xs][xs] pair responses of the tables
  const float2* tw;            // [N] exp(+2 pi i k / N)
  // samples of this launch's channels in the order of the visibilities, staged
  // for the correlators: blocks of 64 antennas x fx_step samples,
  // [n_launch][tiles][steps][planes][64][fx_step]
  int64_t t0, t1;              // time samples of this pass over them
  char* planes;
  double2* Vd;                 // [n_launch][n_ant][n_ant] sums of earlier passes, or null (one pass)
  int first, last;             // first / last pass
  float2* V;                   // [n_launch][n_ant][n_ant] workspace (upper triangle used)
  float2* H;                   // [n_launch][NTP][NL][NL], or [n_launch][L][NL] (one type), workspace
  float2* R;                   // [n_launch][NL][NL] workspace (several types; rows 0 .. L - 1 used)
  float2* Z;                   // [n_launch][L][N] workspace
  float* out;                  // [n_chan][N][N]
  double scale;
};

// One pass over samples t0 .. t1 (a.last: then the image).
hipError_t launch_fx(const FxArgs& a, bool ci4, hipStream_t st);
}  // namespace moff
