// Tables of a context that are made on the device (tables.hip), on the null stream.
#pragma once
#include "common.h"

namespace iwdft {

// Interpolation window of `taps` points of a grid of N: shape beta, transform W0 at 0 (api.hip, grid_window), frequencies up to reach.
struct Window {
  int64_t N;
  double reach, beta, W0;
  int taps;
};
hipError_t make_chirp(float2* c, int64_t Q);  // c[n] = e^{j pi n^2 / Q}, n < Q
hipError_t make_samples(float* dec, int64_t Q, int logN, const Window& w);
hipError_t make_taps(float* taps, int64_t P, int64_t G, double unit, const Window& w);
hipError_t make_token_taps(float* taps, int64_t D, const Window& w);
hipError_t make_token_taps(double* taps, int64_t D, const Window& w);
hipError_t make_gain(float* gain, const Window& w);  // 1 / W of the frequencies 0 .. N / 4
hipError_t make_low(double2* tw, double* gain, const Window& w);

}  // namespace iwdft
