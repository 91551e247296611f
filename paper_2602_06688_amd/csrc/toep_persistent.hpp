// toep_persistent.hpp -- arguments of the persistent pass of the Toeplitz sensors.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pwfs.h"
#include "toep_device.hpp"

namespace pwfs {

// ------------------------------------------------- persistent pass ----
constexpr int kToepMaxHetero = 8;

struct ToepHeteroArgs {
  ToepRowArgs rows[kToepMaxHetero];
  ToepColArgs cols[kToepMaxHetero];
  int ks[kToepMaxHetero];
  int n_items[2][kToepMaxHetero];   // row and column items
  int order[kToepMaxHetero];
  int n_sensors, total, spin_limit;
  int* counters;   // [0] claim, [1 + s] rows done
  int* flag;       // sticky error flag
};
hipError_t toep_hetero_launch(const ToepHeteroArgs& a, int grid, size_t lds, hipStream_t st);
void toep_hetero_limit();

}  // namespace pwfs
