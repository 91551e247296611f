// toep_field.hpp -- the pupil field in the block layout of the Toeplitz passes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pwfs.h"
#include "toep_device.hpp"

namespace pwfs {

constexpr int kToepBlock = 256;

// real part of sample j' of parity q of a line (the imaginary part is 4 floats on)
__device__ __forceinline__ size_t toep_at(int Dq, int line, int jq, int q) {
  return (size_t)(line >> 4) * toep_block_floats(Dq) +
         (((jq >> 3) * 2 + q) * 2 + ((jq >> 2) & 1)) * 128 + 8 * (line & 15) + (jq & 3);
}

struct ToepFieldArgs {
  const float* opd;
  const float* amp;
  float* field;            // [frames][n_lam][Dq / 8] blocks
  long long opd_stride;
  int D, Dh, Dq, n_lam;
  double two_pi_over_lam[PWFS_MAX_LAMBDA];
};

// A exp(i 2 pi OPD / lambda) (phase formed and reduced to [-pi, pi] in float64,
// float32 sincos) in row blocks.  One thread per 2 x 2 block
// of pixels: a sample that is not finite makes its whole block NaN, so both
// parities of its row and column carry it and every output of the frame
// becomes NaN, as it does through a full transform.  The padding is zeroed: the
// passes read it against zero factors.
__device__ __forceinline__ void toep_field_body(const ToepFieldArgs& p, int bid, int tid) {
  const int per = p.Dq * p.Dq;
  const int blocks = (per + kToepBlock - 1) / kToepBlock;
  const int b = bid % blocks, fl = bid / blocks;
  const int lam = fl % p.n_lam, f = fl / p.n_lam;
  const int i = b * kToepBlock + tid;
  if (i >= per) return;
  const int yh = i / p.Dq, xh = i - yh * p.Dq;
  const bool in = yh < p.Dh && xh < p.Dh;
  const float* o = p.opd + (long long)f * p.opd_stride;
  float red[4], amp[4], bad = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int at = in ? (2 * yh + (q >> 1)) * p.D + 2 * xh + (q & 1) : 0;
    const double ph = in ? (double)o[at] * p.two_pi_over_lam[lam] : 0.0;
    const double n = rint(ph * 0.15915494309189533577);
    red[q] = (float)fma(-n, 6.283185307179586477, ph);
    amp[q] = in ? p.amp[at] : 0.f;
    bad += 0.f * red[q];
  }
  float* out = p.field + (size_t)fl * (p.Dq / 8) * toep_block_floats(p.Dq);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float sn, cs;
    sincosf(red[q] + bad, &sn, &cs);
    float* l = out + toep_at(p.Dq, (q >> 1) * p.Dq + yh, xh, q & 1);
    l[0] = amp[q] * cs;
    l[4] = amp[q] * sn;
  }
}

// ------------------------------------------------- persistent pass ----
constexpr int kToepMaxHetero = 8;

struct ToepHeteroArgs {
  ToepFieldArgs field[kToepMaxHetero];
  ToepRowArgs rows[kToepMaxHetero];
  ToepColArgs cols[kToepMaxHetero];
  int ks[kToepMaxHetero];
  int n_items[3][kToepMaxHetero];
  int order[kToepMaxHetero];
  int n_sensors, total, spin_limit;
  int* counters;   // [0] claim, [1 + 2 s] field done, [2 + 2 s] rows done
  int* flag;       // sticky error flag
};
hipError_t toep_hetero_launch(const ToepHeteroArgs& a, int grid, size_t lds, hipStream_t st);
void toep_hetero_limit();

}  // namespace pwfs
