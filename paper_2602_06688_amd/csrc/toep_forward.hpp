// toep_forward.hpp -- kernels and host side of the Toeplitz form of the
// forward model (toep_device.hpp): which sensors take it, its tables and
// scratch, the flat axes of double roofs in its layout, and its launches.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstring>
#include <vector>

#include "fft_device.hpp"
#include "pwfs.h"
#include "pwfs_geom.hpp"
#include "pwfs_internal.hpp"
#include "toep_persistent.hpp"

namespace pwfs {
namespace {

constexpr int kToepBlock = 256;
constexpr double kPiT = 3.14159265358979323846264338327950288;
size_t ta256(size_t x) { return (x + 255) & ~size_t(255); }

struct ToepGeom {
  int KS, Dh, Dq;
};

ToepGeom toep_geom(const pwfs_sensor_desc& d) {
  ToepGeom t;
  t.Dh = d.n_pupil / 2;
  t.KS = (t.Dh + 15) / 16;
  t.Dq = (t.Dh + 7) & ~7;
  return t;
}

// ------------------------------------------------------------- kernels ----
template <int KS>
__global__ __launch_bounds__(kToepRowThreads, 2) void k_toep_rows(ToepRowArgs p) {
  extern __shared__ __align__(16) unsigned char toep_smem[];
  toep_rows_body<KS>(p, blockIdx.x, toep_smem, threadIdx.x);
}

template <int KS, bool SPLIT>
__global__ __launch_bounds__(kToepColThreads, toep_col_waves(KS)) void k_toep_cols(ToepColArgs p) {
  extern __shared__ __align__(16) unsigned char toep_smem[];
  toep_cols_body<KS, SPLIT>(p, blockIdx.x, toep_smem, threadIdx.x);
}

template <int KS>
__global__ __launch_bounds__(kToepColThreads, toep_col_waves(KS)) void k_toep_cols_halves(ToepColArgs p) {
  extern __shared__ __align__(16) unsigned char toep_smem[];
  toep_cols_halves_body<KS>(p, blockIdx.x, toep_smem, threadIdx.x);
}

template <int KS>
__global__ __launch_bounds__(256) void k_toep_sum(ToepColArgs p) {
  toep_sum_body<KS>(p, blockIdx.x, threadIdx.x);
}

template <int KS>
hipError_t toep_rows1(const ToepRowArgs& a, unsigned grid, hipStream_t st) {
  hipLaunchKernelGGL((k_toep_rows<KS>), dim3(grid), dim3(kToepRowThreads), (toep_lds_rows<KS>()), st, a);
  return hipGetLastError();
}
template <int KS>
hipError_t toep_cols1(const ToepColArgs& a, hipStream_t st) {
  const unsigned pairs = (unsigned)((a.lgroups + 1) / 2);
  if (a.n_parts == 1) {
    hipLaunchKernelGGL((k_toep_cols<KS, false>), dim3(pairs), dim3(kToepColThreads),
                       (toep_lds_cols<KS>(false)), st, a);
    return hipGetLastError();
  }
  if (a.halves)   // never with one tile
    hipLaunchKernelGGL((k_toep_cols_halves<(KS > 1 ? KS : 2)>), dim3((unsigned)a.lgroups * a.n_parts), dim3(kToepColThreads),
                       (toep_lds_cols<KS>(true)), st, a);
  else
    hipLaunchKernelGGL((k_toep_cols<KS, true>), dim3(pairs * a.n_parts), dim3(kToepColThreads),
                       (toep_lds_cols<KS>(true)), st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_toep_sum<KS>), dim3((unsigned)(a.lgroups * 4 * KS)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t toep_rows(int KS, const ToepRowArgs& a, unsigned grid, hipStream_t st) {
  switch (KS) {
    case 1: return toep_rows1<1>(a, grid, st);
    case 2: return toep_rows1<2>(a, grid, st);
    case 3: return toep_rows1<3>(a, grid, st);
    case 4: return toep_rows1<4>(a, grid, st);
    case 5: return toep_rows1<5>(a, grid, st);
    case 6: return toep_rows1<6>(a, grid, st);
    case 7: return toep_rows1<7>(a, grid, st);
    case 8: return toep_rows1<8>(a, grid, st);
  }
  return hipErrorInvalidValue;
}
hipError_t toep_cols(int KS, const ToepColArgs& a, hipStream_t st) {
  switch (KS) {
    case 1: return toep_cols1<1>(a, st);
    case 2: return toep_cols1<2>(a, st);
    case 3: return toep_cols1<3>(a, st);
    case 4: return toep_cols1<4>(a, st);
    case 5: return toep_cols1<5>(a, st);
    case 6: return toep_cols1<6>(a, st);
    case 7: return toep_cols1<7>(a, st);
    case 8: return toep_cols1<8>(a, st);
  }
  return hipErrorInvalidValue;
}
template <int KS>
void toep_limit1() {
  const void* fns[] = {(const void*)k_toep_rows<KS>, (const void*)k_toep_cols<KS, false>,
                       (const void*)k_toep_cols<KS, true>, (const void*)k_toep_cols_halves<(KS > 1 ? KS : 2)>};
  for (const void* fn : fns)
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      (void)hipGetLastError();
}
void toep_limits() {
  toep_limit1<1>();
  toep_limit1<2>();
  toep_limit1<3>();
  toep_limit1<4>();
  toep_limit1<5>();
  toep_limit1<6>();
  toep_limit1<7>();
  toep_limit1<8>();
}

// the field in row blocks ([frames][n_lam][Dq / 8]) for arm y of a double roof
__global__ __launch_bounds__(kToepBlock) void k_toep_field(ToepFieldArgs p, float* field, int n_lam) {
  const int per = 2 * p.Dq * p.Dq, blocks = (per + kToepBlock - 1) / kToepBlock;
  const int fl = blockIdx.x / blocks, i = (blockIdx.x - fl * blocks) * kToepBlock + threadIdx.x;
  if (i >= per) return;
  const int line = i / p.Dq;
  toep_field2(p, toep_pixels(p, fl / n_lam, line, i - line * p.Dq), fl % n_lam, line, i - line * p.Dq,
              field + ((size_t)fl * (p.Dq / 8) + (line >> 4)) * toep_block_floats(p.Dq));
}

// The flat axis of a double-roof arm without a field stop is the identity (up
// to unit phases): arm y's row output is the modulated field itself, arm x's
// column output the row output.  Both in the layouts of the Toeplitz passes.
struct ToepIdentArgs {
  const float* field;
  const float2* rx;        // [n_lam][n_a][D]
  float* rbuf;             // [frames][n_lam][cblocks][n_a] blocks
  const int2* kord;
  float* out;
  long long out_stride;
  int D, Dh, Dq, cblocks, N, n_a, n_lam, n_mod, o, win_lo, win_hi;
  float w2[PWFS_MAX_LAMBDA];
};

// Both run one thread per sample of a column block, in the block's own order, so
// that a wavefront's accesses to the row output, which bound them, are one piece
// of 512 bytes.  With the lanes along y, 16 bytes in 512 each, a sensor of 160 px
// and 200 points took 3430 us for 60 frames (FFT passes 3580), now 2315; one of
// 194 px 6580 (5030), now 4940.  Sample `i` of a block: its line, row and offset;
// a workgroup has 256 samples of one block.
struct ToepSample {
  int line, yp, yq, off;
};
__device__ __forceinline__ ToepSample toep_sample(int i) {
  const int r = i & 3, n = (i >> 2) & 15, h = (i >> 6) & 1, q = (i >> 7) & 1, g = i >> 8;
  return {n, q, 8 * g + 4 * h + r, ((2 * g + q) * 2 + h) * 128 + 8 * n + r};
}

// arm y: R[f][lam][a][x][y] = 2^20 E[f][lam][y][x] rx[lam][a][x] (padding of y
// included); one window of columns
__global__ __launch_bounds__(kToepBlock) void k_toep_rows_ident(ToepIdentArgs p) {
  const unsigned parts = p.Dq / 8;
  unsigned r = blockIdx.x / parts;
  const ToepSample t = toep_sample((blockIdx.x - r * parts) * kToepBlock + threadIdx.x);
  const int a = r % p.n_a;
  r /= p.n_a;
  const int cb = r % p.cblocks;
  r /= p.cblocks;
  const int lam = r % p.n_lam;
  const size_t fl = r;   // f n_lam + lam
  const int l = cb * kToepLines + t.line, xp = l >= p.Dq ? 1 : 0, xq = l - xp * p.Dq;
  if (xq >= p.Dh) return;
  const size_t bf = toep_block_floats(p.Dq);
  const float* e = p.field + fl * (p.Dq / 8) * bf + toep_at(p.Dq, t.yp * p.Dq + t.yq, xq, xp);
  const float2 w = p.rx[((long long)lam * p.n_a + a) * p.D + 2 * xq + xp];
  const float2 v = cmul(make_float2(e[0], e[4]), w);
  constexpr float up = (float)(1 << (kToepZExp + kToepKExp));
  float* d = p.rbuf + ((fl * p.cblocks + cb) * p.n_a + a) * bf + t.off;
  d[0] = up * v.x;
  d[4] = up * v.y;
}

// arm x: I[f][o + y][X] = sum_lam w2[lam] sum_points |R[f][lam][key][X][y]|^2
__global__ __launch_bounds__(kToepBlock) void k_toep_cols_ident(ToepIdentArgs p) {
  const unsigned parts = p.Dq / 8;
  const unsigned r = blockIdx.x / parts;
  const ToepSample t = toep_sample((blockIdx.x - r * parts) * kToepBlock + threadIdx.x);
  const int cb = r % p.cblocks;
  const size_t f = r / p.cblocks;
  const int l = cb * kToepLines + t.line, half = l / p.Dq, xq = l - half * p.Dq;   // half: window x 2 + parity
  if (xq >= p.Dh || t.yq >= p.Dh) return;
  const size_t bf = toep_block_floats(p.Dq);
  float acc = 0.f;
  for (int lam = 0; lam < p.n_lam; ++lam) {
    const float* base = p.rbuf + ((f * p.n_lam + lam) * p.cblocks + cb) * p.n_a * bf + t.off;
    float part = 0.f, val = 0.f;
    int prev = -1;
    for (int k = 0; k < p.n_mod; ++k) {
      const int a = p.kord[k].y;
      if (a != prev) {
        const float* s = base + a * bf;
        val = cabs2(make_float2(s[0], s[4]));
        prev = a;
      }
      part += val;
    }
    acc += p.w2[lam] * part;
  }
  const int X = (half >= 2 ? p.win_hi : p.win_lo) + 2 * xq + (half & 1);
  p.out[f * p.out_stride + (long long)(p.o + 2 * t.yq + t.yp) * p.N + X] = acc;
}

}  // namespace

// ---------------------------------------------------------- eligibility ----
// Window-mode sensors without a field stop (the near and the far face of a stop
// are different kernels, which take twice the products) and D <= 256 (the register
// tiles compiled), in FP32 and the split precisions.  All of these take float16 hi
// and lo parts: bfloat16 ones, at the same rate, err by 2.6e-6 where the dense DFT
// products err by 1.3e-6.  The one-term precisions keep their own products, whose
// rounding is their result.
//
// A line costs KS^2 products here and a pair of N-point transforms there.  The
// widest tiles against the shortest transforms that hold them, pupils above 224
// pixels on 512 points, gain nothing from 16 points on (100 frames of 48 points:
// 226 px 2660 us by FFT, 2920; 242 px 2880, 3390; 256 px 2900, 3150; one frame of
// 16: 54 and 64) and stay with the FFT passes; with few points (8: 752 and 737 us;
// 730 and 665) and as double roofs, whose flat axes are copies, they do not.
bool toep_eligible(const pwfs_sensor_desc& d) {
  if (d.precision == PWFS_FP16 || d.precision == PWFS_BF16) return false;
  if ((d.flags & PWFS_F_FULL_PLANE) || d.fov_lod > 0.0 || d.n_pupil > 32 * kToepMaxKS) return false;
  const int points = d.n_mod * (1 + 3 * d.src_rings * (d.src_rings + 1));
  return !(d.precision == PWFS_FP32 && !(d.flags & PWFS_F_DOUBLE_ROOF) && d.n_pupil > 224 && d.n_fft <= 512 &&
           points >= 16);
}

// column blocks per frame and key: windows x 2 parities x Dq lines
static int toep_cblocks(const Geometry& g, const ToepGeom& t) { return g.Nc / g.D * 2 * t.Dq / kToepLines; }

size_t toep_table_bytes(const pwfs_sensor_desc& d) {
  if (!toep_eligible(d)) return 0;
  const ToepGeom t = toep_geom(d);
  const Geometry g = geometry(d);
  return ta256(sizeof(uint16_t) * 2 * toep_table_len(t.KS)) +
         ta256(sizeof(float) * 2 * toep_r_len(t.KS) * (size_t)g.n_lam * g.n_a) +
         ta256(sizeof(float) * 2 * toep_r_len(t.KS) * (size_t)g.n_lam * g.n_mod);
}

// per frame: the row output, then, for the flat axis of a double roof, the field
// (the field block of a pass sits after all frames' row output)
size_t toep_scratch_frame_bytes(const pwfs_sensor_desc& d) {
  const ToepGeom t = toep_geom(d);
  const Geometry g = geometry(d);
  return sizeof(float) * toep_block_floats(t.Dq) * (size_t)g.n_lam * ((size_t)g.n_a * toep_cblocks(g, t) + (sensor_arms(d) == 2 ? t.Dq / 8 : 0));
}

// Unit sums of the split column pass, kept behind a pass's frames.  At most 256
// MiB: beyond that many blocks the chip is full without splitting.
static size_t toep_part_frame_bytes(const ToepGeom& t, const Geometry& g) {
  return sizeof(float) * 2 * 8 * t.KS * 64 * (size_t)toep_cblocks(g, t) * toep_groups(g.n_mod, g.n_lam) * g.n_lam;
}
// Workgroups that share the units of a pair of column blocks in a pass of nf
// frames: as many as make the launch shortest, 1 = the whole form.  One frame of
// the 160 px sensor is 10 workgroups of 48 points otherwise (133 us; 13 us as 160
// workgroups, and 6 us for their sum), while 100 frames of the 64 px one are 400
// (split in two they took 63 us a pass against 53).  Model, from measured passes
// of 1 to 32 frames: a point takes 0.55 + 0.075 KS^2 us with one wavefront on a
// SIMD and 0.12 KS^2 us each where they share it; the split form adds a launch
// (4 us) and a write and a read of the sums at 4 TB/s.
//
// A split pass whose workgroups leave half of the CUs idle takes the half-split
// form, a workgroup per block (one frame of 160 px, the pass: 8 points 13.2 -> 11.9
// us, 16 points 13.4 -> 11.7; a call of 240 px and 8 points 60 -> 53); with more,
// wavefronts share SIMDs and the second rotation of z costs what the halves give.
// A whole pass takes it where that is shorter: a point takes 0.55 + 0.06 KS^2 us
// there and a group's end 0.2 KS us, 0.45 KS in the whole form, which waits for
// its LDS (one frame of 80 px and 6 points, the call: 23.2 -> 19.9 us).
static int toep_parts(const ToepGeom& t, const Geometry& g, int nf, int* per_wg, int* halves) {
  const long long pairs = ((long long)nf * toep_cblocks(g, t) + 1) / 2;
  const int groups = toep_groups(g.n_mod, g.n_lam), units = g.n_lam * groups, waves = toep_col_waves(t.KS);
  const size_t bytes = toep_part_frame_bytes(t, g) * (size_t)nf;
  int parts = 1;
  *per_wg = units;
  *halves = 0;
  if (bytes > ((size_t)256 << 20)) return 1;
  const double k2 = (double)t.KS * t.KS, unit_points = (double)g.n_mod / groups;
  const double extra = 4.0 + 2.0 * (double)bytes / 4e6;
  auto cost = [&](long long wgs, int per) {
    const long long rounds = (wgs + 256 * waves - 1) / (256 * waves);
    const double share = (double)(rounds == 1 ? (wgs + 255) / 256 : waves);
    return unit_points * per * (double)rounds * std::max(0.55 + 0.075 * k2, 0.12 * k2 * share);
  };
  double best = cost(pairs, units);
  for (int s = 2; s <= units; ++s) {
    const int per = (units + s - 1) / s, n = (units + per - 1) / per;
    const double c = cost(pairs * n, per) + extra;
    if (c < best) {
      best = c;
      parts = n;
      *per_wg = per;
    }
  }
  if (t.KS == 1) return parts;
  auto lone = [&](int n) { return 2 * pairs * n <= 256; };
  if (parts > 1) {
    *halves = lone(parts);
  } else {
    best += 0.45 * t.KS * units;   // group ends
    for (int s = 2; s <= units; ++s) {
      const int per = (units + s - 1) / s, n = (units + per - 1) / per;
      const double c = per * (unit_points * (0.55 + 0.06 * k2) + 0.2 * t.KS) + extra;
      if (lone(n) && c < best) {
        best = c;
        parts = n;
        *per_wg = per;
        *halves = 1;
      }
    }
  }
  return parts;
}

// scratch of a pass of at most chunk frames: the frames', and behind them the
// unit sums of a pass that is split (each arm of a double roof is a pass)
size_t toep_scratch_bytes(const pwfs_sensor_desc& d, int chunk) {
  const ToepGeom t = toep_geom(d);
  const size_t scratch = toep_scratch_frame_bytes(d);
  size_t most = scratch * (size_t)chunk;
  for (int a = 0; a < sensor_arms(d); ++a) {
    const Geometry g = sensor_arms(d) == 2 ? arm_geometry(d, a) : geometry(d);
    const size_t frame = toep_part_frame_bytes(t, g);
    for (int nf = 1, per, halves; nf <= chunk && frame * nf <= ((size_t)256 << 20); ++nf)
      if (toep_parts(t, g, nf, &per, &halves) > 1) most = std::max(most, ta256(scratch * nf) + frame * (size_t)nf);
  }
  return most;
}

int toep_frames_per_pass(const pwfs_sensor_desc& d) {
  const ToepGeom t = toep_geom(d);
  const Geometry g = geometry(d);
  // four rounds of resident column workgroups on 256 CUs, just not a fifth
  const int resident = 256 * toep_col_waves(t.KS);   // of 2 blocks each
  return std::max(1, 4 * 2 * resident / toep_cblocks(g, t));
}

int upload_toep_tables(const pwfs_sensor_desc& d, char* dst, hipStream_t st, std::vector<std::vector<char>>& keep) {
  const ToepGeom t = toep_geom(d);
  const Geometry g = geometry(d);
  const int LC = toep_copy_len(t.KS), tl = toep_table_len(t.KS), rl = toep_r_len(t.KS);
  auto c = [&](int n) { return 1.0 / (g.N * std::sin(kPiT * n / g.N)); };
  // the kernels, the rows' factors, the columns' factors: one copy
  const size_t rx_at = ta256(sizeof(uint16_t) * 2 * tl),
               ry_at = rx_at + ta256(sizeof(float) * 2 * rl * (size_t)g.n_lam * g.n_a);
  keep.emplace_back(toep_table_bytes(d), 0);
  std::vector<char>& tab = keep.back();
  uint16_t* A = (uint16_t*)tab.data();
  for (int p = 0; p < 2; ++p)
    for (int w = 0; w < 2; ++w)
      for (int u = 0; u < 32 * t.KS; ++u) {
        // entry u holds the kernel at i' - j' = 16 KS - 1 - u, i - j = 2 (i' - j') + (2 p - 1)
        const int del = 16 * t.KS - 1 - u;
        double v = 0.0;
        if (std::abs(del) < t.Dh) {
          const int n = 2 * del + 2 * p - 1;
          v = (w == 0 ? c(n) - c(n - g.S) : c(n + g.S) - c(n)) * (p ? -1.0 : 1.0) * (double)(1 << kToepKExp);
        }
        const _Float16 hi = (_Float16)v, lo = (_Float16)(v - (double)hi);
        for (int pl = 0; pl < 2; ++pl)
          for (int a = 0; a < 4; ++a)
            if (u - a >= 0) std::memcpy(&A[p * tl + ((w * 2 + pl) * 4 + a) * LC + u - a], pl ? &lo : &hi, 2);
      }
  std::vector<TiltPoint> pts;
  std::vector<double> key_tx;
  tilt_points(d, pts, key_tx);
  double wmax = 0.0;
  for (int l = 0; l < g.n_lam; ++l) wmax = std::max(wmax, d.lambda_weight[l]);
  // factors of one point: register 2 s + j2 = i, lane half h, lane n of 16:
  // sample 8 i + 4 h + (n >> 1 & 3) of parity 1 - p (n < 8) or p, part n & 1
  std::vector<std::complex<double>> z(g.D);
  auto fill = [&](size_t region, size_t at, double tilt, double sc, double sb, double scc) {
    for (int x = g.D / 2; x < g.D; ++x) {
      z[x] = std::polar(1.0, 2.0 * kPiT * sc * tilt * (x - (g.D - 1) / 2.0) / g.D);
      z[g.D - 1 - x] = std::conj(z[x]);
    }
    for (int x = 1; x < g.D; x += 2) z[x] = {-z[x].imag(), z[x].real()};   // odd samples enter times i
    float* R = (float*)(tab.data() + region) + at;
    for (int p = 0; p < 2; ++p)
      for (int jq = 0; jq < t.Dh; ++jq) {
        float* r = R + (size_t)p * rl + (((jq >> 5) * 2 + (jq >> 2 & 1)) * 16 + 2 * (jq & 3)) * 4 + (jq >> 3 & 3);
        const std::complex<double> o = z[2 * jq + 1 - p] * sb, w = z[2 * jq + p] * scc;
        r[0] = (float)o.real();
        r[4] = (float)o.imag();
        r[32] = (float)w.real();
        r[36] = (float)w.imag();
      }
  };
  const double up = std::ldexp(1.0, kToepZExp + kToepKExp);
  for (int l = 0; l < g.n_lam; ++l) {
    const double sc = d.lambda_ref_nm / d.lambda_nm[l];
    const double amp = std::sqrt(d.lambda_weight[l] / wmax);
    for (int a = 0; a < g.n_a; ++a)
      fill(rx_at, ((size_t)l * g.n_a + a) * 2 * rl, key_tx[a], sc, std::ldexp(1.0, kToepZExp), 0.5 * up);
    for (int k = 0; k < g.n_mod; ++k)
      fill(ry_at, ((size_t)l * g.n_mod + k) * 2 * rl, pts[k].ty, sc, amp * std::ldexp(1.0, -kToepKExp), 0.5 * amp);
  }
  if (hipMemcpyAsync(dst, tab.data(), tab.size(), hipMemcpyHostToDevice, st) != hipSuccess) {
    set_last_error("hipMemcpyAsync(Toeplitz tables)");
    return PWFS_EHIP;
  }
  return PWFS_OK;
}

void toep_prepare() {
  toep_limits();
  toep_hetero_limit();
}

namespace {

// Arguments of the passes of one sensor over nf frames.
struct ToepPass {
  ToepRowArgs ra;
  ToepColArgs ca;
  unsigned grid_rows, grid_cols;
};

ToepPass toep_pass(const SensorPlan& sp, const ToepGeom& t, const float* opd, long long opd_stride, float* out,
                   long long out_stride, int nf, float2* rbuf, int row_target) {
  const Geometry& g = sp.g;
  ToepPass tp{};
  float* R = (float*)rbuf;
  const int cblocks = toep_cblocks(g, t);
  const char* tb = (const char*)sp.dev[R_TOEP];
  const uint16_t* atab = (const uint16_t*)tb;
  tb += ta256(sizeof(uint16_t) * 2 * toep_table_len(t.KS));
  const float* rx = (const float*)tb;
  tb += ta256(sizeof(float) * 2 * toep_r_len(t.KS) * (size_t)g.n_lam * g.n_a);
  const float* ry = (const float*)tb;

  ToepRowArgs& ra = tp.ra;
  ToepFieldArgs& fa = ra.field;
  fa.opd = opd;
  fa.amp = (const float*)sp.dev[R_AMP];
  fa.opd_stride = opd_stride;
  fa.D = g.D;
  fa.Dh = t.Dh;
  fa.Dq = t.Dq;
  for (int l = 0; l < g.n_lam; ++l) fa.four_over_lam[l] = 4.0 / sp.desc.lambda_nm[l];
  ra.rbuf = R;
  ra.atab = atab;
  ra.rtab = rx;
  ra.Dh = t.Dh;
  ra.Dq = t.Dq;
  ra.cblocks = cblocks;
  ra.n_a = g.n_a;
  ra.n_lam = g.n_lam;
  ra.lgroups = nf * (t.Dq / 8);
  // split the keys so that a pass has row_target workgroups (two keys at a time each)
  const long long base = (long long)ra.lgroups * g.n_lam;
  const int groups =
      (int)std::min<long long>((g.n_a + 1) / 2, std::max<long long>(1, (row_target + base - 1) / base));
  ra.ag = (g.n_a + groups - 1) / groups;
  ra.n_agroups = (g.n_a + ra.ag - 1) / ra.ag;
  tp.grid_rows = (unsigned)(base * ra.n_agroups);

  ToepColArgs& ca = tp.ca;
  ca.rbuf = R;
  ca.atab = atab;
  ca.rtab = ry;
  ca.kord = (const int2*)sp.dev[R_AK];
  ca.out = out;
  ca.out_stride = out_stride;
  ca.Dh = t.Dh;
  ca.Dq = t.Dq;
  ca.cblocks = cblocks;
  ca.n_a = g.n_a;
  ca.n_lam = g.n_lam;
  ca.n_mod = g.n_mod;
  ca.N = g.N;
  ca.win_lo = g.win_lo;
  ca.win_hi = g.win_hi;
  ca.wy_lo = g.wy_lo;
  ca.wy_hi = g.wy_hi;
  ca.lgroups = nf * cblocks;
  ca.groups = toep_groups(g.n_mod, g.n_lam);
  ca.units = g.n_lam * ca.groups;
  ca.n_parts = 1;
  double wmax = 0.0;
  for (int l = 0; l < g.n_lam; ++l) wmax = std::max(wmax, sp.desc.lambda_weight[l]);
  ca.scale = (float)((sp.arms == 2 ? 0.5 : 1.0) * wmax / ((double)g.n_mod * sp.sumA2) *
                     std::ldexp(1.0, -2 * (kToepZExp + kToepKExp)));
  tp.grid_cols = (unsigned)((ca.lgroups + 1) / 2);
  return tp;
}

int toep_failed(hipError_t e, const char* what) {
  char msg[160];
  snprintf(msg, sizeof msg, "launch %s: %s", what, hipGetErrorString(e));
  set_last_error(msg);
  return PWFS_EHIP;
}

// Whether the scratch of a sensor holds `bytes`, from what a pass is about to be
// given (the layout sized it for every pass that a plan may make).
int toep_scratch_holds(const SensorPlan& sp, size_t bytes) {
  if (bytes <= sp.rbuf_bytes) return PWFS_OK;
  char msg[160];
  snprintf(msg, sizeof msg, "a pass needs %zu bytes of scratch, the plan has %zu", bytes, sp.rbuf_bytes);
  set_last_error(msg);
  return PWFS_EWORKSPACE;
}

size_t toep_lds_of(int KS) {
  switch (KS) {
    case 1: return std::max(toep_lds_rows<1>(), toep_lds_cols<1>(false));
    case 2: return std::max(toep_lds_rows<2>(), toep_lds_cols<2>(false));
    case 3: return std::max(toep_lds_rows<3>(), toep_lds_cols<3>(false));
    case 4: return std::max(toep_lds_rows<4>(), toep_lds_cols<4>(false));
    case 5: return std::max(toep_lds_rows<5>(), toep_lds_cols<5>(false));
    case 6: return std::max(toep_lds_rows<6>(), toep_lds_cols<6>(false));
    case 7: return std::max(toep_lds_rows<7>(), toep_lds_cols<7>(false));
    default: return std::max(toep_lds_rows<8>(), toep_lds_cols<8>(false));
  }
}

}  // namespace

int forward_toep(const SensorPlan& sp, const float* opd, long long opd_stride, float* out, long long out_stride,
                 int nf, float2* rbuf, hipStream_t st, Prof* prof) {
  const Geometry& g = sp.g;
  const ToepGeom t = toep_geom(sp.desc);
  ToepPass tp = toep_pass(sp, t, opd, opd_stride, out, out_stride, nf, rbuf, 512);
  size_t need = toep_scratch_frame_bytes(sp.desc) * (size_t)nf;
  if (sp.ident != 1) {
    tp.ca.n_parts = toep_parts(t, g, nf, &tp.ca.per_wg, &tp.ca.halves);
    tp.ca.part = (float*)((char*)rbuf + ta256(need));
    if (tp.ca.n_parts > 1) need = ta256(need) + toep_part_frame_bytes(t, g) * (size_t)nf;
  }
  if (const int rc = toep_scratch_holds(sp, need)) return rc;
  hipError_t e;
  int slot;
  // behind the pass's row output (the sums of a split pass lie behind it)
  float* field = (float*)rbuf + (size_t)nf * g.n_lam * g.n_a * tp.ca.cblocks * toep_block_floats(t.Dq);
  if (sp.ident == 2) {
    slot = prof->begin(st);
    const unsigned grid = (unsigned)(nf * g.n_lam * ((2 * t.Dq * t.Dq + kToepBlock - 1) / kToepBlock));
    hipLaunchKernelGGL(k_toep_field, dim3(grid), dim3(kToepBlock), 0, st, tp.ra.field, field, g.n_lam);
    if ((e = hipGetLastError()) != hipSuccess) return toep_failed(e, "k_toep_field");
    prof->end(slot, st, K_FIELD);
  }

  ToepIdentArgs ia{};
  if (sp.ident) {
    ia.field = field;
    ia.rx = (const float2*)sp.dev[R_RX];
    ia.rbuf = tp.ra.rbuf;
    ia.kord = tp.ca.kord;
    ia.out = out;
    ia.out_stride = out_stride;
    ia.D = g.D;
    ia.Dh = t.Dh;
    ia.Dq = t.Dq;
    ia.cblocks = tp.ca.cblocks;
    ia.N = g.N;
    ia.n_a = g.n_a;
    ia.n_lam = g.n_lam;
    ia.n_mod = g.n_mod;
    ia.o = g.o;
    ia.win_lo = g.win_lo;
    ia.win_hi = g.win_hi;
    for (int l = 0; l < g.n_lam; ++l)
      ia.w2[l] = (float)(0.5 * sp.desc.lambda_weight[l] / ((double)g.n_mod * sp.sumA2) *
                         std::ldexp(1.0, -2 * (kToepZExp + kToepKExp)));
  }

  slot = prof->begin(st);
  if (sp.ident == 2) {
    const unsigned grid = (unsigned)((long long)nf * g.n_lam * tp.ca.cblocks * g.n_a * (t.Dq / 8));
    hipLaunchKernelGGL(k_toep_rows_ident, dim3(grid), dim3(kToepBlock), 0, st, ia);
    e = hipGetLastError();
  } else {
    e = toep_rows(t.KS, tp.ra, tp.grid_rows, st);
  }
  if (e != hipSuccess) return toep_failed(e, "k_toep_rows");
  prof->end(slot, st, K_ROWS);

  slot = prof->begin(st);
  if (sp.ident == 1) {
    const unsigned grid = (unsigned)((long long)nf * tp.ca.cblocks * (t.Dq / 8));
    hipLaunchKernelGGL(k_toep_cols_ident, dim3(grid), dim3(kToepBlock), 0, st, ia);
    e = hipGetLastError();
  } else {
    e = toep_cols(t.KS, tp.ca, st);
  }
  if (e != hipSuccess) return toep_failed(e, "k_toep_cols");
  prof->end(slot, st, sp.desc.precision == PWFS_FP32 ? K_COLS : K_MFMA);
  return PWFS_OK;
}

// One persistent launch over the Toeplitz sensors of a plan (`which`, indices
// into the plan) for frames [f0, f0 + nf).  `counters` are cleared by the caller.
int forward_toep_hetero(pwfs_plan_s* p, const std::vector<int>& which, const float* opd, int f0, int nf, float* out,
                        int* counters, int* flag, hipStream_t st) {
  ToepHeteroArgs ha{};
  size_t lds = 0;
  std::vector<std::pair<double, int>> cost;
  for (size_t i = 0; i < which.size(); ++i) {
    const SensorPlan& sp = p->s[which[i]];
    const ToepGeom t = toep_geom(sp.desc);
    if (const int rc = toep_scratch_holds(sp, toep_scratch_frame_bytes(sp.desc) * (size_t)nf)) return rc;
    const ToepPass tp = toep_pass(sp, t, opd + sp.opd_offset + (long long)f0 * p->opd_stride,
                                  (long long)p->opd_stride, out + sp.int_offset + (long long)f0 * p->int_stride,
                                  (long long)p->int_stride, nf, sp.rbuf, p->tune.row_groups);
    ha.rows[i] = tp.ra;
    ha.cols[i] = tp.ca;
    ha.ks[i] = t.KS;
    ha.n_items[0][i] = (int)tp.grid_rows;
    ha.n_items[1][i] = (int)tp.grid_cols;
    lds = std::max(lds, toep_lds_of(t.KS));
    cost.push_back({-(double)sp.g.n_mod * sp.g.n_lam * sp.g.D * sp.g.D, (int)i});
    for (int k = 0; k < 2; ++k) ha.total += ha.n_items[k][i];
  }
  std::sort(cost.begin(), cost.end());
  for (size_t i = 0; i < cost.size(); ++i) ha.order[i] = cost[i].second;   // largest sensors claim first
  ha.n_sensors = (int)which.size();
  ha.counters = counters;
  ha.flag = flag;
  ha.spin_limit = p->tune.spin_limit != 0 ? p->tune.spin_limit : (1 << 24);
  const int slot = p->prof.begin(st);
  const hipError_t e = toep_hetero_launch(ha, p->n_cu * std::max(1, p->tune.wg_per_cu), lds, st);
  if (e != hipSuccess) return toep_failed(e, "k_toep_hetero");
  p->prof.end(slot, st, K_HETERO);
  return PWFS_OK;
}

}  // namespace pwfs
