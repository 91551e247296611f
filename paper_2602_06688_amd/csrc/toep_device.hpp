// toep_device.hpp -- the pyramid's transform pair as a real Toeplitz product
// on the matrix cores of gfx950.
//
// One axis of the sensor (pad, half-pixel tilt, DFT, face mask, inverse DFT)
// maps the D pupil samples x_j to the samples e_i of its two image windows.
// The faces are half-planes shifted by -+S/2, and the half-plane projector of
// an N-periodic sequence sampled at half-integer frequencies is, exactly,
//     1/2 delta(n) + i c(n),   c(n) = 1 / (N sin(pi n / N)) for odd n, else 0,
// so, up to one unit phase per output sample,
//     e_i = 1/2 x_i + i sum_j K(i - j) x_j,
//     K(n) = c(n) - c(n - S)  (window at N/2 - S/2),
//     K(n) = c(n + S) - c(n)  (window at N/2 + S/2).
// K is real and couples only samples of opposite parity.  With the odd samples
// multiplied by i on both sides the whole map is real,
//     e_i = 1/2 z_i +- sum_j K(i - j) z_j    (+ even i, - odd i),
// and the real and imaginary parts of a line never mix: 2 D (D / 2) real
// products per part against the 16 D^2 real operations of a dense complex
// operator.  An image only needs |e|^2, so unit phases per row, column or odd
// sample drop out.
//
// Arithmetic.  K and z are split into 16-bit hi and lo parts (x = hi + lo)
// and K z = Kh zh + Kh zl + Kl zh accumulates in float32; the 1/2 z term, half
// of the energy, enters the accumulator in full float32.  K and z are scaled
// by 2^10, so no lo part that matters is a float16 subnormal.  Relative rms error
// against float64, 16 frames of the 160 px sensor: 9.9e-8 of the intensities and
// 1.85e-7 of the slopes (the float32 FFT pair: 2.5e-7 and 1.84e-7); over 50
// unmodulated sensors, whose errors no sum over points averages, 1.5e-7 and
// 1.67e-7 (2.4e-7 and 1.65e-7).
//
// Work split.  A wavefront owns 16 lines (rows, or columns) x (re, im) = the 32
// columns of a 32x32x16 product, and the outputs of one parity p in both
// windows: KS x KS product steps, KS = ceil(D / 32).  A window holds 16 KS rows
// of that parity (its last rows past D / 2 are never stored).
//  * K operand: Toeplitz, so 32 KS numbers per window, plane and parity hold
//    all of it.  They sit in LDS in four copies shifted by one, and every
//    fragment is two aligned 8-byte reads.
//  * z operand: the lines of a block are stored in the order in which the lanes
//    take them (toep_block_floats below), so that every load of a wave is 1 KB in
//    one piece (lines one after the other: 2.1 times the time of the column
//    pass).  The row pass keeps its block in LDS over all keys; the column pass
//    reads each block once per parity, straight into registers.  A lane forms z
//    in registers (the modulation factor is the same for all lines: one register
//    holds it for 8 samples, broadcast along 16 lanes by DPP) and splits the
//    samples of parity 1 - p into its own fragments; the other parity stays
//    float32 for the 1/2 z term.
//  What bounds it.  Rows: the HBM writes of their output (10.2 MB per frame of
//  the 160 px sensor; 200 frames in 410 us, 5.0 TB/s, a large copy's rate; the FFT
//  rows took 930 us).  Columns: by the counters the products are busy for 0.52 of
//  the cycles of a SIMD and the other vector instructions for 0.45; a wavefront
//  forms a point's z before its products, so that the two fill 0.97 of them
//  unless the two wavefronts of a SIMD overlap.  The clock falls to 1.4 - 1.7 GHz
//  (the same launch on zeros is 1.4 times faster); which of the two holds it has
//  not been told apart.  The products come at 0.8 of the rate of a large bf16
//  library product: 200 frames x 48 points in 1.08 - 1.29 ms against 2.30 ms for
//  the FFT columns.  Measured and slower:
//  blocks through LDS (1440 us), the four waves of a block in step with a
//  barrier (1345 us), passes small enough for the 256 MB cache (2200 us).
//  * Accumulator element 4 j + r of a lane is row 8 j + 4 (lane / 32) + r, and
//    the samples of a step are dealt to the lanes in the same order, so a
//    lane's own z are exactly the ones its accumulators need added.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fft_device.hpp"
#include "mfma_gemm.hpp"
#include "phase_device.hpp"
#include "pwfs.h"

namespace pwfs {

constexpr int kToepLines = 16;   // lines of one wavefront
constexpr int kToepMaxKS = 8;    // D <= 256
// Summation groups of a wavelength's modulation points: up to 16 over all
// wavelengths, of at least 3 points (few frames spread them over workgroups; a
// group's end costs a batch about 3% of 3 points).  4 and 5 points make two: one
// chain is the time of a frame alone (160 px, the call: 32.2 and 34.2 us, in two
// groups 27.4 and 29.3, FFT passes 27.0 and 28.2; 16 frames 42.6 and 44.7, 44.7
// and 46.8, FFT 57.8 and 61.7).
__host__ __device__ inline int toep_groups(int n_mod, int n_lam) {
  const int most = n_lam < 16 ? 16 / n_lam : 1, g = n_mod >= 4 && n_mod < 6 ? 2 : n_mod / 3;
  return g < 1 ? 1 : g < most ? g : most;
}

// elements of one shifted copy of a kernel table: 32 KS, rounded so that the
// four copies start 16 LDS banks apart
__host__ __device__ constexpr int toep_copy_len(int KS) {
  int l = 32;
  while (l < 32 * KS) l += 128;
  return l;
}
// uint16 elements of the kernel table of one parity: [window][plane][copy][len]
__host__ __device__ constexpr int toep_table_len(int KS) { return 2 * 2 * 4 * toep_copy_len(KS); }
// float4 loads of the modulation factors of one point; floats per (point, p)
__host__ __device__ constexpr int toep_r_quads(int KS) { return (2 * KS + 3) / 4; }
__host__ __device__ constexpr int toep_r_len(int KS) { return toep_r_quads(KS) * 2 * 16 * 4; }

// powers of two of the scaled operands: z 2^10, K 2^10, accumulators 2^20
constexpr int kToepZExp = 10, kToepKExp = 10;

// A block holds 16 lines: sample 8 i + 4 h + r of parity q, line n / 2, part
// n % 2 (re, im) sits at ((i 2 + q) 2 + h) 128 + 4 n + r, i < Dq / 8 (Dq: D / 2
// rounded up to 8).  Rows of a frame are its lines in the order [parity of
// y][y' < Dq], columns [window][parity of X][X' < Dq]; lines past D / 2 are
// padding.
__host__ __device__ constexpr int toep_block_floats(int Dq) { return Dq / 8 * 512; }

// real part of sample j' of parity q of a line (the imaginary part is 4 floats on)
__device__ __forceinline__ size_t toep_at(int Dq, int line, int jq, int q) {
  return (size_t)(line >> 4) * toep_block_floats(Dq) +
         (((jq >> 3) * 2 + q) * 2 + ((jq >> 2) & 1)) * 128 + 8 * (line & 15) + (jq & 3);
}

struct ToepFieldArgs {
  const float* opd;        // [frames][opd_stride]
  const float* amp;        // [D][D]
  long long opd_stride;
  int D, Dh, Dq;
  double four_over_lam[PWFS_MAX_LAMBDA];
};

// Samples 2 x' and 2 x' + 1 of a line of a frame's rows: A exp(i 2 pi OPD /
// lambda), the phase formed and reduced in float64; out points at the line's block.  A sample that is not finite makes its whole
// 2 x 2 block of pixels NaN, so both parities of its row and column carry it and
// every output of the frame becomes NaN, as it does through a full transform.
// The padding is zeroed: the passes read it against zero factors.
struct ToepPixels {
  float opd[2], amp[2], bad;
};
__device__ __forceinline__ ToepPixels toep_pixels(const ToepFieldArgs& p, int f, int line, int xh) {
  const int yp = line >= p.Dq ? 1 : 0, yh = line - yp * p.Dq;
  const bool in = yh < p.Dh && xh < p.Dh;
  const float* o = p.opd + (long long)f * p.opd_stride;
  const int at = in ? (2 * yh + yp) * p.D + 2 * xh : 0, other = in ? at + (yp ? -p.D : p.D) : 0;
  ToepPixels v;
  v.opd[0] = o[at];
  v.opd[1] = o[at + 1];
  v.bad = 0.f * o[other] + 0.f * o[other + 1];
  v.amp[0] = p.amp[at];
  v.amp[1] = p.amp[at + 1];
  if (!in) v = ToepPixels{};
  return v;
}
__device__ __forceinline__ void toep_field2(const ToepFieldArgs& p, const ToepPixels& v, int lam, int line, int xh,
                                            float* out) {
  const float bad = 0.f * v.opd[0] + 0.f * v.opd[1] + v.bad;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float sn, cs;
    sincos_quarters((double)v.opd[q] * p.four_over_lam[lam], sn, cs);
    float* l = out + toep_at(p.Dq, line & 15, xh, q);
    l[0] = v.amp[q] * cs + bad;
    l[4] = v.amp[q] * sn + bad;
  }
}

struct ToepRowArgs {
  ToepFieldArgs field;
  float* rbuf;             // [frames][n_lam][cblocks][n_a] blocks of columns, 2^20 x the row output
  const uint16_t* atab;    // [2][toep_table_len]
  const float* rtab;       // [n_lam][n_a][2][toep_r_len]
  int Dh, Dq, cblocks, n_a, n_lam;   // cblocks: column blocks per frame and key
  int lgroups;             // row blocks per wavelength (all frames)
  int ag, n_agroups;       // keys per workgroup; key groups
};

struct ToepColArgs {
  const float* rbuf;
  const uint16_t* atab;
  const float* rtab;       // [n_lam][n_mod][2][toep_r_len]
  const int2* kord;        // [n_mod] (point, key), keys ascending
  float* out;
  long long out_stride;
  int Dh, Dq, cblocks, n_a, n_lam, n_mod, N;
  int win_lo, win_hi, wy_lo, wy_hi;
  int lgroups;             // column blocks of all frames
  int groups, units;       // summation groups per wavelength; units = n_lam x groups
  int per_wg, n_parts;     // split form: units per workgroup, workgroups per pair of blocks
  int halves;              // half-split form: workgroups per block
  float* part;             // split form: [units][lgroups][2][8 KS][64] unit sums
  float scale;             // 2^-40 share / (n_mod sum A^2)
};

template <int I>
struct ToepInt {
  static constexpr int value = I;
};

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// z_k = r_k.re x_k + r_k.im y_k for 8 samples, r along the 16 lanes of rr: lane
// 2 k holds r_k.re, lane 2 k + 1 r_k.im, read in place by the DPP row broadcast
// (two instructions per sample; the compiler's own folding leaves the second
// broadcast as a move).  The s_nop covers a DPP read of a register that a
// vector instruction just wrote.
__device__ __forceinline__ void rotate8(float rr, const f32x4_t& xa, const f32x4_t& ya, const f32x4_t& xb,
                                        const f32x4_t& yb, f32x4_t& za, f32x4_t& zb) {
  float z0, z1, z2, z3, z4, z5, z6, z7;
#define PWFS_ROT_M(d, x, l) "v_mul_f32_dpp %" #d ", %8, %" #x " row_newbcast:" #l " row_mask:0xf bank_mask:0xf\n"
#define PWFS_ROT_F(d, y, l) "v_fmac_f32_dpp %" #d ", %8, %" #y " row_newbcast:" #l " row_mask:0xf bank_mask:0xf\n"
  __asm__("s_nop 1\n"
          PWFS_ROT_M(0, 9, 0) PWFS_ROT_M(1, 10, 2) PWFS_ROT_M(2, 11, 4) PWFS_ROT_M(3, 12, 6)
          PWFS_ROT_M(4, 17, 8) PWFS_ROT_M(5, 18, 10) PWFS_ROT_M(6, 19, 12) PWFS_ROT_M(7, 20, 14)
          PWFS_ROT_F(0, 13, 1) PWFS_ROT_F(1, 14, 3) PWFS_ROT_F(2, 15, 5) PWFS_ROT_F(3, 16, 7)
          PWFS_ROT_F(4, 21, 9) PWFS_ROT_F(5, 22, 11) PWFS_ROT_F(6, 23, 13) PWFS_ROT_F(7, 24, 15)
          : "=&v"(z0), "=&v"(z1), "=&v"(z2), "=&v"(z3), "=&v"(z4), "=&v"(z5), "=&v"(z6), "=&v"(z7)
          : "v"(rr), "v"(xa[0]), "v"(xa[1]), "v"(xa[2]), "v"(xa[3]), "v"(ya[0]), "v"(ya[1]), "v"(ya[2]), "v"(ya[3]),
            "v"(xb[0]), "v"(xb[1]), "v"(xb[2]), "v"(xb[3]), "v"(yb[0]), "v"(yb[1]), "v"(yb[2]), "v"(yb[3]));
#undef PWFS_ROT_M
#undef PWFS_ROT_F
  za = f32x4_t{z0, z1, z2, z3};
  zb = f32x4_t{z4, z5, z6, z7};
}
// value of the neighbouring lane (2 n <-> 2 n + 1)
__device__ __forceinline__ float lane_swap(float x) { return dpp_f<0xB1>(x); }

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

// two floats -> packed float16 hi and lo parts
__device__ __forceinline__ void toep_split(float a, float b, uint32_t& hi, uint32_t& lo) {
  const f16x2_t h = __builtin_convertvector(f32x2_t{a, b}, f16x2_t);
  hi = __builtin_bit_cast(uint32_t, h);
  f32x2_t r;   // a - h[0], b - h[1], the float16 operand read in place
  __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r[0]) : "v"(hi), "v"(a));
  __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r[1]) : "v"(hi), "v"(b));
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2_t));
}

// One wavefront's operands for one point and line group.
template <int KS>
struct ToepWave {
  static constexpr int LC = toep_copy_len(KS), PLANE = 4 * LC, WIN = 2 * PLANE, QR = toep_r_quads(KS);
  static constexpr int NM = 3;   // products per step
  u32x4_t bh[KS], bl[KS];  // z of parity 1 - p, 16-bit fragments
  // z of parity p, float32, as 1/2 z in the accumulators' scale, in whole tiles
  // of four 8-sample groups (an odd KS ends in half a tile, used twice)
  f32x16_t zt[(KS + 1) / 2];

  // z = x r of this lane's samples.  x: the block in LDS at the lane's four
  // samples of step 0 and parity 0; q: 1 - p; last: offset of the last 8 samples
  // of a parity (a block without them repeats the 8 before: their factors are
  // zero, as are those of the padding, which holds zeros); rv: factors (register 2 s + j2 holds, along
  // 16 lanes, (re, im) of the 4 samples of parity 1 - p, then of parity p);
  // sgn: -1 on re lanes, +1 on im lanes.
  __device__ __forceinline__ void form(const float* x, int q, int last, const f32x4_t (&rv)[QR], float sgn) {
    f32x4_t xa[2 * KS], xb[2 * KS];
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      const int o = i == 2 * KS - 1 ? last : 512 * i;
      xa[i] = *(const f32x4_t*)(x + o + 256 * q);
      xb[i] = *(const f32x4_t*)(x + o + 256 * (1 - q));
    }
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      const f32x4_t xq = xa[i], xp = xb[i];
      f32x4_t qs, cs, zq;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        qs[r] = sgn * lane_swap(xq[r]);
        cs[r] = sgn * lane_swap(xp[r]);
      }
      f32x4_t zp;
      rotate8(rv[i >> 2][i & 3], xq, qs, xp, cs, zq, zp);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        zt[i >> 2][4 * (i & 3) + r] = zp[r];
        if ((KS & 1) && i >= 2 * KS - 2) zt[i >> 2][4 * (i & 3) + 8 + r] = zp[r];
      }
      uint32_t h0, h1, l0 = 0, l1 = 0;
      toep_split(zq[0], zq[1], h0, l0);
      toep_split(zq[2], zq[3], h1, l1);
      bh[i >> 1][2 * (i & 1)] = h0;
      bh[i >> 1][2 * (i & 1) + 1] = h1;
      bl[i >> 1][2 * (i & 1)] = l0;
      bl[i >> 1][2 * (i & 1) + 1] = l1;
    }
  }

  // lane's offset (elements) into its parity's table for tile 0 of window 0
  __device__ __forceinline__ static int lane_base(int lane) {
    const int lr = lane & 31, h = lane >> 5, a = (3 - lr) & 3;
    return a * LC + (16 * KS - 1 - lr - a) + 4 * h;
  }
  // Tiles: the whole tiles of window 0, for odd KS the last 16 rows of both
  // windows, the whole tiles of window 1.  Window and 8-row group of rows 8 j.
  static constexpr int half = KS / 2;
  static constexpr bool shared(int t) { return (KS & 1) && t == half; }
  static constexpr int win(int t, int j) { return shared(t) ? j >> 1 : t > half - 1 + (KS & 1) ? 1 : 0; }
  static constexpr int tile_in_win(int t) { return t < half ? t : shared(t) ? half : t - half - (KS & 1); }
  static constexpr int group(int t, int j) { return 4 * tile_in_win(t) + (shared(t) ? j & 1 : j); }
  // lane offset of the shared tile beyond tile 0's: rows 16 KS - 16 ... of
  // window 0 on lanes 0-15 of a half, of window 1 on lanes 16-31
  __device__ __forceinline__ static int shared_base(int lane) {
    return (lane & 31) >= 16 ? WIN + 16 - 16 * (KS - 1) : -16 * (KS - 1);
  }

  __device__ __forceinline__ static u32x4_t frag(const uint16_t* a) {
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t lo = *(const u32x2_t*)a, hi = *(const u32x2_t*)(a + 8);
    return u32x4_t{lo[0], lo[1], hi[0], hi[1]};
  }

  // Tiles T0 .. T1 - 1 in turn: use(t, e, v) gets element e of tile t's outputs 1/2 z + K z.
  // The K fragments are read kAhead steps before their products and a tile's
  // outputs are used between the next tile's products; the scheduling barriers
  // keep that order (left to itself the compiler reads each fragment right
  // before its product and waits for it, which doubled the time of this phase).
  static constexpr int kAhead = 2, kRing = kAhead + 1;
  template <int T0 = 0, int T1 = KS, class Use>
  __device__ __forceinline__ void tiles(const uint16_t* tab, int base, int base_s, Use use) const {
    constexpr int steps = (T1 - T0) * KS;
    u32x4_t ah[kRing], al[kRing];
    f32x16_t acc[2];
    int at = 0;
    auto fetch = [&](int step) {
      const int t = T0 + step / KS, s = step % KS, q = step % kRing;
      if (s == 0) {
        at = shared(t) ? base_s : base + (win(t, 0) ? WIN : 0) - 32 * tile_in_win(t);
      }
      ah[q] = frag(tab + at + 16 * s);
      al[q] = frag(tab + at + PLANE + 16 * s);
    };
#pragma unroll
    for (int step = 0; step < kAhead && step < steps; ++step) fetch(step);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = T0; t < T1; ++t) {
      f32x16_t& a = acc[t & 1];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int step = (t - T0) * KS + s, q = step % kRing;
        if (step + kAhead < steps) fetch(step + kAhead);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          a = MfmaTile<1, true>::mma(m < 2 ? ah[q] : al[q], m == 1 ? bl[s] : bh[s], s + m == 0 ? zt[tile_in_win(t)] : a);
          const int k = s * NM + m;   // product of the tile; the previous tile's outputs are dealt over them
          if (t > T0) {
#pragma unroll
            for (int e = 16 * k / (KS * NM); e < 16 * (k + 1) / (KS * NM); ++e) use(t - 1, e, acc[(t & 1) ^ 1][e]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) use(T1 - 1, e, acc[(T1 - 1) & 1][e]);
  }
};

template <int KS>
__host__ __device__ constexpr size_t toep_lds_tab() { return sizeof(uint16_t) * 2 * toep_table_len(KS); }
template <int KS>
__host__ __device__ constexpr size_t toep_lds_block() { return sizeof(float) * 1024 * KS; }

// The kernel tables of both parities into LDS (the caller synchronises).
template <int KS>
__device__ __forceinline__ void toep_stage(uint16_t* s_tab, const uint16_t* tab, int tid, int nt) {
  constexpr int n16 = 2 * toep_table_len(KS) / 8;
  for (int i = tid; i < n16; i += nt) ((u32x4_t*)s_tab)[i] = ((const u32x4_t*)tab)[i];
}

// the wavefront's memory operations have been carried out
__device__ __forceinline__ void toep_landed() { __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------- rows ----
// 4 wavefronts share a row block: 2 parities x alternate keys.  They form the
// block's field in LDS, where it stays for all keys (a pass of its own wrote and
// read it: 31 us per 200 frames of 160 px, and a launch).  Each tile is turned around in LDS (a lane holds one line
// and 16 output samples; a column block wants 4 consecutive lines of one sample)
// and leaves in 16-byte stores, four runs of 256 contiguous bytes per
// instruction.
constexpr int kToepRowThreads = 256;
constexpr int kToepTurn = 32 * 2 * kToepLines;   // floats of one tile

template <int KS>
__host__ __device__ constexpr size_t toep_lds_rows() {
  return toep_lds_tab<KS>() + toep_lds_block<KS>() + 4 * sizeof(float) * kToepTurn;
}

template <int KS>
__device__ __forceinline__ void toep_rows_body(const ToepRowArgs& p, int bid, unsigned char* smem, int tid) {
  using W = ToepWave<KS>;
  uint16_t* s_tab = (uint16_t*)smem;
  float* s_x = (float*)(smem + toep_lds_tab<KS>());
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int par = wave & 1;
  const int lg = bid % p.lgroups;
  bid /= p.lgroups;
  const int agi = bid % p.n_agroups, lam = bid / p.n_agroups;
  const int rblocks = p.Dq / 8, bf = toep_block_floats(p.Dq);
  const int f = lg / rblocks, rb = lg - f * rblocks;
  // the field of the block's lines, 16 lanes side by side along a line; its loads
  // travel while the tables are staged
  ToepPixels px[KS];
#pragma unroll
  for (int i = 0; i < KS; ++i) px[i] = toep_pixels(p.field, f, rb * kToepLines + (tid >> 4), (tid & 15) + 16 * i);
  toep_stage<KS>(s_tab, p.atab, tid, kToepRowThreads);
#pragma unroll
  for (int i = 0; i < KS; ++i)
    if ((tid & 15) + 16 * i < p.Dq)
      toep_field2(p.field, px[i], lam, rb * kToepLines + (tid >> 4), (tid & 15) + 16 * i, s_x);
  __syncthreads();
  float* s_turn = s_x + 1024 * KS + wave * kToepTurn;
  const int a0 = agi * p.ag + (wave >> 1), a1 = min((agi + 1) * p.ag, p.n_a);
  if (a0 >= a1) return;
  const int n = lane & 31, h = lane >> 5, c = n & 1;
  const float sgn = c ? 1.f : -1.f;
  const int base = par * toep_table_len(KS) + W::lane_base(lane), base_s = base + W::shared_base(lane);
  const int last = min(512 * (2 * KS - 1), 512 * (p.Dq / 8 - 1));
  float* dst0 = p.rbuf + ((size_t)f * p.n_lam + lam) * p.n_a * p.cblocks * bf;
  // stores: this lane writes 4 lines y' ... y' + 3 of part lane / 4 % 2 of
  // sample lane / 8 of each 8
  const int srow = lane >> 3, sy = rb * kToepLines + 4 * (lane & 3), syp = sy >= p.Dq ? 1 : 0, syq = sy - syp * p.Dq;
  const int lane_off = ((syq >> 3) * 2 + syp) * 256 + (syq & 4) * 32 + (2 * srow + ((lane >> 2) & 1)) * 4;
  const float* rt = p.rtab + (((size_t)lam * p.n_a + a0) * 2 + par) * toep_r_len(KS) + (h * 16 + (lane & 15)) * 4;
  f32x4_t rv[W::QR];
#pragma unroll
  for (int i = 0; i < W::QR; ++i) rv[i] = *(const f32x4_t*)(rt + i * 128);
  W w;
#pragma unroll 1
  for (int a = a0; a < a1; a += 2) {
    w.form(s_x + 4 * lane, 1 - par, last, rv, sgn);
    rt += a + 2 < a1 ? 4 * toep_r_len(KS) : 0;
#pragma unroll
    for (int i = 0; i < W::QR; ++i) rv[i] = *(const f32x4_t*)(rt + i * 128);
    float* dst = dst0 + (size_t)a * bf;
    // opaque per iteration: the store addresses are then formed by scalar adds
    // where they are used, not hoisted out of the loop into spilled registers
    int dq = __builtin_amdgcn_readfirstlane(p.Dq), cstep = __builtin_amdgcn_readfirstlane(p.n_a * bf);
    __asm__ volatile("" : "+s"(dq), "+s"(cstep));
    auto out = [&](int t) {   // a tile in the turn buffer leaves
      wave_sync();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int win = W::win(t, j), gi = W::group(t, j);
        const f32x4_t v = *(const f32x4_t*)(s_turn + 4 * (lane + 64 * j));
        // the 8 rows are 8 lines of one column block
        const int l8 = win * 2 * dq + par * dq + 8 * gi;
        float* d = dst + (size_t)(l8 >> 4) * cstep + (l8 & 8) * 8;
        if (gi < 2 * KS - 2 || 8 * gi + srow < p.Dh) *(f32x4_t*)(d + lane_off) = v;
      }
      wave_sync();
    };
    w.tiles(s_tab, base, base_s, [&](int t, int e, float v) {
      s_turn[((8 * (e >> 2) + 4 * h + (e & 3)) * 2 + c) * kToepLines + (n >> 1)] = v;
      if (e == 15) out(t);
    });
  }
}

// ------------------------------------------------------------- columns ----
// 4 wavefronts: 2 column blocks x 2 parities.  |e|^2 is summed per group of
// consecutive modulation points in registers (re and im apart), the groups'
// sums, re and im together, in LDS: even lanes keep the even values, odd lanes
// the odd ones.  The block of the next point is touched while this point's
// products run, so that its loads find it in L2.  SPLIT (few frames): the units
// (wavelength, group) of a pair of blocks are spread over workgroups, which
// write their sums apart; toep_sum_body adds them in the same order, so both
// forms give the same bits.  Half-split (a frame or two): 1 column block x 2
// parities x 2 halves of the tiles; with one wavefront on a SIMD a point's chain
// of products is its time, and the halves' second rotation of z costs nothing.
constexpr int kToepColThreads = 256;
// waves per SIMD: the sums and z of KS >= 6 take more than half the register file
__host__ __device__ constexpr int toep_col_waves(int KS) { return KS <= 2 ? 4 : KS <= 5 ? 2 : 1; }

template <int KS>
__host__ __device__ constexpr size_t toep_lds_cols(bool split) {
  return toep_lds_tab<KS>() + (split ? 0 : 4 * sizeof(float) * 8 * KS * 64);
}

template <int KS, bool SPLIT, int T0 = 0, int T1 = KS>
__device__ __forceinline__ void toep_fold(const float (&part)[16 * KS], float* acc, bool first, int c) {
#pragma unroll
  for (int i = 8 * T0; i < 8 * T1; ++i) {
    const float a = part[2 * i] + lane_swap(part[2 * i]);
    const float b = part[2 * i + 1] + lane_swap(part[2 * i + 1]);
    const float v = c ? b : a;
    acc[i * 64] = SPLIT || first ? v : acc[i * 64] + v;
  }
}

// image row of value 2 k + c of a lane of half h, parity par; whether it exists
template <int KS>
__device__ __forceinline__ bool toep_out_row(const ToepColArgs& p, int k, int c, int h, int par, int& Y) {
  using W = ToepWave<KS>;
  const int t = k >> 3, e0 = 2 * (k & 7), j = e0 >> 2, r = e0 & 3;
  const int ii = 8 * W::group(t, j) + 4 * h + r + c;
  Y = (W::win(t, j) ? p.wy_hi : p.wy_lo) + 2 * ii + par;
  return ii < p.Dh;
}

// output column of line l of a frame (window x 2 + parity, X'); whether it exists
__device__ __forceinline__ bool toep_out_col(const ToepColArgs& p, int l, int& X) {
  const int half = l / p.Dq, xq = l - half * p.Dq;
  X = (half >= 2 ? p.win_hi : p.win_lo) + 2 * xq + (half & 1);
  return xq < p.Dh;
}

__device__ __forceinline__ int toep_group_lo(int g, int n_mod, int groups) { return g * n_mod / groups; }

// One wavefront: units u0 .. u1 - 1 of block lg, parity par, tiles T0 .. T1 - 1;
// s_tab is staged.
template <int KS, bool SPLIT, int T0 = 0, int T1 = KS>
__device__ __forceinline__ void toep_cols_wave(const ToepColArgs& p, int lg, int par, int u0, int u1,
                                               unsigned char* smem, int wave, int lane) {
  using W = ToepWave<KS>;
  uint16_t* s_tab = (uint16_t*)smem;
  float* s_acc = (float*)(smem + toep_lds_tab<KS>()) + wave * (8 * KS * 64) + lane;
  const int n = lane & 31, h = lane >> 5, c = n & 1;
  const int bf = toep_block_floats(p.Dq);
  const int f = lg / p.cblocks, cb = lg - f * p.cblocks;
  const size_t lam_stride = (size_t)p.cblocks * p.n_a * bf;
  const float* blk = p.rbuf + (size_t)f * p.n_lam * lam_stride + (size_t)cb * p.n_a * bf;
  const float sgn = c ? 1.f : -1.f;
  const int base = par * toep_table_len(KS) + W::lane_base(lane), base_s = base + W::shared_base(lane);
  const int last = min(512 * (2 * KS - 1), 512 * (p.Dq / 8 - 1));
  // 128-byte lines of a block: this wave touches its half
  const int tl0 = (par * 64 + lane) * 32, tl1 = tl0 + 128 * 32;
  const __attribute__((address_space(4))) int2* kord = (const __attribute__((address_space(4))) int2*)p.kord;
  auto entry = [&](int i) { return make_int2(kord[i].x, kord[i].y); };   // scalar loads
  const float* rt = p.rtab + (size_t)par * toep_r_len(KS) + (h * 16 + (lane & 15)) * 4;
  int lam = u0 / p.groups, g = u0 - lam * p.groups;
  int pos = toep_group_lo(g, p.n_mod, p.groups);
  int2 ka = entry(pos);
  pos = pos + 1 == p.n_mod ? 0 : pos + 1;   // table position of kn, the point after the current one
  int2 kn = entry(pos);
  float part[16 * KS];
  f32x4_t rv[W::QR];
#pragma unroll
  for (int k = 0; k < W::QR; ++k) rv[k] = *(const f32x4_t*)(rt + ((size_t)lam * p.n_mod + ka.x) * 2 * toep_r_len(KS) + k * 128);
  W w;
#pragma unroll 1
  for (int u = u0; u < u1; ++u) {
    const int hi = toep_group_lo(g + 1, p.n_mod, p.groups), count = hi - toep_group_lo(g, p.n_mod, p.groups);
#pragma unroll
    for (int k = 0; k < 16 * KS; ++k) part[k] = 0.f;
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      w.form(blk + lam * lam_stride + (size_t)ka.y * bf + 4 * lane, 1 - par, last, rv, sgn);
      // the next point (wavelength major), and the table entry of the one after it
      const int nl = it + 1 == count && hi == p.n_mod ? min(lam + 1, p.n_lam - 1) : lam;
      ka = kn;
      pos = pos + 1 == p.n_mod ? 0 : pos + 1;
      kn = entry(pos);
      const float* r = rt + ((size_t)nl * p.n_mod + ka.x) * 2 * toep_r_len(KS);
#pragma unroll
      for (int k = 0; k < W::QR; ++k) rv[k] = *(const f32x4_t*)(r + k * 128);
      const float* ahead = blk + nl * lam_stride + (size_t)ka.y * bf;
      const float t0 = ahead[min(tl0, bf - 1)], t1 = ahead[min(tl1, bf - 1)];
      __builtin_amdgcn_s_setprio(2);
      w.template tiles<T0, T1>(
              s_tab, base, base_s,
              [&](int t, int e, float v) { part[16 * t + e] = __builtin_fmaf(v, v, part[16 * t + e]); });
      __builtin_amdgcn_s_setprio(0);
      __asm__ volatile("" ::"v"(t0), "v"(t1));
    }
    if constexpr (SPLIT) {
      toep_fold<KS, true, T0, T1>(part, p.part + ((((size_t)u * p.lgroups + lg) * 2 + par) * 8 * KS) * 64 + lane, true, c);
    } else {
      toep_fold<KS, false>(part, s_acc, u == 0, c);
    }
    lam += hi == p.n_mod ? 1 : 0;
    g = hi == p.n_mod ? 0 : g + 1;
  }
  if constexpr (!SPLIT) {
    int X;
    if (!toep_out_col(p, cb * kToepLines + (n >> 1), X)) return;
    float* out = p.out + (long long)f * p.out_stride + X;
#pragma unroll
    for (int k = 0; k < 8 * KS; ++k) {
      int Y;
      if (toep_out_row<KS>(p, k, c, h, par, Y)) out[(size_t)Y * p.N] = s_acc[k * 64] * p.scale;
    }
  }
}

template <int KS, bool SPLIT>
__device__ __forceinline__ void toep_cols_body(const ToepColArgs& p, int bid, unsigned char* smem, int tid) {
  toep_stage<KS>((uint16_t*)smem, p.atab, tid, kToepColThreads);
  __syncthreads();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pairs = (p.lgroups + 1) / 2;
  const int lg = 2 * (SPLIT ? bid % pairs : bid) + (wave >> 1);
  const int u0 = SPLIT ? bid / pairs * p.per_wg : 0, u1 = SPLIT ? min(u0 + p.per_wg, p.units) : p.units;
  if (lg >= p.lgroups) return;
  toep_cols_wave<KS, SPLIT>(p, lg, wave & 1, u0, u1, smem, wave, lane);
}

template <int KS>
__device__ __forceinline__ void toep_cols_halves_body(const ToepColArgs& p, int bid, unsigned char* smem, int tid) {
  toep_stage<KS>((uint16_t*)smem, p.atab, tid, kToepColThreads);
  __syncthreads();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = bid % p.lgroups, u0 = bid / p.lgroups * p.per_wg, u1 = min(u0 + p.per_wg, p.units);
  constexpr int mid = (KS + 1) / 2;
  if (wave < 2)
    toep_cols_wave<KS, true, 0, mid>(p, lg, wave & 1, u0, u1, smem, wave, lane);
  else
    toep_cols_wave<KS, true, mid, KS>(p, lg, wave & 1, u0, u1, smem, wave, lane);
}

// split form: adds the units of one value of every lane, in order
template <int KS>
__device__ __forceinline__ void toep_sum_body(const ToepColArgs& p, int bid, int tid) {
  // 4 wavefronts, one (block, parity, value) each: a value's 64 lanes
  const int i = bid * 4 + (tid >> 6), lane = tid & 63;
  const int k = i % (8 * KS), bp = i / (8 * KS), par = bp & 1, lg = bp >> 1;
  if (lg >= p.lgroups) return;
  const size_t stride = (size_t)p.lgroups * 2 * 8 * KS * 64;
  const float* v = p.part + (size_t)i * 64 + lane;
  float acc = v[0];
#pragma unroll 8
  for (int u = 1; u < p.units; ++u) acc += v[u * stride];
  const int n = lane & 31, h = lane >> 5, f = lg / p.cblocks;
  int X, Y;
  if (toep_out_col(p, (lg - f * p.cblocks) * kToepLines + (n >> 1), X) &&
      toep_out_row<KS>(p, k, n & 1, h, par, Y))
    p.out[(long long)f * p.out_stride + (size_t)Y * p.N + X] = acc * p.scale;
}

}  // namespace pwfs
