// pwfs_mlp.hip -- matrix-core GEMM entry point and the surrogate network
// (fully connected layers with exact GELU, MSE loss, Adam) for gfx950.
//
// Every product is the "NT" tile engine of mfma_gemm.hpp on bf16 operands
// (one plane: bf16 weights and activations, fp32 accumulation) or on bf16
// hi/lo pairs (three products, ~fp32 accuracy).  Layer l maps P_l -> P_{l+1}
// features (sizes rounded up to 32, padding kept at zero).  Per layer the
// network keeps: fp32 master W [P_{l+1}][P_l] and b, Adam moments, fp32
// gradients, and 16-bit copies of W (rows = outputs) and W^T (rows =
// inputs) so that both the forward product (A W^T) and the backward data
// product (dZ W) read K-contiguous operands.  Activations are stored twice
// by the epilogue that produces them: [batch][features] for the next
// forward product and [features][batch] for the weight-gradient product
// dW = dZ^T A, whose K is the batch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "mfma_gemm.hpp"
#include "pwfs.h"
#include "pwfs_internal.hpp"

namespace pwfs {
namespace {

int mfail(int code, const char* fmt, ...) {
  char msg[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(msg, sizeof msg, fmt, ap);
  va_end(ap);
  set_last_error(msg);
  return code;
}

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }
int up32(int x) { return (x + 31) / 32 * 32; }

// E_PREDICT: the output layer without a target
enum Epi { E_STORE = 0, E_HIDDEN = 1, E_OUTPUT = 2, E_DHIDDEN = 3, E_PREDICT = 4 };

struct GemmArgs {
  const uint16_t* a;
  const uint16_t* b;
  long long a_plane, b_plane, lda, ldb;
  int M, N, K, mtiles, ntiles;
  int xcd_bits, band;     // tile order (tile_order)
  float alpha, beta;      // E_STORE: c = alpha * acc + beta * c (c is not read when beta == 0)
  float* c;               // fp32 output [M][ldc] (E_STORE, E_OUTPUT)
  long long ldc;
  const float* bias;      // [N]
  float* z;               // fp32 pre-activation (E_HIDDEN) or gradient (E_OUTPUT, E_DHIDDEN) [M][ldz]
  long long ldz;
  uint16_t* h;            // 16-bit planes [M][ldh]
  long long h_plane, ldh;
  uint16_t* ht;           // 16-bit planes [N][ldht]
  long long ht_plane, ldht;
  const float* target;    // [M][ldt] (E_OUTPUT with loss)
  long long ldt;
  float tscale, gscale;
  const float* zprev;     // [M][ldzp] (E_DHIDDEN)
  long long ldzp;
  double* loss_part;      // [grid] (E_OUTPUT with loss)
  int planes_out;
  // optional second K segment accumulated into the same tile before the
  // epilogue: acc += A2[M][K2] B2[N][K2]^T (K2 = 0: none)
  const uint16_t* a2;
  const uint16_t* b2;
  long long a2_plane, b2_plane, lda2, ldb2;
  int K2;
};

__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
  return 0.5f * (1.f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * __expf(-0.5f * x * x);
}

__device__ __forceinline__ void put16(uint16_t* base, long long plane, long long off, float v, int planes) {
  if (planes == 2) {
    uint16_t hi, lo;
    split16<false>(v, hi, lo);
    base[off] = hi;
    base[plane + off] = lo;
  } else {
    base[off] = f32_to_bf16_rne(v);
  }
}

// four elements down a column of a transposed 16-bit copy, one 8-byte store
// (off a multiple of 4 elements)
__device__ __forceinline__ void put16x4(uint16_t* base, long long plane, long long off, const float (&v)[4],
                                        int planes) {
  uint16_t hi[4], lo[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (planes == 2) split16<false>(v[r], hi[r], lo[r]);
    else hi[r] = f32_to_bf16_rne(v[r]);
  }
  *(uint2*)(base + off) = make_uint2(hi[0] | (uint32_t)hi[1] << 16, hi[2] | (uint32_t)hi[3] << 16);
  if (planes == 2)
    *(uint2*)(base + plane + off) = make_uint2(lo[0] | (uint32_t)lo[1] << 16, lo[2] | (uint32_t)lo[3] << 16);
}

// What the epilogue of a 32 x 32 tile reads, loaded before its first store: a
// load behind a store waits until the store is done (both count in order), so
// reading the bias beside each store cost a round trip per element (output layer
// of 20000 x 3200: 346 us, the same product without a bias 260 us).
template <int EPI>
struct TileAux {
  float bias = 0.f, v[16];
  // row(e): row of accumulator element e
  template <class Row>
  __device__ __forceinline__ void load(const GemmArgs& p, int n, Row row) {
    if constexpr (EPI == E_HIDDEN || EPI == E_OUTPUT || EPI == E_PREDICT) bias = p.bias[n];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const long long m = min(row(e), p.M - 1);
      v[e] = 0.f;
      if constexpr (EPI == E_STORE) {
        if (p.beta != 0.f) v[e] = p.c[m * p.ldc + n];
      } else if constexpr (EPI == E_OUTPUT) {
        if (p.target) v[e] = p.target[m * p.ldt + n];
      } else if constexpr (EPI == E_DHIDDEN) {
        v[e] = p.zprev[m * p.ldzp + n];
      }
    }
  }
};

// the epilogue of a 32 x 32 tile (column n of this lane; row(e) is the row of
// accumulator element e, of four elements consecutive; rows from p.M on are not
// written) whose accumulated values are val(e); lsum collects the squared error
// (E_OUTPUT with a target).  Transposed copies exist in training only, whose M
// (the batch) and ldht are multiples of 32: they leave in 8-byte stores.
template <int EPI, class Row, class Val>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& p, int n, Row row, Val val, double& lsum) {
  if (n >= p.N) return;
  TileAux<EPI> aux;
  aux.load(p, n, row);
#pragma unroll
  for (int e0 = 0; e0 < 16; e0 += 4) {
    float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = row(e0 + r);
      if (m >= p.M) break;
      const long long mr = m;
      const float v = val(e0 + r);
      if constexpr (EPI == E_STORE) {
        p.c[mr * p.ldc + n] = (p.beta != 0.f) ? p.alpha * v + p.beta * aux.v[e0 + r] : p.alpha * v;
      } else if constexpr (EPI == E_HIDDEN) {
        const float zz = v + aux.bias;
        t[r] = gelu_f(zz);
        put16(p.h, p.h_plane, mr * p.ldh + n, t[r], p.planes_out);
        // the pre-activation and the transposed copy serve the backward
        // pass only (absent in inference)
        if (p.z) p.z[mr * p.ldz + n] = zz;
      } else if constexpr (EPI == E_PREDICT) {
        p.c[mr * p.ldc + n] = p.alpha * (v + aux.bias);
      } else if constexpr (EPI == E_OUTPUT) {
        const float y = v + aux.bias;
        if (p.c) p.c[mr * p.ldc + n] = p.alpha * y;
        if (p.target) {
          const float d = y - aux.v[e0 + r] * p.tscale;
          lsum += (double)d * d;
          t[r] = p.gscale * d;
          p.z[mr * p.ldz + n] = t[r];
          put16(p.h, p.h_plane, mr * p.ldh + n, t[r], p.planes_out);
        }
      } else {  // E_DHIDDEN
        t[r] = v * gelu_grad_f(aux.v[e0 + r]);
        p.z[mr * p.ldz + n] = t[r];
        put16(p.h, p.h_plane, mr * p.ldh + n, t[r], p.planes_out);
      }
    }
    const int m = row(e0);
    if constexpr (EPI != E_STORE && EPI != E_PREDICT)
      if (p.ht && m < p.M) put16x4(p.ht, p.ht_plane, (long long)n * p.ldht + m, t, p.planes_out);
  }
}

// Tile of a workgroup.  Workgroups are dealt to the 8 XCDs in turn: each XCD gets
// a contiguous eighth of the tiles, in columns of `band` = kTileRows row tiles, so
// that the tiles it runs together share their operand rows in its L2.  Row by row
// (xcd_bits 0, band 1) the tiles that run together write whole rows of the output.
// Both by the same arithmetic: a branch here cost a prediction 1.2 %.
constexpr int kTileRows = 4;
__device__ __forceinline__ void tile_of(const GemmArgs& p, int b, int& mt, int& nt) {
  const int mtiles = p.mtiles, ntiles = p.ntiles, mask = (1 << p.xcd_bits) - 1;
  const int total = mtiles * ntiles, q = total >> p.xcd_bits, r = total & mask, x = b & mask;
  const int i = x * q + min(x, r) + (b >> p.xcd_bits);
  const int band = i / (p.band * ntiles), in = i - band * p.band * ntiles;
  const int rows = min(p.band, mtiles - band * p.band);
  nt = in / rows;
  mt = band * p.band + in - nt * rows;
}

// the squared error of a workgroup of 256 lanes
__device__ __forceinline__ void loss_partial(const GemmArgs& p, double lsum, int tid) {
  if (!p.loss_part) return;
  __shared__ double red[256];
  red[tid] = lsum;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) p.loss_part[blockIdx.x] = red[0];
}

template <int NPL, int EPI, int BK>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs p) {
  extern __shared__ u32x4_t lds_raw[];
  uint16_t* lds = (uint16_t*)lds_raw;
  using E = MfmaTile<NPL, false, BK>;
  const int tid = threadIdx.x;
  int mt, nt;
  tile_of(p, blockIdx.x, mt, nt);
  const int m0 = mt * kGemmTile, n0 = nt * kGemmTile;
  typename E::Ops ops;
#pragma unroll
  for (int pl = 0; pl < NPL; ++pl) {
    ops.a[pl] = p.a + pl * p.a_plane + (long long)m0 * p.lda;
    ops.b[pl] = p.b + pl * p.b_plane + (long long)n0 * p.ldb;
  }
  E eng;
  eng.zero();
  eng.run(ops, p.lda, p.M - m0, p.ldb, p.N - n0, p.K, lds, tid);
  if (p.K2 > 0) {
    typename E::Ops ops2;
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
      ops2.a[pl] = p.a2 + pl * p.a2_plane + (long long)m0 * p.lda2;
      ops2.b[pl] = p.b2 + pl * p.b2_plane + (long long)n0 * p.ldb2;
    }
    eng.run(ops2, p.lda2, p.M - m0, p.ldb2, p.N - n0, p.K2, lds, tid);
  }
  double lsum = 0.0;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
    {
      int row0, col;
      E::coord(tid, i, j, 0, row0, col);
      gemm_epilogue<EPI>(p, n0 + col, [&](int e) { return m0 + row0 + 8 * (e >> 2) + (e & 3); },
                         [&](int e) { return eng.value(i, j, e); }, lsum);
    }
  if constexpr (EPI == E_OUTPUT) loss_partial(p, lsum, tid);
}

// Products with few tiles (training batches, short inference batches): 64 x 64
// tiles, one 32 x 32 quarter per wavefront, so that they reach all CUs; their K
// steps are then too short to hide a load, and three of them are kept in flight
// in registers.  Each element sees the matrix products of k_gemm in the same
// order, so both give the same bits.
constexpr int kSmallTile = 64;
template <int NPL, int BK>
constexpr int gemm_small_stage() { return NPL * 2 * kSmallTile * (BK + 8); }   // 16-bit elements, A planes, then B

template <int NPL, int EPI, int BK>
__global__ __launch_bounds__(256) void k_gemm_small(GemmArgs p) {
  using E = MfmaTile<NPL, false, BK>;
  constexpr int DEPTH = 3, CPR = BK / 8, RPP = 256 / CPR, CH = NPL * 2 * kSmallTile / RPP, LROW = BK + 8;
  __shared__ __align__(16) uint16_t lds[2][gemm_small_stage<NPL, BK>()];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  int mt, nt;
  tile_of(p, blockIdx.x, mt, nt);
  const int m0 = mt * kSmallTile, n0 = nt * kSmallTile;
  const int nk1 = p.K / BK, steps = nk1 + p.K2 / BK;
  const int kq = (tid % CPR) * 8;
  // chunk h of a step: stage row tid / CPR + RPP h (A planes, then B planes)
  auto chunk = [&](int h, int s) {
    const int row = tid / CPR + RPP * h, pl = row / kSmallTile % NPL, r = row % kSmallTile;
    const bool is_a = RPP * h < NPL * kSmallTile, seg2 = s >= nk1;
    const long long k = (long long)(seg2 ? s - nk1 : s) * BK + kq;
    if (is_a) {
      const long long ra = min(m0 + r, p.M - 1);
      return *(const u32x4_t*)(seg2 ? p.a2 + pl * p.a2_plane + ra * p.lda2 + k : p.a + pl * p.a_plane + ra * p.lda + k);
    }
    const long long rb = min(n0 + r, p.N - 1);
    return *(const u32x4_t*)(seg2 ? p.b2 + pl * p.b2_plane + rb * p.ldb2 + k : p.b + pl * p.b_plane + rb * p.ldb + k);
  };
  u32x4_t buf[DEPTH][CH];
  auto fetch = [&](u32x4_t (&b)[CH], int s) {   // steps past the end load the last one, unused
#pragma unroll
    for (int h = 0; h < CH; ++h) b[h] = chunk(h, min(s, steps - 1));
  };
  auto stash = [&](const u32x4_t (&b)[CH], uint16_t* stage) {
#pragma unroll
    for (int h = 0; h < CH; ++h) *(u32x4_t*)(stage + (tid / CPR + RPP * h) * LROW + kq) = b[h];
  };
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  auto compute = [&](const uint16_t* stage) {
    const int r = lane & 31, kh = (lane >> 5) * 8;
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      u32x4_t fa[NPL], fb[NPL];
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) {
        fa[pl] = *(const u32x4_t*)(stage + (pl * kSmallTile + wm * 32 + r) * LROW + s * 16 + kh);
        fb[pl] = *(const u32x4_t*)(stage + ((NPL + pl) * kSmallTile + wn * 32 + r) * LROW + s * 16 + kh);
      }
      acc = E::mma(fa[0], fb[0], acc);
      if constexpr (NPL == 2) {
        acc = E::mma(fa[0], fb[1], acc);
        acc = E::mma(fa[1], fb[0], acc);
      }
    }
  };
#pragma unroll
  for (int u = 0; u < DEPTH; ++u) fetch(buf[u], u);
  stash(buf[0], lds[0]);
  fetch(buf[0], DEPTH);
  __syncthreads();
  for (int st = 0; st < steps; st += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      if (st + u >= steps) break;
      compute(lds[(st + u) & 1]);
      stash(buf[(u + 1) % DEPTH], lds[(st + u + 1) & 1]);
      fetch(buf[(u + 1) % DEPTH], st + u + 1 + DEPTH);
      __syncthreads();
    }
  }
  double lsum = 0.0;
  gemm_epilogue<EPI>(p, n0 + wn * 32 + (lane & 31),
                     [&](int e) { return m0 + wm * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); },
                     [&](int e) { return acc[e]; }, lsum);
  if constexpr (EPI == E_OUTPUT) loss_partial(p, lsum, tid);
}

// Large one-plane products (inference passes of the network, big plain
// GEMMs): the wave-specialised workgroup of mfma_gemm.hpp, a 128 x BN tile
// per workgroup with two K steps of operands in flight.  The K segments run
// as one stream of steps (the second segment's after the first's), and the
// consumers' products are those of k_gemm in the same order, so both give
// the same bits.  No loss partials (the product has no target).
constexpr int kGemmWsDepth = 2;

template <int EPI, int BN>
__global__ __launch_bounds__(64 * (2 * BN / 64 + 4)) void k_gemm_ws(GemmArgs p) {
  extern __shared__ u32x4_t lds_raw[];
  uint16_t* lds = (uint16_t*)lds_raw;
  using E = WsEngine<1, false, BN>;
  using W = WsParts<E, BN>;
  constexpr int NC = 2 * BN / 64, BK = E::BK_, CH = W::CH;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int mt, nt;
  tile_of(p, blockIdx.x, mt, nt);
  const int m0 = mt * kGemmTile, n0 = nt * BN;
  const int nk1 = p.K / BK;
  const int steps = nk1 + p.K2 / BK;

  if (wave >= NC) {
    const int pt = tid - 64 * NC;
    long long off1[CH], off2[CH];   // element offset of chunk h in segment 1 and 2 (K step 0)
    int loff[CH];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const int row = W::row(pt, h), kq = W::kq(pt, h);
      if (W::is_a(h)) {
        const long long r = min(m0 + row, p.M - 1);
        off1[h] = r * p.lda + kq;
        off2[h] = r * p.lda2 + kq;
      } else {
        const long long r = min(n0 + row, p.N - 1);
        off1[h] = r * p.ldb + kq;
        off2[h] = r * p.ldb2 + kq;
      }
      loff[h] = W::lds_offset(pt, h);
    }
    ws_produce<E, kGemmWsDepth>(lds, loff, steps, [&](u32x4_t (&b)[CH], int s) {
      const bool seg2 = s >= nk1;
      const long long k0 = (long long)(seg2 ? s - nk1 : s) * BK;
      const uint16_t* A = seg2 ? p.a2 : p.a;
      const uint16_t* B = seg2 ? p.b2 : p.b;
#pragma unroll
      for (int h = 0; h < CH; ++h)
        b[h] = *(const u32x4_t*)((W::is_a(h) ? A : B) + (seg2 ? off2[h] : off1[h]) + k0);
    });
    return;
  }

  // -------------------------------------------------------------- consumer
  const int lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  E eng;
  eng.zero();
  __syncthreads();
  for (int st = 0; st < steps; ++st) {
    eng.compute(lds + (st & 1) * E::STAGE, wm, wn, lane);
    __syncthreads();
  }
  double lsum = 0.0;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      // accumulator layout of the 32 x 32 tile (i, j) of this quarter
      gemm_epilogue<EPI>(p, n0 + wn * 64 + j * 32 + (lane & 31),
                         [&](int e) { return m0 + wm * 64 + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); },
                         [&](int e) { return eng.value(i, j, e); }, lsum);
}

// fp32 [rows][cols] (row stride ld) -> 16-bit planes [rows][ldo], zero padding up
// to Kp columns (a multiple of 4); with dst_t also the transpose [Kp][ldo_t]
// (rows a multiple of 4 then).  Up to two matrices in one launch.
struct SplitArgs {
  const float* src;
  long long ld;
  uint16_t* dst;
  long long plane, ldo;
  int rows, cols, Kp, planes;
  float scale;
  uint16_t* dst_t;
  long long plane_t, ldo_t;
  unsigned wgs;   // workgroups
};
struct SplitPair {
  SplitArgs s[2];
};

// four floats in one access of 4-byte alignment (rows of any length)
struct __attribute__((packed, aligned(4))) Float4 {
  float v[4];
};

// A thread takes four columns of a row in one load, or, with a transpose, four rows of a column: 8-byte stores into the
// transpose, 2-byte ones side by side into the rows.
__global__ __launch_bounds__(256) void k_split(SplitPair a) {
  const bool second = blockIdx.x >= a.s[0].wgs;
  const SplitArgs& p = a.s[second ? 1 : 0];
  const long long i = (long long)(blockIdx.x - (second ? a.s[0].wgs : 0u)) * 256 + threadIdx.x;
  float v[4];
  if (p.dst_t) {
    const long long rq = i / p.Kp;
    const int r = (int)rq * 4, k = (int)(i - rq * p.Kp);
    if (r >= p.rows) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = k < p.cols ? p.src[(long long)(r + q) * p.ld + k] * p.scale : 0.f;
      put16(p.dst, p.plane, (long long)(r + q) * p.ldo + k, v[q], p.planes);
    }
    put16x4(p.dst_t, p.plane_t, (long long)k * p.ldo_t + r, v, p.planes);
    return;
  }
  const int per = p.Kp / 4;
  const long long r = i / per;
  const int k = 4 * (int)(i - r * per);
  if (r >= p.rows) return;
  const float* src = p.src + r * p.ld + k;
  if (k + 4 <= p.cols) {
    const Float4 x = *(const Float4*)src;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = x.v[q] * p.scale;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = k + q < p.cols ? src[q] * p.scale : 0.f;
  }
  put16x4(p.dst, p.plane, r * p.ldo + k, v, p.planes);
}

// Column sums of an fp32 [rows][ld] matrix over its first `rows` rows (ld a
// multiple of 4).  A workgroup takes 16 columns: 4 lanes of 4 columns each, 64
// lanes down the rows, whose sums are added in LDS.  One thread per column was a
// serial chain of loads on 4 to 13 workgroups (236 us for 1024 rows, now 5 us).
constexpr int kColsumCols = 16;
struct ColsumArgs {
  const float* x[8];
  float* out[8];
  int ld[8], cols[8];
  unsigned first[9];   // first workgroup of each layer
  int n, rows;
};
__global__ __launch_bounds__(256) void k_colsum(ColsumArgs p) {
  __shared__ f32x4_t s_sum[64][4];
  const int q = threadIdx.x & 3, r0 = threadIdx.x >> 2;
  int t = 0;
  while (t + 1 < p.n && blockIdx.x >= p.first[t + 1]) ++t;
  const float* x = p.x[t];
  float* out = p.out[t];
  const int ld = p.ld[t], cols = p.cols[t], c = (blockIdx.x - p.first[t]) * kColsumCols + 4 * q;
  f32x4_t s = {0.f, 0.f, 0.f, 0.f};
  if (c < cols)
#pragma unroll 4
    for (int r = r0; r < p.rows; r += 64) s += *(const f32x4_t*)(x + (long long)r * ld + c);
  s_sum[r0][q] = s;
  __syncthreads();
  for (int w = 32; w > 0; w >>= 1) {
    if (r0 < w) s_sum[r0][q] += s_sum[r0 + w][q];
    __syncthreads();
  }
  if (r0 == 0)
    for (int e = 0; e < 4 && c + e < cols; ++e) out[c + e] = s_sum[0][q][e];
}

// one wavefront
__global__ __launch_bounds__(64) void k_loss_reduce(const double* part, int n, float scale, float* loss) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += part[i];
  for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);
  if (threadIdx.x == 0) *loss = (float)(s * scale);
}

struct AdamArgs {
  float* w;        // fp32 master [rows][cols], rows a multiple of 4
  float* m;
  float* v;
  const float* g;
  uint16_t* wq;    // 16-bit planes [rows][cols]    (nullptr for biases)
  uint16_t* wqt;   // 16-bit planes [cols][rows]
  long long plane, plane_t;
  int rows, cols;
};
constexpr int kMaxSegments = 16;   // weights and biases of 8 layers
struct AdamBatch {
  AdamArgs t[kMaxSegments];
  unsigned first[kMaxSegments + 1];   // first workgroup of each tensor
  int n, planes;
  float lr, b1, b2, eps, c1, c2;   // c1 = 1/(1-b1^t), c2 = 1/(1-b2^t)
};

// All tensors in one launch (six for a three-layer network before).  A thread
// takes four rows of a column, so that the transposed copy leaves in 8-byte
// stores.  Bound by the 32 bytes per weight that the step moves.
__global__ __launch_bounds__(256) void k_adam(AdamBatch b) {
  int t = 0;
  while (t + 1 < b.n && blockIdx.x >= b.first[t + 1]) ++t;
  const AdamArgs& p = b.t[t];
  const long long i = (long long)(blockIdx.x - b.first[t]) * 256 + threadIdx.x;
  const int rq = (int)(i / p.cols), c = (int)(i - (long long)rq * p.cols);
  if (4 * rq >= p.rows) return;
  float w4[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const long long at = (long long)(4 * rq + q) * p.cols + c;
    const float g = p.g[at];
    const float m = b.b1 * p.m[at] + (1.f - b.b1) * g;
    const float v = b.b2 * p.v[at] + (1.f - b.b2) * g * g;
    p.m[at] = m;
    p.v[at] = v;
    const float w = p.w[at] - b.lr * (m * b.c1) / (sqrtf(v * b.c2) + b.eps);
    p.w[at] = w;
    w4[q] = w;
    if (p.wq) put16(p.wq, p.plane, at, w, b.planes);
  }
  if (p.wqt) put16x4(p.wqt, p.plane_t, (long long)c * p.rows + 4 * rq, w4, b.planes);
}

// params (packed, unpadded, W as [out][in]) <-> padded master copies, all of them
// in one launch
struct ParamCopyArgs {
  const float* src;
  float* dst;
  int rows, cols, src_ld, dst_ld;
};
struct ParamCopyBatch {
  ParamCopyArgs t[kMaxSegments];
  unsigned first[kMaxSegments + 1];
  int n;
};
// a thread copies four columns of a row in one access
__global__ __launch_bounds__(256) void k_copy2d(ParamCopyBatch b) {
  int t = 0;
  while (t + 1 < b.n && blockIdx.x >= b.first[t + 1]) ++t;
  const ParamCopyArgs& p = b.t[t];
  const int i = (int)(blockIdx.x - b.first[t]) * 256 + threadIdx.x, per = (p.cols + 3) / 4;
  const int r = i / per, c = 4 * (i - r * per);
  if (r >= p.rows) return;
  const float* src = p.src + (long long)r * p.src_ld + c;
  float* dst = p.dst + (long long)r * p.dst_ld + c;
  if (c + 4 <= p.cols) {
    *(Float4*)dst = *(const Float4*)src;
  } else {
    for (int q = 0; q < 4 && c + q < p.cols; ++q) dst[q] = src[q];
  }
}

__global__ __launch_bounds__(256) void k_row_rms(const float* x, long long ld, int rows, int cols, float* out) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  double s = 0.0;
  for (int c = 0; c < cols; ++c) {
    const double v = x[(long long)r * ld + c];
    s += v * v;
  }
  out[r] = (float)sqrt(s / cols);
}

template <int NPL, int EPI, int BK>
int gemm_launch(const GemmArgs& a0, hipStream_t st) {
  GemmArgs a = a0;
  a.mtiles = (a.M + kGemmTile - 1) / kGemmTile;
  a.ntiles = (a.N + kGemmTile - 1) / kGemmTile;
  static bool lds_set = false;
  if (!lds_set) {
    if (hipFuncSetAttribute((const void*)k_gemm<NPL, EPI, BK>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)MfmaTile<NPL, false, BK>::lds_bytes()) != hipSuccess)
      (void)hipGetLastError();
    lds_set = true;
  }
  const size_t lds = MfmaTile<NPL, false, BK>::lds_bytes();
  hipLaunchKernelGGL((k_gemm<NPL, EPI, BK>), dim3((unsigned)(a.mtiles * a.ntiles)), dim3(256), lds, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_gemm: %s", hipGetErrorString(e));
  return PWFS_OK;
}

template <int NPL, int EPI, int BK>
int gemm_small_launch(const GemmArgs& a0, hipStream_t st) {
  GemmArgs a = a0;
  a.mtiles = (a.M + kSmallTile - 1) / kSmallTile;
  a.ntiles = (a.N + kSmallTile - 1) / kSmallTile;
  hipLaunchKernelGGL((k_gemm_small<NPL, EPI, BK>), dim3((unsigned)(a.mtiles * a.ntiles)), dim3(256), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_gemm_small: %s", hipGetErrorString(e));
  return PWFS_OK;
}

// One-plane products whose K is a multiple of 64 take K steps of 64 (8
// matrix products per wavefront between barriers instead of 4, so load
// latency hides behind them; same products in the same order, same bits).
// Two-plane products keep steps of 32 (their 80 KB stages allow two
// workgroups per CU; 64 would allow one).
template <int EPI, int BN>
int gemm_ws_launch(const GemmArgs& a0, hipStream_t st) {
  GemmArgs a = a0;
  a.mtiles = (a.M + kGemmTile - 1) / kGemmTile;
  a.ntiles = (a.N + BN - 1) / BN;
  const size_t lds = WsEngine<1, false, BN>::lds_bytes();
  static bool lds_set = false;
  if (!lds_set) {
    if (hipFuncSetAttribute((const void*)k_gemm_ws<EPI, BN>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess)
      (void)hipGetLastError();
    lds_set = true;
  }
  hipLaunchKernelGGL((k_gemm_ws<EPI, BN>), dim3((unsigned)(a.mtiles * a.ntiles)), dim3(64 * (2 * BN / 64 + 4)), lds,
                     st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_gemm_ws: %s", hipGetErrorString(e));
  return PWFS_OK;
}

// One-plane products with at least two rounds of wave-specialised
// workgroups on the chip (one per CU) and no loss epilogue take the
// wave-specialised tiles: 128 x 256 where that still gives four rounds,
// else 128 x 128.  The rest (two-plane products, the loss and gradient
// epilogues) take the 256-lane tiles, and so do hidden layers of at least two
// rounds of them (two workgroups share a CU): the GELU of one (43 us of vector
// issue for 20000 x 1024) runs beside the products of the other.  Predictions of a
// 500-h-h-3200 network, 256-lane and wave-specialised hidden layers: 20000
// samples, h = 1024: 440 and 451 us; h = 2048: 711 and 737; 32768, h = 1024: 562
// and 577.  With 664 tiles, 1.3 rounds, the wave-specialised ones are 1 % faster.
constexpr int kWsMinTiles = 512, kWsWideTiles = 1024, kSharedMinTiles = 1024;

// Products of few 128 x 128 tiles take 64 x 64 tiles, which reach all CUs and move
// twice the operand bytes per product.  Plain stores and predictions do up to 320
// tiles (1000 x 3072 x 1000, 192 tiles: 28 us -> 26; 1000 x 5120 x 1000, 320: 33
// either way; 3000 x 2600 x 1000, 504: 36 -> 44; 2048 x 3584 x 2000, 448: 57 ->
// 84), the epilogues of a training step up to two rounds of the chip: their reads
// and stores run beside the products of the other tiles on a CU (a step of 5120
// samples, 500-1024-1024-64, hidden layers of 320 tiles: 258 us; in 128-tiles
// 320).  Two-plane products do three times the work per load and only gain while
// tiles leave CUs idle (1000 x 3072 x 256, 192 tiles: 0.98; 400 x 7596 x 576, 240
// tiles: 38 us in 128-tiles, 44 us in 64-tiles).
template <int EPI>
bool small_tiles(int planes, int M, int N) {
  const long long tiles = (long long)((M + kGemmTile - 1) / kGemmTile) * ((N + kGemmTile - 1) / kGemmTile);
  return tiles < (planes == 2 ? 192 : EPI == E_STORE || EPI == E_PREDICT ? 320 : 512);
}

// Products whose time is the stores of the output gain nothing from operand rows
// in an XCD's L2 and lose the whole rows: those of one K step (one plane, 1000 x
// 25600 x 64: 33.9 us by rows, 35.9 in XCD bands; K = 256: 51.1, 49.2), of one row
// tile (x3, 100 x 25600 x 256: 25.8, 33) and of two or three, if they are more than
// a round of the chip (300 x 25600 x 256: 40.3, 43.7; 256 x 12800 x 256, 200 tiles:
// 26.3, 25.2; four, 500 x 25600 x 500: 77.4, 76.0).
void tile_order(GemmArgs& a) {
  const long long mt = (a.M + kGemmTile - 1) / kGemmTile, nt = (a.N + kGemmTile - 1) / kGemmTile;
  const bool by_row = a.K + a.K2 <= 64 || mt == 1 || (mt < kTileRows && mt * nt > 256);
  a.xcd_bits = by_row ? 0 : 3;
  a.band = by_row ? 1 : kTileRows;
}

template <int EPI>
int gemm_dispatch(int planes, const GemmArgs& a0, hipStream_t st) {
  if constexpr (EPI == E_OUTPUT)
    if (!a0.target) return gemm_dispatch<E_PREDICT>(planes, a0, st);
  GemmArgs a = a0;
  tile_order(a);
  if (small_tiles<EPI>(planes, a.M, a.N)) {
    if (planes == 2) return gemm_small_launch<2, EPI, 32>(a, st);
    if (a.K % 64 != 0 || a.K2 % 64 != 0) return gemm_small_launch<1, EPI, 32>(a, st);
    return gemm_small_launch<1, EPI, 64>(a, st);
  }
  if (planes == 2) return gemm_launch<2, EPI, 32>(a, st);
  if (a.K % 64 != 0 || a.K2 % 64 != 0) return gemm_launch<1, EPI, 32>(a, st);
  if constexpr (EPI != E_DHIDDEN && EPI != E_OUTPUT) {
    const long long mt = (a.M + kGemmTile - 1) / kGemmTile, tiles = mt * ((a.N + 127) / 128);
    if (!(EPI == E_HIDDEN && tiles >= kSharedMinTiles)) {
      if (mt * ((a.N + 255) / 256) >= kWsWideTiles) return gemm_ws_launch<EPI, 256>(a, st);
      if (tiles >= kWsMinTiles) return gemm_ws_launch<EPI, 128>(a, st);
    }
  }
  return gemm_launch<1, EPI, 64>(a, st);
}

SplitArgs split_args(const float* src, long long ld, int rows, int cols, int Kp, uint16_t* dst, long long plane,
                     long long ldo, int planes, float scale) {
  SplitArgs s{src, ld, dst, plane, ldo, rows, cols, Kp, planes, scale, nullptr, 0, 0, 0};
  s.wgs = (unsigned)(((long long)rows * (Kp / 4) + 255) / 256);
  return s;
}

int split_launch(const SplitArgs& s0, const SplitArgs& s1, hipStream_t st) {
  const SplitPair p{{s0, s1}};
  hipLaunchKernelGGL(k_split, dim3(s0.wgs + s1.wgs), dim3(256), 0, st, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_split: %s", hipGetErrorString(e));
  return PWFS_OK;
}

int planes_of(int precision) { return precision == PWFS_BF16X3 ? 2 : 1; }

}  // namespace
}  // namespace pwfs

using namespace pwfs;

// ================================================================ GEMM ABI ==
extern "C" int pwfs_gemm_workspace_size(int M, int N, int K, int precision, size_t* bytes) {
  if (!bytes || M < 1 || N < 1 || K < 1) return mfail(PWFS_EINVAL, "bad GEMM sizes");
  if (precision != PWFS_BF16 && precision != PWFS_BF16X3) return mfail(PWFS_EUNSUPPORTED, "precision");
  const size_t Kp = up32(K), pl = planes_of(precision);
  *bytes = a256(2 * pl * (size_t)M * Kp) + a256(2 * pl * (size_t)N * Kp);
  return PWFS_OK;
}

namespace pwfs {
namespace {

// C = alpha A B^T + beta C with the operand planes in `ws` (>= the
// pwfs_gemm_workspace_size bytes, 256-byte aligned; checked by the callers).
// k_split writes every element of both planes, K padding included, so the
// workspace needs no clearing.
int gemm_run(const float* A, long long lda, const float* B, long long ldb, float* C, long long ldc, int M, int N,
             int K, float alpha, float beta, int precision, void* ws, hipStream_t st) {
  const int Kp = up32(K), pl = planes_of(precision);
  uint16_t* a16 = (uint16_t*)ws;
  uint16_t* b16 = (uint16_t*)((char*)ws + a256(2 * pl * (size_t)M * Kp));
  const long long ap = (long long)M * Kp, bp = (long long)N * Kp;
  int rc;
  if ((rc = split_launch(split_args(A, lda, M, K, Kp, a16, ap, Kp, pl, 1.f),
                         split_args(B, ldb, N, K, Kp, b16, bp, Kp, pl, 1.f), st)))
    return rc;
  GemmArgs g{};
  g.a = a16;
  g.b = b16;
  g.a_plane = ap;
  g.b_plane = bp;
  g.lda = Kp;
  g.ldb = Kp;
  g.M = M;
  g.N = N;
  g.K = Kp;
  g.alpha = alpha;
  g.beta = beta;
  g.c = C;
  g.ldc = ldc;
  return gemm_dispatch<E_STORE>(pl, g, st);
}

int gemm_args_check(const float* A, long long lda, const float* B, long long ldb, float* C, long long ldc, int M,
                    int N, int K, int precision, size_t* need) {
  int rc = pwfs_gemm_workspace_size(M, N, K, precision, need);
  if (rc) return rc;
  if (!A || !B || !C) return mfail(PWFS_EINVAL, "NULL device pointer");
  if (lda < K || ldb < K || ldc < N) return mfail(PWFS_EINVAL, "leading dimension too small");
  return PWFS_OK;
}

// ------------------------------------------- static scratch of the GEMM ----
// pwfs_gemm_noalloc keeps its operand planes in this file-scope device array
// instead of a caller workspace.  Every GPU the library runs on holds its own
// copy for the life of the process.  In host code the array's name is only a
// stand-in: its device address is looked up once per device with
// hipGetSymbolAddress (with that device current) and only that address is
// passed to kernels.
constexpr size_t kGemmScratchBytes = PWFS_GEMM_NOALLOC_MAX_BYTES;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char scratch[kGemmScratchBytes];

std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

int scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return mfail(PWFS_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return mfail(PWFS_EUNSUPPORTED, "device index %d >= %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return mfail(PWFS_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    if (!p || ((uintptr_t)p & 255)) return mfail(PWFS_EHIP, "static scratch has no aligned device address");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return PWFS_OK;
}

}  // namespace
}  // namespace pwfs

extern "C" int pwfs_gemm(const float* A, long long lda, const float* B, long long ldb, float* C, long long ldc,
                         int M, int N, int K, float alpha, float beta, int precision, void* ws, size_t ws_bytes,
                         void* stream) {
  size_t need = 0;
  int rc = gemm_args_check(A, lda, B, ldb, C, ldc, M, N, K, precision, &need);
  if (rc) return rc;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return mfail(PWFS_EWORKSPACE, "workspace");
  return gemm_run(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, precision, ws, (hipStream_t)stream);
}

extern "C" int pwfs_gemm_noalloc(const float* A, long long lda, const float* B, long long ldb, float* C,
                                 long long ldc, int M, int N, int K, float alpha, float beta, int precision,
                                 void* stream) {
  size_t need = 0;
  int rc = gemm_args_check(A, lda, B, ldb, C, ldc, M, N, K, precision, &need);
  if (rc) return rc;
  if (need > kGemmScratchBytes)
    return mfail(PWFS_EWORKSPACE, "operand planes need %zu bytes; the static scratch holds %zu", need,
                 kGemmScratchBytes);
  void* ws = nullptr;
  if ((rc = scratch_of_current_device(&ws))) return rc;
  return gemm_run(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, precision, ws, (hipStream_t)stream);
}

extern "C" int pwfs_row_rms(const float* x, long long ld, int rows, int cols, float* out, void* stream) {
  if (!x || !out || rows < 1 || cols < 1 || ld < cols) return mfail(PWFS_EINVAL, "bad arguments");
  hipLaunchKernelGGL(k_row_rms, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, (hipStream_t)stream, x, ld,
                     rows, cols, out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_row_rms: %s", hipGetErrorString(e));
  return PWFS_OK;
}

// ================================================================= MLP ABI ==
struct pwfs_mlp_s {
  int L = 0, Bm = 0, precision = 0, planes = 1;
  long long step = 0;                        // Adam steps taken
  std::vector<int> n, P;                     // true and padded sizes, L + 1 each
  // per layer l (0..L-1)
  std::vector<float*> W, b, mW, vW, mb, vb, gW, gb;
  std::vector<uint16_t*> Wq, Wqt;            // planes [P_{l+1}][P_l], [P_l][P_{l+1}]
  // per layer boundary j (0..L): activation planes and transposes; z, dz fp32
  std::vector<uint16_t*> H, Ht, G, Gt;
  std::vector<float*> Z, dZ;
  float* Y = nullptr;
  // fixed linear term of inference (pwfs_mlp_set_linear): C [P_L][P_0] fp32
  // and its 16-bit planes holding C / c_scale (c_scale = the out_scale they
  // were made for, 0 = stale)
  float* C = nullptr;
  uint16_t* Cq = nullptr;
  bool have_linear = false;
  float c_scale = 0.f;
  double* loss_part = nullptr;
  int loss_parts = 0;
  bool have_grad = false;
};

namespace {

struct MlpLayout {
  size_t total = 0;
  std::vector<size_t> off;
};

// sizes of every region, in order; `cb` is called with each region's bytes
// squared-error partials: one per tile of the output layer, the small ones at most
int loss_parts_of(int Bm, int P) { return ((Bm + kSmallTile - 1) / kSmallTile) * ((P + kSmallTile - 1) / kSmallTile); }

template <class CB>
void mlp_regions(int L, const std::vector<int>& P, int Bm, int planes, CB cb) {
  for (int l = 0; l < L; ++l) {
    const size_t w = (size_t)P[l + 1] * P[l], bb = (size_t)P[l + 1];
    for (int r = 0; r < 4; ++r) cb(4 * w);     // W, mW, vW, gW
    for (int r = 0; r < 4; ++r) cb(4 * bb);    // b, mb, vb, gb
    cb(2 * planes * w);                        // Wq
    cb(2 * planes * w);                        // Wqt
  }
  for (int j = 0; j <= L; ++j) {
    const size_t a = (size_t)Bm * P[j];
    cb(2 * planes * a);  // H
    cb(2 * planes * a);  // Ht
    cb(2 * planes * a);  // G
    cb(2 * planes * a);  // Gt
    cb(4 * a);           // Z
    cb(4 * a);           // dZ
  }
  cb(4 * (size_t)Bm * P[L]);                   // Y
  cb(4 * (size_t)P[L] * P[0]);                 // C
  cb(2 * planes * (size_t)P[L] * P[0]);        // Cq
  cb(8 * (size_t)loss_parts_of(Bm, P[L]));     // loss partials
}

int mlp_check(int L, const int32_t* sizes, int Bm, int precision, std::vector<int>& n, std::vector<int>& P) {
  if (L < 1 || L > 8 || !sizes) return mfail(PWFS_EINVAL, "n_layers must be in [1, 8]");
  if (Bm < 32 || Bm % 32) return mfail(PWFS_EINVAL, "max_batch must be a positive multiple of 32");
  if (precision != PWFS_BF16 && precision != PWFS_BF16X3) return mfail(PWFS_EUNSUPPORTED, "precision");
  n.assign(sizes, sizes + L + 1);
  P.resize(L + 1);
  for (int j = 0; j <= L; ++j) {
    if (n[j] < 1 || n[j] > 65536) return mfail(PWFS_EINVAL, "layer size out of range");
    P[j] = up32(n[j]);
  }
  return PWFS_OK;
}

}  // namespace

extern "C" int pwfs_mlp_workspace_size(int L, const int32_t* sizes, int max_batch, int precision, size_t* bytes) {
  std::vector<int> n, P;
  int rc = mlp_check(L, sizes, max_batch, precision, n, P);
  if (rc) return rc;
  if (!bytes) return mfail(PWFS_EINVAL, "bytes is NULL");
  size_t tot = 0;
  mlp_regions(L, P, max_batch, planes_of(precision), [&](size_t b) { tot += a256(b); });
  *bytes = tot;
  return PWFS_OK;
}

extern "C" int pwfs_mlp_create(int L, const int32_t* sizes, int max_batch, int precision, void* ws, size_t ws_bytes,
                               void* stream, pwfs_mlp_t* out) {
  size_t need = 0;
  int rc = pwfs_mlp_workspace_size(L, sizes, max_batch, precision, &need);
  if (rc) return rc;
  if (!out) return mfail(PWFS_EINVAL, "out is NULL");
  *out = nullptr;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return mfail(PWFS_EWORKSPACE, "workspace missing, small or misaligned");
  pwfs_mlp_s* m = new (std::nothrow) pwfs_mlp_s();
  if (!m) return mfail(PWFS_EINVAL, "out of host memory");
  mlp_check(L, sizes, max_batch, precision, m->n, m->P);
  m->L = L;
  m->Bm = max_batch;
  m->precision = precision;
  m->planes = planes_of(precision);
  std::vector<char*> reg;
  size_t off = 0;
  mlp_regions(L, m->P, max_batch, m->planes, [&](size_t b) {
    reg.push_back((char*)ws + off);
    off += a256(b);
  });
  size_t r = 0;
  for (int l = 0; l < L; ++l) {
    m->W.push_back((float*)reg[r++]);
    m->mW.push_back((float*)reg[r++]);
    m->vW.push_back((float*)reg[r++]);
    m->gW.push_back((float*)reg[r++]);
    m->b.push_back((float*)reg[r++]);
    m->mb.push_back((float*)reg[r++]);
    m->vb.push_back((float*)reg[r++]);
    m->gb.push_back((float*)reg[r++]);
    m->Wq.push_back((uint16_t*)reg[r++]);
    m->Wqt.push_back((uint16_t*)reg[r++]);
  }
  for (int j = 0; j <= L; ++j) {
    m->H.push_back((uint16_t*)reg[r++]);
    m->Ht.push_back((uint16_t*)reg[r++]);
    m->G.push_back((uint16_t*)reg[r++]);
    m->Gt.push_back((uint16_t*)reg[r++]);
    m->Z.push_back((float*)reg[r++]);
    m->dZ.push_back((float*)reg[r++]);
  }
  m->Y = (float*)reg[r++];
  m->C = (float*)reg[r++];
  m->Cq = (uint16_t*)reg[r++];
  m->loss_part = (double*)reg[r++];
  m->loss_parts = loss_parts_of(max_batch, m->P[L]);
  // everything starts at zero: padding of every buffer must stay zero
  const hipError_t e = hipMemsetAsync(ws, 0, need, (hipStream_t)stream);
  if (e != hipSuccess) {
    delete m;
    return mfail(PWFS_EHIP, "hipMemsetAsync: %s", hipGetErrorString(e));
  }
  *out = m;
  return PWFS_OK;
}

extern "C" int pwfs_mlp_param_count(pwfs_mlp_t m, size_t* count) {
  if (!m || !count) return mfail(PWFS_EINVAL, "NULL argument");
  size_t c = 0;
  for (int l = 0; l < m->L; ++l) c += (size_t)m->n[l + 1] * m->n[l] + m->n[l + 1];
  *count = c;
  return PWFS_OK;
}

namespace {

// collects copies and issues them kMaxSegments at a time
struct Copies {
  ParamCopyBatch b{};
  void add(const float* src, int src_ld, float* dst, int dst_ld, int rows, int cols) {
    b.t[b.n] = {src, dst, rows, cols, src_ld, dst_ld};
    b.first[b.n + 1] = b.first[b.n] + (unsigned)(((long long)rows * ((cols + 3) / 4) + 255) / 256);
    ++b.n;
  }
  int launch(hipStream_t st) {
    hipLaunchKernelGGL(k_copy2d, dim3(b.first[b.n]), dim3(256), 0, st, b);
    b.n = 0;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return mfail(PWFS_EHIP, "launch k_copy2d: %s", hipGetErrorString(e));
    return PWFS_OK;
  }
};

// refresh the 16-bit weight copies from the fp32 masters (Adam with lr = 0
// on zero moments would do the same; this is explicit)
int refresh_q(pwfs_mlp_t m, int l, hipStream_t st) {
  const int rows = m->P[l + 1], cols = m->P[l];
  SplitArgs a = split_args(m->W[l], cols, rows, cols, cols, m->Wq[l], (long long)rows * cols, cols, m->planes, 1.f);
  a.dst_t = m->Wqt[l];
  a.plane_t = (long long)rows * cols;
  a.ldo_t = rows;
  return split_launch(a, SplitArgs{}, st);
}

}  // namespace

extern "C" int pwfs_mlp_set_params(pwfs_mlp_t m, const float* params, void* stream) {
  if (!m || !params) return mfail(PWFS_EINVAL, "NULL argument");
  hipStream_t st = (hipStream_t)stream;
  size_t off = 0;
  int rc;
  Copies cp;
  for (int l = 0; l < m->L; ++l) {
    const int no = m->n[l + 1], ni = m->n[l];
    cp.add(params + off, ni, m->W[l], m->P[l], no, ni);
    off += (size_t)no * ni;
    cp.add(params + off, no, m->b[l], no, 1, no);
    off += no;
  }
  if ((rc = cp.launch(st))) return rc;
  for (int l = 0; l < m->L; ++l) {
    const size_t w = (size_t)m->P[l + 1] * m->P[l];
    if (hipMemsetAsync(m->mW[l], 0, 4 * w, st) != hipSuccess || hipMemsetAsync(m->vW[l], 0, 4 * w, st) != hipSuccess ||
        hipMemsetAsync(m->mb[l], 0, 4 * (size_t)m->P[l + 1], st) != hipSuccess ||
        hipMemsetAsync(m->vb[l], 0, 4 * (size_t)m->P[l + 1], st) != hipSuccess)
      return mfail(PWFS_EHIP, "hipMemsetAsync");
    if ((rc = refresh_q(m, l, st))) return rc;
  }
  m->step = 0;
  m->have_grad = false;
  return PWFS_OK;
}

extern "C" int pwfs_mlp_get_params(pwfs_mlp_t m, float* params, void* stream) {
  if (!m || !params) return mfail(PWFS_EINVAL, "NULL argument");
  hipStream_t st = (hipStream_t)stream;
  size_t off = 0;
  Copies cp;
  for (int l = 0; l < m->L; ++l) {
    const int no = m->n[l + 1], ni = m->n[l];
    cp.add(m->W[l], m->P[l], params + off, ni, no, ni);
    off += (size_t)no * ni;
    cp.add(m->b[l], no, params + off, no, 1, no);
    off += no;
  }
  return cp.launch(st);
}

extern "C" int pwfs_mlp_set_linear(pwfs_mlp_t m, const float* C, void* stream) {
  if (!m) return mfail(PWFS_EINVAL, "NULL argument");
  if (!C) {
    m->have_linear = false;
    return PWFS_OK;
  }
  const int no = m->n[m->L], ni = m->n[0];
  // rows and columns past the true sizes stay zero (the workspace is cleared at create)
  Copies cp;
  cp.add(C, ni, m->C, m->P[0], no, ni);
  if (const int rc = cp.launch((hipStream_t)stream)) return rc;
  m->have_linear = true;
  m->c_scale = 0.f;
  return PWFS_OK;
}

// the Adam moments, each packed like the parameters: m, then v
extern "C" int pwfs_mlp_get_state(pwfs_mlp_t m, float* moments, long long* step, void* stream) {
  if (!m || !moments || !step) return mfail(PWFS_EINVAL, "NULL argument");
  hipStream_t st = (hipStream_t)stream;
  size_t count = 0;
  pwfs_mlp_param_count(m, &count);
  int rc;
  for (int which = 0; which < 2; ++which) {
    size_t off = which * count;
    Copies cp;
    for (int l = 0; l < m->L; ++l) {
      const int no = m->n[l + 1], ni = m->n[l];
      cp.add(which ? m->vW[l] : m->mW[l], m->P[l], moments + off, ni, no, ni);
      off += (size_t)no * ni;
      cp.add(which ? m->vb[l] : m->mb[l], no, moments + off, no, 1, no);
      off += no;
    }
    if ((rc = cp.launch(st))) return rc;
  }
  *step = m->step;
  return PWFS_OK;
}

extern "C" int pwfs_mlp_set_state(pwfs_mlp_t m, const float* moments, long long step, void* stream) {
  if (!m || !moments) return mfail(PWFS_EINVAL, "NULL argument");
  if (step < 0) return mfail(PWFS_EINVAL, "step must be >= 0");
  hipStream_t st = (hipStream_t)stream;
  size_t count = 0;
  pwfs_mlp_param_count(m, &count);
  int rc;
  for (int which = 0; which < 2; ++which) {
    size_t off = which * count;
    Copies cp;
    for (int l = 0; l < m->L; ++l) {
      const int no = m->n[l + 1], ni = m->n[l];
      cp.add(moments + off, ni, which ? m->vW[l] : m->mW[l], m->P[l], no, ni);
      off += (size_t)no * ni;
      cp.add(moments + off, no, which ? m->vb[l] : m->mb[l], no, 1, no);
      off += no;
    }
    if ((rc = cp.launch(st))) return rc;
  }
  m->step = step;
  return PWFS_OK;
}

namespace {

// forward through all layers; the output epilogue optionally forms the loss
// gradient against `target`
int mlp_forward(pwfs_mlp_t m, const float* x, int batch, float* y, float out_scale, const float* target,
                float tscale, hipStream_t st) {
  const int L = m->L, pl = m->planes;
  int rc;
  // input activations (and their transpose, used by dW of layer 0)
  const long long a0 = (long long)m->Bm * m->P[0];
  SplitArgs xs = split_args(x, m->n[0], batch, m->n[0], m->P[0], m->H[0], a0, m->P[0], pl, 1.f);
  if (target) {   // batch is a multiple of 32
    xs.dst_t = m->Ht[0];
    xs.plane_t = a0;
    xs.ldo_t = m->Bm;
  }
  if ((rc = split_launch(xs, SplitArgs{}, st))) return rc;
  for (int l = 0; l < L; ++l) {
    GemmArgs g{};
    g.a = m->H[l];
    g.a_plane = (long long)m->Bm * m->P[l];
    g.lda = m->P[l];
    g.b = m->Wq[l];
    g.b_plane = (long long)m->P[l + 1] * m->P[l];
    g.ldb = m->P[l];
    g.M = batch;
    g.N = m->n[l + 1];
    g.K = m->P[l];
    g.bias = m->b[l];
    g.planes_out = pl;
    const long long ap = (long long)m->Bm * m->P[l + 1];
    if (l + 1 < L) {
      g.z = target ? m->Z[l + 1] : nullptr;
      g.ldz = m->P[l + 1];
      g.h = m->H[l + 1];
      g.h_plane = ap;
      g.ldh = m->P[l + 1];
      g.ht = target ? m->Ht[l + 1] : nullptr;
      g.ht_plane = ap;
      g.ldht = m->Bm;
      if ((rc = gemm_dispatch<E_HIDDEN>(pl, g, st))) return rc;
    } else {
      g.alpha = out_scale;
      g.c = y;
      g.ldc = m->n[L];
      if (!target && m->have_linear) {
        // y = out_scale (h W^T + b) + x C^T as one product: the planes of
        // C / out_scale extend K after the layer's own weights
        if (m->c_scale != out_scale) {
          const int PL = m->P[L], P0 = m->P[0];
          if ((rc = split_launch(
                   split_args(m->C, P0, PL, P0, P0, m->Cq, (long long)PL * P0, P0, pl, 1.f / out_scale), SplitArgs{}, st)))
            return rc;
          m->c_scale = out_scale;
        }
        g.a2 = m->H[0];
        g.a2_plane = a0;
        g.lda2 = m->P[0];
        g.b2 = m->Cq;
        g.b2_plane = (long long)m->P[L] * m->P[0];
        g.ldb2 = m->P[0];
        g.K2 = m->P[0];
      }
      if (target) {
        g.target = target;
        g.ldt = m->n[L];
        g.tscale = tscale;
        g.gscale = 2.f / ((float)batch * (float)m->n[L]);
        g.z = m->dZ[L];
        g.ldz = m->P[L];
        g.h = m->G[L];
        g.h_plane = ap;
        g.ldh = m->P[L];
        g.ht = m->Gt[L];
        g.ht_plane = ap;
        g.ldht = m->Bm;
        g.loss_part = m->loss_part;
      }
      if ((rc = gemm_dispatch<E_OUTPUT>(pl, g, st))) return rc;
    }
  }
  return PWFS_OK;
}

}  // namespace

extern "C" int pwfs_mlp_forward(pwfs_mlp_t m, const float* x, int batch, float* y, float out_scale, void* stream) {
  if (!m || !x || !y) return mfail(PWFS_EINVAL, "NULL argument");
  if (batch < 1 || batch > m->Bm) return mfail(PWFS_ESTATE, "batch outside [1, max_batch]");
  if (m->have_linear && !(out_scale != 0.f && std::isfinite(out_scale)))
    return mfail(PWFS_EINVAL, "out_scale must be finite and non-zero with a linear term");
  return mlp_forward(m, x, batch, y, out_scale, nullptr, 1.f, (hipStream_t)stream);
}

extern "C" int pwfs_mlp_grad(pwfs_mlp_t m, const float* x, const float* t, int batch, float tscale, float* loss,
                             float* grads, void* stream) {
  if (!m || !x || !t) return mfail(PWFS_EINVAL, "NULL argument");
  if (batch < 32 || batch > m->Bm || batch % 32)
    return mfail(PWFS_ESTATE, "training batch must be a multiple of 32 in [32, max_batch]");
  hipStream_t st = (hipStream_t)stream;
  const int L = m->L, pl = m->planes;
  int rc = mlp_forward(m, x, batch, m->Y, 1.f, t, tscale, st);
  if (rc) return rc;
  const int tile = small_tiles<E_OUTPUT>(pl, batch, m->n[L]) ? kSmallTile : kGemmTile;
  const int tiles = ((batch + tile - 1) / tile) * ((m->n[L] + tile - 1) / tile);
  if (loss) {
    hipLaunchKernelGGL(k_loss_reduce, dim3(1), dim3(64), 0, st, m->loss_part, tiles,
                       1.f / ((float)batch * (float)m->n[L]), loss);
    if (hipGetLastError() != hipSuccess) return mfail(PWFS_EHIP, "launch k_loss_reduce");
  }
  ColsumArgs cs{};   // bias gradients of all layers, after the last product
  cs.rows = batch;
  for (int l = L - 1; l >= 0; --l) {
    // dW_l = G_{l+1}^T H_l : A = Gt_{l+1} [n_{l+1}][batch], B = Ht_l [P_l][batch], K = batch
    GemmArgs g{};
    g.a = m->Gt[l + 1];
    g.a_plane = (long long)m->Bm * m->P[l + 1];
    g.lda = m->Bm;
    g.b = m->Ht[l];
    g.b_plane = (long long)m->Bm * m->P[l];
    g.ldb = m->Bm;
    g.M = m->n[l + 1];
    g.N = m->P[l];
    g.K = batch;
    g.alpha = 1.f;
    g.c = m->gW[l];
    g.ldc = m->P[l];
    if ((rc = gemm_dispatch<E_STORE>(pl, g, st))) return rc;
    cs.x[cs.n] = m->dZ[l + 1];
    cs.out[cs.n] = m->gb[l];
    cs.ld[cs.n] = m->P[l + 1];
    cs.cols[cs.n] = m->n[l + 1];
    cs.first[cs.n + 1] = cs.first[cs.n] + (unsigned)((m->n[l + 1] + kColsumCols - 1) / kColsumCols);
    ++cs.n;
    if (l == 0) break;
    // G_l = (G_{l+1} W_l) * gelu'(Z_l) : A = G_{l+1} [batch][P_{l+1}], B = Wqt_l [P_l][P_{l+1}]
    GemmArgs d{};
    d.a = m->G[l + 1];
    d.a_plane = (long long)m->Bm * m->P[l + 1];
    d.lda = m->P[l + 1];
    d.b = m->Wqt[l];
    d.b_plane = (long long)m->P[l + 1] * m->P[l];
    d.ldb = m->P[l + 1];
    d.M = batch;
    d.N = m->n[l];
    d.K = m->P[l + 1];
    d.zprev = m->Z[l];
    d.ldzp = m->P[l];
    d.z = m->dZ[l];
    d.ldz = m->P[l];
    d.h = m->G[l];
    d.h_plane = (long long)m->Bm * m->P[l];
    d.ldh = m->P[l];
    d.ht = m->Gt[l];
    d.ht_plane = (long long)m->Bm * m->P[l];
    d.ldht = m->Bm;
    d.planes_out = pl;
    if ((rc = gemm_dispatch<E_DHIDDEN>(pl, d, st))) return rc;
  }
  hipLaunchKernelGGL(k_colsum, dim3(cs.first[cs.n]), dim3(256), 0, st, cs);
  if (hipGetLastError() != hipSuccess) return mfail(PWFS_EHIP, "launch k_colsum");
  m->have_grad = true;
  if (grads) {
    size_t off = 0;
    Copies cp;
    for (int l = 0; l < L; ++l) {
      const int no = m->n[l + 1], ni = m->n[l];
      cp.add(m->gW[l], m->P[l], grads + off, ni, no, ni);
      off += (size_t)no * ni;
      cp.add(m->gb[l], no, grads + off, no, 1, no);
      off += no;
    }
    if ((rc = cp.launch(st))) return rc;
  }
  return PWFS_OK;
}

extern "C" int pwfs_mlp_adam(pwfs_mlp_t m, float lr, float beta1, float beta2, float eps, void* stream) {
  if (!m) return mfail(PWFS_EINVAL, "NULL argument");
  if (!m->have_grad) return mfail(PWFS_ESTATE, "no gradient: call pwfs_mlp_grad first");
  if (!(lr >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
    return mfail(PWFS_EINVAL, "bad Adam hyper-parameters");
  hipStream_t st = (hipStream_t)stream;
  m->step += 1;
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, m->step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, m->step)));
  AdamBatch b{};
  b.planes = m->planes;
  b.lr = lr;
  b.b1 = beta1;
  b.b2 = beta2;
  b.eps = eps;
  b.c1 = c1;
  b.c2 = c2;
  auto add = [&](const AdamArgs& a) {
    b.t[b.n] = a;
    b.first[b.n + 1] = b.first[b.n] + (unsigned)(((long long)(a.rows / 4) * a.cols + 255) / 256);
    ++b.n;
  };
  for (int l = 0; l < m->L; ++l) {
    const int rows = m->P[l + 1], cols = m->P[l];
    const long long w = (long long)rows * cols;
    add({m->W[l], m->mW[l], m->vW[l], m->gW[l], m->Wq[l], m->Wqt[l], w, w, rows, cols});
    add({m->b[l], m->mb[l], m->vb[l], m->gb[l], nullptr, nullptr, 0, 0, rows, 1});
  }
  hipLaunchKernelGGL(k_adam, dim3(b.first[b.n]), dim3(256), 0, st, b);
  if (hipGetLastError() != hipSuccess) return mfail(PWFS_EHIP, "launch k_adam");
  return PWFS_OK;
}

extern "C" void pwfs_mlp_destroy(pwfs_mlp_t m) { delete m; }
