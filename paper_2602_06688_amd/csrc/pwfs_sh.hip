// pwfs_sh.hip -- Shack-Hartmann wavefront sensor (the paper's SH processing
// object, Table 4; its FFT workload shapes in Table 2, e.g. 314 subapertures
// of 56 x 56 for the SCAO SH).
//
// One workgroup per (frame, subaperture), everything in LDS:
//   E[y][x]  = A exp(i 2 pi OPD / lambda) on the b x b block (phase formed and
//              reduced in float64);
//   T[y][u]  = sum_x E[y][x] W[u][x]          (b x M)
//   F[v][u]  = sum_y W[v][y] T[y][u]          (M x M, never stored)
//   pixel P  = sum over its rebin x rebin focal samples of |F|^2, in a fixed
//              order; then the centre of gravity of the n_pix x n_pix pixels.
// W[u][x] = exp(-2 pi i (u - M/2 + 1/2)(x - (b-1)/2) / M) puts the focal
// samples at half-integer frequencies (a flat wavefront's spot sits on the
// corner of the four central samples).  A 2-D DFT of a b x b block onto
// M x M samples as two small products needs no radix plan for M = 56 or 240.
//
// Both indices of W = c + i s are centred, so W[u][b-1-x] = W[M-1-u][x] =
// conj W[u][x].  With E+- = E(x) +- E(b-1-x), x < h = ceil(b / 2) (a middle
// element enters E+ once and E- as zero),
//   T[u] = C + i S,  T[M-1-u] = C - i S,  C = sum E+ c,  S = sum E- s,
// half the terms, each a complex number times a real one, and two samples from
// one pair of sums: 2 b real multiply-adds per two samples instead of 8 b.  The
// same holds for F along v, with T folded along y as it is stored.
//
// Polychromatic sensor (Table 4: PolyChromSH): the workgroup runs the three
// steps once per sampled wavelength lambda_l, with that wavelength's phase and
// its table W_l (frequencies scaled by s = lambda_ref / lambda_l: the focal
// samples are fixed in angle), and adds w_l s^2 |F_l|^2 / (M^2 sum A^2) into
// the pixels in wavelength order before the centre of gravity.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <complex>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "pwfs.h"
#include "pwfs_internal.hpp"
#include "phase_device.hpp"

namespace pwfs {
namespace {

constexpr int kShBlock = 256;
constexpr double kPiSh = 3.14159265358979323846264338327950288;

int sfail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  set_last_error(buf);
  return code;
}

struct ShArgs {
  const float* opd;        // [frames][D][D]
  const float* amp;        // [D][D]
  const float2* W;         // [n_lam][ceil(M / 2)][ceil(b / 2)]
  const uint8_t* valid;    // [n][n]
  float* pixels;           // [frames][n][n][k][k] or nullptr
  float* slopes;           // [frames][2][n][n]
  int D, n, b, M, r, k, n_lam, tpp_log2;
  float wnorm[PWFS_MAX_LAMBDA];             // w_l s_l^2 / (M^2 sum A^2) (monochromatic: 1 / (M^2 sum A^2))
  double four_over_lam[PWFS_MAX_LAMBDA];
};

// Folded sizes: h = ceil(b / 2) samples, ceil(M / 2) frequencies.  The rows of
// the (c, s) table in LDS have an odd stride, so that the rows that consecutive
// lanes read in the T product start on different banks.
__host__ __device__ constexpr int sh_half(int n) { return (n + 1) / 2; }
__host__ __device__ constexpr int sc_stride(int h) { return h | 1; }

// Threads per pair of pixels (pr, pc), (k-1-pr, pc) in the pixel loop: the
// largest power of two that keeps kShBlock threads busy without exceeding r.
__host__ __device__ inline int sh_tpp(int pairs, int r) {
  int tpp = 1;
  while (tpp * 2 * pairs <= kShBlock && tpp * 2 <= r) tpp *= 2;
  return tpp;
}

size_t sh_lds(int b, int M, int k, int nt) {
  const size_t h = sh_half(b);
  return sizeof(float4) * (h * M + 2 * h * h) + sizeof(float2) * ((size_t)sh_half(M) * sc_stride((int)h) + (size_t)b * b) +
         sizeof(float) * ((size_t)k * k + 1 + 2 * nt);
}

// H: the folded subaperture width at compile time.  A thread of a pixel pair
// keeps NC focal columns of the folded T in registers while the pair's table
// rows stream past (the lanes of one pixel row read the same ones), so a row read
// from LDS serves 2 NC samples.  NC = 4 pays where a thread owns at least four
// columns (r >= 4 tpp), for H <= 4.  NT = 128 where the pairs fill no more (the
// 8 x 8 pixels of 56 samples).  Bound by vector issue: 4 H + 8 instructions per
// two samples, where the unfolded complex products took 8 b + 4.  68 x 68
// subapertures of 7 pixels onto 240 x 240, 10 frames: 1270 -> 510 us; 20 x 20 of
// 8 pixels onto 56 x 56, 500 frames: 655 -> 290 us.
template <int H, int NC, int NT>
__global__ __launch_bounds__(NT) void k_sh(ShArgs p) {
  extern __shared__ float4 sh_mem[];
  // i / d for 0 <= i < 2^18, d <= 512, by the reciprocal (the quotient's distance
  // to an integer is at least 1 / (2 d)): an integer division is 25 instructions
  auto quot = [](int i, float inv) { return (int)(((float)i + 0.5f) * inv); };
  const int tid = threadIdx.x;
  const int sub = blockIdx.x % (p.n * p.n), f = blockIdx.x / (p.n * p.n);
  const int si = sub / p.n, sj = sub % p.n;
  const int b = p.b, M = p.M, r = p.r, k = p.k, hm = sh_half(M);
  const int kk = k * k;
  float* pix_out = p.pixels ? p.pixels + ((size_t)f * p.n * p.n + sub) * kk : nullptr;
  float* sl = p.slopes + (size_t)f * 2 * p.n * p.n;
  if (!p.valid[sub]) {   // invalid subaperture: zero slopes (and pixels)
    if (tid == 0) {
      sl[sub] = 0.f;
      sl[p.n * p.n + sub] = 0.f;
    }
    if (pix_out)
      for (int i = tid; i < kk; i += NT) pix_out[i] = 0.f;
    return;
  }
  constexpr int CW = sc_stride(H);
  float4* sT = sh_mem;                       // [H][M]: T+ (re, im), T- (re, im) of rows y, b-1-y
  float4* sF = sT + H * M;                   // [H][H][2]: E folded along y (+, -); each (x+ re, im, x- re, im)
  float2* sC = (float2*)(sF + 2 * H * H);    // [hm][CW] (c, s)
  float2* sE = sC + hm * CW;                 // [b][b]
  float* sP = (float*)(sE + b * b);          // [kk] pixel values
  float2* sR = (float2*)(sP + (kk + 1) / 2 * 2);   // [NT] partial sums of a pair

  const float* opd = p.opd + (size_t)f * p.D * p.D;
  // one pass per wavelength; the pixel loop's last barrier frees the LDS for the
  // next one
  for (int l = 0; l < p.n_lam; ++l) {
    for (int i = tid; i < hm * H; i += NT) sC[(i / H) * CW + i % H] = p.W[(size_t)l * hm * H + i];
    for (int i = tid; i < b * b; i += NT) {
      const int y = b == 2 * H ? i / (2 * H) : i / (2 * H - 1), x = i - y * b;
      const size_t g = (size_t)(si * b + y) * p.D + sj * b + x;
      float sn, cs;
      sincos_quarters((double)opd[g] * p.four_over_lam[l], sn, cs);
      const float a = p.amp[g];
      sE[i] = make_float2(a * cs, a * sn);
    }
    __syncthreads();
    for (int i = tid; i < H * H; i += NT) {
      const int y = i / H, x = i % H, yb = b - 1 - y, xb = b - 1 - x;
      const float2 e00 = sE[y * b + x];
      const float2 z = make_float2(0.f, 0.f);
      const float2 e01 = xb != x ? sE[y * b + xb] : z;
      const float2 e10 = yb != y ? sE[yb * b + x] : z;
      const float2 e11 = xb != x && yb != y ? sE[yb * b + xb] : z;
      // along x: the middle element is E+ itself, and no E-
      const bool mx = xb == x, my = yb == y;
      const float2 p0 = make_float2(e00.x + e01.x, e00.y + e01.y), p1 = make_float2(e10.x + e11.x, e10.y + e11.y);
      const float2 m0 = mx ? z : make_float2(e00.x - e01.x, e00.y - e01.y);
      const float2 m1 = mx ? z : make_float2(e10.x - e11.x, e10.y - e11.y);
      sF[2 * i] = make_float4(p0.x + p1.x, p0.y + p1.y, m0.x + m1.x, m0.y + m1.y);
      // 0 x: a sample that is not finite stays in the row's both folds
      sF[2 * i + 1] = my ? make_float4(0.f * p0.x, 0.f * p0.y, 0.f * m0.x, 0.f * m0.y)
                         : make_float4(p0.x - p1.x, p0.y - p1.y, m0.x - m1.x, m0.y - m1.y);
    }
    __syncthreads();
    // T+-[y][u], T+-[y][M-1-u]
    const float inv_hm = 1.f / (float)hm, inv_k = 1.f / (float)k;
    for (int i = tid; i < H * hm; i += NT) {
      const int y = quot(i, inv_hm), u = i - y * hm;
      const float2* w = sC + u * CW;
      const float4* e = sF + 2 * H * y;
      float cr = 0.f, ci = 0.f, sr = 0.f, sii = 0.f, dr = 0.f, di = 0.f, tr = 0.f, ti = 0.f;
#pragma unroll
      for (int x = 0; x < H; ++x) {
        const float2 cs = w[x];
        const float4 a = e[2 * x], d = e[2 * x + 1];
        cr = fmaf(a.x, cs.x, cr);
        ci = fmaf(a.y, cs.x, ci);
        sr = fmaf(a.z, cs.y, sr);
        sii = fmaf(a.w, cs.y, sii);
        dr = fmaf(d.x, cs.x, dr);
        di = fmaf(d.y, cs.x, di);
        tr = fmaf(d.z, cs.y, tr);
        ti = fmaf(d.w, cs.y, ti);
      }
      // C + i S and C - i S
      sT[y * M + u] = make_float4(cr - sii, ci + sr, dr - ti, di + tr);
      sT[y * M + M - 1 - u] = make_float4(cr + sii, ci - sr, dr + ti, di - tr);
    }
    __syncthreads();
    // pixels: tpp threads per pixel pair share its focal columns s, s + tpp, ...
    // (fixed order).  The two pixels' rows v and M-1-v come from one pair of
    // sums; with k odd the middle pixel row is its own pair, over half its rows,
    // and the middle v of an odd M is its own mirror image.
    const int pairs = sh_half(k) * k;
    const int tpp = 1 << p.tpp_log2;
    for (int base = 0; base < pairs * tpp; base += NT) {
      const int slot = base + tid;
      const int P = slot >> p.tpp_log2, s = slot - (P << p.tpp_log2);
      const int pr = quot(P, inv_k), pc = P - pr * k;
      const bool mid = 2 * pr == k - 1;
      float acc1 = 0.f, acc2 = 0.f;
      if (P < pairs) {
        const int rows = mid ? r / 2 : r;
        for (int u0 = s; u0 < r; u0 += NC * tpp) {
          float4 tc[NC][H];
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const bool in = u0 + c * tpp < r;
            const int u = pc * r + (in ? u0 + c * tpp : u0);
#pragma unroll
            for (int y = 0; y < H; ++y) tc[c][y] = in ? sT[y * M + u] : make_float4(0.f, 0.f, 0.f, 0.f);
          }
          auto row = [&](int v, bool both) {
            const float2* w = sC + v * CW;
            float cr[NC], ci[NC], sr[NC], sii[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) cr[c] = ci[c] = sr[c] = sii[c] = 0.f;
#pragma unroll
            for (int y = 0; y < H; ++y) {
              const float2 cs = w[y];
#pragma unroll
              for (int c = 0; c < NC; ++c) {
                cr[c] = fmaf(cs.x, tc[c][y].x, cr[c]);
                ci[c] = fmaf(cs.x, tc[c][y].y, ci[c]);
                sr[c] = fmaf(cs.y, tc[c][y].z, sr[c]);
                sii[c] = fmaf(cs.y, tc[c][y].w, sii[c]);
              }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              const float ar = cr[c] - sii[c], ai = ci[c] + sr[c];
              acc1 = fmaf(ar, ar, fmaf(ai, ai, acc1));
              if (both) {
                const float br = cr[c] + sii[c], bi = ci[c] - sr[c];
                acc2 = fmaf(br, br, fmaf(bi, bi, acc2));
              }
            }
          };
          for (int vv = 0; vv < rows; ++vv) row(pr * r + vv, true);
          if (mid && (r & 1)) row(pr * r + rows, false);
        }
      }
      sR[tid] = make_float2(acc1, acc2);
      __syncthreads();
      if (s == 0 && P < pairs) {
        float2 v = sR[tid];
        for (int q = 1; q < tpp; ++q) {
          v.x += sR[tid + q].x;
          v.y += sR[tid + q].y;
        }
        if (mid) v.x += v.y;
        const int P2 = (k - 1 - pr) * k + pc;
        sP[P] = (l == 0 ? 0.f : sP[P]) + v.x * p.wnorm[l];
        if (!mid) sP[P2] = (l == 0 ? 0.f : sP[P2]) + v.y * p.wnorm[l];
      }
      __syncthreads();
    }
  }   // wavelengths
  // centre of gravity: the first wavefront sums the pixels lane-strided,
  // then a fixed butterfly of cross-lane adds (no workgroup barriers)
  if (tid >= 64) return;
  float t0 = 0.f, tx = 0.f, ty = 0.f;
  const float c0 = 0.5f * (float)(k - 1);
  for (int P = tid; P < kk; P += 64) {
    const float v = sP[P];
    t0 += v;
    const int py = quot(P, 1.f / (float)k);
    tx = fmaf(v, (float)(P - py * k) - c0, tx);
    ty = fmaf(v, (float)py - c0, ty);
    if (pix_out) pix_out[P] = v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    t0 += __shfl_xor(t0, off, 64);
    tx += __shfl_xor(tx, off, 64);
    ty += __shfl_xor(ty, off, 64);
  }
  if (tid == 0) {
    sl[sub] = t0 > 0.f ? tx / t0 : 0.f;
    sl[p.n * p.n + sub] = t0 > 0.f ? ty / t0 : 0.f;
  }
}

// calls fn(kernel, threads) with the kernel of a folded width, for a thread that
// owns `cols` columns of a pixel
template <int H, class Fn>
void sh_pick(int h, int cols, bool narrow, Fn fn) {
  if constexpr (H <= 16) {
    if (h != H) return sh_pick<H + 1>(h, cols, narrow, fn);
    constexpr int NC = H <= 8 ? 2 : 1;
    if constexpr (H <= 4)
      if (cols >= 4) return narrow ? fn(k_sh<H, 4, 128>, 128) : fn(k_sh<H, 4, kShBlock>, kShBlock);
    return narrow ? fn(k_sh<H, NC, 128>, 128) : fn(k_sh<H, NC, kShBlock>, kShBlock);
  }
}

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace
}  // namespace pwfs

using namespace pwfs;

struct pwfs_sh_s {
  pwfs_sh_desc d;
  int D, n, b, M, r, k, max_frames, n_valid, n_lam;
  float wnorm[PWFS_MAX_LAMBDA];
  double four_over_lam[PWFS_MAX_LAMBDA];
  float* amp = nullptr;
  float2* W = nullptr;
  uint8_t* valid = nullptr;
  size_t lds = 0;
  bool narrow = false;   // 128 threads
  int tpp_log2 = 0;
  int cols = 1;          // focal columns of a pixel per thread
};

extern "C" int pwfs_sh_validate(const pwfs_sh_desc* d) {
  if (!d) return sfail(PWFS_EINVAL, "NULL description");
  if (d->pad_ != 0) return sfail(PWFS_EINVAL, "reserved fields must be 0");
  if (d->n_lambda < 0 || d->n_lambda > PWFS_MAX_LAMBDA)
    return sfail(PWFS_EINVAL, "n_lambda must be in [0, %d]", PWFS_MAX_LAMBDA);
  if (d->n_pupil < 2 || d->n_subap < 1 || d->n_pupil % d->n_subap)
    return sfail(PWFS_EINVAL, "n_pupil must be a positive multiple of n_subap");
  const int b = d->n_pupil / d->n_subap;
  if (b > 32) return sfail(PWFS_EUNSUPPORTED, "subaperture of %d px (> 32) not supported", b);
  if (d->n_fft < 2 || d->n_fft > 512) return sfail(PWFS_EINVAL, "n_fft must be in [2, 512]");
  if (d->rebin < 1 || d->n_fft % d->rebin) return sfail(PWFS_EINVAL, "rebin must divide n_fft");
  if (!(d->obstruction >= 0.0 && d->obstruction < 1.0)) return sfail(PWFS_EINVAL, "obstruction must be in [0, 1)");
  if (!(d->lambda_nm > 0.0) || !std::isfinite(d->lambda_nm)) return sfail(PWFS_EINVAL, "lambda_nm must be > 0");
  if (d->n_lambda >= 2) {
    double wsum = 0.0;
    for (int l = 0; l < d->n_lambda; ++l) {
      if (!(d->lambdas_nm[l] >= d->lambda_nm) || !std::isfinite(d->lambdas_nm[l]))
        return sfail(PWFS_EINVAL, "lambdas_nm[%d] must be finite and >= lambda_nm (the reference)", l);
      if (!(d->lambda_weights[l] >= 0.0)) return sfail(PWFS_EINVAL, "lambda_weights[%d] must be >= 0", l);
      wsum += d->lambda_weights[l];
    }
    if (std::fabs(wsum - 1.0) > 1e-9) return sfail(PWFS_EINVAL, "lambda_weights must sum to 1");
  }
  const int k = d->n_fft / d->rebin;
  // What is admitted goes by the size of unfolded tables, in at most 150 KiB.  The
  // folded ones are smaller from b = 4 on and a little larger for b = 1 and 3: at
  // most 152 KiB of what is admitted (b = 1, n_fft = 382, rebin 2).
  const size_t wide = (size_t)(b % 2 == 0 ? b + 1 : b), tall = (size_t)(d->n_fft <= 256 ? 257 : d->n_fft);
  const size_t lds = sizeof(float2) * ((size_t)d->n_fft * wide + (size_t)b * tall + (size_t)b * b) +
                     sizeof(float) * ((size_t)k * k + kShBlock);
  if (lds > 150 * 1024 || sh_lds(b, d->n_fft, k, kShBlock) > 160 * 1024)
    return sfail(PWFS_EUNSUPPORTED, "subaperture tables exceed the LDS (n_fft x b too large)");
  return PWFS_OK;
}

extern "C" int pwfs_sh_workspace_size(const pwfs_sh_desc* d, int max_frames, size_t* bytes) {
  int rc = pwfs_sh_validate(d);
  if (rc) return rc;
  if (!bytes || max_frames < 1) return sfail(PWFS_EINVAL, "bad arguments");
  const int D = d->n_pupil, n = d->n_subap, b = D / n;
  const int nl = d->n_lambda >= 2 ? d->n_lambda : 1;
  *bytes = a256(sizeof(float) * D * D) + a256(sizeof(float2) * nl * d->n_fft * b) + a256((size_t)n * n);
  return PWFS_OK;
}

extern "C" int pwfs_sh_plan(const pwfs_sh_desc* d, int max_frames, void* ws, size_t ws_bytes, void* stream,
                            pwfs_sh_t* out) {
  size_t need = 0;
  int rc = pwfs_sh_workspace_size(d, max_frames, &need);
  if (rc) return rc;
  if (!out) return sfail(PWFS_EINVAL, "out is NULL");
  *out = nullptr;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return sfail(PWFS_EWORKSPACE, "workspace missing, small or misaligned");
  const int D = d->n_pupil, n = d->n_subap, b = D / n, M = d->n_fft;
  // pupil (pixel centres at i - (D-1)/2, inside if eps R <= r <= R) and valid map (>= half lit)
  std::vector<float> A((size_t)D * D);
  const double R = D / 2.0, Ro = d->obstruction * R;
  double sA2 = 0.0;
  for (int y = 0; y < D; ++y)
    for (int x = 0; x < D; ++x) {
      const double cy = y - (D - 1) / 2.0, cx = x - (D - 1) / 2.0, r2 = cx * cx + cy * cy;
      A[(size_t)y * D + x] = (r2 <= R * R && r2 >= Ro * Ro) ? 1.f : 0.f;
      sA2 += A[(size_t)y * D + x];
    }
  std::vector<uint8_t> V((size_t)n * n);
  int nv = 0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      int c = 0;
      for (int y = 0; y < b; ++y)
        for (int x = 0; x < b; ++x) c += A[(size_t)(i * b + y) * D + j * b + x] != 0.f;
      V[(size_t)i * n + j] = 2 * c >= b * b;
      nv += V[(size_t)i * n + j];
    }
  if (nv == 0) return sfail(PWFS_EINVAL, "no valid subaperture");
  // per wavelength: W_l[u][x] with the frequency scale s_l = lambda_ref / lambda_l
  const int nl = d->n_lambda >= 2 ? d->n_lambda : 1;
  const int hm = sh_half(M), hb = sh_half(b);   // the other entries are conjugates
  std::vector<float2> W((size_t)nl * hm * hb);
  std::vector<double> scale(nl, 1.0), lam(nl, d->lambda_nm), wgt(nl, 1.0);
  for (int l = 0; l < nl && d->n_lambda >= 2; ++l) {
    lam[l] = d->lambdas_nm[l];
    wgt[l] = d->lambda_weights[l];
    scale[l] = d->lambda_nm / d->lambdas_nm[l];
  }
  for (int l = 0; l < nl; ++l)
    for (int u = 0; u < hm; ++u)
      for (int x = 0; x < hb; ++x) {
        const double a = -2.0 * kPiSh * (u - M / 2.0 + 0.5) * (x - (b - 1) / 2.0) * scale[l] / M;
        W[((size_t)l * hm + u) * hb + x] = make_float2((float)std::cos(a), (float)std::sin(a));
      }
  pwfs_sh_s* s = new (std::nothrow) pwfs_sh_s();
  if (!s) return sfail(PWFS_EINVAL, "out of host memory");
  s->d = *d;
  s->D = D;
  s->n = n;
  s->b = b;
  s->M = M;
  s->r = d->rebin;
  s->k = M / d->rebin;
  s->max_frames = max_frames;
  s->n_valid = nv;
  s->n_lam = nl;
  for (int l = 0; l < nl; ++l) {
    s->wnorm[l] = (float)(wgt[l] * scale[l] * scale[l] / ((double)M * M * sA2));
    s->four_over_lam[l] = 4.0 / lam[l];
  }
  char* p = (char*)ws;
  s->amp = (float*)p;
  p += a256(sizeof(float) * D * D);
  s->W = (float2*)p;
  p += a256(sizeof(float2) * nl * M * b);
  s->valid = (uint8_t*)p;
  const int pairs = sh_half(s->k) * s->k, tpp = sh_tpp(pairs, s->r);
  while ((1 << s->tpp_log2) < tpp) ++s->tpp_log2;
  s->narrow = pairs * tpp <= 128;
  s->cols = s->r / tpp;
  s->lds = sh_lds(b, M, s->k, s->narrow ? 128 : kShBlock);
  hipStream_t st = (hipStream_t)stream;
  if (hipMemcpyAsync(s->amp, A.data(), A.size() * sizeof(float), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(s->W, W.data(), W.size() * sizeof(float2), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(s->valid, V.data(), V.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    delete s;
    return sfail(PWFS_EHIP, "uploading the sensor tables failed");
  }
  sh_pick<1>(hb, s->cols, s->narrow, [](void (*fn)(ShArgs), int) {
    if (hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      (void)hipGetLastError();
  });
  *out = s;
  return PWFS_OK;
}

extern "C" int pwfs_sh_forward(pwfs_sh_t s, const float* opd, int nf, float* pixels, float* slopes, void* stream) {
  if (!s) return sfail(PWFS_EINVAL, "plan is NULL");
  if (!opd || !slopes) return sfail(PWFS_EINVAL, "NULL device pointer");
  if (nf < 1 || nf > s->max_frames) return sfail(PWFS_ESTATE, "n_frames %d outside [1, max_frames]", nf);
  ShArgs a{};
  a.opd = opd;
  a.amp = s->amp;
  a.W = s->W;
  a.valid = s->valid;
  a.pixels = pixels;
  a.slopes = slopes;
  a.D = s->D;
  a.n = s->n;
  a.b = s->b;
  a.M = s->M;
  a.r = s->r;
  a.k = s->k;
  a.n_lam = s->n_lam;
  a.tpp_log2 = s->tpp_log2;
  for (int l = 0; l < s->n_lam; ++l) {
    a.wnorm[l] = s->wnorm[l];
    a.four_over_lam[l] = s->four_over_lam[l];
  }
  const unsigned grid = (unsigned)((long long)nf * s->n * s->n);
  hipStream_t st = (hipStream_t)stream;
  sh_pick<1>(sh_half(s->b), s->cols, s->narrow, [&](void (*fn)(ShArgs), int threads) {
    hipLaunchKernelGGL(fn, dim3(grid), dim3((unsigned)threads), s->lds, st, a);
  });
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return sfail(PWFS_EHIP, "launch k_sh: %s", hipGetErrorString(e));
  return PWFS_OK;
}

extern "C" int pwfs_sh_query(pwfs_sh_t s, int32_t* n_valid, int32_t* n_pix) {
  if (!s || !n_valid || !n_pix) return sfail(PWFS_EINVAL, "NULL argument");
  *n_valid = s->n_valid;
  *n_pix = s->k;
  return PWFS_OK;
}

extern "C" void pwfs_sh_destroy(pwfs_sh_t s) { delete s; }
