// Training losses of the framework (Sec. V, implementation details): the
// photometric loss w_l1 * L1 + w_ssim * (1 - SSIM) of the 3D-GS model
// (0.8 / 0.2) and the volume regularisation sum_i Prod(s_i) of the
// Scaffold-GS model (weight 0.01).
//
// SSIM (Wang et al. 2004, the standard form the paper refers to): an 11 x 11
// Gaussian window (sigma 1.5), C1 = 0.01^2, C2 = 0.03^2, windowed statistics
// as a same-size correlation with zeros outside the image, per channel
// image, averaged over all images and pixels.  Its gradient needs the window
// correlation twice: once for the statistics, once (the adjoint; the window
// is symmetric) for the three per-pixel derivative maps
//   dS/dmu_x = S (2 mu_y / A1 - 2 mu_y / A2 - 2 mu_x / B1 + 2 mu_x / B2),
//   dS/dE[x^2] = -S / B2,  dS/dE[xy] = 2 S / A2,
// with A1 = 2 mu_x mu_y + C1, A2 = 2 s_xy + C2, B1 = mu_x^2 + mu_y^2 + C1,
// B2 = s_xx + s_yy + C2, so dS/dx = w * m0 + 2 x (w * m1) + y (w * m2).
//
// Large images (tiles_cheaper): one kernel does both correlations.  A block of 256 threads walks down a
// strip of kOutW = 236 output columns (236 + 2 x 10 image columns, one per
// thread), two image rows per step:
//   - the rows' (m, d, m^2, d^2) with m = (x + y) / 2 and d = x - y go to LDS
//     as one float4 per column; a thread pair (columns 2p, 2p + 1) shares the
//     horizontal sums: its even thread takes the first row and its odd thread
//     the second, each for both columns, from 12 float4 reads instead of
//     2 x 11, and the two swap the halves that the other needs (quad permute);
//   - the vertical sums are kept in registers as transposed filters
//     (s[i] <- s[i + 1] + g h), so nothing but a new row enters per step;
//   - the derivative maps (scaled by -w_ssim / n) of the rows that this
//     completes go to LDS in the next step, are summed the same way, and the
//     completed rows of the image gradient are written with the L1 term.
// Of m and d, mu_x mu_y = E[m]^2 - E[d]^2 / 4, s_xx + s_yy = 2 var m + var d / 2
// and 2 s_xy = 2 var m - var d / 2: four correlations instead of the five of
// x, y, x^2, y^2, x y, and the rounding of var m enters A2 and B2 alike (error
// of the gradient against 64 bits: 8.4e-7, the five maps' 8.9e-7).  The LDS
// rows are double-buffered: one barrier per step.
// A block's strip is as long as leaves about two blocks per compute unit; it
// runs 20 rows more than it writes (the two windows' rows above and below).
// Bound by vector ALU work (about 220 instructions per pixel of the padded
// strip; the tiled two-pass form moved the three maps through memory and its
// LDS reads, four words apart, conflicted four ways).  Three 1600 x 1066
// planes with the loss sum: 129 us before, 72 us now; about 480 blocks
// measured best (256: 87 us, 768: 75 us, 1,024: 82 us).
// Each block leaves one partial loss sum per term; a final block adds them in
// double, in a fixed order.
#include "octgs_internal.h"

namespace octgs {

namespace {

constexpr int kR = 5, kTaps = 2 * kR + 1;
constexpr int kOutW = kBlock - 4 * kR;  // output columns of a block
constexpr float kC1 = 0.0001f, kC2 = 0.0009f;
// Rows that a block writes: long strips amortise the 2 x 10 extra rows, short
// ones fill the chip.  Two blocks of 4 waves per compute unit keep the vector
// ALUs busy, so a strip grows until there are about 512 blocks.  kUnroll steps
// of two rows are unrolled, the vertical filters' period of 10 rows, so that
// their states rotate through the registers without a move; a block takes
// rows / 2 + 11 steps, so rows is 8 more than a multiple of 10.
constexpr int kUnroll = (kTaps - 1) / 2, kMinRows = 8, kMaxRows = 128, kWantBlocks = 512;

__device__ __forceinline__ int64_t block_index() {
  return ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
}

int strip_rows(int64_t n_images, int32_t height, int32_t width) {
  const int64_t cols = (width + kOutW - 1) / kOutW;
  // strips per column of blocks, at least one, so that cols * n_images * strips
  // is at most kWantBlocks
  const int64_t strips = std::max<int64_t>(kWantBlocks / std::max<int64_t>(cols * n_images, 1), 1);
  const int64_t rows = (height + strips - 1) / strips;
  const int64_t fit = kMinRows + (std::max<int64_t>(rows - kMinRows, 0) + 5) / 10 * 10;
  return (int)std::min<int64_t>(fit, kMaxRows);
}

int64_t ssim_blocks(int64_t n_images, int32_t height, int32_t width) {
  const int rows = strip_rows(n_images, height, width);
  return (int64_t)((width + kOutW - 1) / kOutW) * ((height + rows - 1) / rows) * n_images;
}

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

struct SsimArgs {
  const float *x, *y;
  float *m0, *m1, *m2;  // derivative maps (workspace; tiled passes)
  float *part;  // per-block loss partial sums: [2][blocks] (workspace)
  float *dimg, *loss;
  int H, W, rows;
  float w_l1, w_ssim, inv_n;
  float g[kTaps];
};

// The two rows' window sums of NM maps at this thread's column: src[row] holds
// the maps of column base + 2p.., base = first tap of the pair's even column.
// Lane pairs differ in the row they read, so the rows are an odd number of
// float4s apart (no bank conflicts).
template <int NM>
__device__ __forceinline__ void pair_sums(const float4 *src, const float (&g)[kTaps], bool odd,
                                          float (&r0)[NM], float (&r1)[NM]) {
  float l[NM], r[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) l[m] = r[m] = 0.0f;
#pragma unroll
  for (int q = 0; q <= kTaps; ++q) {
    const float4 v = src[q];
    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if (q < kTaps) l[m] = fma_(g[q < kTaps ? q : 0], e[m], l[m]);
      if (q > 0) r[m] = fma_(g[q > 0 ? q - 1 : 0], e[m], r[m]);
    }
  }
  // even thread: own row 0 of its column, row 1 from its partner; odd alike
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const float got = __uint_as_float(dpp_u<kDppXor1>(__float_as_uint(odd ? l[m] : r[m])));
    r0[m] = odd ? got : l[m];
    r1[m] = odd ? r[m] : got;
  }
}

// One row through the vertical filter: returns the window sum that it
// completes (the row kR above) and shifts the partial sums.
__device__ __forceinline__ float fir(float (&s)[kTaps - 1], const float (&g)[kTaps], float h) {
  const float out = fma_(g[0], h, s[0]);
#pragma unroll
  for (int i = 0; i < kTaps - 2; ++i) s[i] = fma_(g[i + 1], h, s[i + 1]);
  s[kTaps - 2] = g[kTaps - 1] * h;
  return out;
}

__global__ __launch_bounds__(kBlock) void k_ssim(SsimArgs a) {
  // thread t: image column x0 - 10 + t, maps and output of column x0 - 5 + t
  // (the last 10 threads' windows run past the block's columns; no output
  // reads them)
  constexpr int kPitch = kBlock + 2 * kR + 1;  // float4s; odd
  __shared__ float4 ra[2][2 * kPitch], rb[2][2 * kPitch];
  __shared__ float red[4];
  const int t = threadIdx.x, p2 = t & ~1;
  const bool odd = t & 1;
  const int x0 = blockIdx.x * kOutW, y0 = blockIdx.y * a.rows;
  const int ca = x0 - 2 * kR + t, cm = x0 - kR + t;
  const int64_t base = (int64_t)blockIdx.z * a.H * a.W;
  const float *x = a.x + base, *y = a.y + base;
  const bool in_ca = ca >= 0 && ca < a.W, in_cm = cm >= 0 && cm < a.W;
  const uint32_t oa = min(max(ca, 0), a.W - 1), om = min(max(cm, 0), a.W - 1);
  const bool out_col = t >= kR && t < kR + kOutW && cm < a.W;
  const float coef = -a.w_ssim * a.inv_n, l1 = a.w_l1 * a.inv_n;
  for (int i = t; i < 2 * kPitch; i += kBlock) {
    const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    ra[0][i] = ra[1][i] = rb[0][i] = rb[1][i] = z;
  }
  __syncthreads();
  // start of an image row, clamped: loads are unconditional, so they stay in
  // flight until their use
  auto row_at = [&](int row) { return (int64_t)min(max(row, 0), a.H - 1) * a.W; };
  float sa[4][kTaps - 1], sb[3][kTaps - 1];
#pragma unroll
  for (int i = 0; i < kTaps - 1; ++i) {
#pragma unroll
    for (int m = 0; m < 4; ++m) sa[m][i] = 0.0f;
#pragma unroll
    for (int m = 0; m < 3; ++m) sb[m][i] = 0.0f;
  }
  float px[2], py[2];  // the next two rows
  int r = y0 - 2 * kR;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    px[k] = x[row_at(r + k) + oa];
    py[k] = y[row_at(r + k) + oa];
  }
  float4 mrow[2];
  mrow[0] = mrow[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float acc_s = 0.0f, acc_l1 = 0.0f;
  // in the step that takes rows r, r + 1: statistics and maps of rows r - 5,
  // r - 4; maps of rows r - 7, r - 6 enter the second window; gradient of
  // rows r - 12, r - 11
  const int steps = a.rows / 2 + kTaps;
  const int y1 = min(y0 + a.rows, a.H);
  for (int it = 0; it < steps; it += kUnroll)
#pragma unroll
  for (int u = 0; u < kUnroll; ++u, r += 2) {
    float4 *wa = ra[(it + u) & 1], *wb = rb[(it + u) & 1];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bool in = in_ca && r + k >= 0 && r + k < a.H;
      const float vx = in ? px[k] : 0.0f, vy = in ? py[k] : 0.0f;
      const float vm = 0.5f * (vx + vy), vd = vx - vy;
      wa[k * kPitch + t] = make_float4(vm, vd, vm * vm, vd * vd);
      wb[k * kPitch + kR + t] = mrow[k];
    }
    __syncthreads();
    // the next rows, and the image at the gradient's rows
    float ox[2], oy[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t o = row_at(r - 12 + k) + om, q = row_at(r + 2 + k) + oa;
      ox[k] = x[o];
      oy[k] = y[o];
      px[k] = x[q];
      py[k] = y[q];
    }
    float h0[4], h1[4], g0[3], g1[3];
    pair_sums<4>(wa + (odd ? kPitch : 0) + p2, a.g, odd, h0, h1);
    pair_sums<3>(wb + (odd ? kPitch : 0) + p2, a.g, odd, g0, g1);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float st[4], cv[3];
#pragma unroll
      for (int m = 0; m < 4; ++m) st[m] = fir(sa[m], a.g, k ? h1[m] : h0[m]);
#pragma unroll
      for (int m = 0; m < 3; ++m) cv[m] = fir(sb[m], a.g, k ? g1[m] : g0[m]);
      // SSIM at row r - 5 + k.  With 1 / (B1 B2) =: iB, S = A1 A2 iB,
      //   S / A1 = A2 iB, S / A2 = A1 iB, S / B1 = S B2 iB, S / B2 = S B1 iB
      {
        const int row = r - kR + k;
        const float mx = fma_(0.5f, st[1], st[0]), my = fma_(-0.5f, st[1], st[0]);
        const float mm = st[0] * st[0], dd = st[1] * st[1];
        const float vm = st[2] - mm, vd = st[3] - dd;
        const float A1 = fma_(2.0f, mm, -0.5f * dd) + kC1, B1 = fma_(2.0f, mm, 0.5f * dd) + kC1;
        const float A2 = fma_(2.0f, vm, -0.5f * vd) + kC2, B2 = fma_(2.0f, vm, 0.5f * vd) + kC2;
        const float iB = 1.0f / (B1 * B2);
        const float S = A1 * A2 * iB, SiB = S * iB;
        const bool in = in_cm && row >= 0 && row < a.H;
        const float c = in ? coef : 0.0f;
        mrow[k].x = in ? c * 2.0f * fma_(my * (A2 - A1), iB, mx * (B1 - B2) * SiB) : 0.0f;
        mrow[k].y = in ? c * -(SiB * B1) : 0.0f;
        mrow[k].z = in ? c * (2.0f * A1 * iB) : 0.0f;
        if (out_col && row >= y0 && row < y1) acc_s += S;
      }
      const int ro = r - 12 + k;
      if (out_col && ro >= y0 && ro < y1) {
        const float X = ox[k], Y = oy[k], d = X - Y;
        const float sg = d > 0.0f ? l1 : (d < 0.0f ? -l1 : 0.0f);
        a.dimg[base + (int64_t)ro * a.W + cm] =
            fma_(2.0f * X, cv[1], fma_(Y, cv[2], cv[0])) + sg;
        acc_l1 += fabsf(d);
      }
    }
  }
  acc_s = block_sum_f(acc_s, red);
  if (t == 0) a.part[block_index()] = coef * acc_s;
  __syncthreads();
  acc_l1 = block_sum_f(acc_l1, red);
  if (t == 0) a.part[(int64_t)gridDim.x * gridDim.y * gridDim.z + block_index()] = l1 * acc_l1;
}

// ---- small images: two tiled passes -----------------------------------------
// A strip takes rows / 2 + 11 steps of about a microsecond one after the other
// however small the image, so an image that does not fill the chip with strips
// is done in 64 x 16 tiles instead, all at once: pass 1 writes the three
// derivative maps to the workspace, pass 2 correlates them.  Each stages its
// input with a 5-pixel halo in LDS and runs the window as a horizontal then a
// vertical sweep, each thread producing four adjacent outputs from one
// register window.
constexpr int kSW = 64, kSH = 16;
constexpr int kRW = kSW + 2 * kR, kRH = kSH + 2 * kR;  // 74 x 26 staged region

int64_t tile_blocks(int64_t n_images, int32_t height, int32_t width) {
  return (int64_t)((width + kSW - 1) / kSW) * ((height + kSH - 1) / kSH) * n_images;
}

// Tiles or strips, whichever has less to do for the planes at hand: a strip is
// 256 columns wide however narrow its plane, so what counts is the padded work,
// not the pixels.  Either form costs what its fullest compute unit runs, a
// strip 0.87 us per step of two rows and a tile (both passes) 5.5 us, and the
// tiles 4 us more around that (a second launch, three maps).  Calls of up to
// 1.6M elements stay in tiles: there the strips' steps, one after the other, are
// no less than the tiles even where they fill the chip.  Measured (us, tiles /
// strips):
//   3 x 51 x 88 15 / 24, 3 x 480 x 640 35 / 48, 3 x 540 x 960 (1.56M) 42 / 43;
//   wide planes: 3 x 720 x 1280 73 / 52, 3 x 1066 x 1600 122 / 72, 3 x 600 x
//     4000 167 / 124, 2 x 900 x 1000 52 / 42, 6 x 500 x 600 55 / 42;
//   narrow ones: 400 x 64 x 64 51 / 89, 1,600 x 32 x 32 78 / 286, 7,000 x 16 x 16
//     148 / 486, 16 x 1000 x 128 56 / 78, 3 x 20000 x 64 92 / 137, 24 x 300 x 240
//     55 / 78 (two strips of 236 columns), 12 x 400 x 480 65 / 78;
//   alike: 12 x 400 x 472 64 / 64, 48 x 200 x 200 66 / 64, 3 x 2000 x 300 55 / 51.
constexpr int64_t kTileElements = 1600000;

bool tiles_cheaper(int64_t n_images, int32_t height, int32_t width) {
  const int64_t cus = 256, steps = strip_rows(n_images, height, width) / 2 + kTaps;
  const int64_t strips = (ssim_blocks(n_images, height, width) + cus - 1) / cus * steps;
  return tile_blocks(n_images, height, width) * (5.5 / cus) + 4.0 <= strips * 0.87;
}

// Do the two ranges of n floats share memory?
bool overlap(const float *a, const float *b, int64_t n) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b, bytes = (uintptr_t)n * sizeof(float);
  return x < y ? y - x < bytes : x - y < bytes;
}

// Stage `nmaps` planes of the (kRH x kRW) region around the block's tile
// (zeros outside the image).
template <int NM>
__device__ __forceinline__ void stage(const float *const *src, int64_t base, int H, int W,
                                      float (*dst)[kRH][kRW]) {
  const int x0 = blockIdx.x * kSW - kR, y0 = blockIdx.y * kSH - kR;
  for (int i = threadIdx.x; i < kRH * kRW; i += kBlock) {
    const int r = i / kRW, c = i - r * kRW;
    const int gy = y0 + r, gx = x0 + c;
    const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
    const int64_t o = base + (int64_t)(in ? gy : 0) * W + (in ? gx : 0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const float v = src[m][o];
      dst[m][r][c] = in ? v : 0.0f;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_ssim_fwd(SsimArgs a) {
  __shared__ float in[2][kRH][kRW];
  __shared__ float hs[5][kRH][kSW];
  __shared__ float red[4];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.z * a.H * a.W;
  {
    const float *src[2] = {a.x, a.y};
    stage<2>(src, base, a.H, a.W, in);
  }
  __syncthreads();
  // horizontal sweep: rows of the region, 4 outputs per task
  for (int task = t; task < kRH * (kSW / 4); task += kBlock) {
    const int r = task / (kSW / 4), j0 = (task % (kSW / 4)) * 4;
    float xv[kTaps + 3], yv[kTaps + 3];
#pragma unroll
    for (int q = 0; q < kTaps + 3; ++q) {
      xv[q] = in[0][r][j0 + q];
      yv[q] = in[1][r][j0 + q];
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f, s4 = 0.0f;
#pragma unroll
      for (int q = 0; q < kTaps; ++q) {
        const float X = xv[o + q], Y = yv[o + q];
        const float gX = a.g[q] * X, gY = a.g[q] * Y;
        s0 += gX;
        s1 += gY;
        s2 = fma_(gX, X, s2);
        s3 = fma_(gY, Y, s3);
        s4 = fma_(gX, Y, s4);
      }
      hs[0][r][j0 + o] = s0; hs[1][r][j0 + o] = s1; hs[2][r][j0 + o] = s2;
      hs[3][r][j0 + o] = s3; hs[4][r][j0 + o] = s4;
    }
  }
  __syncthreads();
  // vertical sweep: 4 rows per thread at one column; SSIM and its partials
  const int j = t % kSW, r0 = (t / kSW) * 4;
  float st[5][4];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    float v[kTaps + 3];
#pragma unroll
    for (int q = 0; q < kTaps + 3; ++q) v[q] = hs[k][r0 + q][j];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < kTaps; ++q) s = fma_(a.g[q], v[o + q], s);
      st[k][o] = s;
    }
  }
  const int gx = blockIdx.x * kSW + j;
  const float coef = -a.w_ssim * a.inv_n;
  float acc = 0.0f;
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int gy = blockIdx.y * kSH + r0 + o;
    if (gx < a.W && gy < a.H) {
      const float mx = st[0][o], my = st[1][o];
      const float sxx = st[2][o] - mx * mx, syy = st[3][o] - my * my, sxy = st[4][o] - mx * my;
      const float A1 = fma_(2.0f * mx, my, kC1), A2 = fma_(2.0f, sxy, kC2);
      const float B1 = fma_(mx, mx, fma_(my, my, kC1)), B2 = sxx + syy + kC2;
      const float iA1 = 1.0f / A1, iA2 = 1.0f / A2, iB1 = 1.0f / B1, iB2 = 1.0f / B2;
      const float S = A1 * A2 * iB1 * iB2;
      acc += S;
      const int64_t o_ = base + (int64_t)gy * a.W + gx;
      a.m0[o_] = coef * S * 2.0f * (my * (iA1 - iA2) + mx * (iB2 - iB1));
      a.m1[o_] = coef * (-S * iB2);
      a.m2[o_] = coef * (2.0f * S * iA2);
    }
  }
  acc = block_sum_f(acc, red);
  if (t == 0) a.part[block_index()] = coef * acc;
}

__global__ __launch_bounds__(kBlock) void k_ssim_bwd(SsimArgs a) {
  __shared__ float in[3][kRH][kRW];
  __shared__ float hs[3][kRH][kSW];
  __shared__ float red[4];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.z * a.H * a.W;
  {
    const float *src[3] = {a.m0, a.m1, a.m2};
    stage<3>(src, base, a.H, a.W, in);
  }
  __syncthreads();
  for (int task = t; task < kRH * (kSW / 4); task += kBlock) {
    const int r = task / (kSW / 4), j0 = (task % (kSW / 4)) * 4;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      float v[kTaps + 3];
#pragma unroll
      for (int q = 0; q < kTaps + 3; ++q) v[q] = in[m][r][j0 + q];
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < kTaps; ++q) s = fma_(a.g[q], v[o + q], s);
        hs[m][r][j0 + o] = s;
      }
    }
  }
  __syncthreads();
  const int j = t % kSW, r0 = (t / kSW) * 4;
  float cv[3][4];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    float v[kTaps + 3];
#pragma unroll
    for (int q = 0; q < kTaps + 3; ++q) v[q] = hs[m][r0 + q][j];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < kTaps; ++q) s = fma_(a.g[q], v[o + q], s);
      cv[m][o] = s;
    }
  }
  const int gx = blockIdx.x * kSW + j;
  const float l1 = a.w_l1 * a.inv_n;
  float acc = 0.0f;
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int gy = blockIdx.y * kSH + r0 + o;
    if (gx < a.W && gy < a.H) {
      const int64_t o_ = base + (int64_t)gy * a.W + gx;
      const float X = a.x[o_], Y = a.y[o_];
      const float d = X - Y;
      const float sg = d > 0.0f ? l1 : (d < 0.0f ? -l1 : 0.0f);
      a.dimg[o_] = fma_(2.0f * X, cv[1][o], fma_(Y, cv[2][o], cv[0][o])) + sg;
      acc += fabsf(d);
    }
  }
  acc = block_sum_f(acc, red);
  if (t == 0) a.part[(int64_t)gridDim.x * gridDim.y * gridDim.z + block_index()] = l1 * acc;
}

// One block: *loss += w_ssim + the per-block partial sums, added in double
// in a fixed order (the loss is the same bit for bit on every run).
__global__ __launch_bounds__(kBlock) void k_loss_finish(const float *__restrict__ part, int64_t n,
                                                        float base, float *__restrict__ loss) {
  // eight loads in flight per thread: the kernel is one block's latency
  constexpr int kU = 8;
  __shared__ double red[kBlock / kWave];
  double s = 0.0;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += kU * kBlock) {
    float v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = part[min(i0 + u * kBlock, n - 1)];
#pragma unroll
    for (int u = 0; u < kU; ++u) s += i0 + u * kBlock < n ? (double)v[u] : 0.0;
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
  if (__lane_id() == 0) red[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0)
    *loss = (float)((double)*loss + (double)base + ((red[0] + red[1]) + (red[2] + red[3])));
}

// L1 only (w_ssim = 0): elementwise, four independent elements per step; dimg
// may be x or y.
__global__ __launch_bounds__(kBlock) void k_l1_only(const float *x, const float *y, int64_t n,
                                                    float scale, float *dimg, float *loss) {
  __shared__ float red[4];
  float acc = 0.0f;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < n; i0 += 4 * stride) {
    float d[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = min(i0 + u * stride, n - 1);
      d[u] = x[i] - y[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * stride;
      if (i < n) {
        dimg[i] = d[u] > 0.0f ? scale : (d[u] < 0.0f ? -scale : 0.0f);
        acc += fabsf(d[u]);
      }
    }
  }
  acc = block_sum_f(acc, red);
  if (threadIdx.x == 0 && acc != 0.0f) atomicAdd(loss, acc * scale);
}

// Volume regularisation over the rendered slots (opacity > 0).
__global__ __launch_bounds__(kBlock) void k_volume(const float *__restrict__ g, int64_t cap,
                                                   const uint32_t *__restrict__ count, float w,
                                                   float *__restrict__ dg, float *__restrict__ loss) {
  __shared__ float red[4];
  const int64_t n = min((int64_t)*count, cap);
  float acc = 0.0f;
  for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < n;
       s += (int64_t)gridDim.x * kBlock) {
    const float op = g[10 * cap + s];
    const float s0 = g[3 * cap + s], s1 = g[4 * cap + s], s2 = g[5 * cap + s];
    if (op > 0.0f) {
      acc = fma_(s0 * s1, s2, acc);
      dg[3 * cap + s] += w * (s1 * s2);
      dg[4 * cap + s] += w * (s0 * s2);
      dg[5 * cap + s] += w * (s0 * s1);
    }
  }
  acc = block_sum_f(acc, red);
  if (threadIdx.x == 0 && acc != 0.0f) atomicAdd(loss, w * acc);
}

}  // namespace

}  // namespace octgs

using namespace octgs;

extern "C" {

size_t octgs_photometric_workspace_bytes(int64_t n_images, int32_t height, int32_t width) {
  if (n_images < 0 || height < 0 || width < 0) return 0;
  // Three maps and two partial sums per tile, as the tiled passes use, or two
  // partial sums per strip (a strip covers the whole of a small image, but the
  // last ones of a row or column of strips may be of one pixel's width).
  if (n_images == 0 || height == 0 || width == 0) return 256;
  return (size_t)std::max(3 * n_images * (int64_t)height * width +
                              2 * tile_blocks(n_images, height, width),
                          2 * ssim_blocks(n_images, height, width)) * sizeof(float) + 256;
}

int octgs_photometric_loss_grad(const float *img, const float *target, int64_t n_images,
                                int32_t height, int32_t width, float w_l1, float w_ssim,
                                float *dimg, float *loss, void *ws, size_t ws_bytes,
                                octgs_stream stream) {
  if (n_images < 0 || height < 0 || width < 0) return OCTGS_EINVAL;
  const int64_t n = n_images * (int64_t)height * width;
  if (n == 0) return OCTGS_OK;
  if (!img || !target || !dimg || !loss) return OCTGS_EINVAL;
  if (n_images > 65535 || !(w_l1 >= 0.0f) || !(w_ssim >= 0.0f)) return OCTGS_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (w_ssim == 0.0f) {
    const int grid = (int)std::min<int64_t>((n + kBlock - 1) / kBlock, 512);
    hipLaunchKernelGGL(k_l1_only, dim3(grid), dim3(kBlock), 0, s, img, target, n,
                       (float)(w_l1 / (double)n), dimg, loss);
    return hipGetLastError() == hipSuccess ? OCTGS_OK : OCTGS_EHIP;
  }
  if (!ws) return OCTGS_EINVAL;
  if (ws_bytes < octgs_photometric_workspace_bytes(n_images, height, width)) return OCTGS_ENOSPC;
  SsimArgs a;
  a.x = img; a.y = target;
  // A strip reads rows of its neighbours as halo while those write theirs, so a
  // gradient that is written over an image takes the tiled passes: the second
  // reads the images only where it writes.  (Planes too high for a grid of tiles
  // are left to the strips.)
  const bool tiled = n <= kTileElements || overlap(dimg, img, n) || overlap(dimg, target, n) ||
                     ((height + kSH - 1) / kSH <= 65535 && tiles_cheaper(n_images, height, width));
  a.m0 = (float *)ws; a.m1 = a.m0 + n; a.m2 = a.m1 + n;
  a.part = tiled ? a.m2 + n : (float *)ws;
  a.dimg = dimg; a.loss = loss;
  a.H = height; a.W = width;
  a.rows = strip_rows(n_images, height, width);
  a.w_l1 = w_l1; a.w_ssim = w_ssim; a.inv_n = (float)(1.0 / (double)n);
  double gs[kTaps], sum = 0.0;
  for (int q = 0; q < kTaps; ++q) {
    const double d = q - kR;
    gs[q] = std::exp(-d * d / (2.0 * 1.5 * 1.5));
    sum += gs[q];
  }
  for (int q = 0; q < kTaps; ++q) a.g[q] = (float)(gs[q] / sum);
  int64_t parts;
  if (tiled) {
    const dim3 grid((width + kSW - 1) / kSW, (height + kSH - 1) / kSH, (unsigned)n_images);
    hipLaunchKernelGGL(k_ssim_fwd, grid, dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_ssim_bwd, grid, dim3(kBlock), 0, s, a);
    parts = tile_blocks(n_images, height, width);
  } else {
    const dim3 grid((width + kOutW - 1) / kOutW, (height + a.rows - 1) / a.rows, (unsigned)n_images);
    hipLaunchKernelGGL(k_ssim, grid, dim3(kBlock), 0, s, a);
    parts = ssim_blocks(n_images, height, width);
  }
  hipLaunchKernelGGL(k_loss_finish, dim3(1), dim3(kBlock), 0, s, a.part, 2 * parts, w_ssim, loss);
  return hipGetLastError() == hipSuccess ? OCTGS_OK : OCTGS_EHIP;
}

int octgs_volume_loss_grad(const octgs_gaussians *g, float weight, float *d_gauss, float *loss,
                           octgs_stream stream) {
  if (!g || !g->data || !g->count || g->capacity < 0 || !d_gauss || !loss) return OCTGS_EINVAL;
  if (g->capacity == 0) return OCTGS_OK;
  const int grid = (int)std::min<int64_t>((g->capacity + kBlock - 1) / kBlock, 512);
  hipLaunchKernelGGL(k_volume, dim3(grid), dim3(kBlock), 0, (hipStream_t)stream, g->data,
                     g->capacity, g->count, weight, d_gauss, loss);
  return hipGetLastError() == hipSuccess ? OCTGS_OK : OCTGS_EHIP;
}

}  // extern "C"
