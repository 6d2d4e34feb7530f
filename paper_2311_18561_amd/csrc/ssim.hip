// SSIM term of the training loss (Sec. 3.4 objective, weight lambda_r): the
// structural similarity of Wang et al. with an 11 x 11 Gaussian window
// (sigma 1.5), zero padding and C1 = 0.01^2, C2 = 0.03^2, per channel and
// pixel:
//   S = (2 mx my + C1)(2 sxy + C2) / ((mx^2 + my^2 + C1)(sxx + syy + C2))
// with mx = G*x, sxx = G*(x^2) - mx^2, sxy = G*(x y) - mx my (G* the window).
// y (the target) takes no gradient.
//
// One 256-thread workgroup per tile of 32 x 32 pixels and channel.  The
// forward stages the tile's 42 x 42 halo of x and y in LDS, filters four maps
// separably (of the second moments S asks only sxy and sxx + syy, the
// variance of x - y plus 2 sxy, so the maps are x, y, (x - y)^2 and x y; where
// x = y the two factors cancel exactly), and writes S and the three partial
// derivatives dS/dmx, dS/d(G*x^2), dS/d(G*xy) that the adjoint needs.  The
// adjoint stages the upstream gradient times those partials on the halo,
// filters them the same way (the window is symmetric, so the zero-padded
// filter is its own adjoint) and forms
//   dL/dx = G*(g dS/dmx) + 2 x G*(g dS/dExx) + y G*(g dS/dExy).
#include <cmath>

#include "pvg_internal.hpp"

namespace pvg {

namespace {

constexpr int kR = 5;  // window radius
constexpr int kTW = 32, kTH = 32;  // tile
constexpr int kV = 4;              // rows of a thread's outputs in the column pass
constexpr int kRows = kTH + 2 * kR, kCols = kTW + 2 * kR;
constexpr int kRun = 8;            // columns of a thread's outputs in the row pass
// LDS row strides: the staged maps are read 16 bytes at a time, 20 values for
// 8 outputs; of the filtered rows a wave reads two sets of 32 columns 8 rows
// apart, which 36 places on different banks.
constexpr int kSrcStride = 44, kMidStride = 36;
static_assert(kTW / kRun * kRows <= 256, "one item of the row pass per thread");
static_assert(kTW * kTH == 256 * kV && kTH == 8 * kV, "one item of the column pass per thread");
constexpr float kC1 = 0.0001f, kC2 = 0.0009f;

struct Window {
  float w[2 * kR + 1];
};

// Workgroup b takes tile (b mod 8) * per + b / 8: workgroups are dealt to the
// eight XCDs in turn, so each XCD gets a contiguous band of tiles and the
// halos that neighbouring tiles share stay in its L2.  Tiles past the end
// (the grid is 8 per) exit at once.
__device__ __forceinline__ int64_t band_tile(int64_t b, int64_t total) {
  const int64_t per = (total + 7) / 8;
  return (b % 8) * per + b / 8;
}

// The SSIM kernels may fuse multiply-adds and use the hardware reciprocal:
// no decision depends on their rounding (the bar is a tolerance), and with
// contraction off they were bound by the separate multiplies and adds of the
// window sums and the IEEE division sequences.
//
// Bound: with an output per thread the passes were bound by LDS, 11 reads a
// map, pass and output.  A thread now filters 8 neighbouring columns from 18
// staged values and 4 rows from 14, in registers, and the row pass's results
// take the place of the staged maps in LDS, so that six workgroups fit a CU
// where two did (adjoint: three).  Loads go out together, ahead of the first
// LDS store.  Per 1920x1280 image of three channels, us: forward 135 -> 56,
// adjoint 83 -> 57 (their reads and writes alone: 36 and 42).  Tiles of 48
// rows 59 and 59, of 24 rows 62 and 60; a branch around each load 72 and 69.
// Taking (x - y)^2 for x^2 and y^2 lowers the map's error against 64 bits from
// 6.2e-6 to 4.8e-6 of its norm (640x960, noise 0.1), the gradient's from
// 2.5e-6 to 1.9e-6.

// Rows y0 .. y0 + kRows, columns x0 .. x0 + kCols of kM maps, a row per wave;
// zeros outside the image.  load(offset, values) reads kL values at an offset
// in the image (the nearest pixel's for those outside, so that all loads can
// be in flight together), map(values, maps) forms the maps.
template <int kL, int kM, class Load, class Map>
__device__ __forceinline__ void stage(float (*src)[kRows][kSrcStride], int x0, int y0, int H, int W, Load load,
                                      Map map) {
  constexpr int kIts = (kRows + 3) / 4;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane >= kSrcStride) return;
  const int px = x0 + lane, cx = min(max(px, 0), W - 1);
  const bool inx = px >= 0 && px < W;
  float v[kIts][kL];
#pragma unroll
  for (int it = 0; it < kIts; ++it)
    load(static_cast<int64_t>(min(max(y0 + wid + 4 * it, 0), H - 1)) * W + cx, v[it]);
#pragma unroll
  for (int it = 0; it < kIts; ++it) {
    const int r = wid + 4 * it, py = y0 + r;
    if (r >= kRows) break;
    float m[kM];
    map(v[it], m);
#pragma unroll
    for (int q = 0; q < kM; ++q) src[q][r][lane] = inx && py >= 0 && py < H ? m[q] : 0.0f;
  }
}

// Window sums along a row of kN maps, kRun outputs each, over the maps that
// expand(staged values, values) forms from the kM staged ones.
template <int kM, int kN, class Expand>
__device__ __forceinline__ void filter_row(const float (*src)[kRows][kSrcStride], int r, int c0, const float* w,
                                           float (&acc)[kN][kRun], Expand expand) {
#pragma clang fp contract(fast)
#pragma unroll
  for (int m = 0; m < kN; ++m)
#pragma unroll
    for (int o = 0; o < kRun; ++o) acc[m][o] = 0.0f;
#pragma unroll
  for (int i4 = 0; i4 < kRun + 2 * kR; i4 += 4) {
    float4 q[kM];
#pragma unroll
    for (int m = 0; m < kM; ++m) q[m] = *reinterpret_cast<const float4*>(&src[m][r][c0 + i4]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i4 + u;
      float in[kM], v[kN];
#pragma unroll
      for (int m = 0; m < kM; ++m) in[m] = u == 0 ? q[m].x : u == 1 ? q[m].y : u == 2 ? q[m].z : q[m].w;
      expand(in, v);
#pragma unroll
      for (int o = 0; o < kRun; ++o)
        if (i >= o && i - o <= 2 * kR) {
#pragma unroll
          for (int m = 0; m < kN; ++m) acc[m][o] += w[i - o] * v[m];
        }
    }
  }
}

template <int kN>
__device__ __forceinline__ void store_row(float (*mid)[kRows][kMidStride], int r, int c0, const float (&acc)[kN][kRun]) {
#pragma unroll
  for (int m = 0; m < kN; ++m) {
    float4* d = reinterpret_cast<float4*>(&mid[m][r][c0]);
    d[0] = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
    d[1] = make_float4(acc[m][4], acc[m][5], acc[m][6], acc[m][7]);
  }
}

// Window sums down column c of kN maps, kV outputs from row r0 on.
template <int kN>
__device__ __forceinline__ void filter_column(const float (*mid)[kRows][kMidStride], int r0, int c, const float* w,
                                              float (&acc)[kN][kV]) {
#pragma clang fp contract(fast)
#pragma unroll
  for (int m = 0; m < kN; ++m)
#pragma unroll
    for (int o = 0; o < kV; ++o) acc[m][o] = 0.0f;
#pragma unroll
  for (int i = 0; i < kV + 2 * kR; ++i)
#pragma unroll
    for (int m = 0; m < kN; ++m) {
      const float v = mid[m][r0 + i][c];
#pragma unroll
      for (int o = 0; o < kV; ++o)
        if (i >= o && i - o <= 2 * kR) acc[m][o] += w[i - o] * v;
    }
}

// The thread's items: (row, first column) of the row pass, (first row,
// column) of the column pass, where a wave takes two sets of rows 2 kV apart.
__device__ __forceinline__ int row_item() { return threadIdx.x / (kTW / kRun); }
__device__ __forceinline__ int run_item() { return threadIdx.x % (kTW / kRun) * kRun; }
__device__ __forceinline__ int column_item() { return threadIdx.x % kTW; }
__device__ __forceinline__ int first_row_item() {
  const int wid = threadIdx.x >> 6;
  return kV * ((wid & 1) + 4 * (wid >> 1) + (threadIdx.x & 32 ? 2 : 0));
}

union FwdLds {
  float src[2][kRows][kSrcStride];
  float mid[4][kRows][kMidStride];
};

__global__ void __launch_bounds__(256) k_ssim_fwd(const float* __restrict__ x, const float* __restrict__ y, int H,
                                                  int W, int GX, int64_t ntiles, Window win,
                                                  float* __restrict__ smap, float* __restrict__ part) {
#pragma clang fp contract(fast)
  __shared__ __align__(16) FwdLds lds;
  const int ch = blockIdx.y;
  const int64_t HW = static_cast<int64_t>(H) * W;
  const float* xc = x + ch * HW;
  const float* yc = y + ch * HW;
  const int64_t tile = band_tile(blockIdx.x, ntiles);
  if (tile >= ntiles) return;  // the whole workgroup, before any barrier
  const int x0 = static_cast<int>(tile % GX) * kTW - kR, y0 = static_cast<int>(tile / GX) * kTH - kR;
  float w[2 * kR + 1];
#pragma unroll
  for (int k = 0; k <= 2 * kR; ++k) w[k] = win.w[k];
  stage<2, 2>(
      lds.src, x0, y0, H, W,
      [&](int64_t o, float* v) {
        v[0] = xc[o];
        v[1] = yc[o];
      },
      [](const float* v, float* m) {
        m[0] = v[0];
        m[1] = v[1];
      });
  __syncthreads();
  {
    const int r = row_item(), c0 = run_item();
    float acc[4][kRun];
    if (r < kRows)
      filter_row<2, 4>(lds.src, r, c0, w, acc, [](const float* in, float* v) {
#pragma clang fp contract(fast)
        v[0] = in[0];
        v[1] = in[1];
        v[2] = (in[0] - in[1]) * (in[0] - in[1]);
        v[3] = in[0] * in[1];
      });
    __syncthreads();
    if (r < kRows) store_row<4>(lds.mid, r, c0, acc);
  }
  __syncthreads();
  const int64_t CHW = static_cast<int64_t>(gridDim.y) * HW;
  const int c = column_item(), r0 = first_row_item();
  float f[4][kV];
  filter_column<4>(lds.mid, r0, c, w, f);
  const int px = x0 + kR + c;
#pragma unroll
  for (int j = 0; j < kV; ++j) {
    const int py = y0 + kR + r0 + j;
    if (py >= H || px >= W) continue;
    const float mx = f[0][j], my = f[1][j];
    const float sxy = f[3][j] - mx * my, dm = mx - my;
    const float A = 2.0f * mx * my + kC1, B = 2.0f * sxy + kC2;
    // mx^2 + my^2 = 2 mx my + dm^2, sxx + syy = 2 sxy + the variance of x - y
    const float Cc = A + dm * dm, D = B + (f[2][j] - dm * dm);
    // C >= C1 and D near sxx + syy + C2 > 0: neither is ever 0
    const float iC = __builtin_amdgcn_rcpf(Cc), iD = __builtin_amdgcn_rcpf(D);
    const float Q = iC * iD;
    const float S = (A * B) * Q;
    const int64_t o = ch * HW + static_cast<int64_t>(py) * W + px;
    if (smap) smap[o] = S;
    // dS/dmx (through A, B, C, D), dS/d(G*x^2) (through D), dS/d(G*xy) (through
    // B); no division by A or B, which may pass through 0
    part[o] = 2.0f * my * (B - A) * Q + 2.0f * mx * S * (iD - iC);
    part[CHW + o] = -S * iD;
    part[2 * CHW + o] = 2.0f * A * Q;
  }
}

union BwdLds {
  float src[3][kRows][kSrcStride];
  float mid[3][kRows][kMidStride];
};

__global__ void __launch_bounds__(256) k_ssim_bwd(const float* __restrict__ g, const float* __restrict__ x,
                                                  const float* __restrict__ y, const float* __restrict__ part, int H,
                                                  int W, int GX, int64_t ntiles, Window win, float* __restrict__ dx) {
#pragma clang fp contract(fast)
  __shared__ __align__(16) BwdLds lds;
  const int ch = blockIdx.y;
  const int64_t HW = static_cast<int64_t>(H) * W;
  const int64_t CHW = static_cast<int64_t>(gridDim.y) * HW;
  const int64_t tile = band_tile(blockIdx.x, ntiles);
  if (tile >= ntiles) return;  // the whole workgroup, before any barrier
  const int x0 = static_cast<int>(tile % GX) * kTW - kR, y0 = static_cast<int>(tile / GX) * kTH - kR;
  float w[2 * kR + 1];
#pragma unroll
  for (int k = 0; k <= 2 * kR; ++k) w[k] = win.w[k];
  const float* gc = g + ch * HW;
  const float* pc = part + ch * HW;
  stage<4, 3>(
      lds.src, x0, y0, H, W,
      [&](int64_t o, float* v) {
        v[0] = gc[o];
        v[1] = pc[o];
        v[2] = pc[CHW + o];
        v[3] = pc[2 * CHW + o];
      },
      [](const float* v, float* m) {
        m[0] = v[0] * v[1];
        m[1] = v[0] * v[2];
        m[2] = v[0] * v[3];
      });
  __syncthreads();
  {
    const int r = row_item(), c0 = run_item();
    float acc[3][kRun];
    if (r < kRows)
      filter_row<3, 3>(lds.src, r, c0, w, acc, [](const float* in, float* v) {
        v[0] = in[0];
        v[1] = in[1];
        v[2] = in[2];
      });
    __syncthreads();
    if (r < kRows) store_row<3>(lds.mid, r, c0, acc);
  }
  __syncthreads();
  const int c = column_item(), r0 = first_row_item();
  float f[3][kV];
  filter_column<3>(lds.mid, r0, c, w, f);
  const int px = x0 + kR + c;
#pragma unroll
  for (int j = 0; j < kV; ++j) {
    const int py = y0 + kR + r0 + j;
    if (py < H && px < W) {
      const int64_t o = ch * HW + static_cast<int64_t>(py) * W + px;
      dx[o] = f[0][j] + 2.0f * x[o] * f[1][j] + y[o] * f[2][j];
    }
  }
}

Window gaussian_window() {
  Window win;
  double w[2 * kR + 1], sum = 0.0;
  for (int k = 0; k <= 2 * kR; ++k) {
    const double d = k - kR;
    w[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
    sum += w[k];
  }
  for (int k = 0; k <= 2 * kR; ++k) win.w[k] = static_cast<float>(w[k] / sum);
  return win;
}

}  // namespace

hipError_t launch_ssim_fwd(const float* x, const float* y, int C, int H, int W, float* smap, float* part,
                           hipStream_t st) {
  if (static_cast<int64_t>(H) * W * C == 0) return hipSuccess;
  const int GX = (W + kTW - 1) / kTW, GY = (H + kTH - 1) / kTH;
  const int64_t ntiles = static_cast<int64_t>(GX) * GY;
  hipLaunchKernelGGL(k_ssim_fwd, dim3(static_cast<unsigned>(8 * ((ntiles + 7) / 8)), C), dim3(256), 0, st, x, y, H,
                     W, GX, ntiles, gaussian_window(), smap, part);
  return hipGetLastError();
}

hipError_t launch_ssim_bwd(const float* g, const float* x, const float* y, const float* part, int C, int H, int W,
                           float* dx, hipStream_t st) {
  if (static_cast<int64_t>(H) * W * C == 0) return hipSuccess;
  const int GX = (W + kTW - 1) / kTW, GY = (H + kTH - 1) / kTH;
  const int64_t ntiles = static_cast<int64_t>(GX) * GY;
  hipLaunchKernelGGL(k_ssim_bwd, dim3(static_cast<unsigned>(8 * ((ntiles + 7) / 8)), C), dim3(256), 0, st, g, x, y,
                     part, H, W, GX, ntiles, gaussian_window(), dx);
  return hipGetLastError();
}

}  // namespace pvg
