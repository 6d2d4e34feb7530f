// Per-tile alpha blending (Sec. 3.1, Eq. (3)) and its adjoint on gfx950.
//
// One 64-lane wavefront owns one 16x16 tile (in the forward, a half or a
// quarter of one where the image has few tiles); lane l shades the four
// pixels of column l % 16 in rows l / 16 + {0, 4, 8, 12}.  The tile's depth-ordered list
// is walked in batches of 64 Gaussians: each lane gathers one Gaussian's
// record (2D mean, conic, opacity, colour) into LDS and every lane then reads
// the batch back as broadcasts.  A pixel stops before the Gaussian that would
// take its transmittance below 1e-4; the wave leaves the list as soon as a
// ballot shows all 256 pixels done.
//
// The adjoint walks the list backwards from the wave's last contributor,
// recovering each pixel's transmittance by division, sums the four pixels'
// screen-space gradients per lane and reduces them across the wave, four
// pairs at a time.  Each (Gaussian, tile) pair's nine sums are stored, without atomics, at the pair's
// index in emission order (a Gaussian's pairs are contiguous there) and
// flagged in a byte array; a gather kernel then adds each Gaussian's flagged
// pairs.  Device-scope float atomics resolve
// at the memory side on this chip and cost three times the rest of the
// kernel, and the atomic-free sums are bitwise reproducible.
//
// Tiles reach the eight XCDs in row-sized chunks dealt round-robin
// (xcd_tile), which balances the XCDs' work and keeps a chunk's shared
// Gaussians in one L2.
#include <climits>
#include <type_traits>

#include "blend.hpp"

namespace pvg {

// Waves per tile of the forward walk, by the launch's tiles (batched: its
// bound).  The chip has 1,024 SIMDs and a wave alone issues at about a third
// of a SIMD's rate, so a launch needs several waves a SIMD; a split tile
// walks its list once per strip, which costs the per-pair work again.
// The lines lie where rectangle lists, whose strips also pay the tile test,
// break even; culled lists gain from a split for a while longer.  us, 20,000 /
// 200,000 Gaussians of a box:
//   117 tiles, whole - halves - quarters: culled 103 - 56 - 40 / 73 - 43 - 31
//   1,024 tiles, halves - quarters: culled 45 - 39 / 39 - 36, rectangles 51 - 53 / 51 - 52
//   4,096 tiles, whole - halves: culled 84 - 75 / 78 - 74, rectangles 95 - 97 / 94 - 99
//   8,160 tiles, whole - halves: culled 120 - 119 / 119 - 121, rectangles 146 - 157 / 142 - 159
static int forward_parts(int64_t tiles) { return tiles <= 1024 ? 4 : tiles <= 4096 ? 2 : 1; }

// Pairs per group of the walk: enough independent work for a lane with one
// pixel, few enough live weights for one with four.
constexpr int forward_group(int px) { return px == 1 ? 8 : 4; }

// kCh: also blend each Gaussian's camera depth, mean velocity and
// staticness into the channels the view asks for (the flexible rendering of
// Sec. 3.1, with these in place of the colour).
// kPx: pixels per lane.  A wave takes kPx / 4 of a tile, a strip of 4 kPx of
// its rows (forward_parts has the rule): block b is strip b mod (4 / kPx) of
// its tile, and each wave walks the tile's list by itself.
// Of rectangle lists (kCulled false) only the Gaussians that the tile test
// keeps are walked, as in the adjoint and the feature kernels.  A strip also
// leaves out those that cannot reach it, by rect_reachable: the adjoint walks
// whole tiles, so a pair left out here that a pixel would use is divided out
// of T there and credited with a gradient.
template <bool kCount, bool kCulled, bool kCh, int kPx>
__global__ void __launch_bounds__(64) k_render_fwd(ViewSet vs, Geom geom, const uint32_t* __restrict__ vals,
                                                   const uint32_t* __restrict__ ranges,
                                                   unsigned long long* pair_counter) {
  constexpr int kParts = 4 / kPx;
  constexpr bool kTest = !kCulled || kParts > 1;  // not every listed Gaussian is walked
  constexpr int kGroup = forward_group(kPx);
  __shared__ float2 s_xy[64];
  __shared__ float4 s_co[64];
  __shared__ float4 s_rgb[64];  // rgb and the list position (as int bits)
  __shared__ float s_z[kCh ? 64 : 1];
  __shared__ float4 s_fv[kCh ? 64 : 1];  // v~ and rho
  const int64_t ntiles = live_tiles(vs);
  const int64_t tile = xcd_tile(static_cast<int64_t>(blockIdx.x) / (8 * kParts) * 8 + (blockIdx.x & 7), vs.total_tiles);
  const int part = static_cast<int>(blockIdx.x >> 3) % kParts;
  if (tile >= ntiles) return;
  const View& v = view_at(vs, view_of_tile(vs, tile));
  const int64_t local = tile - v.tile_off;
  const int tx = static_cast<int>(local % v.GX), ty = static_cast<int>(local / v.GX);
  const int row0 = ty * kTile + 4 * kPx * part;  // the strip's first row
  if (row0 >= v.H) return;
  const int lane = threadIdx.x;
  const int px = tx * kTile + (lane & 15);
  const int py0 = row0 + (lane >> 4);
  const float fpx = static_cast<float>(px);
  float X0, X1, Y0, Y1;
  tile_bounds(tx, ty, v.W, v.H, X0, X1, Y0, Y1);
  const float S0 = static_cast<float>(row0), S1 = static_cast<float>(min(v.H, row0 + 4 * kPx) - 1);  // the strip's rows
  const uint64_t lt = (1ull << lane) - 1ull;
  float T[kPx], Cr[kPx], Cg[kPx], Cb[kPx], Dz[kPx], V0[kPx], V1[kPx], V2[kPx], Rh[kPx];
  float Aw[kPx];  // sum T alpha, the normalized depth's denominator
  int last[kPx];
  float thr[kPx];       // alpha a pair needs to be used: 1/255, or infinity once the pixel has stopped
  uint64_t live = 0;    // lanes with a pixel that has not stopped
#pragma unroll
  for (int k = 0; k < kPx; ++k) {
    T[k] = 1.0f; Cr[k] = 0.0f; Cg[k] = 0.0f; Cb[k] = 0.0f; last[k] = 0;
    Dz[k] = 0.0f; V0[k] = 0.0f; V1[k] = 0.0f; V2[k] = 0.0f; Rh[k] = 0.0f; Aw[k] = 0.0f;
    const bool in = px < v.W && py0 + 4 * k < v.H;
    thr[k] = in ? kAlphaMin : kNever;
    live |= __ballot(in);
  }
  auto blend = [&](int k, const float4& cc, float gz, const float4& gv, float w) {
    Cr[k] = fmaf(cc.x, w, Cr[k]);
    Cg[k] = fmaf(cc.y, w, Cg[k]);
    Cb[k] = fmaf(cc.z, w, Cb[k]);
    if (kCh) {
      Dz[k] = fmaf(gz, w, Dz[k]);
      Aw[k] += w;
      V0[k] = fmaf(gv.x, w, V0[k]);
      V1[k] = fmaf(gv.y, w, V1[k]);
      V2[k] = fmaf(gv.z, w, V2[k]);
      Rh[k] = fmaf(gv.w, w, Rh[k]);
    }
  };
  const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
  long long evaluated = 0;
  for (uint32_t b0 = start; b0 < end && live; b0 += 64) {
    const uint32_t idx = b0 + lane;
    bool keep = false, plain = true;
    float2 m;
    float4 co, c;
    float z = 0.0f;
    float4 fv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (idx < end) {
      const uint32_t g = vals[idx];
      m = reinterpret_cast<const float2*>(geom.xy)[g];
      co = reinterpret_cast<const float4*>(geom.conic_op)[g];
      c = make_float4(geom.rgb[3 * g], geom.rgb[3 * g + 1], geom.rgb[3 * g + 2],
                      __int_as_float(static_cast<int>(idx - start) + 1));
      if (kCh) {
        z = geom.depth[g];
        if (geom.feat) fv = reinterpret_cast<const float4*>(geom.feat)[g];
      }
      keep = kCulled || tile_reachable(m.x, m.y, co.x, co.y, co.z, co.w, X0, X1, Y0, Y1);
      if (kParts > 1) keep = keep && rect_reachable(m.x, m.y, co.x, co.y, co.z, co.w, X0, X1, S0, S1);
      plain = !keep || pair_is_plain(m, co);
    }
    const uint64_t km = __ballot(keep);
    const int cnt = __popcll(km);
    if (keep) {
      const int slot = __popcll(km & lt);
      s_xy[slot] = m;
      s_co[slot] = pair_coefs(co.x, co.y, co.z, co.w);
      s_rgb[slot] = c;
      if (kCh) {
        s_z[slot] = z;
        s_fv[slot] = fv;
      }
    }
    if (lane >= cnt && lane < (cnt + kGroup - 1) / kGroup * kGroup) {
      // padding up to a whole group (the lane may also have filled a slot
      // below cnt): opacity 0 gives alpha = 0, which no pixel uses, and
      // finite values keep the blends' products at 0
      s_xy[lane] = make_float2(0.0f, 0.0f);
      s_co[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s_rgb[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (kCh) {
        s_z[lane] = 0.0f;
        s_fv[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
    }
    __syncthreads();
    // Pairs go in groups of kGroup.  The walk is bound by VALU issue, so the
    // common path holds only what every pixel needs: a stopped pixel is one
    // whose threshold no alpha passes, an unused pair takes alpha = 0 (which
    // leaves T and the sums as they are), and whether a pixel stops is asked
    // once per group (T only falls, so its value behind the group tells).  A
    // tile's pixels stop within a few pairs of each other (0.5 pairs before
    // the tile's end on average on the 1M-Gaussian driving path, 5 on the
    // 200k box), so only a walk's last groups take the second path, pair by
    // pair with the stop test.
    auto walk = [&](auto plain_pairs) {
      constexpr bool kPlain = decltype(plain_pairs)::value;
      for (int j0 = 0;; j0 += kGroup) {
        bool stopped = false;
        for (; j0 < cnt; j0 += kGroup) {
          float w[kGroup][kPx], Tn[kPx];
          bool ok[kGroup][kPx];
#pragma unroll
          for (int k = 0; k < kPx; ++k) Tn[k] = T[k];
#pragma unroll
          for (int u = 0; u < kGroup; ++u) {
            const float2 gm = s_xy[j0 + u];
            const float4 gc = s_co[j0 + u];
            const float dx = gm.x - fpx;
            const float c1 = gc.y * dx, c0 = (gc.x * dx) * dx;
#pragma unroll
            for (int k = 0; k < kPx; ++k) {
              const float dy = gm.y - static_cast<float>(py0 + 4 * k);
              const float p2 = pair_exp2(gc.z, c1, c0, dy);
              const float raw = gc.w * __builtin_amdgcn_exp2f(p2);
              const float alpha = kPlain ? raw : fminf(kAlphaMax, raw);
              ok[u][k] = !(alpha < thr[k]) && (kPlain || !(p2 > 0.0f));
              const float au = ok[u][k] ? alpha : 0.0f;
              w[u][k] = au * Tn[k];
              Tn[k] = Tn[k] * (1.0f - au);
            }
          }
          bool stops = false;
#pragma unroll
          for (int k = 0; k < kPx; ++k) stops = stops || Tn[k] < kTMin;
          if (__any(stops)) {
            stopped = true;
            break;
          }
#pragma unroll
          for (int u = 0; u < kGroup; ++u) {
            const float4 cc = s_rgb[j0 + u];
            const float gz = kCh ? s_z[j0 + u] : 0.0f;
            const float4 gv = kCh ? s_fv[j0 + u] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const int pos = kTest ? __float_as_int(cc.w) : static_cast<int>(b0 - start) + j0 + u + 1;
#pragma unroll
            for (int k = 0; k < kPx; ++k) {
              if (kCount) evaluated += (thr[k] < 1.0f && j0 + u < cnt) ? 1 : 0;
              blend(k, cc, gz, gv, w[u][k]);
              last[k] = ok[u][k] ? pos : last[k];
            }
          }
#pragma unroll
          for (int k = 0; k < kPx; ++k) T[k] = Tn[k];
        }
        if (!stopped) return;
#pragma unroll 1
        for (int j4 = j0; j4 < j0 + kGroup; j4 += 4) {
#pragma unroll 1
          for (int j = j4; j < j4 + 4; ++j) {
            const float2 gm = s_xy[j];
            const float4 gc = s_co[j];
            const float4 cc = s_rgb[j];
            const float gz = kCh ? s_z[j] : 0.0f;
            const float4 gv = kCh ? s_fv[j] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const int pos = kTest ? __float_as_int(cc.w) : static_cast<int>(b0 - start) + j + 1;
            const float dx = gm.x - fpx;
            const float c1 = gc.y * dx, c0 = (gc.x * dx) * dx;
            bool on = false;
#pragma unroll
            for (int k = 0; k < kPx; ++k) {
              if (kCount) evaluated += (thr[k] < 1.0f && j < cnt) ? 1 : 0;
              const float dy = gm.y - static_cast<float>(py0 + 4 * k);
              const float p2 = pair_exp2(gc.z, c1, c0, dy);
              const float raw = gc.w * __builtin_amdgcn_exp2f(p2);
              const float alpha = kPlain ? raw : fminf(kAlphaMax, raw);
              const bool pass = !(alpha < thr[k]) && (kPlain || !(p2 > 0.0f));
              const float Tp = T[k] * (1.0f - alpha);
              const bool stop = pass && Tp < kTMin, use = pass && !stop;
              blend(k, cc, gz, gv, use ? alpha * T[k] : 0.0f);
              T[k] = use ? Tp : T[k];
              last[k] = use ? pos : last[k];
              thr[k] = stop ? kNever : thr[k];
              on = on || thr[k] < 1.0f;
            }
            live = __ballot(on);
          }
          if (!live) return;  // the next four pairs are not blended: their values may be NaN
        }
      }
    };
    if (__all(plain)) walk(std::true_type{});
    else walk(std::false_type{});
    __syncthreads();
  }
  const int64_t HW = static_cast<int64_t>(v.W) * v.H;
#pragma unroll
  for (int k = 0; k < kPx; ++k) {
    const int py = py0 + 4 * k;
    if (px < v.W && py < v.H) {
      const int64_t o = static_cast<int64_t>(py) * v.W + px;
      v.img[o] = Cr[k] + T[k] * v.bg[0];
      v.img[HW + o] = Cg[k] + T[k] * v.bg[1];
      v.img[2 * HW + o] = Cb[k] + T[k] * v.bg[2];
      v.final_T[o] = T[k];
      v.n_contrib[o] = last[k];
      if (v.opacity_img) v.opacity_img[o] = 1.0f - T[k];
      if (kCh) {
        // every contributor has alpha >= 1/255, so the sum is 0 exactly when none did
        if (v.depth_img) v.depth_img[o] = !v.depth_norm ? Dz[k] : (Aw[k] > 0.0f ? Dz[k] / Aw[k] : 0.0f);
        if (v.vbar_img) {
          v.vbar_img[o] = V0[k];
          v.vbar_img[HW + o] = V1[k];
          v.vbar_img[2 * HW + o] = V2[k];
        }
        if (v.rho_img) v.rho_img[o] = Rh[k];
      }
    }
  }
  if (kCount && pair_counter) {
    long long e = evaluated;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
    if (lane == 0) atomicAdd(pair_counter, static_cast<unsigned long long>(e));
  }
}

// kCh: the view also carries upstream gradients of the depth, velocity and
// staticness channels and/or of final_T (each may be null); records then hold
// five more sums (d z, d v~, d rho).
//
// Bound: vector issue (a 1M-Gaussian 1920x1280 view walks 1.2M pairs of 256
// pixels; its records are 60 MB).  Four pairs form a group: their pixel work
// is unrolled back to front, and their 36 (56) sums are folded together
// (group_sum_store), which takes a third of the instructions of folding each
// pair's nine by DPP.  A batch whose pairs cannot clamp (pair_is_plain) walks
// without the clamp's tests, a group behind every pixel's last contributor
// without the position's.  Mean per view, us: 1M 382 -> 329 (channels 497 ->
// 465), 200k at 960x640 164 -> 135.  Three waves a SIMD (141 registers;
// channels 168, a few words spilled): at four the plain kernel is even at 1M
// and 4% slower on 1280x720, at five, which spills, 7%; channels at two 5%.
//
// The order of every sum is fixed by design, pair by pair and pixel by pixel:
// near the camera a Gaussian's gradient is the difference of sums many
// thousand times its size, so another order moves single elements by more
// than 1e-3 of their size.  The two products of the mean's gradient are
// written as fused multiply-adds for the same reason: left to contraction,
// which product is rounded first depends on the instantiation.
template <bool kCount, bool kCulled, bool kCh>
__global__ void __launch_bounds__(64, 3) k_render_bwd(ViewSet vs, Geom geom, Lists lists, float* rec,
                                                   uint8_t* vis, unsigned long long* pair_counter) {
  // The gradient arithmetic may fuse multiply-adds.  Every branch decision
  // (exponent sign, alpha thresholds) comes from pair_coefs, pair_exp2 (its
  // FMAs explicit) and single products, which fuse with nothing, so the
  // adjoint takes the forward's.
#pragma clang fp contract(fast)
  const uint32_t* __restrict__ vals = lists.vals;
  const uint32_t* __restrict__ ranges = lists.ranges;
  constexpr int kG = 4;                 // pairs per group
  constexpr int kSums = kCh ? 14 : 9;   // also the record stride
  __shared__ float2 s_xy[64];
  __shared__ float4 s_co[64];   // -A, -B, -C and 1 / o
  __shared__ float4 s_q[64];    // pair_coefs of the conic and the opacity
  __shared__ float4 s_rgb[64];  // rgb and the 0-based list position (as int bits)
  __shared__ float s_z[kCh ? 64 : 1];
  __shared__ float4 s_fv[kCh ? 64 : 1];
  __shared__ __align__(16) float s_red[kSums * kG * kRedStride];
  __shared__ float s_acc[64][kSums];
  const int64_t ntiles = live_tiles(vs);
  const int64_t tile = xcd_tile(blockIdx.x, vs.total_tiles);
  if (tile >= ntiles) return;
  const View& v = view_at(vs, view_of_tile(vs, tile));
  const int64_t local = tile - v.tile_off;
  const int tx = static_cast<int>(local % v.GX), ty = static_cast<int>(local / v.GX);
  const int lane = threadIdx.x;
  const int px = tx * kTile + (lane & 15);
  const int py0 = ty * kTile + (lane >> 4);
  const float fpx = static_cast<float>(px);
  float X0, X1, Y0, Y1;
  tile_bounds(tx, ty, v.W, v.H, X0, X1, Y0, Y1);
  const uint64_t lt = (1ull << lane) - 1ull;
  const int64_t HW = static_cast<int64_t>(v.W) * v.H;
  float T[kPix], rr[kPix], gr[kPix], gg[kPix], gb[kPix];
  float gd[kPix], gv0[kPix], gv1[kPix], gv2[kPix], gh[kPix];  // channel gradients: z, v~, rho
  int last[kPix];
  float thr[kPix];  // alpha a pair needs to be used: 1/255, or infinity outside the image
  int lmax = 0, lmin = INT_MAX;
#pragma unroll
  for (int k = 0; k < kPix; ++k) {
    const int py = py0 + 4 * k;
    float gt = 0.0f;
    gd[k] = 0.0f; gv0[k] = 0.0f; gv1[k] = 0.0f; gv2[k] = 0.0f; gh[k] = 0.0f;
    thr[k] = kNever;
    if (px < v.W && py < v.H) {
      const int64_t o = static_cast<int64_t>(py) * v.W + px;
      thr[k] = kAlphaMin;
      T[k] = v.final_T[o];
      last[k] = v.n_contrib[o];
      lmin = min(lmin, last[k]);
      gr[k] = v.dL_dimg[o];
      gg[k] = v.dL_dimg[HW + o];
      gb[k] = v.dL_dimg[2 * HW + o];
      if (kCh) {
        if (v.dL_dT) gt = v.dL_dT[o];
        if (v.dL_dO) gt -= v.dL_dO[o];  // O = 1 - final_T
        if (v.dL_ddepth) {
          gd[k] = v.dL_ddepth[o];
          if (v.depth_norm) {
            // D / A with A = sum T alpha = 1 - final_T: d/dD = 1 / A and, the
            // sum telescoping, d/d final_T = (D / A) / A
            const float A = 1.0f - T[k];
            const float ia = A > 0.0f ? 1.0f / A : 0.0f;
            gt = fmaf(gd[k] * v.depth_img[o], ia, gt);
            gd[k] *= ia;
          }
        }
        if (v.dL_dvbar) {
          gv0[k] = v.dL_dvbar[o];
          gv1[k] = v.dL_dvbar[HW + o];
          gv2[k] = v.dL_dvbar[2 * HW + o];
        }
        if (v.dL_drho) gh[k] = v.dL_drho[o];
      }
    } else {
      T[k] = 1.0f; last[k] = 0; gr[k] = 0.0f; gg[k] = 0.0f; gb[k] = 0.0f;
    }
    // the blend behind the last contributor: the background colour, and for
    // final_T a channel that is 0 on every Gaussian and 1 behind them all
    rr[k] = v.bg[0] * gr[k] + v.bg[1] * gg[k] + v.bg[2] * gb[k] + gt;
    lmax = max(lmax, last[k]);
  }
  lmax = wave_max(lmax);
  lmin = -wave_max(-lmin);
  const uint32_t start = ranges[2 * tile];
  lmax = min(lmax, static_cast<int>(ranges[2 * tile + 1] - start));  // never read past the tile's list
  long long evaluated = 0;
  for (int hi = lmax; hi > 0; hi -= 64) {
    const int lo = max(0, hi - 64);
    bool keep = false, plain = true;
    uint32_t g = 0;
    float2 m;
    float4 co, c;
    float z = 0.0f;
    float4 fv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (lane < hi - lo) {
      g = vals[start + lo + lane];
      m = reinterpret_cast<const float2*>(geom.xy)[g];
      co = reinterpret_cast<const float4*>(geom.conic_op)[g];
      c = make_float4(geom.rgb[3 * g], geom.rgb[3 * g + 1], geom.rgb[3 * g + 2], __int_as_float(lo + lane));
      if (kCh) {
        z = geom.depth[g];
        if (geom.feat) fv = reinterpret_cast<const float4*>(geom.feat)[g];
      }
      keep = kCulled || tile_reachable(m.x, m.y, co.x, co.y, co.z, co.w, X0, X1, Y0, Y1);
      plain = !keep || pair_is_plain(m, co);
    }
    const uint64_t km = __ballot(keep);
    const int cnt = __popcll(km);
    const int slot = __popcll(km & lt);
    if (keep) {
      s_xy[slot] = m;
      // the negated conic and 1 / o for the record sums (one reciprocal per
      // Gaussian and batch rather than per pair)
      s_co[slot] = make_float4(-co.x, -co.y, -co.z, co.w > 0.0f ? __builtin_amdgcn_rcpf(co.w) : 0.0f);
      s_q[slot] = pair_coefs(co.x, co.y, co.z, co.w);
      s_rgb[slot] = c;
      if (kCh) {
        s_z[slot] = z;
        s_fv[slot] = fv;
      }
    }
    if (lane >= cnt && lane < (cnt + kG - 1) / kG * kG) {  // padding pairs, which no pixel uses
      s_xy[lane] = make_float2(0.0f, 0.0f);
      s_co[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s_q[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s_rgb[lane] = make_float4(0.0f, 0.0f, 0.0f, __int_as_float(INT_MAX));
      if (kCh) {
        s_z[lane] = 0.0f;
        s_fv[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
    }
    __syncthreads();
    uint64_t used = 0;  // pairs of the batch that some pixel uses
    // One group of pairs j0 .. j0 + 3.  kPlain: no pair of the batch needs the
    // clamp or the exponent's sign; kAll: every pixel is past its last
    // contributor's position, so the list position needs no test.
    auto group = [&](auto plain_pairs, auto all_pixels, int j0) {
      constexpr bool kPlain = decltype(plain_pairs)::value, kAll = decltype(all_pixels)::value;
      float h[kSums][2];  // the pairs' sums folded over the half-waves: pairs 0 | 1 and 2 | 3
#pragma unroll
      for (int half = 1; half >= 0; --half) {
        if (!kAll && half == 1 && j0 + 2 >= cnt) {  // both padding, half of the walk where lists are short
#pragma unroll
          for (int q = 0; q < kSums; ++q) h[q][1] = 0.0f;
          continue;
        }
        float a[2][kSums];
#pragma unroll
        for (int sub = 1; sub >= 0; --sub) {
          const int u = 2 * half + sub, j = j0 + u;
          const float2 gm = s_xy[j];
          const float4 gc = s_co[j];
          const float4 gq = s_q[j];
          const float4 cc = s_rgb[j];
          const float gz = kCh ? s_z[j] : 0.0f;
          const float4 gf = kCh ? s_fv[j] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          const int pos = __float_as_int(cc.w);
          // The lane's four pixels share the column offset dx.  Per pixel the
          // power gradient is gp = alpha dL/dalpha (zero where the pair is unused
          // or alpha is clamped); the lane sums s0 = sum gp, s1 = sum gp dy and
          // s2 = sum gp dy^2, from which the moments of gp in (dx, dy) follow.
          // An unused pair takes alpha = 0, which leaves T (rcp(1) is exact)
          // and the colour behind it unchanged, so no selects are needed.
          const float dx = gm.x - fpx;
          const float c1 = gq.y * dx, c0 = (gq.x * dx) * dx;
          float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, cr = 0.0f, cgr = 0.0f, cb = 0.0f;
          float cz = 0.0f, cv0 = 0.0f, cv1 = 0.0f, cv2 = 0.0f, ch = 0.0f;
          uint64_t any = 0;
#pragma unroll
          for (int k = 0; k < kPix; ++k) {
            if (kCount) evaluated += (thr[k] < 1.0f && j < cnt && (kAll || pos < last[k])) ? 1 : 0;
            const float dy = gm.y - static_cast<float>(py0 + 4 * k);
            const float p2 = pair_exp2(gq.z, c1, c0, dy);
            const float raw = gq.w * __builtin_amdgcn_exp2f(p2);
            const float alpha = kPlain ? raw : fminf(kAlphaMax, raw);
            bool ok = !(alpha < thr[k]);
            if (!kPlain) ok = ok && !(p2 > 0.0f);
            if (!kAll) ok = ok && pos < last[k];
            any |= __ballot(ok);
            const float au = ok ? alpha : 0.0f;
            const float om = 1.0f - au;
            T[k] *= __builtin_amdgcn_rcpf(om);
            float cg = cc.x * gr[k] + cc.y * gg[k] + cc.z * gb[k];
            if (kCh) {  // the channels blend like a colour
              cg = fmaf(gz, gd[k], cg);
              cg = fmaf(gf.x, gv0[k], cg);
              cg = fmaf(gf.y, gv1[k], cg);
              cg = fmaf(gf.z, gv2[k], cg);
              cg = fmaf(gf.w, gh[k], cg);
            }
            const float d = cg - rr[k];
            const float dal = T[k] * d;
            const float w = au * T[k];
            cr = fmaf(w, gr[k], cr);
            cgr = fmaf(w, gg[k], cgr);
            cb = fmaf(w, gb[k], cb);
            if (kCh) {
              cz = fmaf(w, gd[k], cz);
              cv0 = fmaf(w, gv0[k], cv0);
              cv1 = fmaf(w, gv1[k], cv1);
              cv2 = fmaf(w, gv2[k], cv2);
              ch = fmaf(w, gh[k], ch);
            }
            rr[k] = fmaf(au, d, rr[k]);  // alpha c + (1 - alpha) rr
            const float gp = (!kPlain && raw > kAlphaMax ? 0.0f : au) * dal;
            s0 += gp;
            s1 = fmaf(dy, gp, s1);
            s2 = fmaf(dy * dy, gp, s2);
          }
          used |= any ? 1ull << j : 0ull;
          // power = -(A dx^2 + C dy^2)/2 - B dx dy and d(mean) = d(dx, dy); the
          // exponential's own gradient, sum G dL/dalpha over unclamped pairs, is
          // s0 / o (there alpha = o G)
          const float sx = dx * s0;
          a[sub][0] = kCh ? fmaf(gc.x, sx, gc.y * s1) : fmaf(gc.y, s1, gc.x * sx);
          a[sub][1] = kCh ? fmaf(gc.y, sx, gc.z * s1) : fmaf(gc.z, s1, gc.y * sx);
          a[sub][2] = -0.5f * (dx * sx);
          a[sub][3] = -(dx * s1);
          a[sub][4] = -0.5f * s2;
          a[sub][5] = s0 * gc.w;  // gc.w = 1 / o (0 for o = 0)
          a[sub][6] = cr;
          a[sub][7] = cgr;
          a[sub][8] = cb;
          if constexpr (kCh) {
            a[sub][9] = cz;
            a[sub][10] = cv0;
            a[sub][11] = cv1;
            a[sub][12] = cv2;
            a[sub][13] = ch;
          }
        }
#pragma unroll
        for (int q = 0; q < kSums; ++q) h[q][half] = swap_sum32(a[0][q], a[1][q]);
      }
      group_sum_store<kSums>(h, lane, s_red, &s_acc[j0][0]);
    };
    auto walk = [&](auto plain_pairs) {
      int j0 = (cnt - 1) / kG * kG;
      if (cnt == 0) return;
      for (; j0 >= 0; j0 -= kG) {  // until every pixel is past its last contributor
        const int p_hi = __builtin_amdgcn_readfirstlane(__float_as_int(s_rgb[j0 + kG - 1].w));
        if (p_hi < lmin) break;  // (a padding pair's position is never below)
        group(plain_pairs, std::false_type{}, j0);
      }
      for (; j0 >= 0; j0 -= kG) group(plain_pairs, std::true_type{}, j0);
    };
    if (__all(plain)) walk(std::true_type{});
    else walk(std::false_type{});
    __syncthreads();
    if (keep && (used >> slot & 1ull)) {
      // record of this (Gaussian, tile) pair at its emission-order index,
      // flagged for the gather (pairs no pixel used keep flag 0, no record)
      const uint32_t e = record_index<kCulled>(lists, geom, v, g, m, tx, ty);
      if (static_cast<int64_t>(e) < lists.capacity) {
        float* dst = rec + kSums * static_cast<int64_t>(e);
#pragma unroll
        for (int q = 0; q < kSums; ++q) dst[q] = s_acc[slot][q];
        vis[e] = 1;
      }
    }
    __syncthreads();
  }
  if (kCount && pair_counter) {
    long long e = evaluated;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
    if (lane == 0) atomicAdd(pair_counter, static_cast<unsigned long long>(e));
  }
}

// Per visible Gaussian: the index range of its pairs (first[g] and the
// listed count: its rectangle's tiles, or, for culled lists, up to the end
// of its last row) and the sum of the flagged records.
// kCh: the records hold the five channel sums too (d z, d v~, d rho); g2d
// slots 9..13 receive them, or zeros.
template <bool kCulled, bool kCh>
__global__ void __launch_bounds__(256) k_grad_gather(ViewSet vs, Geom geom, Lists lists,
                                                     const float* __restrict__ rec,
                                                     const uint8_t* __restrict__ vis, float* g2d) {
  constexpr int kSums = kCh ? 14 : 9;
  __shared__ uint32_t s_queue[256][3];  // wave-gathered Gaussians from the front, block-gathered from the back
  __shared__ uint32_t s_idx[4][1024];   // per wave: flagged pair indices of one round
  __shared__ float s_part[4][16];       // per wave: its share of a block-gathered Gaussian's sums
  __shared__ int s_qn, s_hn;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (tid == 0) { s_qn = 0; s_hn = 0; }
  __syncthreads();
  const int64_t gi = static_cast<int64_t>(blockIdx.x) * 256 + tid;
  const bool visible = gi < live_gauss(vs) && geom.radius[gi] > 0;
  uint32_t e0 = 0, cnt = 0;
  if (visible) record_range<kCulled>(vs, geom, lists, gi, e0, cnt);
  if (visible && cnt <= kShortRange) {
    float acc[16];
    gather_range<kSums>(e0, cnt, rec, vis, acc);
    float* dst = g2d + kG2DStride * gi;
#pragma unroll
    for (int c = 0; c < 14; ++c) dst[c] = acc[c];
  } else if (visible) {
    const int q = cnt > kHugeRange ? 255 - atomicAdd(&s_hn, 1) : atomicAdd(&s_qn, 1);
    s_queue[q][0] = static_cast<uint32_t>(gi);
    s_queue[q][1] = e0;
    s_queue[q][2] = cnt;
  }
  __syncthreads();
  const int qn = s_qn, hn = s_hn;
  for (int qi = wid; qi < qn; qi += 4) {
    const uint32_t g = s_queue[qi][0];
    float acc[16], red[4];
    gather_range_wave<kSums>(s_queue[qi][1], s_queue[qi][2], lane, rec, vis, s_idx[wid], acc);
    wave_sum16(acc, red);
    if ((lane & 15) == 0) {
      const int r = lane >> 4;
      float* dst = g2d + kG2DStride * static_cast<int64_t>(g);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int qq = 4 * k + 2 * (r & 1) + (r >> 1);
        if (qq < 14) dst[qq] = red[k];
      }
    }
  }
  // block-gathered Gaussians, one at a time: wave w sums rounds w, w + 4, ...
  // and the four shares are added in wave order
  for (int h = 0; h < hn; ++h) {
    const uint32_t g = s_queue[255 - h][0], he0 = s_queue[255 - h][1], hcnt = s_queue[255 - h][2];
    float acc[16], red[4];
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[c] = 0.0f;
    for (uint32_t r0 = 1024u * static_cast<uint32_t>(wid); r0 < hcnt; r0 += 4096u) {
      float part[16];
      gather_range_wave<kSums>(he0 + r0, min(1024u, hcnt - r0), lane, rec, vis, s_idx[wid], part);
#pragma unroll
      for (int c = 0; c < 16; ++c) acc[c] += part[c];
    }
    wave_sum16(acc, red);
    if ((lane & 15) == 0) {
      const int r = lane >> 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) s_part[wid][4 * k + 2 * (r & 1) + (r >> 1)] = red[k];
    }
    __syncthreads();
    if (tid < 14) g2d[kG2DStride * static_cast<int64_t>(g) + tid] = ((s_part[0][tid] + s_part[1][tid]) + s_part[2][tid]) + s_part[3][tid];
    __syncthreads();
  }
}

hipError_t launch_render_fwd(const ViewSet& vs, const Geom& geom, const uint32_t* vals, const uint32_t* ranges,
                             bool culled, hipStream_t s) {
  if (vs.total_tiles == 0) return hipSuccess;
  StageScope scope(PVG_STAGE_RENDER_FWD, s);
  const int parts = forward_parts(vs.total_tiles);
  const dim3 grid(static_cast<unsigned>(parts * render_grid(vs.total_tiles)));
  unsigned long long* cnt = profile_work_counter(PVG_STAGE_RENDER_FWD);
  // channels are single-view only
  const bool ch = !vs.table && (vs.one.depth_img || vs.one.vbar_img || vs.one.rho_img);
  auto pick = [&](auto count, auto channels) {
    constexpr bool kCount = decltype(count)::value, kCh = decltype(channels)::value;
    return parts == 4   ? (culled ? k_render_fwd<kCount, true, kCh, 1> : k_render_fwd<kCount, false, kCh, 1>)
           : parts == 2 ? (culled ? k_render_fwd<kCount, true, kCh, 2> : k_render_fwd<kCount, false, kCh, 2>)
                        : (culled ? k_render_fwd<kCount, true, kCh, 4> : k_render_fwd<kCount, false, kCh, 4>);
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  auto k = ch ? (cnt ? pick(yes, yes) : pick(no, yes)) : (cnt ? pick(yes, no) : pick(no, no));
  hipLaunchKernelGGL(k, grid, dim3(64), 0, s, vs, geom, vals, ranges, cnt);
  return hipGetLastError();
}

hipError_t launch_render_bwd(const ViewSet& vs, const Geom& geom, const Lists& lists, float* rec, uint8_t* vis,
                             int64_t vis_bytes, float* g2d, hipStream_t s) {
  if (vs.total_tiles == 0) return hipSuccess;
  const bool culled = lists.culled;
  // channel gradients are single-view only
  const bool ch =
      !vs.table && (vs.one.dL_ddepth || vs.one.dL_dT || vs.one.dL_dO || vs.one.dL_dvbar || vs.one.dL_drho);
  {
    StageScope scope(PVG_STAGE_RENDER_BWD, s);
    // clear the flags (a fill kernel: no memset node in a captured graph)
    hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(vis), 0u, vis_bytes / 4, s);
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>(render_grid(vs.total_tiles)));
    unsigned long long* cnt = profile_work_counter(PVG_STAGE_RENDER_BWD);
    auto k = ch ? (cnt ? (culled ? k_render_bwd<true, true, true> : k_render_bwd<true, false, true>)
                       : (culled ? k_render_bwd<false, true, true> : k_render_bwd<false, false, true>))
                : (cnt ? (culled ? k_render_bwd<true, true, false> : k_render_bwd<true, false, false>)
                       : (culled ? k_render_bwd<false, true, false> : k_render_bwd<false, false, false>));
    hipLaunchKernelGGL(k, grid, dim3(64), 0, s, vs, geom, lists, rec, vis, cnt);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (vs.total_gauss == 0) return hipSuccess;
  StageScope scope(PVG_STAGE_GRAD_GATHER, s);
  hipLaunchKernelGGL(ch ? (culled ? k_grad_gather<true, true> : k_grad_gather<false, true>)
                        : (culled ? k_grad_gather<true, false> : k_grad_gather<false, false>),
                     dim3(static_cast<unsigned>((vs.total_gauss + 255) / 256)), dim3(256), 0, s, vs, geom, lists, rec,
                     vis, g2d);
  return hipGetLastError();
}

}  // namespace pvg
