// Rendering loss with the D-SSIM term (Sec. 3.3, Eq. (5): L_render is the 3DGS weighted sum of
// L1 and D-SSIM): SSIM per colour channel with an 11 x 11 Gaussian window (sigma 1.5), zero
// padding, C1 = 0.01^2, C2 = 0.03^2, averaged over all pixels and channels of a view; its gradient
// and the L1 part's, in one pass over the images.
//
// One 256-thread block per (54 x 22 region, channel).  The region and a 10-pixel halo of both
// images are staged in LDS; four window moments are filtered: E[x], E[y], E[xy] and E[(x - y)^2],
// which give the denominators as the numerators plus (mu_x - mu_y)^2 and the variance of x - y (SSIM
// needs the two variances' sum only, and where x is near y, as in training, this form keeps the
// digits that E[x^2] - mu_x^2 loses).  They are filtered separably over the region and a 5-pixel
// halo, rows first (a thread filters four consecutive columns of a row from 14 loaded values), then
// columns (eight consecutive rows of a column from 18); per pixel the SSIM value and its derivatives
// with respect to the three moments that depend on the rendered image (E[x], E[x^2], E[xy]), scaled
// by dL/dS = -lambda w_s / (3 H W), go to LDS and are filtered back the same way (the window is
// symmetric, so the adjoint of the zero-padded filter is the same filter):
// dL/dx = L1 part + F*a + 2 x F*b + y F*c.  Per-region partial sums of the SSIM map and of |x - y|
// (no same-address atomics) are folded per view by the loss.  The window sums use fused
// multiply-adds in window order (this term is compared within a tolerance).
//
// Bound by vector issue: 256 multiply-adds per value, of which a third repeats the halo's moments.
// Three kernels (L1; moments, writing 36 bytes of derivatives per pixel; their filter) took 264 us
// for two 1080p images, their multiply-adds at half rate for taking the window from scalar
// registers; this one takes 152 us, and 690 us instead of 1,280 us for 16 training images.  What
// carried it, in us: one pass 253, eight-byte LDS reads 200, each stage's result in the place of its
// input (25 KB of LDS, five blocks per CU instead of three) 168, four moments instead of five 152.
#include "clod_internal.h"

namespace clod {

constexpr int kHalo = 5;
constexpr int kWin = 2 * kHalo + 1;
constexpr int kOutW = kSsimRegionW, kOutH = kSsimRegionH;           // outputs of a region
constexpr int kMapW = kOutW + 2 * kHalo, kMapH = kOutH + 2 * kHalo;  // SSIM map of a region: 64 x 32
constexpr int kStW = kMapW + 2 * kHalo, kStH = kMapH + 2 * kHalo;    // staged pixels: 74 x 42
constexpr int kQ = 4;                      // outputs per task along a row,
constexpr int kQc = 8, kQb = 6;            // along a column of the map, of the region
constexpr int kL = kWin + kQ - 1;          // 14 inputs per four outputs
constexpr int kXyStride = 74, kMapStride = 66, kBackW = (kOutW + kQ - 1) / kQ * kQ;
constexpr int kRowTasks = kStH * (kMapW / kQ), kRowRounds = (kRowTasks + kBlock - 1) / kBlock;       // 672, 3
constexpr int kBackRowTasks = kMapH * (kBackW / kQ), kBackColTasks = kOutW * ((kOutH + kQb - 1) / kQb);  // 448, 216
constexpr float kC1 = 0.0001f;             // 0.01^2
constexpr float kC2 = 0.0009f;             // 0.03^2
static_assert(kMapW == 64 && kMapW * (kMapH / kQc) == kBlock && kBackColTasks <= kBlock, "one column task per thread");
static_assert(kMapW - kQ + kL <= kXyStride && kBackW - kQ + kL <= kMapStride, "row reads stay in their row");

struct Region {
  int v, x0, y0;
};

// View and pixel origin of region r (binary search of the views' first regions).
__device__ __forceinline__ Region region_of(const DevView* views, int V, uint32_t r) {
  int lo = 0, hi = V - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].rgn_base <= r) lo = mid; else hi = mid - 1;
  }
  const DevView& Vw = views[lo];
  const int rx = (Vw.width + kOutW - 1) / kOutW;
  const int local = (int)(r - Vw.rgn_base);
  return Region{lo, (local % rx) * kOutW, (local / rx) * kOutH};
}

// Eight-byte LDS reads, kept from being merged: 16-byte reads of 16 lanes to a row meet in the banks
// unless the rows follow each other (8.4 to 11 cycles instead of 4.6; 8-byte reads always take 3).
typedef float Pair __attribute__((ext_vector_type(2)));
typedef const volatile __attribute__((address_space(3))) Pair LdsPair;
// Each stage's result replaces its input, which every thread has in registers by then.
struct __attribute__((aligned(16))) SsimLds {
  union {
    float xy[2][kStH][kXyStride];        // staged images
    float rows[2][kStH][kMapW];          // row sums of a moment, double buffered
    float map[3][kMapH][kMapStride];     // derivatives
    float back[3][kMapH][kBackW];        // row sums of the derivatives
  };
  float red[4][2];
};
static_assert(sizeof(SsimLds) <= 160 * 1024 / 6, "LDS for six blocks per CU");

// 1 / x to within an ulp (x normal): hardware reciprocal and a Newton step.
__device__ __forceinline__ float near_rcp(float x) {
  const float y = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, y, 1.0f), y, y);
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_ssim(const DevView* __restrict__ views, int V,
                                                 const float* __restrict__ rgb, const float* __restrict__ target,
                                                 SsimWindow win, float lambda, float s_max,
                                                 float* __restrict__ dL_drgb, float* __restrict__ part) {
  __shared__ SsimLds S;
  const uint32_t region = blockIdx.x;
  const int ch = blockIdx.y, t = (int)threadIdx.x;
  const Region R = region_of(views, V, region);
  const DevView& Vw = views[R.v];
  const int x0 = R.x0, y0 = R.y0;
  const int W = Vw.width, H = Vw.height;
  const int64_t HW = (int64_t)W * H;
  const int64_t img = 3ll * Vw.pix_base + (int64_t)ch * HW;
  // The window in vector registers: a multiply-add with a scalar operand issues at half the rate.
  float g[kHalo + 1];
#pragma unroll
  for (int k = 0; k <= kHalo; ++k) {
    g[k] = win.g[k];
    asm volatile("" : "+v"(g[k]));
  }
  auto tap = [&](int k) { return g[k <= kHalo ? k : 2 * kHalo - k]; };   // (symmetric)
  // Staging, every load issued before the first LDS store: wave w takes rows w, w + 4, ... (lane:
  // column), then the block the columns past 64.
  {
    constexpr int kRest = kStW - 64, kMain = (kStH + 3) / 4, kTail = (kStH * kRest + kBlock - 1) / kBlock;
    const float* __restrict__ xp = rgb + img;
    const float* __restrict__ yp = target + img;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int gx = x0 - 2 * kHalo + lane;
    const bool inx = (gx >= 0) & (gx < W);
    float lx[kMain + kTail], ly[kMain + kTail];
#pragma unroll
    for (int q = 0; q < kMain; ++q) {
      const int gy = y0 - 2 * kHalo + wave + 4 * q;   // uniform
      const bool in = inx & (gy >= 0) & (gy < H) & (wave + 4 * q < kStH);
      lx[q] = in ? xp[gy * W + gx] : 0.f;
      ly[q] = in ? yp[gy * W + gx] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kTail; ++q) {
      const int idx = t + q * kBlock, r = idx / kRest, c = 64 + idx - r * kRest;
      const int hx = x0 - 2 * kHalo + c, hy = y0 - 2 * kHalo + r;
      const bool in = (idx < kStH * kRest) & (hx < W) & (hy >= 0) & (hy < H);   // (hx >= 44)
      lx[kMain + q] = in ? xp[hy * W + hx] : 0.f;
      ly[kMain + q] = in ? yp[hy * W + hx] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kMain; ++q) {
      if (wave + 4 * q < kStH) {
        S.xy[0][wave + 4 * q][lane] = lx[q];
        S.xy[1][wave + 4 * q][lane] = ly[q];
      }
    }
#pragma unroll
    for (int q = 0; q < kTail; ++q) {
      const int idx = t + q * kBlock, r = idx / kRest, c = 64 + idx - r * kRest;
      if (idx < kStH * kRest) {
        S.xy[0][r][c] = lx[kMain + q];
        S.xy[1][r][c] = ly[kMain + q];
      }
    }
  }
  __syncthreads();
  // Rows: task (r, c0) filters columns c0 .. c0 + 3 of staged row r.
  float h[kRowRounds][4][kQ];   // x, y, x y, (x - y)^2
#pragma unroll
  for (int q = 0; q < kRowRounds; ++q) {
    const int task = t + q * kBlock;
    if (task < kRowTasks) {
      const int r = task / (kMapW / kQ), c0 = (task % (kMapW / kQ)) * kQ;
      float xs[kL], ys[kL];
      // (Pairs: 16-byte reads of rows that do not follow each other meet in the banks.)
#pragma unroll
      for (int k = 0; k < kL; k += 2) {
        const Pair a = *(LdsPair*)&S.xy[0][r][c0 + k];
        const Pair b = *(LdsPair*)&S.xy[1][r][c0 + k];
        xs[k] = a.x; xs[k + 1] = a.y;
        ys[k] = b.x; ys[k + 1] = b.y;
      }
#pragma unroll
      for (int j = 0; j < kQ; ++j)
#pragma unroll
        for (int m = 0; m < 4; ++m) h[q][m][j] = 0.f;
#pragma unroll
      for (int i = 0; i < kL; ++i) {
        const float xv = xs[i], yv = ys[i], xy = xv * yv, d = xv - yv, dd = d * d;
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
          const int k = i - j;
          if (k >= 0 && k < kWin) {
            h[q][0][j] = fmaf(tap(k), xv, h[q][0][j]);
            h[q][1][j] = fmaf(tap(k), yv, h[q][1][j]);
            h[q][2][j] = fmaf(tap(k), xy, h[q][2][j]);
            h[q][3][j] = fmaf(tap(k), dd, h[q][3][j]);
          }
        }
      }
    }
  }
  __syncthreads();
  // Columns: the thread filters rows r0 .. r0 + 7 of map column c, a moment at a time.
  const int c = t % kMapW, r0 = (t / kMapW) * kQc;
  float mom[4][kQc];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    float (*rows)[kMapW] = S.rows[m & 1];
#pragma unroll
    for (int q = 0; q < kRowRounds; ++q) {
      const int task = t + q * kBlock;
      if (task < kRowTasks)
        *reinterpret_cast<float4*>(&rows[task / (kMapW / kQ)][(task % (kMapW / kQ)) * kQ]) =
            make_float4(h[q][m][0], h[q][m][1], h[q][m][2], h[q][m][3]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kQc; ++j) mom[m][j] = 0.f;
#pragma unroll
    for (int i = 0; i < kWin + kQc - 1; ++i) {
      const float x = rows[r0 + i][c];
#pragma unroll
      for (int j = 0; j < kQc; ++j)
        if (i - j >= 0 && i - j < kWin) mom[m][j] = fmaf(tap(i - j), x, mom[m][j]);
    }
  }
  __syncthreads();
  // The SSIM map and its derivatives (0 outside the image).
  const float w_s = w_s_weight(Vw.s_v, s_max);
  const float up = -lambda * w_s / (3.0f * (float)HW);
  float s = 0.f;
  const int px = x0 - kHalo + c;
  const bool inx = (px >= 0) & (px < W), ownx = inx & (c >= kHalo) & (c < kHalo + kOutW);
#pragma unroll
  for (int j = 0; j < kQc; ++j) {
    const int r = r0 + j, py = y0 - kHalo + r;
    const bool iny = (py >= 0) & (py < H);
    const float mx = mom[0][j], my = mom[1][j], md = mx - my;
    const float A1 = 2.f * mx * my + kC1, A2 = 2.f * (mom[2][j] - mx * my) + kC2;
    const float B1 = A1 + md * md, B2 = A2 + (mom[3][j] - md * md);
    const float r1 = near_rcp(B1), r2 = near_rcp(B2), inv = r1 * r2;
    const float sv = A1 * A2 * inv;
    // dS/d(mu_x), dS/d(sigma_x^2), dS/d(sigma_xy), then the chain to the moments.
    const float d_mu = (2.f * my * A2) * inv - sv * (2.f * mx) * r1;
    const float d_var = -sv * r2;
    const float d_cov = 2.f * A1 * inv;
    const float u = inx & iny ? up : 0.f;
    S.map[0][r][c] = u * (d_mu - 2.f * mx * d_var - my * d_cov);
    S.map[1][r][c] = u * d_var;
    S.map[2][r][c] = u * d_cov;
    s += ownx & iny & (r >= kHalo) & (r < kHalo + kOutH) ? sv : 0.f;
  }
  __syncthreads();
  // Back: rows of the map (columns past it hold other rows' or stale values, which only reach
  // outputs past the region), then columns.
  constexpr int kBackRounds = (kBackRowTasks + kBlock - 1) / kBlock;
  float hb[kBackRounds][3][kQ];
#pragma unroll
  for (int q = 0; q < kBackRounds; ++q) {
    const int task = t + q * kBlock;
    if (task < kBackRowTasks) {
      const int r = task / (kBackW / kQ), c0 = (task % (kBackW / kQ)) * kQ;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        float xs[kL];
#pragma unroll
        for (int k = 0; k < kL; k += 2) {
          const Pair v = *(LdsPair*)&S.map[m][r][c0 + k];
          xs[k] = v.x; xs[k + 1] = v.y;
        }
#pragma unroll
        for (int j = 0; j < kQ; ++j) hb[q][m][j] = 0.f;
#pragma unroll
        for (int i = 0; i < kL; ++i)
#pragma unroll
          for (int j = 0; j < kQ; ++j)
            if (i - j >= 0 && i - j < kWin) hb[q][m][j] = fmaf(tap(i - j), xs[i], hb[q][m][j]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kBackRounds; ++q) {
    const int task = t + q * kBlock;
    if (task < kBackRowTasks) {
      const int r = task / (kBackW / kQ), c0 = (task % (kBackW / kQ)) * kQ;
#pragma unroll
      for (int m = 0; m < 3; ++m)
        *reinterpret_cast<float4*>(&S.back[m][r][c0]) = make_float4(hb[q][m][0], hb[q][m][1], hb[q][m][2], hb[q][m][3]);
    }
  }
  __syncthreads();
  const float scale = (1.0f - lambda) * w_s / (float)(3 * HW);   // of the L1 part's sign
  float l1 = 0.f;
  const int bc = t % kOutW, b0 = (t / kOutW) * kQb;
  if (t < kBackColTasks && x0 + bc < W) {
    // The pixels are read again (cache hits): requested before the sums.
    float x[kQb], y[kQb], f[3][kQb];
    const int64_t at = img + (int64_t)(y0 + b0) * W + x0 + bc;
#pragma unroll
    for (int j = 0; j < kQb; ++j) {
      const bool in = (b0 + j < kOutH) & (y0 + b0 + j < H);
      x[j] = in ? rgb[at + (int64_t)j * W] : 0.f;
      y[j] = in ? target[at + (int64_t)j * W] : 0.f;
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
      for (int j = 0; j < kQb; ++j) f[m][j] = 0.f;
#pragma unroll
      for (int i = 0; i < kWin + kQb - 1; ++i) {
        const float v = S.back[m][b0 + i < kMapH ? b0 + i : kMapH - 1][bc];   // (past it: rows past the region only)
#pragma unroll
        for (int j = 0; j < kQb; ++j)
          if (i - j >= 0 && i - j < kWin) f[m][j] = fmaf(tap(i - j), v, f[m][j]);
      }
    }
#pragma unroll
    for (int j = 0; j < kQb; ++j) {
      if (b0 + j < kOutH && y0 + b0 + j < H) {
        const float diff = x[j] - y[j];
        l1 += fabsf(diff);
        const float sign = diff > 0.f ? scale : (diff < 0.f ? -scale : 0.f);
        dL_drgb[at + (int64_t)j * W] = sign + (f[0][j] + 2.f * x[j] * f[1][j] + y[j] * f[2][j]);
      }
    }
  }
  s = wave_sum(s);
  l1 = wave_sum(l1);
  if (lane_id() == 0) { S.red[t >> 6][0] = s; S.red[t >> 6][1] = l1; }
  __syncthreads();
  if (t < 2) part[2 * (3 * (int64_t)region + ch) + t] = S.red[0][t] + S.red[1][t] + S.red[2][t] + S.red[3][t];
}

hipError_t launch_ssim(const Layout& L, void* ws, const float* rgb, const float* target, float lambda,
                       float s_max, float* part, float* dL_drgb, hipStream_t s) {
  if (L.ssim_regions == 0) return hipSuccess;
  SsimWindow win;
  double g[kWin], sum = 0.0;
  for (int k = 0; k < kWin; ++k) {
    const double d = (double)(k - kHalo);
    g[k] = exp(-d * d / (2.0 * 1.5 * 1.5));
    sum += g[k];
  }
  for (int k = 0; k < kWin; ++k) win.g[k] = (float)(g[k] / sum);
  const DevView* views = (const DevView*)((char*)ws + L.vinfo);
  hipLaunchKernelGGL(k_ssim, dim3(L.ssim_regions, 3), dim3(kBlock), 0, s, views, L.V, rgb, target, win, lambda, s_max,
                     dL_drgb, part);
  return hipGetLastError();
}

}  // namespace clod
