// Per-Gaussian stages: view setup, frustum maximum of the camera distance (Sec. 3.2),
// attenuated opacity of Eq. (2) with the LoD mask, EWA projection / cull / tile rectangle /
// SH colour (Sec. 3.1), and the standalone multi-view LoD counter.
//
// Reads are plane-major (structure of arrays): consecutive lanes read consecutive floats of
// a plane, so every wave load is a full 256-byte coalesced transaction.  One thread owns one
// Gaussian and loops over the views of the batch, so parameters are read once per batch.
#include "clod_internal.h"

namespace clod {

// Derives per-view constants on the device (graph-replay safe: reads only views_dev).  With `hdr`
// non-NULL the workspace header is cleared as well (a new projection).  One wave, a view per lane:
// the running bases are wave scans (one thread walking the views took 12 us for five views and
// 57 us for 64, on every render's critical path).
__device__ __forceinline__ void view_setup_body(const ViewSetupArgs& a, Blk b) {
  const clod_view* __restrict__ views = a.views;
  const int V = a.V;
  const clod_params& prm = a.prm;
  DevView* __restrict__ out = a.out;
  if (b.id != 0 || threadIdx.x >= 64u) return;
  const int lane = (int)threadIdx.x;
  if (a.hdr && lane < kHdrWords)
    a.hdr[lane] = lane == kHdrKeyBase ? (unsigned long long)__float_as_uint(prm.near_z) : 0ull;
  uint32_t tile_base = 0, pix_base = 0, loss_base = 0, rgn_base = 0, row_base = 0;
  int lead = 0;
  // Same camera: every field the positions, projections and colours depend on, bit for bit.
  auto same_camera = [](const clod_view& p, const clod_view& q) {
    uint32_t diff = 0;
    for (int j = 0; j < 9; ++j) diff |= __float_as_uint(p.W[j]) ^ __float_as_uint(q.W[j]);
    for (int j = 0; j < 3; ++j)
      diff |= (__float_as_uint(p.t[j]) ^ __float_as_uint(q.t[j])) | (__float_as_uint(p.c[j]) ^ __float_as_uint(q.c[j]));
    diff |= (__float_as_uint(p.fx) ^ __float_as_uint(q.fx)) | (__float_as_uint(p.fy) ^ __float_as_uint(q.fy)) |
            (__float_as_uint(p.cx) ^ __float_as_uint(q.cx)) | (__float_as_uint(p.cy) ^ __float_as_uint(q.cy));
    diff |= (uint32_t)((p.width ^ q.width) | (p.height ^ q.height) | (p.frame_width ^ q.frame_width) |
                       (p.frame_height ^ q.frame_height) | (p.vx ^ q.vx) | (p.vy ^ q.vy));
    return diff == 0u;
  };
  for (int v0 = 0; v0 < V; v0 += 64) {
    const int v = v0 + lane;
    const bool valid = v < V;
    const clod_view& cv = views[valid ? v : V - 1];
    const uint64_t starts = ballot64(valid && (v == 0 || !same_camera(cv, views[v - 1])));
    const uint64_t upto = starts & (lanemask_lt() | (1ull << lane));
    DevView d;
    d.cam_lead = upto ? v0 + 63 - __builtin_clzll(upto) : lead;
    lead = starts ? v0 + 63 - __builtin_clzll(starts) : lead;
    for (int j = 0; j < 9; ++j) d.W[j] = cv.W[j];
    for (int j = 0; j < 3; ++j) { d.t[j] = cv.t[j]; d.c[j] = cv.c[j]; }
    d.fx = cv.fx; d.fy = cv.fy; d.cx = cv.cx; d.cy = cv.cy;
    d.s_v = cv.s_v;
    // A viewport keeps its frame's frustum: the limits come from the frame size.
    const bool vp = cv.frame_width > 0 || cv.frame_height > 0;
    const int fw = vp ? cv.frame_width : cv.width, fh = vp ? cv.frame_height : cv.height;
    d.limx = prm.guard * ((0.5f * (float)fw) / cv.fx);
    d.limy = prm.guard * ((0.5f * (float)fh) / cv.fy);
    d.ftiles_x = (fw + kTile - 1) / kTile;
    d.ftiles_y = (fh + kTile - 1) / kTile;
    d.vx = vp ? cv.vx : 0;
    d.vy = vp ? cv.vy : 0;
    d.tau_sv = prm.tau * cv.s_v;
    d.width = cv.width;
    d.height = cv.height;
    d.tiles_x = (cv.width + kTile - 1) / kTile;
    d.tiles_y = (cv.height + kTile - 1) / kTile;
    // Bound for the counting pass (count_body): a Gaussian of largest scale s at depth z and
    // tangents (tx, ty) has projected variances of at most geo_k (1 + tx^2 + ty^2) (s / z)^2 +
    // dilation (the largest row sum of |W W^T| bounds the norm of W W^T).  Infinite, so that every
    // projection is evaluated, where the pixel error of its approximate centre is not far below
    // the margin it uses.
    {
      float wb = 0.f;
      for (int r = 0; r < 3; ++r) {
        float row = 0.f;
        for (int q = 0; q < 3; ++q)
          row += fabsf(cv.W[3 * r] * cv.W[3 * q] + cv.W[3 * r + 1] * cv.W[3 * q + 1] + cv.W[3 * r + 2] * cv.W[3 * q + 2]);
        wb = row > wb ? row : wb;
      }
      const float f = fmaxf(cv.fx, cv.fy), extent = prm.guard * (float)(fw > fh ? fw : fh);
      const bool ok = wb < 4.0f && f < 1e6f && extent < 1e5f && fabsf(cv.cx) < 1e5f && fabsf(cv.cy) < 1e5f;
      d.geo_k = ok ? 1.001f * wb * f * f : __builtin_inff();
    }
    d.budget = cv.budget;
    d.mkey = 0ull;
    // Running bases: the sums over the views before this one.
    auto before = [&](uint32_t mine, uint32_t& base) {
      uint32_t inc = valid ? mine : 0u;
      const uint32_t own = inc;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(inc, o, 64);
        if (lane >= o) inc += up;
      }
      const uint32_t first = base + inc - own;
      base += __shfl(inc, 63, 64);
      return first;
    };
    const uint32_t px = (uint32_t)(cv.width * cv.height);
    d.tile_base = before((uint32_t)(d.tiles_x * d.tiles_y), tile_base);
    d.rgn_base = before((uint32_t)(((cv.width + kSsimRegionW - 1) / kSsimRegionW) *
                                   ((cv.height + kSsimRegionH - 1) / kSsimRegionH)), rgn_base);
    d.pix_base = before(px, pix_base);
    d.loss_block_base = before((3u * px + kLossChunk - 1) / kLossChunk, loss_base);
    d.row_base = before((uint32_t)d.tiles_y, row_base);
    if (valid) out[v] = d;
  }
}
__global__ void k_view_setup(ViewSetupArgs a) { view_setup_body(a, grid_blk()); }

__device__ __forceinline__ void fill_body(const FillArgs& a, Blk b) {
  for (int64_t i = (int64_t)b.id * kBlock + threadIdx.x; i < a.count; i += (int64_t)b.n * kBlock) a.p[i] = a.value;
}
__global__ __launch_bounds__(kBlock) void k_fill_u32(FillArgs a) { fill_body(a, grid_blk()); }

// Folds the G per-block partials of view v (every thread of the block takes part).  With kpart: the maximum squared distance, stored as the key
// bits(sqrt(max)) << 32 (0 if the frustum is empty).  With cpart: the counts (sum; also to
// counts_dev when non-NULL), the kept ratio eta = n_mask / n of Eq. (4) (to eta_dev when
// non-NULL; binary32 quotient of the counts converted to binary32) and the lowest index at d_max
// (min), which completes the low half of that key.
__device__ __forceinline__ void fold_view(int v, const uint32_t* __restrict__ kpart, const uint32_t* __restrict__ cpart,
                          int G, int V, int64_t n, unsigned long long* __restrict__ dmax_key,
                          unsigned long long* __restrict__ counts, int64_t* __restrict__ counts_dev,
                          float* __restrict__ eta_dev) {
  __shared__ unsigned long long sm[4][4];
  __shared__ uint32_t smin[4];
  unsigned long long key = 0ull, c0 = 0, c1 = 0, c2 = 0;
  uint32_t imin = 0xFFFFFFFFu;
  for (int b = threadIdx.x; b < G; b += kBlock) {
    if (kpart) {
      const unsigned long long k = kpart[(int64_t)b * V + v];
      key = k > key ? k : key;
    }
    if (cpart) {
      const uint32_t* c = cpart + ((int64_t)b * V + v) * 4;
      c0 += c[0];
      c1 += c[1];
      c2 += c[2];
      imin = c[3] < imin ? c[3] : imin;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long ok = __shfl_xor(key, o, 64);
    key = ok > key ? ok : key;
    c0 += __shfl_xor(c0, o, 64);
    c1 += __shfl_xor(c1, o, 64);
    c2 += __shfl_xor(c2, o, 64);
    const uint32_t om = __shfl_xor(imin, o, 64);
    imin = om < imin ? om : imin;
  }
  const int w = threadIdx.x >> 6;
  if (lane_id() == 0) { sm[w][0] = key; sm[w][1] = c0; sm[w][2] = c1; sm[w][3] = c2; smin[w] = imin; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int j = 1; j < 4; ++j) {
      key = sm[j][0] > key ? sm[j][0] : key;
      c0 += sm[j][1]; c1 += sm[j][2]; c2 += sm[j][3];
      imin = smin[j] < imin ? smin[j] : imin;
    }
    if (kpart) {
      const float d2 = __uint_as_float((uint32_t)key);
      dmax_key[v] = key ? (unsigned long long)__float_as_uint(__builtin_sqrtf(d2)) << 32 : 0ull;
    }
    if (cpart) {
      counts[3 * v] = c0; counts[3 * v + 1] = c1; counts[3 * v + 2] = c2;
      if (counts_dev) {
        counts_dev[3 * v] = (int64_t)c0; counts_dev[3 * v + 1] = (int64_t)c1; counts_dev[3 * v + 2] = (int64_t)c2;
      }
      if (eta_dev) eta_dev[v] = n > 0 ? (float)c1 / (float)n : 0.0f;
      const unsigned long long dk = dmax_key[v];
      if (dk) dmax_key[v] = (dk & 0xFFFFFFFF00000000ull) | (unsigned long long)(0xFFFFFFFFu - imin);
    }
  }
  __syncthreads();
}

// Block v folds view v.
__device__ __forceinline__ void fold_body(const FoldArgs& a, Blk b) {
  zero_words(a.clear, a.clear_words, b);
  fold_view((int)b.id, a.kpart, a.cpart, a.G, a.V, a.n, a.dmax_key, a.counts, a.counts_dev, a.eta_dev);
}
__global__ __launch_bounds__(kBlock) void k_reduce_partials(FoldArgs a) { fold_body(a, grid_blk()); }

// Per-block partials instead of global atomics: block b owns the contiguous chunk
// [b*C, (b+1)*C) of Gaussians and writes one partial per view (the frustum-max key, the three
// counts); k_reduce_partials folds them per view (one block per view).  Same-address atomics
// from every wave
// serialise in L2 and would dominate these otherwise bandwidth-bound kernels.

// Frustum maximum of the squared distance per view, as the float bits (order-preserving for
// non-negative values; 0 = no Gaussian in the frustum).  fold_view turns the maximum
// into the key bits(d_max) << 32 (d_max its correctly rounded root, the largest distance),
// and k_classify finds the lowest index at that distance, which completes the key with
// 2^32 - 1 - index (so that ties resolve to the lowest index).
// words: LDS of kCamWords V words.
__device__ __forceinline__ void frustum_max_body(const FrustumArgs& a, Blk b, uint32_t* words) {
  constexpr int kVG = 8;      // views per group (keys held in registers)
  constexpr int kItems = 4;   // Gaussians per thread per round, loaded before any is used
  __shared__ uint32_t sm[kVG][4];
  const float* __restrict__ mean = a.mean;
  const int64_t n = a.n;
  const DevView* __restrict__ views = a.views;
  const int V = a.V;
  const float near_z = a.near_z;
  uint32_t* __restrict__ part = a.part;   // [G][V]
  CamLds* cam = reinterpret_cast<CamLds*>(words);
  for (int v = threadIdx.x; v < V; v += kBlock) cam[v] = cam_lds(views[v]);
  __syncthreads();
  int64_t lo, hi;
  block_chunk(n, b, lo, hi);
  for (int v0 = 0; v0 < V; v0 += kVG) {
    const int vn = V - v0 < kVG ? V - v0 : kVG;
    // A view whose camera run started earlier in this group takes its lead's maximum (same
    // camera, same frustum, same distances) instead of evaluating the Gaussians again.
    uint32_t shared = 0u;   // bit vv: view v0 + vv copies its lead's key
#pragma unroll
    for (int vv = 0; vv < kVG; ++vv)
      if (vv < vn && views[v0 + vv].cam_lead != v0 + vv && views[v0 + vv].cam_lead >= v0) shared |= 1u << vv;
    uint32_t key[kVG];
#pragma unroll
    for (int vv = 0; vv < kVG; ++vv) key[vv] = 0u;
    for (int64_t b0 = lo; b0 < hi; b0 += (int64_t)kItems * kBlock) {
      // Past the chunk's end the last Gaussian is taken again (the maximum stays).
      float px[kItems], py[kItems], pz[kItems];
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const int64_t j = b0 + (int64_t)k * kBlock + threadIdx.x, i = j < hi ? j : hi - 1;
        px[k] = mean[i];
        py[k] = mean[n + i];
        pz[k] = mean[2 * n + i];
      }
      const int kn = hi - b0 >= kItems * kBlock ? kItems : (int)((hi - b0 + kBlock - 1) / kBlock);   // uniform
#pragma unroll
      for (int vv = 0; vv < kVG; ++vv) {
        if (vv >= vn) break;
        if ((shared >> vv) & 1u) continue;
        const CamLds Vw = cam[v0 + vv];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
          if (k >= kn) continue;
          float x, y, z, ex, ey, ez;
          to_camera(Vw, px[k], py[k], pz[k], x, y, z);
          const uint32_t kk = __float_as_uint(cam_distance2(Vw, px[k], py[k], pz[k], ex, ey, ez));
          const uint32_t key2 = kk > key[vv] ? kk : key[vv];
          key[vv] = in_frustum(Vw, x, y, z, near_z) ? key2 : key[vv];
        }
      }
    }
    // (A run's views are consecutive: each shared view copies the one before it.)
#pragma unroll
    for (int vv = 1; vv < kVG; ++vv)
      if ((shared >> vv) & 1u) key[vv] = key[vv - 1];
#pragma unroll
    for (int vv = 0; vv < kVG; ++vv) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const uint32_t other = __shfl_xor(key[vv], o, 64);
        key[vv] = other > key[vv] ? other : key[vv];
      }
      if (lane_id() == 0) sm[vv][threadIdx.x >> 6] = key[vv];
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)vn) {
      const int vv = threadIdx.x;
      part[(int64_t)b.id * V + v0 + vv] = max(max(sm[vv][0], sm[vv][1]), max(sm[vv][2], sm[vv][3]));
    }
    __syncthreads();
  }
}
__global__ __launch_bounds__(kBlock) void k_frustum_max(FrustumArgs a) {
  extern __shared__ __align__(16) uint32_t words_dyn[];
  frustum_max_body(a, grid_blk(), words_dyn);
}

// log2(e) q at which the contract's exponential of -q becomes 0 (q = 86).
constexpr float kZeroExp = 124.0717f;

// Factors of Eq. (2) for the loops below, beside the camera in LDS (every block fills its own table).
__device__ __forceinline__ CamLds classify_cam(const DevView& Vw, unsigned long long dk) {
  CamLds L = cam_lds(Vw);
  const float dmax = dmax_from_key(dk);   // frustum maximum (1 if empty)
  L.k[0] = dmax;
  L.k[1] = 1.0f / dmax;
  L.k[2] = Vw.s_v;
  return L;
}
// A view without a budget whose threshold is 0 keeps every alpha'' above 0.
__device__ __forceinline__ bool zero_threshold(const DevView& Vw) { return Vw.budget <= 0 && Vw.tau_sv == 0.0f; }
// Counting: (s_v / d_max)^2 (NaN: no estimate), log2 of the mask's threshold, and the squared
// distance below which a Gaussian cannot hold the frustum maximum.  zeros: some view of the batch has
// a threshold of 0 (see lod_item).
__device__ __forceinline__ CamLds count_cam(const DevView& Vw, unsigned long long dk, float eps, bool zeros) {
  CamLds L = cam_lds(Vw);
  const float dmax = dmax_from_key(dk), r = Vw.s_v / dmax, kv = r * r;
  // The mask keeps alpha'' above tau s_v, or above (or at) the value of the budget's smallest key.
  const float thr = Vw.budget > 0 ? __uint_as_float((uint32_t)(Vw.mkey >> 32)) : Vw.tau_sv;
  const bool zero = zero_threshold(Vw), all = Vw.budget > 0 && Vw.mkey == 0ull;   // all: the budget is the whole scene
  const bool ok = in_exponents<100>(kv) && eps > 1e-36f && (zero || (thr >= 0x1p-100f && !zeros));
  L.k[0] = all ? 0.0f : ok ? kv : __builtin_nanf("");
  L.k[1] = all ? -__builtin_inff() : zero ? -kZeroExp : __builtin_amdgcn_logf(thr);
  L.k[2] = dk ? (dmax * 0.999999f) * dmax : __builtin_inff();
  return L;
}
// Whether some view has a threshold of 0 (every thread of the block takes part; s_v is 1 or more).
__device__ __forceinline__ bool any_zero_threshold(const DevView* views, int V, float tau) {
  if (tau > 0.0f) return false;
  bool z = false;
  for (int v = threadIdx.x; v < V; v += kBlock) z = z || zero_threshold(views[v]);
  return __builtin_amdgcn_readfirstlane(__syncthreads_or(z ? 1 : 0)) != 0;
}

// Whether Gaussian i at distance d, in the frustum, holds the frustum maximum: its index competes
// for the lowest.
__device__ __forceinline__ void dmax_tie(uint32_t* imin, float d, unsigned long long dk, int64_t i) {
  if (dk != 0ull && __float_as_uint(d) == (uint32_t)(dk >> 32)) atomicMin(imin, (uint32_t)i);
}

// Appends the wave's lanes with `put` to the block's list segment (order arbitrary).
__device__ __forceinline__ void list_append(uint32_t* list, uint32_t* sbase, bool put, int64_t i, uint64_t lt) {
  const uint64_t bw = ballot64(put);
  if (bw == 0ull) return;
  uint32_t at = 0;
  if (lane_id() == 0) at = atomicAdd(sbase, (uint32_t)__popcll(bw));
  at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
  if (put) list[at + (uint32_t)__popcll(bw & lt)] = (uint32_t)i;
}

// Pass 1 over every Gaussian (block b owns the chunk [b*C, (b+1)*C)): per view the frustum
// flag, Eq. (2) and the LoD mask (alpha'' and the F/M flags written for every (view,
// Gaussian)), F and M counts, and the Gaussians that are in some view's
// frustum and kept by its mask appended to the block's segment of the work list (order
// within a segment is arbitrary).  Outside those, nothing else is computed, so the heavy
// pass below runs on full waves instead of the ~40% of lanes a whole-scene pass keeps busy.
//
// A thread takes four Gaussians at a time, so that a view's constants (scalar loads) and the LDS
// counters are paid once per 256 of them and four chains run side by side; the root and the two
// quotients of Eq. (2) are the forms of sqrt_normal and div_normal wherever the arguments allow.
// One Gaussian at a time, its view's constants read lane by lane behind each branch, it spent three
// quarters of its wave cycles waiting: 107 us for six views of 3M, 162 us for 16 of 2M, 57 us for
// one of 6M; now 64, 81 and 38 us, of which the stores of alpha'' and the flags and the reads
// (20 + 5 V bytes per Gaussian) are 30, 40 and 30 us at the 5.1 TB/s of a large copy.
// words: LDS of kClassifyWords V words ([V] CamLds, [V] counts F | M << 32, [V] lowest index at d_max).
constexpr int kClassifyWords = 3 + kCamWords;
template <bool kLaunch>
__device__ __forceinline__ void classify_body(const ClassifyArgs& a, Blk b, uint32_t* words) {
  constexpr int kItems = 4;
  __shared__ uint32_t sbase;
  const clod_scene& sc = a.sc;
  const DevView* __restrict__ views = a.views;
  const int V = a.V;
  const clod_params& prm = a.prm;
  const unsigned long long* __restrict__ dmax_key = a.dmax_key;
  const int64_t n = sc.n;
  CamLds* cam = reinterpret_cast<CamLds*>(words);
  unsigned long long* cnt = reinterpret_cast<unsigned long long*>(words + kCamWords * V);
  uint32_t* imin = words + (kCamWords + 2) * V;
  for (int j = threadIdx.x; j < V; j += kBlock) {
    cnt[j] = 0ull;
    imin[j] = 0xFFFFFFFFu;
    cam[j] = classify_cam(views[j], dmax_key[j]);
  }
  if (threadIdx.x == 0) sbase = 0;
  __syncthreads();
  int64_t lo, hi;
  block_chunk(n, b, lo, hi);
  const uint64_t lt = lanemask_lt();
  for (int64_t b0 = lo; b0 < hi; b0 += kItems * kBlock) {
    const int kn = hi - b0 >= kItems * kBlock ? kItems : (int)((hi - b0 + kBlock - 1) / kBlock);   // uniform
    float mx[kItems], my[kItems], mz[kItems], alpha[kItems], den[kItems], rden[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const int64_t j = b0 + k * kBlock + threadIdx.x, i = j < hi ? j : hi - 1;
      mx[k] = sc.mean[i]; my[k] = sc.mean[n + i]; mz[k] = sc.mean[2 * n + i];
      alpha[k] = sc.opacity[i]; den[k] = sc.decay[i];
    }
    uint32_t any = 0;   // bit k: item k is in some view's frustum and kept
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      alpha[k] = sigmoid_c(alpha[k]);
      den[k] = decay_den(den[k], prm.eps);   // view independent
      rden[k] = 1.0f / den[k];
    }
    uint64_t vm[kItems];   // lanes with a Gaussian
#pragma unroll
    for (int k = 0; k < kItems; ++k) vm[k] = ballot64(b0 + k * kBlock + threadIdx.x < hi);
    // The camera's part (frustum flag, distance, d / d_max) of the previous view, reused by the
    // views of the same camera run (which have the same frustum maximum).
    int lead = -1;
    uint64_t F[kItems];
    float d[kItems], dn[kItems];
    for (int v = 0; v < V; ++v) {
      const DevView Vw = view_at<kLaunch>(views, v);
      const CamLds C = cam[v];
      const float dmax = C.k[0], rdmax = C.k[1], s_v = C.k[2];
      uint32_t nF = 0, nM = 0, kept = 0;
      const bool fresh = Vw.cam_lead != lead;
      lead = Vw.cam_lead;
      // Lanes whose arguments the short forms do not take, or at the frustum maximum.
      uint64_t special = ballot64(!in_exponents<40>(dmax));
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        if (k < kn) {
          const int64_t i = b0 + k * kBlock + threadIdx.x;
          if (fresh) {
            float x, y, z, ex, ey, ez;
            to_camera(C, mx[k], my[k], mz[k], x, y, z);
            F[k] = frustum_mask(C, x, y, z, prm.near_z) & vm[k];
            const float d2 = cam_distance2(C, mx[k], my[k], mz[k], ex, ey, ez);
            d[k] = sqrt_normal(d2);
            dn[k] = div_normal(d[k], dmax, rdmax);
            special |= ballot64(!in_exponents<80>(d2));
          }
          const float u = dn[k] * s_v, num = u * u;
          const float q = div_normal(num, den[k], rden[k]);
          const float a2 = alpha[k] * (q > 86.0f ? 0.0f : cexp_core(-q));
          special |= ballot64(!in_exponents<60>(num)) | ballot64(!in_exponents<60>(den[k])) | (ballot64(d[k] == dmax) & F[k]);
          const uint64_t M = (Vw.budget > 0 ? ballot64(lod_key(a2, i) >= Vw.mkey) : ballot64(a2 > Vw.tau_sv)) & vm[k];
          const uint32_t fl = (__builtin_amdgcn_inverse_ballot_w64(F[k]) ? 1u : 0u) |
                              (__builtin_amdgcn_inverse_ballot_w64(M) ? 2u : 0u);
          if (__builtin_amdgcn_inverse_ballot_w64(vm[k])) {
            const int64_t f = (int64_t)v * n + i;
            a.alpha[f] = a2;
            a.flags[f] = (uint8_t)fl;
          }
          kept |= fl == 3u ? 1u << k : 0u;
          nF += (uint32_t)__popcll(F[k]);
          nM += (uint32_t)__popcll(M);
        }
      }
      if (special) {
        // Once more with the general forms, from the planes; nothing is handed to the next view.
        nF = nM = kept = 0u;
        lead = -1;
        for (int k = 0; k < kn; ++k) {
          const int64_t i = b0 + k * kBlock + threadIdx.x;
          bool Fk = false, M = false;
          if (i < hi) {
            const float px = sc.mean[i], py = sc.mean[n + i], pz = sc.mean[2 * n + i];
            float x, y, z, ex, ey, ez, al, q;
            to_camera(Vw, px, py, pz, x, y, z);
            Fk = in_frustum(Vw, x, y, z, prm.near_z);
            const float dk = cam_distance(Vw, px, py, pz, ex, ey, ez);
            if (Fk) dmax_tie(&imin[v], dk, dmax_key[v], i);
            const float a2 = attenuated(dk, dmax, Vw.s_v, sc.decay[i], sc.opacity[i], prm.eps, al, q);
            M = lod_kept(Vw, a2, i);
            const int64_t f = (int64_t)v * n + i;
            a.alpha[f] = a2;
            a.flags[f] = (uint8_t)((Fk ? 1 : 0) | (M ? 2 : 0));
          }
          kept |= Fk && M ? 1u << k : 0u;
          nF += (uint32_t)__popcll(ballot64(Fk));
          nM += (uint32_t)__popcll(ballot64(M));
        }
      }
      any |= kept;
      if (lane_id() == 0 && (nF | nM)) atomicAdd(&cnt[v], (unsigned long long)nF | (unsigned long long)nM << 32);
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k)
      list_append(a.list + lo, &sbase, (any >> k) & 1u, b0 + k * kBlock + threadIdx.x, lt);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < V; j += kBlock) {
    uint32_t* c = a.cpart + ((int64_t)b.id * V + j) * 4;   // [G][V][4]
    c[0] = (uint32_t)cnt[j];
    c[1] = (uint32_t)(cnt[j] >> 32);
    c[3] = imin[j];
  }
  if (threadIdx.x == 0) a.lcount[b.id] = sbase;
}
__global__ __launch_bounds__(kBlock) void k_classify(ClassifyArgs a) {
  extern __shared__ __align__(16) uint32_t words_dyn[];
  classify_body<true>(a, grid_blk(), words_dyn);
}

// Counting without rendering (clod_lod_count): nothing of Eq. (2) or of the projection is stored,
// only compared with a threshold, so both are estimated first and evaluated only where the estimate
// leaves the comparison open.  The counts are those of the full evaluation.  64 views of 6M
// Gaussians: 1,198 us for the masks and 509 us for the projections in full, now 559 us (two thirds
// of it vector issue) and 193 us.
//
// Mask: alpha'' > threshold is log2(alpha) - q log2(e) > log2(threshold), where the left side needs
// no root, quotient or exponential per view.  alpha'' of the contract differs from the exact value
// by a factor within 2^(5e-6 q + 1e-6) (q's roundings, E's 2 ulp, the last product), and the
// estimate's by less than that (hardware log2 and reciprocal, five products; a product that underflows
// is off by 2^-149 / eps at most), both far inside the margin below; NaN and any case the factors
// cannot express (count_cam) stay open.
//
// A threshold of 0 keeps alpha'' > 0, which ends where the contract's exponential does, at log2(e) q =
// kZeroExp, for every alpha above 2^-20 (the product is then at least 2^-145).  In a batch with such
// views la is 0, or NaN for the fainter Gaussians, and the views' threshold is 2^-kZeroExp; a budget
// of the whole scene keeps everything (kv = 0).  Other views of such a batch get no estimate.  16 views of
// 6M Gaussians with tau = 0 took 697 us in full and 1,008 us with every mask left open, now 358 us;
// with budgets of the whole scene 960, 1,075 and now 432 us.
struct LodItem {
  float la, iden;   // log2(alpha), log2(e) / (2 max(sigma_d, 0)^2 + eps)
};
__device__ __forceinline__ LodItem lod_item(float opac, float decay, float eps, bool zeros) {
  const float la = __builtin_amdgcn_logf(sigmoid_c(opac));
  return LodItem{!zeros ? la : la > -20.0f ? 0.0f : __builtin_nanf(""),
                 1.44269504088896341f * __builtin_amdgcn_rcpf(decay_den(decay, eps))};
}
// (Lane masks of the wave.)
__device__ __forceinline__ void mask_estimate(const LodItem& I, const CamLds& L, float d2, uint64_t& kept, uint64_t& dropped) {
  const float x = (d2 * L.k[0]) * I.iden, y = I.la - L.k[1];
  kept = ballot64(fmaf_(x, 1.00001f, 1e-4f) < y);
  dropped = ballot64(fmaf_(x, 0.99999f, -1e-4f) > y);
}
__device__ __forceinline__ bool mask_exact(const clod_scene& sc, const DevView& Vw, unsigned long long dk, float d2,
                                           float eps, int64_t i) {
  float alpha, q;
  return lod_kept(Vw, attenuated(__builtin_sqrtf(d2), dmax_from_key(dk), Vw.s_v, sc.decay[i], sc.opacity[i], eps, alpha, q), i);
}

// Projection of a Gaussian in the frustum: rendered if det > 0 and its rectangle meets the viewport.
// Both projected variances are at most B (DevView::geo_k, the largest scale).  Centre inside the
// viewport: the rectangle holds its tile, and det >= dilation^2 in exact arithmetic, while the
// binary32 evaluation errs by at most 5e-5 B^2 (35 roundings along the chain, times the sums of
// absolute values, at most 6 B each).  Centre farther outside than 3 sqrt(2 B) + 1, which bounds the
// radius: no tile.  Anything else stays open, as do rotations or scales that are not plain numbers.
__device__ __forceinline__ float geo_item(const clod_scene& sc, int64_t i) {   // largest scale squared, inf: open
  const int64_t n = sc.n;
  const float l0 = sc.log_scale[i], l1 = sc.log_scale[n + i], l2 = sc.log_scale[2 * n + i];
  const float qw = sc.quat[i], qx = sc.quat[n + i], qy = sc.quat[2 * n + i], qz = sc.quat[3 * n + i];
  const float n2 = qw * qw + qx * qx + qy * qy + qz * qz, ls = l0 + l1 + l2;
  const float s2 = 1.001f * __builtin_amdgcn_exp2f(2.88539008177792681f * fmaxf(l0, fmaxf(l1, l2)));
  return (n2 > 1e-30f) & (n2 < 1e30f) & (ls == ls) ? s2 : __builtin_inff();
}
__device__ __forceinline__ void geo_estimate(const DevView& Vw, float s2, float dil, float x, float y, float z,
                                             uint64_t& in, uint64_t& out) {
  const float iz = __builtin_amdgcn_rcpf(z), tx = x * iz, ty = y * iz;
  const float B = fmaf_(Vw.geo_k * s2, fmaf_(tx, tx, fmaf_(ty, ty, 1.0f)) * (iz * iz), dil);
  const float u = fmaf_(Vw.fx, tx, Vw.cx - (float)Vw.vx), v = fmaf_(Vw.fy, ty, Vw.cy - (float)Vw.vy);
  const float far = fmaxf(fmaxf(-u, u - (float)(kTile * Vw.tiles_x)), fmaxf(-v, v - (float)(kTile * Vw.tiles_y)));
  in = ballot64(u > 0.5f) & ballot64(u < (float)Vw.width - 0.5f) & ballot64(v > 0.5f) &
       ballot64(v < (float)Vw.height - 0.5f) & ballot64(1e-4f * (B * B) < dil * dil);
  // (For NaN none of the comparisons holds.)
  out = ballot64(far > fmaf_(4.25f, __builtin_amdgcn_sqrtf(B), 2.0f)) & ~in;
}

// Pass 1 of the counting: F and M counts, the decided part of the rendered counts, and the Gaussians
// whose projection is open in some view appended to the block's list segment.
// words: LDS of kCountWords V words ([V] CamLds, [V] counts F | M << 32, [V] lowest index at d_max,
// [V] rendered).
constexpr int kCountWords = 4 + kCamWords;
__device__ __forceinline__ void count_body(const ClassifyArgs& a, Blk b, uint32_t* words) {
  constexpr int kItems = 4;
  __shared__ uint32_t sbase;
  const clod_scene& sc = a.sc;
  const DevView* __restrict__ views = a.views;
  const int V = a.V;
  const clod_params& prm = a.prm;
  const unsigned long long* __restrict__ dmax_key = a.dmax_key;
  const int64_t n = sc.n;
  CamLds* cam = reinterpret_cast<CamLds*>(words);
  unsigned long long* cnt = reinterpret_cast<unsigned long long*>(words + kCamWords * V);
  uint32_t* imin = words + (kCamWords + 2) * V;
  uint32_t* rend = imin + V;
  const bool zeros = any_zero_threshold(views, V, prm.tau);
  for (int j = threadIdx.x; j < V; j += kBlock) {
    cnt[j] = 0ull;
    imin[j] = 0xFFFFFFFFu;
    rend[j] = 0u;
    cam[j] = count_cam(views[j], dmax_key[j], prm.eps, zeros);
  }
  if (threadIdx.x == 0) sbase = 0;
  __syncthreads();
  int64_t lo, hi;
  block_chunk(n, b, lo, hi);
  const uint64_t lt = lanemask_lt();
  for (int64_t b0 = lo; b0 < hi; b0 += kItems * kBlock) {
    const int kn = hi - b0 >= kItems * kBlock ? kItems : (int)((hi - b0 + kBlock - 1) / kBlock);   // uniform
    float mx[kItems], my[kItems], mz[kItems], s2[kItems];
    LodItem it[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const int64_t j = b0 + k * kBlock + threadIdx.x, i = j < hi ? j : hi - 1;
      mx[k] = sc.mean[i]; my[k] = sc.mean[n + i]; mz[k] = sc.mean[2 * n + i];
      it[k] = LodItem{sc.opacity[i], sc.decay[i]};
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) it[k] = lod_item(it[k].la, it[k].iden, prm.eps, zeros);
    uint64_t vm[kItems];   // lanes with a Gaussian
#pragma unroll
    for (int k = 0; k < kItems; ++k) vm[k] = ballot64(b0 + k * kBlock + threadIdx.x < hi);
    uint32_t have = 0, open = 0;   // bit k: s2[k] read (uniform); some view's projection is open
    for (int v = 0; v < V; ++v) {
      const DevView Vw = view_at<true>(views, v);
      const CamLds C = cam[v];
      uint32_t nF = 0, nM = 0, nR = 0, opened = 0;
      uint64_t special = 0;   // lanes whose mask is open, or that may hold the frustum maximum
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        if (k < kn) {
          float x, y, z, ex, ey, ez;
          to_camera(C, mx[k], my[k], mz[k], x, y, z);
          const uint64_t F = frustum_mask(C, x, y, z, prm.near_z) & vm[k];
          const float d2 = cam_distance2(C, mx[k], my[k], mz[k], ex, ey, ez);
          uint64_t kept, dropped;
          mask_estimate(it[k], C, d2, kept, dropped);
          special |= (vm[k] & ~(kept | dropped)) | (F & ballot64(d2 >= C.k[2]));
          const uint64_t M = vm[k] & kept, FM = F & M;
          nF += (uint32_t)__popcll(F);
          nM += (uint32_t)__popcll(M);
          if (FM) {
            if (!((have >> k) & 1u)) {
              uint32_t at = k * kBlock + threadIdx.x;
              asm volatile("" : "+v"(at));   // (keeps these addresses out of the registers until here)
              const int64_t i = b0 + at;
              s2[k] = geo_item(sc, i < hi ? i : hi - 1);
              have |= 1u << k;
            }
            uint64_t in, out;
            geo_estimate(Vw, s2[k], prm.dilation, x, y, z, in, out);
            nR += (uint32_t)__popcll(FM & in);
            opened |= __builtin_amdgcn_inverse_ballot_w64(FM & ~(in | out)) ? 1u << k : 0u;
          }
        }
      }
      if (special) {
        // Once more with the mask evaluated in full where it is open.
        nF = nM = nR = opened = 0u;
        for (int k = 0; k < kn; ++k) {
          const int64_t j = b0 + k * kBlock + threadIdx.x, i = j < hi ? j : hi - 1;
          const uint64_t valid = ballot64(j < hi);
          const float px = sc.mean[i], py = sc.mean[n + i], pz = sc.mean[2 * n + i];
          float x, y, z, ex, ey, ez;
          to_camera(C, px, py, pz, x, y, z);
          const uint64_t F = frustum_mask(C, x, y, z, prm.near_z) & valid;
          const float d2 = cam_distance2(C, px, py, pz, ex, ey, ez);
          if (__builtin_amdgcn_inverse_ballot_w64(F)) dmax_tie(&imin[v], __builtin_sqrtf(d2), dmax_key[v], i);
          uint64_t kept, dropped;
          mask_estimate(lod_item(sc.opacity[i], sc.decay[i], prm.eps, zeros), C, d2, kept, dropped);
          const uint64_t M = (kept | (ballot64(mask_exact(sc, Vw, dmax_key[v], d2, prm.eps, i)) & ~dropped)) & valid;
          uint64_t in, out;
          geo_estimate(Vw, geo_item(sc, i), prm.dilation, x, y, z, in, out);
          nF += (uint32_t)__popcll(F);
          nM += (uint32_t)__popcll(M);
          nR += (uint32_t)__popcll(F & M & in);
          opened |= __builtin_amdgcn_inverse_ballot_w64(F & M & ~(in | out)) ? 1u << k : 0u;
        }
      }
      open |= opened;
      if (lane_id() == 0 && (nF | nM)) {
        atomicAdd(&cnt[v], (unsigned long long)nF | (unsigned long long)nM << 32);
        if (nR) atomicAdd(&rend[v], nR);
      }
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k)
      list_append(a.list + lo, &sbase, (open >> k) & 1u, b0 + k * kBlock + threadIdx.x, lt);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < V; j += kBlock) {
    uint32_t* c = a.cpart + ((int64_t)b.id * V + j) * 4;   // [G][V][4]
    c[0] = (uint32_t)cnt[j];
    c[1] = (uint32_t)(cnt[j] >> 32);
    c[2] = rend[j];
    c[3] = imin[j];
  }
  if (threadIdx.x == 0) a.lcount[b.id] = sbase;
}
__global__ __launch_bounds__(kBlock) void k_count(ClassifyArgs a) {
  extern __shared__ __align__(16) uint32_t words_dyn[];
  count_body(a, grid_blk(), words_dyn);
}

// The work list: G segments (block g's at g * per, its length in lcount[g]).  Every block scans the
// lengths (G <= kMaxProjBlocks: eight per thread) into soff[0 .. kMaxProjBlocks], the segments'
// first entries (past the last segment the number of entries); returns that number.
constexpr int kSegWords = kMaxProjBlocks + 1;
__device__ __forceinline__ uint32_t scan_segments(const uint32_t* __restrict__ lcount, int G, uint32_t* soff) {
  __shared__ uint32_t sm[4];
  constexpr int kPer = kMaxProjBlocks / kBlock;
  static_assert(kPer * kBlock == kMaxProjBlocks, "segment scan layout");
  const int j0 = threadIdx.x * kPer;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    c[k] = j0 + k < G ? lcount[j0 + k] : 0u;
    sum += c[k];
  }
  uint32_t tot;
  uint32_t off = block_exclusive_scan(sum, sm, tot);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    soff[j0 + k] = off;
    off += c[k];
  }
  if (threadIdx.x == 0) soff[kMaxProjBlocks] = tot;
  __syncthreads();
  return tot;
}
// The Gaussian of entry e (of the wave's first entry e0 onwards, e0 uniform and below the number of
// entries): the wave finds the segment of e0 with two 64-wide comparisons (a binary search is eleven
// dependent LDS reads), and the lanes walk on from there.
__device__ __forceinline__ int64_t list_entry(const uint32_t* __restrict__ list, const uint32_t* soff, int64_t per,
                                              uint32_t e0, uint32_t e) {
  constexpr uint32_t kFine = kMaxProjBlocks / 64;
  const uint32_t lane = lane_id();
  const uint32_t c = (uint32_t)__popcll(ballot64(soff[lane * kFine] <= e0)) - 1u;   // soff[0] = 0
  const uint32_t f = (uint32_t)__popcll(ballot64(lane < kFine && soff[c * kFine + (lane % kFine)] <= e0)) - 1u;
  uint32_t s = c * kFine + f;
  while (soff[s + 1] <= e) ++s;
  return (int64_t)list[(int64_t)s * per + (e - soff[s])];
}

// Pass 2 of the counting, over the listed Gaussians: the open projections evaluated in full.
// sdyn: LDS of kSegWords + kCountWords V words ([V] CamLds, segment offsets, [V] rendered counts).
__device__ __forceinline__ void count_rest_body(const ProjectArgs& a, Blk b, uint32_t* sdyn) {
  const clod_scene& sc = a.sc;
  const DevView* __restrict__ views = a.views;
  const int V = a.V, G = (int)b.n;
  const clod_params& prm = a.prm;
  const int64_t n = sc.n;
  CamLds* cam = reinterpret_cast<CamLds*>(sdyn);
  uint32_t* soff = sdyn + kCamWords * V;
  uint32_t* scnt = soff + kSegWords;
  const bool zeros = any_zero_threshold(views, V, prm.tau);
  for (int j = threadIdx.x; j < V; j += kBlock) {
    scnt[j] = 0u;
    cam[j] = count_cam(views[j], a.dmax_key[j], prm.eps, zeros);
  }
  const uint32_t L = scan_segments(a.lcount, G, soff);
  const int64_t per = (n + G - 1) / G;
  for (int64_t base = (int64_t)b.id * kBlock + (threadIdx.x & ~63u); base < L; base += (int64_t)G * kBlock) {
    const uint32_t e0 = (uint32_t)base, e = min(e0 + lane_id(), L - 1u);
    const uint64_t valid = ballot64(e0 + lane_id() < L);
    const int64_t i = list_entry(a.list, soff, per, e0, e);
    const float mx = sc.mean[i], my = sc.mean[n + i], mz = sc.mean[2 * n + i];
    const LodItem it = lod_item(sc.opacity[i], sc.decay[i], prm.eps, zeros);
    const float s2 = geo_item(sc, i);
    const float s0 = cexp(sc.log_scale[i]), s1 = cexp(sc.log_scale[n + i]), s2c = cexp(sc.log_scale[2 * n + i]);
    float Rm[9], S[9], w_, x_, y_, z_, rn;
    quat_rot(sc.quat[i], sc.quat[n + i], sc.quat[2 * n + i], sc.quat[3 * n + i], Rm, w_, x_, y_, z_, rn);
    cov3(Rm, s0, s1, s2c, S);
    for (int v = 0; v < V; ++v) {
      const DevView Vw = view_at<true>(views, v);
      const CamLds C = cam[v];
      float x, y, z, ex, ey, ez;
      to_camera(C, mx, my, mz, x, y, z);
      uint64_t in, out, kept, dropped;
      geo_estimate(Vw, s2, prm.dilation, x, y, z, in, out);
      const uint64_t F = frustum_mask(C, x, y, z, prm.near_z) & valid & ~(in | out);
      if (!F) continue;
      const float d2 = cam_distance2(C, mx, my, mz, ex, ey, ez);
      mask_estimate(it, C, d2, kept, dropped);
      const uint64_t open = F & ~dropped;
      bool R = false;
      if (__builtin_amdgcn_inverse_ballot_w64(open)) {
        Proj P;
        R = ewa(Vw, x, y, z, S, prm.dilation, P) &&
            (__builtin_amdgcn_inverse_ballot_w64(kept) || mask_exact(sc, Vw, a.dmax_key[v], d2, prm.eps, i));
      }
      const uint32_t nR = (uint32_t)__popcll(ballot64(R));
      if (lane_id() == 0 && nR) atomicAdd(&scnt[v], nR);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < V; j += kBlock) a.cpart[((int64_t)b.id * V + j) * 4 + 2] += scnt[j];
}
__global__ __launch_bounds__(kBlock) void k_count_rest(ProjectArgs a) {
  extern __shared__ __align__(16) uint32_t words_dyn[];
  count_rest_body(a, grid_blk(), words_dyn);
}

// Pass 2 over the work list (entries spread evenly over the blocks): per listed Gaussian the
// EWA projection, cull and rectangle in the views that keep it (the flags and alpha'' of pass 1),
// remembering which views render it; then the colour of each rendering view is evaluated from its
// SH coefficients.  Records (with depth, rectangle and tiles touched in their fourth quad) are
// written for rendered (view, Gaussian) pairs only.  The pass waits for its gathers more than it
// computes: the parameters and the first flags of an entry are all requested before any is used.
// Eq. (2) is read, not evaluated again, and no plane address outlives its use (the 3K addresses of
// plane-major coefficients, formed ahead of the loop, left two waves per SIMD): six views of 3M
// 168 -> 152 us, 5 views of a camera 47 -> 40 us, 16 views of 2M with plane-major coefficients
// 336 -> 245 us.
// sdyn: LDS of kSegWords + V words ([kSegWords] segment offsets, then [V] rendered counts).
template <int DEG, bool kPacked, bool kLaunch>
__device__ __forceinline__ void project_body(const ProjectArgs& a, Blk b, uint32_t* sdyn) {
  const clod_scene& sc = a.sc;
  const DevView* __restrict__ views = a.views;
  const int V = a.V;
  const clod_params& prm = a.prm;
  uint8_t* __restrict__ flags = a.flags;
  const float* __restrict__ alpha = a.alpha;
  float4* __restrict__ rec = a.rec;
  constexpr int K = (DEG + 1) * (DEG + 1);
  const int64_t n = sc.n;
  const int G = (int)b.n;
  uint32_t* soff = sdyn;
  uint32_t* scnt = sdyn + kSegWords;
  for (int j = threadIdx.x; j < V; j += kBlock) scnt[j] = 0;
  const uint32_t L = scan_segments(a.lcount, G, soff);
  const int64_t per = (n + G - 1) / G;   // chunk length of the first pass
  for (int64_t base = (int64_t)b.id * kBlock + (threadIdx.x & ~63u); base < L; base += (int64_t)G * kBlock) {
    const uint32_t e0 = (uint32_t)base, e = min(e0 + lane_id(), L - 1u);
    const bool valid = e0 + lane_id() < L;
    const int64_t i = list_entry(a.list, soff, per, e0, e);
    const float mx = sc.mean[i], my = sc.mean[n + i], mz = sc.mean[2 * n + i];
    const float l0 = sc.log_scale[i], l1 = sc.log_scale[n + i], l2 = sc.log_scale[2 * n + i];
    const float qw = sc.quat[i], qx = sc.quat[n + i], qy = sc.quat[2 * n + i], qz = sc.quat[3 * n + i];
    float S[9];   // 3D covariance (view independent)
    // The projection (and below the colour) of the last camera run evaluated: views of one run
    // share them (only alpha'' and the mask depend on s_v).
    int geo_lead = -1, col_lead = -1;
    Proj P;
    float z = 0.f;
    bool pok = false, have_cov = false;
    float col[3] = {0.f, 0.f, 0.f};
    uint8_t cfl = 0;
    for (int v0 = 0; v0 < V; v0 += 32) {
      const int vn = V - v0 < 32 ? V - v0 : 32;
      uint32_t kmask = 0, rmask = 0;   // views of the group that keep the Gaussian; that render it
#pragma unroll 8
      for (int vv = 0; vv < vn; ++vv)
        kmask |= (flags[(int64_t)(v0 + vv) * n + i] & 3u) == 3u ? 1u << vv : 0u;
      if (!valid) kmask = 0;
      if (!have_cov) {
        have_cov = true;
        float Rm[9], w_, x_, y_, z_, rn;
        quat_rot(qw, qx, qy, qz, Rm, w_, x_, y_, z_, rn);
        cov3(Rm, cexp(l0), cexp(l1), cexp(l2), S);
      }
      for (int vv = 0; vv < vn; ++vv) {
        const bool kept = ((kmask >> vv) & 1u) != 0u;
        if (!ballot64(kept)) continue;
        const int v = v0 + vv;
        const DevView Vw = view_at<kLaunch>(views, v);
        bool R = false;
        if (kept) {
          const int64_t f = (int64_t)v * n + i;
          const float a2 = alpha[f];
          if (Vw.cam_lead != geo_lead) {
            float x, y;
            to_camera(Vw, mx, my, mz, x, y, z);
            pok = ewa(Vw, x, y, z, S, prm.dilation, P);
            geo_lead = Vw.cam_lead;
          }
          R = pok;
          if (R) {
            rec[kRecQuads * f] = make_float4(P.u, P.v, a2, P.rad);
            rec[kRecQuads * f + 1] = make_float4(P.A, P.B, P.C, 0.f);
            // Depth, tile rectangle and tiles touched: the fourth quad, so the record is
            // written whole (no partial 64-byte segments, no separate scattered planes).
            rec[kRecQuads * f + 3] =
                make_float4(z, __uint_as_float((uint32_t)P.x0 | ((uint32_t)P.x1 << 16)),
                            __uint_as_float((uint32_t)P.y0 | ((uint32_t)P.y1 << 16)),
                            __uint_as_float((uint32_t)((P.x1 - P.x0) * (P.y1 - P.y0))));
          }
        }
        rmask |= (R ? 1u : 0u) << vv;
        const uint64_t bR = ballot64(R);
        if (lane_id() == 0 && bR) atomicAdd(&scnt[v], (uint32_t)__popcll(bR));
      }
      if (rmask) {
        // Plane-major coefficients are gathered once into registers (read again for every rendering
        // view, whose lanes differ, they cost 456 us instead of 245 for 16 views of 2M); a packed
        // per-Gaussian block is instead re-read for every rendering view (cache hits after the
        // first one, float4 chunks when 3K % 4 == 0), which keeps the kernel at half the registers.
        // Either way each channel accumulates in coefficient order.
        float shc[kPacked ? 1 : 3 * K];
        if constexpr (!kPacked) {
          int64_t at = i;
          asm volatile("" : "+v"(at));   // (keeps the 3K addresses from being formed ahead of the loop)
#pragma unroll
          for (int k = 0; k < 3 * K; ++k) shc[k] = sc.sh[(int64_t)k * n + at];
        }
        uint32_t m = rmask;
        while (m) {
          const int vv = __builtin_ctz(m);
          m &= m - 1;
          const int v = v0 + vv;
          const DevView& Vw = views[v];
          const int64_t f = (int64_t)v * n + i;
          if (Vw.cam_lead != col_lead) {
          col_lead = Vw.cam_lead;
          float ex, ey, ez;
          const float d = cam_distance(Vw, mx, my, mz, ex, ey, ez);
          const float id = 1.0f / d;
          float Yb[16];
          sh_basis(DEG, ex * id, ey * id, ez * id, Yb);
          float acc[3];
          if constexpr (kPacked) {
            const float* src = sc.sh_packed + (int64_t)i * (3 * K);
            if constexpr ((3 * K) % 4 == 0) {
              const float4* src4 = reinterpret_cast<const float4*>(src);
#pragma unroll
              for (int q = 0; q < (3 * K) / 4; ++q) {
                const float4 c4 = src4[q];
                const float cv[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const int idx = 4 * q + e, k = idx / 3, ch = idx % 3;
                  acc[ch] = k == 0 ? cv[e] * Yb[0] : fmaf_(cv[e], Yb[k], acc[ch]);
                }
              }
            } else {
#pragma unroll
              for (int idx = 0; idx < 3 * K; ++idx) {
                const int k = idx / 3, ch = idx % 3;
                acc[ch] = k == 0 ? src[idx] * Yb[0] : fmaf_(src[idx], Yb[k], acc[ch]);
              }
            }
          } else {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
              float a = shc[ch] * Yb[0];
#pragma unroll
              for (int k = 1; k < K; ++k) a = fmaf_(shc[3 * k + ch], Yb[k], a);
              acc[ch] = a;
            }
          }
          cfl = 1u | 2u | 4u;   // rendered implies in frustum and kept
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) {
            const float cv = acc[ch] + 0.5f;
            if (!(cv > 0.0f)) cfl |= (uint8_t)(8 << ch);
            col[ch] = fmaxf(cv, 0.0f);
          }
          }
          rec[kRecQuads * f + 2] = make_float4(col[0], col[1], col[2], 0.f);
          flags[f] = cfl;
        }
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < V; j += kBlock) a.cpart[((int64_t)b.id * V + j) * 4 + 2] = scnt[j];
}

// Plane-major coefficients.
template <int DEG>
__global__ __launch_bounds__(kBlock) void k_project(ProjectArgs a) {
  extern __shared__ uint32_t sdyn[];
  project_body<DEG, false, true>(a, grid_blk(), sdyn);
}

// Packed coefficients: fits 128 registers, so four waves per SIMD hide the gather latency.
template <int DEG>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_project_packed(ProjectArgs a) {
  extern __shared__ uint32_t sdyn[];
  project_body<DEG, true, true>(a, grid_blk(), sdyn);
}

// Budgeted LoD (a view with budget K, 0 < K < n): the K-th largest selection key.  alpha'' (as
// bits) is found by an MSD radix select in three levels of 11, 11 and 10 bits; among equal
// alpha'' the lowest indices are kept, so the last stage finds the index at the remaining rank.
//   k_select_first  level 0: counts of the leading digit (LDS counts, added to the view's bins)
//   k_select_hist   levels 1 and 2: counts of the level's digit over the keys that share the digits
//                   found so far
//   k_select_hist   level 3: keys equal to the threshold per chunk of the view's Gaussians
//   k_select_pick   the chunk and then the index at the rank; the threshold key to the view
// Every block finds the digits of the levels before its own itself from the view's bins, so no
// launch sits between the levels.  Level 0 computes alpha'' exactly as the projection does and,
// where there is a plane for it (not in the counting entry points), stores it for the other
// levels to read instead of computing it again.  Five launches; the eight 8-bit levels over the
// whole 64-bit key that these replaced took sixteen and computed alpha'' eight times (3M
// Gaussians in four viewports: 540 us, now 114 us).  K >= n keeps everything (threshold 0).
//
// Level 0 is bound by vector issue and, at its end, by the atomics of its blocks' bins.  A block
// takes its Gaussians through up to four views, so that sigmoid and reciprocal denominator are
// formed once for them and the distance once per camera run, with the short root and quotients of
// k_classify where the arguments allow (else once more with the general forms): 45 us for the four
// viewports, against 68 us a view at a time with the general forms.  Three blocks' worth of parts per
// CU: with 512 parts 50 us (too few waves), with 1024 48 us and with 2048 76 us (their bins).
__device__ __forceinline__ int64_t select_chunk(int64_t n) {   // Gaussians per chunk
  const int64_t c = (n + kSelBlocks - 1) / kSelBlocks;
  return (c + kBlock - 1) / kBlock * kBlock;
}
// The digits of the first `levels` levels (as the leading bits of a key) and the rank, from the
// largest, among the keys that share them.
__device__ __forceinline__ void select_derive(const uint32_t* __restrict__ hist, int levels, int64_t budget,
                                              uint32_t& prefix, uint32_t& rank, uint32_t* sm) {
  __shared__ uint32_t found[2];
  constexpr int kPer = kSelBins / kBlock;
  prefix = 0u;
  rank = (uint32_t)budget;   // 0 < budget < n < 2^32
  for (int l = 0; l < levels; ++l) {
    // Thread t takes the digits kSelBins - 1 - (8 t + k), so a scan over them counts from the top.
    const uint32_t* h = hist + l * kSelBins + (kSelBins - kPer * (1 + (int)threadIdx.x));
    uint32_t c[kPer], s = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) { c[k] = h[kPer - 1 - k]; s += c[k]; }
    uint32_t total;
    uint32_t ex = block_exclusive_scan(s, sm, total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (ex < rank && rank <= ex + c[k]) {
        found[0] = kSelBins - 1u - (kPer * threadIdx.x + (uint32_t)k);
        found[1] = rank - ex;
      }
      ex += c[k];
    }
    __syncthreads();
    prefix = (prefix << (l < 2 ? 11 : 10)) | found[0];
    rank = found[1];
    __syncthreads();
  }
}
__device__ __forceinline__ uint32_t select_bits(const SelectArgs& a, const DevView& Vw, float dmax, int64_t v, int64_t i) {
  const int64_t n = a.sc.n;
  if (a.alpha && a.level > 0) return __float_as_uint(a.alpha[v * n + i]);
  float ex, ey, ez;
  const float d = cam_distance(Vw, a.sc.mean[i], a.sc.mean[n + i], a.sc.mean[2 * n + i], ex, ey, ez);
  float alpha, q;
  return __float_as_uint(attenuated(d, dmax, Vw.s_v, a.sc.decay[i], a.sc.opacity[i], a.prm.eps, alpha, q));
}

struct SelectLds {
  uint32_t h[kSelViews][kSelBins];   // (the levels after the first use one row)
};
// Block b of ceil(V / kSelViews) * kSelFirst: part b % kSelFirst of the Gaussians, in the views of
// group b / kSelFirst.
__device__ __forceinline__ void select_first_body(const SelectArgs& a, Blk b, SelectLds& S) {
  constexpr int kItems = 4;
  __shared__ float vk[kSelViews][6];   // camera centre, d_max, its reciprocal, s_v
  const int v0 = (int)(b.id / kSelFirst) * kSelViews;
  const uint32_t part = b.id % kSelFirst;
  const clod_scene& sc = a.sc;
  const int64_t n = sc.n;
  int64_t per = (n + kSelFirst - 1) / kSelFirst;
  per = (per + kBlock - 1) / kBlock * kBlock;
  const int64_t lo = part * per, hi = lo + per < n ? lo + per : n;
  if (lo >= n) return;
  uint32_t active = 0;   // uniform: views of the group that select
  for (int w = 0; w < kSelViews && v0 + w < a.V; ++w) {
    const int64_t k = a.views[v0 + w].budget;
    active |= k > 0 && k < n ? 1u << w : 0u;
  }
  if (active == 0u) return;
  for (uint32_t j = threadIdx.x; j < kSelViews * kSelBins; j += kBlock) (&S.h[0][0])[j] = 0u;
  if (threadIdx.x < kSelViews && ((active >> threadIdx.x) & 1u)) {
    const int w = (int)threadIdx.x;
    const float dmax = dmax_from_key(a.dmax_key[v0 + w]);
    for (int j = 0; j < 3; ++j) vk[w][j] = a.views[v0 + w].c[j];
    vk[w][3] = dmax;
    vk[w][4] = 1.0f / dmax;
    vk[w][5] = a.views[v0 + w].s_v;
  }
  __syncthreads();
  for (int64_t b0 = lo; b0 < hi; b0 += kItems * kBlock) {
    float mx[kItems], my[kItems], mz[kItems], alpha[kItems], den[kItems], rden[kItems], dn[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const int64_t j = b0 + k * kBlock + threadIdx.x, i = j < hi ? j : hi - 1;
      mx[k] = sc.mean[i]; my[k] = sc.mean[n + i]; mz[k] = sc.mean[2 * n + i];
      alpha[k] = sc.opacity[i]; den[k] = sc.decay[i];
    }
    uint64_t own = 0;   // lanes whose arguments the short forms do not take, whatever the view
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      alpha[k] = sigmoid_c(alpha[k]);
      den[k] = decay_den(den[k], a.prm.eps);
      rden[k] = 1.0f / den[k];
      own |= ballot64(!in_exponents<60>(den[k]));
    }
    int lead = -1;         // camera run whose distances dn holds
    uint64_t far = 0;      // lanes whose distance the short forms do not take
#pragma unroll 1
    for (int w = 0; w < kSelViews; ++w) {
      if (!((active >> w) & 1u)) continue;
      const int v = v0 + w;
      if (a.views[v].cam_lead != lead) {
        lead = a.views[v].cam_lead;
        const float c0 = vk[w][0], c1 = vk[w][1], c2 = vk[w][2], dmax = vk[w][3], rdmax = vk[w][4];
        far = ballot64(!in_exponents<40>(dmax));
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
          const float ex = mx[k] - c0, ey = my[k] - c1, ez = mz[k] - c2;   // as cam_distance2
          const float d2 = fmaf_(ex, ex, fmaf_(ey, ey, ez * ez));
          dn[k] = div_normal(sqrt_normal(d2), dmax, rdmax);
          far |= ballot64(!in_exponents<80>(d2));
        }
      }
      const float s_v = vk[w][5];
      uint64_t special = own | far;
      uint32_t key[kItems];
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const float u = dn[k] * s_v, num = u * u;
        const float q = div_normal(num, den[k], rden[k]);
        special |= ballot64(!in_exponents<60>(num));
        key[k] = __float_as_uint(alpha[k] * (q > 86.0f ? 0.0f : cexp_core(-q)));
      }
      if (special) {   // the general forms, for the whole wave
        const float dmax = vk[w][3];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
          float ex, ey, ez, q;
          const float d = cam_distance(a.views[v], mx[k], my[k], mz[k], ex, ey, ez);
          key[k] = __float_as_uint(attenuated_pre(d, dmax, s_v, alpha[k], den[k], q));
        }
      }
      uint32_t zeros = 0;   // keys of digit 0: half the scene may be (alpha'' flushed to 0)
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const int64_t i = b0 + k * kBlock + threadIdx.x;
        if (i < hi) {
          if (a.alpha) a.alpha[(int64_t)v * n + i] = __uint_as_float(key[k]);
          const uint32_t d = (key[k] >> 21) & 2047u;
          if (d != 0u) atomicAdd(&S.h[w][d], 1u);
          zeros += d == 0u ? 1u : 0u;
        }
      }
      zeros = wave_sum(zeros);
      if (lane_id() == 0 && zeros) atomicAdd(&S.h[w][0], zeros);
    }
  }
  __syncthreads();
  // (Each block starts at bins of its own: blocks end together, and met at the same ones.)
  for (uint32_t j0 = threadIdx.x; j0 < kSelViews * kSelBins; j0 += kBlock) {
    const uint32_t j = (j0 + part * kBlock) % (kSelViews * kSelBins);
    const uint32_t w = j / kSelBins, c = S.h[w][j % kSelBins];
    if (c) atomicAdd(a.hist + (size_t)(v0 + (int)w) * kSelWords + j % kSelBins, c);
  }
}
__global__ __launch_bounds__(kBlock) void k_select_first(SelectArgs a) {
  __shared__ SelectLds S;
  select_first_body(a, grid_blk(), S);
}
// Block b of V * kSelBlocks: chunk b % kSelBlocks of view b / kSelBlocks.
__device__ __forceinline__ void select_hist_body(const SelectArgs& a, Blk b, uint32_t* h) {
  __shared__ uint32_t sm[4];
  const int v = (int)(b.id / kSelBlocks);
  const uint32_t chunk = b.id % kSelBlocks;
  const DevView& Vw = a.views[v];
  const int64_t n = a.sc.n;
  if (Vw.budget <= 0 || Vw.budget >= n) return;
  const int64_t per = select_chunk(n), lo = chunk * per, hi = lo + per < n ? lo + per : n;
  if (lo >= n) return;
  uint32_t* __restrict__ hist = a.hist + (size_t)v * kSelWords;
  for (uint32_t j = threadIdx.x; j < kSelBins; j += kBlock) h[j] = 0u;
  __syncthreads();
  uint32_t prefix, rank;
  select_derive(hist, a.level, Vw.budget, prefix, rank, sm);
  const int shift = a.level == 1 ? 10 : 0;
  const uint32_t mask = a.level == 3 ? 0u : a.level == 2 ? 1023u : 2047u;
  const float dmax = dmax_from_key(a.dmax_key[v]);
  uint32_t zeros = 0;   // keys of digit 0 (half the scene may be: alpha'' flushed to 0)
  constexpr int kItems = 4;   // Gaussians per thread and round, read before any is used
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kItems * kBlock) {
    uint32_t k[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = i0 + j * kBlock;
      k[j] = select_bits(a, Vw, dmax, v, i < hi ? i : hi - 1);
    }
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = i0 + j * kBlock;
      if (i >= hi) break;
      const bool in = a.level == 3 ? k[j] == prefix : (k[j] >> (a.level == 1 ? 21 : 10)) == prefix;
      const uint32_t d = (k[j] >> shift) & mask;
      if (in && d != 0u) atomicAdd(&h[d], 1u);
      zeros += in && d == 0u ? 1u : 0u;
    }
  }
  zeros = wave_sum(zeros);
  if (lane_id() == 0 && zeros) atomicAdd(&h[0], zeros);
  __syncthreads();
  if (a.level == 3) {
    if (threadIdx.x == 0) hist[3 * kSelBins + chunk] = h[0];
    return;
  }
  for (uint32_t j = threadIdx.x; j < kSelBins; j += kBlock)
    if (h[j]) atomicAdd(&hist[a.level * kSelBins + j], h[j]);
}
__global__ __launch_bounds__(kBlock) void k_select_hist(SelectArgs a) {
  __shared__ uint32_t h[kSelBins];
  select_hist_body(a, grid_blk(), h);
}

// Block v: the index of view v's last kept Gaussian among those at the threshold.
__device__ __forceinline__ void select_pick_body(const SelectArgs& a, Blk b) {
  __shared__ uint32_t sm[4];
  __shared__ uint32_t found[2];
  const int v = (int)b.id;
  const DevView& Vw = a.views[v];
  const int64_t n = a.sc.n;
  if (Vw.budget <= 0) return;
  if (Vw.budget >= n) {
    if (threadIdx.x == 0) a.views_out[v].mkey = 0ull;
    return;
  }
  uint32_t* hist = a.hist + (size_t)v * kSelWords;
  uint32_t prefix, rank;
  select_derive(hist, 3, Vw.budget, prefix, rank, sm);
  // The chunk that holds the rank-th equal key (lowest index first).
  const int64_t per = select_chunk(n);
  const uint32_t chunks = (uint32_t)((n + per - 1) / per);
  static_assert(kSelBlocks <= 4 * kBlock, "four chunks per thread");
  uint32_t c[4], s = 0, total;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t q = 4 * threadIdx.x + k;
    c[k] = q < chunks ? hist[3 * kSelBins + q] : 0u;
    s += c[k];
  }
  uint32_t ex = block_exclusive_scan(s, sm, total);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (ex < rank && rank <= ex + c[k]) { found[0] = 4 * threadIdx.x + k; found[1] = rank - ex; }
    ex += c[k];
  }
  __syncthreads();
  const uint32_t chunk = found[0];
  rank = found[1];
  const float dmax = dmax_from_key(a.dmax_key[v]);
  const int64_t lo = chunk * per, hi = lo + per < n ? lo + per : n;
  for (int64_t i0 = lo; i0 < hi; i0 += kBlock) {
    const int64_t i = i0 + threadIdx.x;
    const bool eq = i < hi && select_bits(a, Vw, dmax, v, i) == prefix;
    const uint32_t before = block_exclusive_scan(eq ? 1u : 0u, sm, total);
    if (eq && before + 1u == rank) a.views_out[v].mkey = ((unsigned long long)prefix << 32) | (0xFFFFFFFFu - (uint32_t)i);
    if (rank <= total) break;
    rank -= total;
  }
}
__global__ __launch_bounds__(kBlock) void k_select_pick(SelectArgs a) { select_pick_body(a, grid_blk()); }

// The bins start clear (the frustum maximum's fold clears them).
hipError_t launch_lod_select(const clod_scene& sc, DevView* vinfo, int V, clod_params prm,
                             const unsigned long long* dmax_key, uint32_t* hist, float* alpha, const Sink& out) {
  if (sc.n == 0) return hipSuccess;
  Stage h{};
  h.block = kBlock;
  hipError_t e = hipSuccess;
  for (int level = 0; level < 5 && e == hipSuccess; ++level) {
    h.kind = level == 0 ? kStSelectFirst : level < 4 ? kStSelectHist : kStSelectPick;
    h.items = (uint32_t)(level == 0 ? kSelFirst * ((V + kSelViews - 1) / kSelViews) : level < 4 ? kSelBlocks * V : V);
    h.a.select = SelectArgs{sc, vinfo, vinfo, V, prm, dmax_key, hist, alpha, level, 0};
    e = out.put(h);
  }
  return e;
}

// Blocks of the per-Gaussian passes: four Gaussians per thread and more where the scene fills the
// chip that way, one per thread in small scenes.
int proj_blocks(int64_t n) {
  int64_t g = (n + 4 * kBlock - 1) / (4 * kBlock), least = (n + kBlock - 1) / kBlock;
  if (least > 512) least = 512;
  if (g < least) g = least;
  if (g < 1) g = 1;
  if (g > kMaxProjBlocks) g = kMaxProjBlocks;
  return (int)g;
}

hipError_t launch_view_setup(const clod_view* views_dev, int V, clod_params prm, DevView* vinfo,
                             unsigned long long* hdr, const Sink& out) {
  Stage st{};
  st.kind = kStViewSetup;
  st.items = 1;
  st.block = 64;
  st.a.view_setup = ViewSetupArgs{views_dev, V, prm, vinfo, hdr};
  return out.put(st);
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, const Sink& out) {
  if (count <= 0) return hipSuccess;
  int64_t g = (count + kBlock - 1) / kBlock;
  if (g > 4096) g = 4096;
  Stage st{};
  st.kind = kStFill;
  st.items = (uint32_t)g;
  st.block = kBlock;
  st.a.fill = FillArgs{p, value, count};
  return out.put(st);
}

static Stage fold_stage(const uint32_t* kpart, const uint32_t* cpart, int G, int V,
                        unsigned long long* dmax_key, unsigned long long* counts, int64_t* counts_dev, int64_t n,
                        float* eta_dev, uint32_t* clear, uint32_t clear_words) {
  Stage st{};
  st.kind = kStFold;
  st.items = (uint32_t)V;
  st.block = kBlock;
  st.a.fold = FoldArgs{kpart, cpart, G, V, dmax_key, counts, counts_dev, n, eta_dev, clear, clear_words};
  return st;
}

hipError_t launch_frustum_max(const clod_scene& sc, const DevView* vinfo, int V, float near_z,
                              uint32_t* kpart, unsigned long long* dmax_key, uint32_t* clear,
                              uint32_t clear_words, const Sink& out) {
  if (sc.n == 0) return launch_fill_u32((uint32_t*)dmax_key, 0u, 2 * (int64_t)V, out);
  const int G = proj_blocks(sc.n);
  Stage st{};
  st.kind = kStFrustumMax;
  st.items = (uint32_t)G;
  st.block = kBlock;
  st.lds = (uint32_t)(kCamWords * V * sizeof(uint32_t));
  st.a.frustum = FrustumArgs{sc.mean, sc.n, vinfo, V, near_z, kpart};
  hipError_t e = out.put(st);
  if (e == hipSuccess)
    e = out.put(fold_stage(kpart, nullptr, G, V, dmax_key, nullptr, nullptr, sc.n, nullptr, clear, clear_words));
  return e;
}

template <bool kWrite>
static hipError_t project_impl(const clod_scene& sc, const DevView* vinfo, int V, clod_params prm,
                               unsigned long long* dmax_key, uint32_t* cpart, unsigned long long* counts,
                               int64_t* counts_dev, float* eta_dev, uint8_t* flags, float* alpha, float4* rec,
                               uint32_t* list, uint32_t* lcount, uint32_t* clear, uint32_t clear_words,
                               const Sink& out) {
  if (sc.n == 0) {
    hipError_t e = launch_fill_u32((uint32_t*)counts, 0u, 6 * (int64_t)V, out);
    if (e == hipSuccess && counts_dev) e = launch_fill_u32((uint32_t*)counts_dev, 0u, 6 * (int64_t)V, out);
    if (e == hipSuccess && eta_dev) e = launch_fill_u32((uint32_t*)eta_dev, 0u, (int64_t)V, out);
    return e;
  }
  const int G = proj_blocks(sc.n);
  Stage c{};
  c.kind = kStClassify;
  c.items = (uint32_t)G;
  c.block = kBlock;
  c.lds = (uint32_t)((kWrite ? kClassifyWords : kCountWords) * V * sizeof(uint32_t));
  c.a.classify = ClassifyArgs{sc, vinfo, V, kWrite ? 1 : 0, prm, dmax_key, cpart, flags, alpha, list, lcount};
  hipError_t e = out.put(c);
  if (e != hipSuccess) return e;
  // Packed SH is only read when records are written.
  Stage p{};
  p.kind = kStProject;
  p.items = (uint32_t)G;
  p.block = kBlock;
  p.lds = (uint32_t)((kSegWords + (kWrite ? 1 : kCountWords) * V) * sizeof(uint32_t));
  p.a.project = ProjectArgs{sc, vinfo, V, prm, dmax_key, cpart, list, lcount, flags, alpha, rec, kWrite ? 1 : 0,
                            kWrite && sc.sh_packed != nullptr ? 1 : 0};
  e = out.put(p);
  if (e != hipSuccess) return e;
  // Counts to the workspace and the caller, and the argmax index into the d_max key.
  return out.put(fold_stage(nullptr, cpart, G, V, dmax_key, counts, counts_dev, sc.n, eta_dev, clear, clear_words));
}

hipError_t launch_project(const clod_scene& sc, const DevView* vinfo, int V, clod_params prm,
                          unsigned long long* dmax_key, uint32_t* cpart, unsigned long long* counts,
                          int64_t* counts_dev, float* eta_dev, uint8_t* flags, float* alpha, float4* rec,
                          uint32_t* list, uint32_t* lcount, uint32_t* clear, uint32_t clear_words, const Sink& out) {
  return project_impl<true>(sc, vinfo, V, prm, dmax_key, cpart, counts, counts_dev, eta_dev, flags, alpha, rec, list,
                            lcount, clear, clear_words, out);
}

hipError_t launch_lod_count(const clod_scene& sc, const DevView* vinfo, int V, clod_params prm,
                            unsigned long long* dmax_key, uint32_t* cpart, unsigned long long* counts,
                            int64_t* counts_dev, float* eta_dev, uint32_t* list, uint32_t* lcount,
                            const Sink& out) {
  return project_impl<false>(sc, vinfo, V, prm, dmax_key, cpart, counts, counts_dev, eta_dev, nullptr, nullptr,
                             nullptr, list, lcount, nullptr, 0, out);
}

// One kernel per stage kind of this file (the template instance the arguments select).
hipError_t launch_project_stage(const Stage& st, hipStream_t s) {
  const dim3 g(st.items), blk(st.block);
  switch (st.kind) {
    case kStViewSetup: hipLaunchKernelGGL(k_view_setup, g, blk, 0, s, st.a.view_setup); break;
    case kStFill: hipLaunchKernelGGL(k_fill_u32, g, blk, 0, s, st.a.fill); break;
    case kStFrustumMax: hipLaunchKernelGGL(k_frustum_max, g, blk, st.lds, s, st.a.frustum); break;
    case kStFold: hipLaunchKernelGGL(k_reduce_partials, g, blk, 0, s, st.a.fold); break;
    case kStClassify:
      if (st.a.classify.write) hipLaunchKernelGGL(k_classify, g, blk, st.lds, s, st.a.classify);
      else hipLaunchKernelGGL(k_count, g, blk, st.lds, s, st.a.classify);
      break;
    case kStProject: {
      const ProjectArgs& a = st.a.project;
      auto kern = a.packed ? k_project_packed<3> : k_project<3>;
      switch (a.sc.sh_degree) {
        case 0: kern = a.packed ? k_project_packed<0> : k_project<0>; break;
        case 1: kern = a.packed ? k_project_packed<1> : k_project<1>; break;
        case 2: kern = a.packed ? k_project_packed<2> : k_project<2>; break;
        default: break;
      }
      if (!a.write) kern = k_count_rest;
      hipLaunchKernelGGL(kern, g, blk, st.lds, s, a);
      break;
    }
    case kStSelectFirst: hipLaunchKernelGGL(k_select_first, g, blk, 0, s, st.a.select); break;
    case kStSelectHist: hipLaunchKernelGGL(k_select_hist, g, blk, 0, s, st.a.select); break;
    case kStSelectPick: hipLaunchKernelGGL(k_select_pick, g, blk, 0, s, st.a.select); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace clod
