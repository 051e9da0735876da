// Per-tile front-to-back blending (Sec. 3.1, Eq. (1)) and its adjoint.
//
// One 256-thread workgroup (4 wave64) per 16x16 tile; wave w owns the 8x8 quadrant
// (w & 1, w >> 1) and lane l its pixel (l & 7, l >> 3).  Entries of the tile's sorted list
// are staged in LDS (one per lane or thread, a coalesced gather of the records) and read back
// as LDS broadcasts; entries that provably cannot reach a quadrant are dropped for it (see
// block_reached).  Blocks take tiles longest list first (the order clod_bin_sort computes),
// so the long tiles, not stragglers, start the launch.  Long lists (store_long_tiles) are blended with
// 4x4-pixel blocks per wave (four workgroups per tile); a stage before the blend marks per entry the
// blocks it may reach, and each block's wave walks only those entries.
#include "clod_internal.h"

namespace clod {

// XCD-aware launch order.  Consecutive workgroups are dispatched round-robin over the eight
// XCDs, each with its own L2, so tiles next to each other in the launch order (the same list
// length class, neighbours in the frame, sharing many records) would each fetch the shared
// records into a different L2.  Block b instead takes position
// ((b/8/C)*8 + b%8)*C + (b/8)%C of the tile order: runs of C consecutive positions stay on one
// XCD while the launch as a whole still proceeds in order (longest lists first).  The grid is
// rounded up to a multiple of 8C; the map is a bijection on it and blocks past the last tile
// exit at once.
constexpr uint32_t kXcds = 8, kXcdRun = 16;
constexpr uint32_t kLongMaskBlocks = 1024;   // grid of the long-tile mask stage

__device__ __forceinline__ uint32_t xcd_tile_pos(uint32_t b) {
  const uint32_t x = b % kXcds, j = b / kXcds, r = j / kXcdRun, i = j % kXcdRun;
  return (r * kXcds + x) * kXcdRun + i;
}

__host__ __device__ inline uint32_t xcd_grid(uint32_t tiles) {
  return (tiles + kXcds * kXcdRun - 1) / (kXcds * kXcdRun) * (kXcds * kXcdRun);
}

// Long tiles are taken by four workgroups each, in runs of eight tiles (one tile per XCD).
__host__ __device__ inline uint32_t long_grid(uint32_t long_tiles) {
  return (4 * long_tiles + 4 * kXcds - 1) / (4 * kXcds) * (4 * kXcds);
}

// The long (or masked) tiles of this blend: the first *count positions of the tile order (written by
// the tile ordering stage), within the bound the launch was sized for.
__device__ __forceinline__ uint32_t long_tiles(const uint32_t* count, uint32_t bound) {
  const uint32_t nl = *count;
  return nl < bound ? nl : bound;
}

__device__ __forceinline__ int view_of_tile(const DevView* views, int V, uint32_t tile) {
  int lo = 0, hi = V - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_base <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Per-entry power cut.  An entry contributes to a pixel only if alpha'' E(power) >= fl(1/255).
// E(p) <= 1 for p <= 0 and E never decreases by more than 2^-23 relative between neighbouring
// inputs, so for power < cut = ln(1 / (255 alpha'')) - 0.01 the product is below
// (1/255) e^-0.01 (1 + 3 2^-23) < 1/255: the contract skips the pair.  The cut is formed as
// (ln(1/255) - 0.01) - ln 2 log2(alpha'') with the hardware log2, whose error here (about
// 1e-6 absolute for alpha'' in [1/255, 1]) the 0.01 margin absorbs.  cut > 0 means the entry
// is skipped at every pixel; alpha'' = 0 (or a flushed subnormal) gives cut = +inf.
__device__ __forceinline__ float entry_cut(float a2) {
  constexpr float kC0 = -5.551263545158426f;   // ln(1/255) - 0.01
  constexpr float kLn2 = 0.6931471805599453f;
  return kC0 - kLn2 * __builtin_amdgcn_logf(a2);
}

// Minimum over the box [X0, X1] x [Y0, Y1] of q(dx, dy) = A dx^2 + 2 B dx dy + C dy^2 (the
// conic's quadratic form, positive definite): 0 if the box holds the origin, else the least of
// the four edge minima (each a clamped 1-D vertex).  The vertices use the hardware reciprocal:
// q along an edge exceeds its minimum by a term quadratic in the vertex offset, so a
// relative offset of a few 2^-24 stays negligible next to the allowance below.
__device__ __forceinline__ float box_qmin(float A, float B, float C, float X0, float X1, float Y0, float Y1) {
  if (X0 <= 0.0f && X1 >= 0.0f && Y0 <= 0.0f && Y1 >= 0.0f) return 0.0f;
  const float bc = B * __builtin_amdgcn_rcpf(C), ba = B * __builtin_amdgcn_rcpf(A);
  auto qf = [&](float dx, float dy) { return fmaf(A * dx, dx, fmaf(C * dy, dy, 2.0f * B * dx * dy)); };
  const float yx0 = fminf(fmaxf(-bc * X0, Y0), Y1), yx1 = fminf(fmaxf(-bc * X1, Y0), Y1);
  const float xy0 = fminf(fmaxf(-ba * Y0, X0), X1), xy1 = fminf(fmaxf(-ba * Y1, X0), X1);
  return fminf(fminf(qf(X0, yx0), qf(X1, yx1)), fminf(qf(xy0, Y0), qf(xy1, Y1)));
}

// Second, tighter test for a quadrant: the entry is dropped if the quadratic form stays above
// 2.5 |cut| over the box of the quadrant's pixel centres (widened by 1e-3 px for the rounding
// of the box edges).  With AC / (AC - B^2) <= 5e4 the binary32 evaluation is within 1.2 % of
// the exact form (and the vertex rounding is negligible), so the exact minimum exceeds
// 2.4 |cut| and the same argument as the circle test applies.
// kB x kB pixel block with corner (x0, y0).
template <int kB = 8>
__device__ __forceinline__ bool ellipse_reaches(float u, float v, float A, float B, float C, float cut,
                                                float x0, float y0) {
  constexpr float kHi = (float)kB - 0.499f;
  const float X0 = (x0 + 0.499f) - u, X1 = (x0 + kHi) - u;
  const float Y0 = (y0 + 0.499f) - v, Y1 = (y0 + kHi) - v;
  return box_qmin(A, B, C, X0, X1, Y0, Y1) < 2.5f * -cut;
}

// Conservative cull of a staged entry for the kB x kB pixel block with corner (x0, y0) (an 8x8
// quadrant, a 4x4 block of a long tile): 1 if the entry may touch it.  A pixel centre p farther than
// sqrt(2.4 |cut|) rad / 3 + 0.5 from the 2D mean has exact quadratic form
// d^T Q d > 2.4 |cut| (rad >= 3 sqrt(lambda_max)), i.e. exact power < -1.2 |cut|.  The binary32
// power differs from the exact one by a factor common to the conic (the rounding of det,
// <= 2u r) plus independent roundings amplified by at most r = AC / (AC - B^2); with
// r <= 5e4 the total stays below 4%, so the evaluated power is below cut and the pair is
// skipped.  (The radius uses the hardware square root: its relative error of a few 2^-24
// is far inside that slack.)  Culled pairs are therefore exactly pairs the pixel loop would have skipped.
// Entries with a worse conditioned conic are never culled spatially.
template <int kB>
__device__ __forceinline__ uint32_t block_reached(float u, float v, float A, float B, float C, float rad,
                                                   float cut, float x0, float y0) {
  if (!(cut <= 0.0f)) return 0u;   // never live (a NaN cut included: no power reaches it)
  const float ac = A * C;
  const float det = ac - B * B;
  if (!(det > 2e-5f * ac) || !(rad < 1e6f)) return 1u;
  constexpr float kHi = (float)kB - 0.5f;
  const float rc = __builtin_amdgcn_sqrtf(2.4f * -cut) * rad * (1.0f / 3.0f) + 0.5f;
  const float ddx = fmaxf(0.0f, fmaxf(x0 + 0.5f - u, u - (x0 + kHi)));
  const float ddy = fmaxf(0.0f, fmaxf(y0 + 0.5f - v, v - (y0 + kHi)));
  return (ddx * ddx + ddy * ddy <= rc * rc && ellipse_reaches<kB>(u, v, A, B, C, cut, x0, y0)) ? 1u : 0u;
}

// Long tiles (store_long_tiles) are blended with 4x4-pixel blocks per wave: a wave walks only the
// entries that may reach its block, and sixteen waves share the tile instead of four.  The tile
// order puts them first (longest first): they are taken by the leading workgroups of the launch.
// They get their block tests from k_long_mask and their waves walk compacted lists (where the bit
// planes find no room, in the resident server, and for all but the longest in full batches, the
// waves test the entries themselves).

// Forward blend.  Each wave owns one 8x8 quadrant of a tile (lane l: pixel (l & 7, l >> 3))
// and runs on its own: it takes 64 entries of the tile's sorted list at a time (one entry per
// lane, a coalesced gather), stages the ones that can touch its quadrant in its private LDS
// slice, compacted in list order, and walks them with the next entry's LDS reads issued
// before the current entry's arithmetic.  A wave stops after the batch in which its 64
// pixels saturate, independently of the other quadrants; the only block barrier is the
// final reduction of the optional pair counters.
struct TileLds {
  float4 st[4][3][64];   // per wave: (u, v, hA, nB), (hC, alpha'', r, g), (b, cut, list position, -)
  uint32_t q[4][256];    // per wave: ring of the list positions that reach its 4x4 block (long tiles)
};

// One tile, at position pos of the batch's tile order, by the 256 threads of the block (four
// independent waves).  Shared by the per-batch launch (k_blend_fwd) and the persistent server.
// kB = 8: the four waves take the tile's four 8x8 quadrants.  kB = 4: the four waves take the
// 4x4 blocks 4 sub .. 4 sub + 3 of the tile (row-major over its 4 x 4 blocks); lane 16 g + p
// takes pixel p of the block, and the lanes of row 0 (g = 0) own the results.
template <bool kCount, int kB = 8>
__device__ __forceinline__ void blend_tile(const BlendArgs& a, uint32_t pos, TileLds& S, uint32_t sub = 0) {
  auto& st = S.st;
  const DevView* __restrict__ views = a.views;
  const int V = a.V;
  const uint32_t tiles_total = a.tiles_total;
  const int64_t VN = a.VN;
  const float4* __restrict__ rec = a.rec;
  const uint2* __restrict__ ranges = a.ranges;
  const uint32_t* __restrict__ svals = a.svals;
  const float bg0 = a.bg0, bg1 = a.bg1, bg2 = a.bg2;
  float* __restrict__ rgb = a.rgb;
  float* __restrict__ Tout = a.T;
  uint32_t* __restrict__ lastout = a.last;
  unsigned long long* __restrict__ pair_part = a.pair_part;
  const uint32_t* __restrict__ order = a.order;
  const uint32_t t = threadIdx.x;
  if (a.hdr[kHdrOverflow]) return;
  if (pos >= tiles_total) return;
  // The long tiles are taken as 4x4 blocks.
  if ((kB == 8) != (pos >= long_tiles(a.nlong, a.long_max))) return;
  const int tile_i = (int)order[pos];
  const int v = view_of_tile(views, V, (uint32_t)tile_i);
  const DevView& Vw = views[v];
  const int local = tile_i - (int)Vw.tile_base;
  const int tx = local % Vw.tiles_x, ty = local / Vw.tiles_x;
  const int wave = (int)(t >> 6);
  const uint32_t lane = lane_id();
  const int blk = kB == 8 ? wave : (int)sub * 4 + wave;
  const int qx0 = tx * kTile + (blk % (kTile / kB)) * kB, qy0 = ty * kTile + (blk / (kTile / kB)) * kB;
  const uint32_t pl = kB == 4 ? (lane & 15u) : lane;   // the lane's pixel within the block
  const int px = qx0 + (int)(pl % kB);
  const int py = qy0 + (int)(pl / kB);
  const bool inside = px < Vw.width && py < Vw.height;
  const bool own = inside && (kB == 8 || lane < 16u);
  // Pixel centres and quadrant corners in frame coordinates (the viewport origin added).
  const float pcx = (float)(px + Vw.vx) + 0.5f, pcy = (float)(py + Vw.vy) + 0.5f;
  const float fqx = (float)(qx0 + Vw.vx), fqy = (float)(qy0 + Vw.vy);
  const uint2 rg = ranges[tile_i];
  const float kSkip = 0.0039215688593685627f;   // fl(1/255)
  const float kTmin = 9.99999974737875163e-05f; // fl(1e-4)
  float4* s0 = st[wave][0];
  float4* s1 = st[wave][1];
  float4* s2 = st[wave][2];
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  uint32_t last = 0, term = 0xFFFFFFFFu, nexp = 0, nblend = 0;
  // Lanes whose pixel has terminated (or lies outside the frame), as a wave-uniform mask: the
  // per-entry predicates below are formed as lane masks and turned back into execution masks
  // with inverse ballots, so the termination bookkeeping stays in scalar registers.  (4x4 blocks:
  // the 16 pixels' bits four times, once per row of lanes.)
  uint64_t dm = ballot64(!inside);
  // 4x4 blocks: the n entries of a batch that may reach the block (staged compacted in list
  // order, slots 0 .. n-1), four at a time.  Row g of the wave evaluates entry g of the group for
  // the block's 16 pixels (power, live test, exponential, clamp, skip test: four exponentials side
  // by side) and keeps its opacity, or 0 where the contract skips the pair.  The opacities then go
  // to all rows (whole-wave row swaps), and every row takes the four entries in list order through
  // the same transmittance, row c adding up colour channel c: the contract's operations in its
  // order, an opacity of 0 leaving T and the sums as they are (T * 1 and fma(c, 0, sum); colours
  // are finite here).  T never grows, so if no pixel is below the termination threshold after the
  // group, none was inside it; else (at most once per pixel) the group is taken again from the
  // state before it, one entry at a time with the contract's termination test.  `last` is kept by
  // the row that evaluated the entry (the largest of a pixel's four counts).
  // A wave walks these lists all but alone on its SIMD, so the chain of a group is what counts: with
  // the tests, masks and branches of every entry in it a group took 740 cycles, and the longest
  // of the 6M far frame's 6,500-entry chains set its 558 us; now 300.
  auto walk4 = [&](const uint32_t n, const bool finite) {
    const uint32_t row = lane >> 4;
    struct Set {
      float4 a; float2 c; float2 b;   // (u, v, -A/2, -B), (-C/2, alpha''), (cut, list position)
    };
    const float* colour = row == 0u ? &s1[0].z : row == 1u ? &s1[0].w : &s2[0].x;
    auto load = [&](const uint32_t k, Set& q) {
      const uint32_t fr = k + row;
      q.a = s0[fr];
      q.c = *reinterpret_cast<const float2*>(&s1[fr].x);
      q.b = *reinterpret_cast<const float2*>(&s2[fr].y);
    };
    auto group = [&](const uint32_t k, const Set& q) {
      // The row's channel of the four entries: requested here, there before the opacities are.  (In
      // the two sets they took eight registers more, and the kernel spilled: 382 us for the five-frame
      // batch of 3M at seven waves per SIMD, now 371.)
      float col[4];
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) col[e] = colour[4u * (k + e)];
      const float dx = q.a.x - pcx, dy = q.a.y - pcy;
      const float power = fmaf_(q.a.z * dx, dx, fmaf_(q.c.x * dy, dy, (q.a.w * dx) * dy));
      const uint32_t left = n - k;   // slots at or past n hold stale entries
      const uint64_t slots = left >= 4u ? ~0ull : (1ull << (16u * left)) - 1ull;
      const uint64_t live = ballot64(__builtin_amdgcn_fmed3f(power, q.b.x, 0.0f) == power) & ~dm & slots;
      if (live == 0ull) return;
      const float al = fminf(0.99f, q.c.y * cexp_core(power));
      const uint64_t um = ballot64(al >= kSkip) & live;
      if (um == 0ull) {
        if (kCount) nexp += __builtin_amdgcn_inverse_ballot_w64(live) ? 1u : 0u;
        return;
      }
      const float am = __builtin_amdgcn_inverse_ballot_w64(um) ? al : 0.0f;
      // Rows 0 .. 3 of am to every row.
      const auto x32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(am), __float_as_uint(am), false, false);
      const auto x01 = __builtin_amdgcn_permlane16_swap(x32[0], x32[0], false, false);
      const auto x23 = __builtin_amdgcn_permlane16_swap(x32[1], x32[1], false, false);
      const float al4[4] = {__uint_as_float(x01[0]), __uint_as_float(x01[1]), __uint_as_float(x23[0]), __uint_as_float(x23[1])};
      const uint32_t count = __float_as_uint(q.b.y) + 1u;
      float Tn = T, sum = cr;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = al4[e] * Tn;
        sum = fmaf_(col[e], w, sum);
        Tn = Tn * (1.0f - al4[e]);
      }
      if ((ballot64(Tn < kTmin) & ~dm) == 0ull && finite) {
        T = Tn;
        cr = sum;
        last = __builtin_amdgcn_inverse_ballot_w64(um) ? count : last;
        if (kCount) {
          nexp += __builtin_amdgcn_inverse_ballot_w64(live) ? 1u : 0u;
          nblend += __builtin_amdgcn_inverse_ballot_w64(um) ? 1u : 0u;
        }
        return;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t rows = 0xFFFFull << (16 * e);
        const uint64_t lm = live & rows & ~dm;   // pairs of entry e
        const uint64_t take = ballot64(al4[e] > 0.0f) & ~dm, ends = ballot64(T * (1.0f - al4[e]) < kTmin) & take;
        if (__builtin_amdgcn_inverse_ballot_w64(take & ~ends)) {
          const float w = al4[e] * T;
          cr = fmaf_(col[e], w, cr);
          T = T * (1.0f - al4[e]);
        }
        last = __builtin_amdgcn_inverse_ballot_w64(take & ~ends & rows) ? count : last;
        if (kCount) {
          if (__builtin_amdgcn_inverse_ballot_w64(ends)) term = __float_as_uint(s2[k + (uint32_t)e].z);
          nexp += __builtin_amdgcn_inverse_ballot_w64(lm) ? 1u : 0u;
          nblend += __builtin_amdgcn_inverse_ballot_w64(take & ~ends & rows) ? 1u : 0u;
        }
        dm |= ends;
      }
    };
    // Two register sets in alternation, as below.
    Set A, B;
    load(0u, A);
    for (uint32_t k = 0; k < n; k += 8) {
      load(k + 4u, B);   // (k + 4 <= 60)
      group(k, A);
      load(k + 8u < 60u ? k + 8u : 60u, A);
      if (k + 4u < n) group(k + 4u, B);
      if (dm == ~0ull) break;
    }
  };
  // One batch of up to 64 entries, its records (g0, g1, g2) already in registers, lane l's
  // at list position j: staged in this wave's LDS slice, culled against the quadrant, then
  // walked.  The entries of a premasked long tile arrive already compacted to those that may reach
  // the 4x4 block (relc); elsewhere the batch is 64 consecutive entries and is culled here.
  const bool pre = kB == 4 && pos < long_tiles(a.npre, a.pre_max);
  // next() runs between the staging and the walk: it requests the next batch's records, into the
  // same registers.
  auto batch = [&](const uint32_t j, const float4& g0, const float4& g1, const float4& g2,
                   const bool relc, auto&& next) {
    bool rel = false;
    float cut = 0.0f;
    if (kB == 4 && pre) {
      rel = relc;
      if (rel) {
        s0[lane] = make_float4(g0.x, g0.y, -0.5f * g1.x, -g1.y);
        s1[lane] = make_float4(-0.5f * g1.z, g0.z, g2.x, g2.y);
        s2[lane] = make_float4(g2.z, entry_cut(g0.z), __uint_as_float(j - rg.x), 0.f);
      }
    } else if (j < rg.y) {
      cut = entry_cut(g0.z);
      rel = (block_reached<kB>(g0.x, g0.y, g1.x, g1.y, g1.z, g0.w, cut, fqx, fqy)) != 0u;
    }
    uint64_t mask = ballot64(rel);
    // The entries that may reach the quadrant (block) are staged compacted, in list order
    // (slot = rank of the lane among them), so that the walks below step a counter.  (Those of
    // a premasked tile are the leading lanes already.)
    if (!(kB == 4 && pre)) {
      if (rel) {
        const uint32_t slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        s0[slot] = make_float4(g0.x, g0.y, -0.5f * g1.x, -g1.y);
        s1[slot] = make_float4(-0.5f * g1.z, g0.z, g2.x, g2.y);
        s2[slot] = make_float4(g2.z, cut, __uint_as_float(j - rg.x), 0.f);
      }
    }
    const uint32_t n = (uint32_t)__builtin_popcountll(mask);
    if (kB == 8 && (n & 1u) && lane == 63u) {
      s0[n] = make_float4(__builtin_nanf(""), __builtin_nanf(""), 0.0f, 0.0f);
      s2[n] = make_float4(0.0f, __builtin_inff(), 0.0f, 0.0f);
    }
    if (kB == 4 && lane >= n && lane < ((n + 3u) & ~3u)) {   // the last group's empty slots: colour 0
      s1[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s2[lane] = make_float4(0.0f, __builtin_inff(), 0.0f, 0.0f);
    }
    // The staged entries are read by other lanes of this wave: wait for the LDS writes.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if constexpr (kB == 4) {
      // Colours are at least 0 (or NaN, which fails the comparison as infinity does).
      const uint64_t odd = ballot64(rel && !(g2.x < __builtin_inff() && g2.y < __builtin_inff() && g2.z < __builtin_inff()));
      next();
      walk4(n, odd == 0ull);
      return;
    }
    next();
    if (mask == 0ull) return;
    // One entry: the contract's skip, exponential, clamp, termination and blend.  Below the
    // entry's cut (or above 0) the contract skips the pair whatever E returns; live pairs have
    // power in [cut, 0] with cut >= ln(1/255) - 0.01, inside cexp_core's range.  Once some
    // lane is live, every lane evaluates E (an exec-mask region around it would cost scalar
    // instructions and save no vector ones); the skip and termination tests then run on the
    // whole wave and are masked with the live set, so al and Tn of other lanes are never used.
    auto pair = [&](const float4& a, const float4& c, const float4& bc) {
      const float dx = a.x - pcx, dy = a.y - pcy;
      const float power = fmaf_(a.z * dx, dx, fmaf_(c.x * dy, dy, (a.w * dx) * dy));
      // cut <= power <= 0 as one test: a staged entry has cut <= 0 (block_reached culls the
      // others), so the median of (power, cut, 0) is power exactly then; a NaN power (the
      // padding entry) compares unequal.
      const uint64_t lm = ballot64(__builtin_amdgcn_fmed3f(power, bc.y, 0.0f) == power) & ~dm;
      if (lm == 0ull) return;
      const float al = fminf(0.99f, c.y * cexp_core(power));
      const float Tn = T * (1.0f - al);
      // al is never NaN (fminf returns 0.99 for a NaN product) and T is in (0, 1], so
      // Tn >= fl(1e-4) is exactly the negation of the contract's termination test.
      const uint64_t um = ballot64(al >= kSkip) & lm;
      const uint64_t km = ballot64(Tn >= kTmin);
      const uint64_t bm = um & km;
      dm |= um & ~km;
      const uint32_t pos = __float_as_uint(bc.z);
      if (__builtin_amdgcn_inverse_ballot_w64(bm)) {
        const float w = al * T;
        cr = fmaf_(c.z, w, cr);
        cg = fmaf_(c.w, w, cg);
        cb = fmaf_(bc.x, w, cb);
        T = Tn;
        last = pos + 1u;
      }
      if (kCount) {   // work counters only when asked for (they cost the per-entry loop)
        if (__builtin_amdgcn_inverse_ballot_w64(um & ~km)) term = pos;
        nexp += __builtin_amdgcn_inverse_ballot_w64(lm) ? 1u : 0u;
        nblend += __builtin_amdgcn_inverse_ballot_w64(bm) ? 1u : 0u;
      }
    };
    // Two register sets in alternation: the LDS reads of the next entry are in flight while
    // the current one is evaluated, with no copies between iterations.  The walk takes the
    // slots two at a time; an odd count is padded with slot n, given a NaN position and a cut
    // of +inf (so no pixel is live for it) before the wave barrier above.  (Slots past that hold stale
    // entries: they may be read ahead, within the slice, but are never walked.)
    // The saturation of all 64 pixels is checked per batch, by the caller: within a batch the
    // loop has no exit test but its count.
    float4 a0 = s0[0], c0 = s1[0], b0 = s2[0];
    for (uint32_t k = 0; k < n; k += 2) {
      const float4 a1 = s0[k + 1u], c1 = s1[k + 1u], b1 = s2[k + 1u];
      pair(a0, c0, b0);
      const uint32_t k2 = k + 2u < 63u ? k + 2u : 63u;
      a0 = s0[k2]; c0 = s1[k2]; b0 = s2[k2];
      pair(a1, c1, b1);
    }
  };
  // Software pipeline over the batches: while one batch is walked, the records of the next and the
  // sorted indices of the one after are in flight (index -> record is two dependent memory latencies
  // per batch, which few resident waves -- a far frame's handful of long tiles -- cannot hide).  A
  // batch's records leave their registers when it is staged, so one set of them is enough (two, in
  // alternation, cost eight waves' worth of registers per CU).  Every load is issued (positions past
  // the list end read its last entry, which is not staged), so the wait counts stay static.
  if (rg.y > rg.x) {
    const uint32_t jmax = rg.y - 1;
    auto index_at = [&](uint32_t q) {
      const uint32_t f = svals[q < jmax ? q : jmax];
      return (int64_t)f < VN ? f : 0u;   // defensive: the sort only emits indices < V*n
    };
    if (kB == 4 && pre) {
      // The wave scans its block's bit plane (one word per 64 entries, read
      // with scalar loads: they do not enter the vector-memory wait count, so the pipeline's
      // gathers stay in flight while it scans), appends the positions of the entries that may
      // reach the block to its LDS ring, and takes them 64 at a time into the same two-set
      // pipeline (indices two batches ahead, records one), so that it gathers, stages and walks
      // only those entries.  (The planes are written by an earlier launch, and the scalar
      // cache is invalidated when a launch starts; the resident serving kernel, which runs a
      // job's stages in one launch, does not take this path.)
      typedef const __attribute__((address_space(4))) unsigned long long* ConstWords;
      // (readfirstlane returns int: each half goes through uint32_t so that the low half is
      // not sign-extended into the high one.)
      const uint64_t pa = (uint64_t)(uintptr_t)(a.lplane + (int64_t)blk * a.pw + (rg.x >> 6) + (uint32_t)tile_i);
      const uint64_t pu = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(pa >> 32)) << 32) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pa);
      const ConstWords plane = (ConstWords)(uintptr_t)pu;
      const uint32_t nwords = ((rg.y - rg.x) + 63u) >> 6;
      uint32_t* __restrict__ ring = S.q[wave];
      uint32_t head = 0, tail = 0, wi = 0;
      auto fill = [&]() {
        while (tail - head < 192u && wi < nwords) {
          const unsigned long long word = plane[wi];
          const uint32_t lo = (uint32_t)word, hi = (uint32_t)(word >> 32);
          if ((word >> lane) & 1ull)
            ring[(tail + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))) & 255u] =
                rg.x + 64u * wi + lane;
          tail += (uint32_t)__builtin_popcountll(word);
          ++wi;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      };
      // The next (up to) 64 positions of the ring, one per lane (v: the lane holds one).
      auto take = [&](uint32_t& q, bool& v) {
        fill();
        const uint32_t n = tail - head < 64u ? tail - head : 64u;
        v = lane < n;
        q = v ? ring[(head + lane) & 255u] : rg.x;
        head += n;
      };
      // Ring positions lie in [rg.x, rg.y) (clamped all the same: they come from LDS, so the
      // clamp costs no memory wait); the record indices read there are the sort's own and are
      // not clamped (a clamp of each loaded index would make the wave wait for every gather in
      // flight).
      auto index_of = [&](uint32_t q) { return svals[q < jmax ? q : jmax]; };
      uint32_t q, qn;
      bool v, vn;
      take(q, v);
      uint32_t f = index_of(q);
      float4 g0 = rec[kRecQuads * (int64_t)f], g1 = rec[kRecQuads * (int64_t)f + 1], g2 = rec[kRecQuads * (int64_t)f + 2];
      take(qn, vn);
      f = index_of(qn);
      while (ballot64(v) != 0ull && dm != ~0ull) {
        batch(q, g0, g1, g2, v, [&]() {
          g0 = rec[kRecQuads * (int64_t)f];
          g1 = rec[kRecQuads * (int64_t)f + 1];
          g2 = rec[kRecQuads * (int64_t)f + 2];
          q = qn;
          v = vn;
          take(qn, vn);
          f = index_of(qn);
        });
      }
    } else {
      uint32_t f = index_at(rg.x + lane);
      float4 g0 = rec[kRecQuads * (int64_t)f], g1 = rec[kRecQuads * (int64_t)f + 1], g2 = rec[kRecQuads * (int64_t)f + 2];
      f = index_at(rg.x + 64 + lane);
      for (uint32_t base = rg.x; base < rg.y && dm != ~0ull; base += 64) {
        batch(base + lane, g0, g1, g2, false, [&]() {
          g0 = rec[kRecQuads * (int64_t)f];
          g1 = rec[kRecQuads * (int64_t)f + 1];
          g2 = rec[kRecQuads * (int64_t)f + 2];
          f = index_at(base + 128 + lane);
        });
      }
    }
  }
  if constexpr (kB == 4) {   // a channel per row; the counts of the rows folded
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
      const uint32_t q = __shfl_xor(last, o, 64);
      last = q > last ? q : last;
    }
    const uint32_t row = lane >> 4;
    if (inside && row < 3u)
      rgb[3 * (int64_t)Vw.pix_base + (int64_t)row * Vw.width * Vw.height + (int64_t)py * Vw.width + px] =
          fmaf_(T, row == 0u ? bg0 : row == 1u ? bg1 : bg2, cr);
  }
  if (own) {
    const int64_t P = (int64_t)Vw.pix_base;
    const int64_t HW = (int64_t)Vw.width * Vw.height;
    const int64_t p = (int64_t)py * Vw.width + px;
    if constexpr (kB == 8) {
    rgb[3 * P + p] = fmaf_(T, bg0, cr);
    rgb[3 * P + HW + p] = fmaf_(T, bg1, cg);
    rgb[3 * P + 2 * HW + p] = fmaf_(T, bg2, cb);
    }
    Tout[P + p] = T;
    lastout[P + p] = last;
  }
  if (kCount) {
    // Pairs the contract's per-pixel loop evaluates: up to and including the terminating
    // entry, else the whole list.  The four wave totals are added to the tile's (zeroed)
    // partials.
    const unsigned long long ev = !own ? 0ull : (term != 0xFFFFFFFFu ? (unsigned long long)term + 1ull
                                                                         : (unsigned long long)(rg.y - rg.x));
    const unsigned long long es = wave_sum(ev);
    const unsigned long long x = wave_sum((unsigned long long)nexp);
    const unsigned long long bl = wave_sum((unsigned long long)nblend);
    if (lane == 0) {
      atomicAdd(pair_part + 3 * (int64_t)tile_i, es);
      atomicAdd(pair_part + 3 * (int64_t)tile_i + 1, x);
      atomicAdd(pair_part + 3 * (int64_t)tile_i + 2, bl);
    }
  }
}

// Long tiles, per entry of their lists: the 4x4 blocks of the tile the entry may reach (the
// blend's own block test, run once per entry here instead of once per entry in each of the
// tile's sixteen waves, which all walk these lists to the end in the far views of a large
// scene), as sixteen bit planes: per block, one bit per entry, 64 entries per word.  The tiles'
// 64-entry chunks are numbered through 256 tiles at a time (a block scan of their counts), and wave
// w of the grid takes the chunks w, w + W, ..., writing a chunk's sixteen words (lane b the word of
// block b).  (Every wave walking the list of tiles for its own chunks, a chain of loads per tile,
// took 480 us for 150 tiles of 1.9M entries; now 72 us for 300 of 2.3M.)
__device__ __forceinline__ void long_mask_body(const LongMaskArgs& a, Blk b) {
  __shared__ uint32_t first[kBlock + 1], start[kBlock], len[kBlock], tile[kBlock], sm[4];
  __shared__ float ox[kBlock], oy[kBlock];
  if (a.hdr[kHdrOverflow]) return;
  const uint32_t nl = long_tiles(a.npre, a.pre_max);
  const uint32_t lane = lane_id(), t = threadIdx.x;
  const uint32_t gw = b.id * (kBlock / 64u) + (t >> 6), GW = b.n * (kBlock / 64u);
  for (uint32_t p0 = 0; p0 < nl; p0 += kBlock) {
    uint32_t chunks = 0;
    if (p0 + t < nl) {
      const uint32_t tile_i = a.order[p0 + t];
      const DevView& Vw = a.views[view_of_tile(a.views, a.V, tile_i)];
      const int local = (int)(tile_i - Vw.tile_base);
      const uint2 rg = a.ranges[tile_i];
      ox[t] = (float)(local % Vw.tiles_x * kTile + Vw.vx);
      oy[t] = (float)(local / Vw.tiles_x * kTile + Vw.vy);
      start[t] = rg.x;
      len[t] = rg.y - rg.x;
      tile[t] = tile_i;
      chunks = (len[t] + 63u) >> 6;
    }
    uint32_t total;
    first[t] = block_exclusive_scan(chunks, sm, total);
    if (t == 0) first[kBlock] = total;
    __syncthreads();
    for (uint32_t c = gw; c < total; c += GW) {
      uint32_t lo = 0, hi = kBlock - 1;   // last tile whose first chunk is at most c
      while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (first[mid] <= c) lo = mid; else hi = mid - 1;
      }
      const uint32_t word = c - first[lo], e = 64u * word + lane;
      uint32_t m = 0u;
      if (e < len[lo]) {
        uint32_t f = a.svals[start[lo] + e];
        if ((int64_t)f >= a.VN) f = 0u;   // defensive: the sort only emits indices < V*n
        const float4 g0 = a.rec[kRecQuads * (int64_t)f], g1 = a.rec[kRecQuads * (int64_t)f + 1];
        const float cut = entry_cut(g0.z);
#pragma unroll
        for (int q = 0; q < 16; ++q)
          m |= block_reached<4>(g0.x, g0.y, g1.x, g1.y, g1.z, g0.w, cut, ox[lo] + (float)(q % 4 * 4),
                                 oy[lo] + (float)(q / 4 * 4)) << q;
      }
      unsigned long long mine = 0ull;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const unsigned long long w = ballot64(((m >> q) & 1u) != 0u);
        if (lane == (uint32_t)q) mine = w;
      }
      if (lane < 16u) a.lplane[(int64_t)lane * a.pw + (start[lo] >> 6) + tile[lo] + word] = mine;
    }
    __syncthreads();
  }
}
__global__ __launch_bounds__(kBlock) void k_long_mask(LongMaskArgs a) { long_mask_body(a, grid_blk()); }

// Long tiles: four workgroups per tile, on one XCD (workgroups b, b + 8, b + 16, b + 24 take
// the same tile: consecutive workgroups go round-robin to the eight XCDs).
__device__ __forceinline__ void long_item(uint32_t b, uint32_t& pos, uint32_t& sub) {
  const uint32_t x = b % kXcds, j = b / kXcds;
  sub = j % 4;
  pos = x + kXcds * (j / 4);
}

// Item b of the blend stage: the leading long_grid(long_tiles) items take the long tiles as
// 4x4 blocks, the next xcd_grid(tiles) items one tile each in the XCD-aware order (both in one
// launch, so that the long tiles run beside the others).  Items past these (the launch is
// sized for the most long tiles the pair capacity allows) map past the last tile and exit.
template <bool kCount>
__device__ __forceinline__ void blend_item(const BlendArgs& a, uint32_t b, TileLds& S) {
  const uint32_t lb = long_grid(long_tiles(a.nlong, a.long_max));
  if (b < lb) {
    uint32_t pos, sub;
    long_item(b, pos, sub);
    blend_tile<kCount, 4>(a, pos, S, sub);
  } else {
    blend_tile<kCount>(a, xcd_tile_pos(b - lb), S);
  }
}

// Items a blend stage needs once the tile order is known (the resident kernel sizes its
// claims by it; a per-stage launch covers the bound instead).
__device__ __forceinline__ uint32_t blend_items(const BlendArgs& a) {
  return long_grid(long_tiles(a.nlong, a.long_max)) + xcd_grid(a.tiles_total);
}

// Per-batch launch: one workgroup per tile (four per long tile).  Seven waves per SIMD, 72 registers
// (six cost 2 to 4 % on frames without long tiles); the counting instance needs 78, so six.
template <bool kCount>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kCount ? 6 : 7))) void k_blend_fwd(BlendArgs a) {
  __shared__ TileLds S;
  blend_item<kCount>(a, blockIdx.x, S);
}

// Sums the per-tile pair partials into the caller's counters (one block, three atomics).
__device__ __forceinline__ void reduce_pairs_body(const ReducePairsArgs& r, Blk) {
  __shared__ unsigned long long sm[4][3];
  const unsigned long long* __restrict__ part = r.part;
  unsigned long long* __restrict__ out = r.out;
  unsigned long long a = 0, b = 0, c = 0;
  for (uint32_t t = threadIdx.x; t < r.tiles; t += kBlock) {
    a += part[3 * (int64_t)t]; b += part[3 * (int64_t)t + 1]; c += part[3 * (int64_t)t + 2];
  }
  a = wave_sum(a); b = wave_sum(b); c = wave_sum(c);
  if (lane_id() == 0) { sm[threadIdx.x >> 6][0] = a; sm[threadIdx.x >> 6][1] = b; sm[threadIdx.x >> 6][2] = c; }
  __syncthreads();
  if (threadIdx.x < 3) atomicAdd(out + threadIdx.x, sm[0][threadIdx.x] + sm[1][threadIdx.x] + sm[2][threadIdx.x] + sm[3][threadIdx.x]);
}
__global__ __launch_bounds__(kBlock) void k_reduce_pairs(ReducePairsArgs r) { reduce_pairs_body(r, grid_blk()); }

hipError_t launch_blend_fwd(const Layout& L, void* ws, const BlendBufs& bb, clod_params prm, float* rgb, float* T,
                            uint32_t* last, int64_t* pairs, const Sink& out) {
  if (L.tiles_total == 0) return hipSuccess;
  char* w = (char*)ws;
  unsigned long long* part = pairs ? (unsigned long long*)(w + L.pair_part) : nullptr;
  if (part) {
    hipError_t e = launch_fill_u32((uint32_t*)part, 0u, 6 * (int64_t)L.tiles_total, out);
    if (e != hipSuccess) return e;
  }
  // The long tiles' bit planes (16 planes of pw words) must fit the arrays the tile-id sort left free,
  // else each wave tests the entries itself.
  const uint32_t pw = (uint32_t)((bb.cap + 63) / 64 + (int64_t)L.tiles_total + 1);
  const bool planes_fit = (size_t)16 * pw * sizeof(unsigned long long) <= bb.spare_bytes;
  const uint32_t long_max = long_tile_bound(bb.cap, L.tiles_total, planes_fit);
  const uint32_t* tord = (const uint32_t*)(w + L.tord);
  const uint32_t* nlong = tord + (planes_fit ? kTileLongWord : kTileLongBareWord);
  const uint32_t pre_max = planes_fit ? long_max : 0u;
  if (pre_max > 0) {
    Stage m{};
    m.kind = kStLongMask;
    m.items = kLongMaskBlocks;
    m.block = kBlock;
    m.a.long_mask = LongMaskArgs{(const DevView*)(w + L.vinfo), L.V, (const uint2*)(w + L.ranges),
                                 (const uint32_t*)(w + L.order), tord + kTileMaskedWord, bb.svals,
                                 (const float4*)(w + L.rec), L.VN, (const unsigned long long*)(w + L.hdr),
                                 bb.spare, pw, pre_max};
    const hipError_t e = out.put(m);
    if (e != hipSuccess) return e;
  }
  Stage st{};
  st.kind = kStBlend;
  st.items = long_grid(long_max) + xcd_grid(L.tiles_total);
  st.block = kBlock;
  st.a.blend = BlendArgs{(const DevView*)(w + L.vinfo), L.V, L.tiles_total, L.VN, (const float4*)(w + L.rec),
                         (const uint2*)(w + L.ranges), bb.svals, (const unsigned long long*)(w + L.hdr), prm.bg[0],
                         prm.bg[1], prm.bg[2], rgb, T, last, part, (const uint32_t*)(w + L.order),
                         nlong, tord + kTileMaskedWord, long_max, part ? 1 : 0, bb.spare, pw, pre_max};
  hipError_t e = out.put(st);
  if (e == hipSuccess && part) {
    Stage r{};
    r.kind = kStReducePairs;
    r.items = 1;
    r.block = kBlock;
    r.a.reduce_pairs = ReducePairsArgs{(const unsigned long long*)part, L.tiles_total, (unsigned long long*)pairs};
    e = out.put(r);
  }
  return e;
}

hipError_t launch_blend_stage(const Stage& st, hipStream_t s) {
  const dim3 g(st.items), blk(st.block);
  switch (st.kind) {
    case kStBlend:
      if (st.a.blend.count) hipLaunchKernelGGL(k_blend_fwd<true>, g, blk, 0, s, st.a.blend);
      else hipLaunchKernelGGL(k_blend_fwd<false>, g, blk, 0, s, st.a.blend);
      break;
    case kStReducePairs: hipLaunchKernelGGL(k_reduce_pairs, g, blk, 0, s, st.a.reduce_pairs); break;
    case kStLongMask: hipLaunchKernelGGL(k_long_mask, g, blk, 0, s, st.a.long_mask); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- adjoint
// Back-to-front over each pixel's blended entries (positions < last), recomputing every
// decision exactly as the forward; transmittance is recovered by division
// (T_k = T_{k+1} / (1 - a_k)); the normalised colour of everything behind entry k obeys
// R_{k-1} = c_k a_k + (1 - a_k) R_k with R = background after the last entry, so
// dC/da_k = T_k (c_k - R_k); only g . R (g = dL/dC of the pixel) is needed, and it obeys the
// same recurrence.
// Same quadrant mapping, batches and compacted walk as the forward (culled entries are ones the
// forward skipped), from the last entry some pixel of the quadrant blended to the first.
//
// The four waves of a tile share nothing but their CU's first-level cache, where the records that
// one gathers are found by the others.  A blended entry gives per pixel two numbers, h = dL/da E(power) (0 where the clamp holds)
// and w = a T, from which its nine partials are sums over the pixels: five moments a'' sum h dx,
// h dy, h dx^2, h dx dy, h dy^2 (linear in which are the partials of u, v and the conic), sum h, and
// the colours sum w g.  Reducing the nine over the wave for each entry took 25 exchanges at four
// to eight issue cycles each, half of the walk.  Instead the wave writes (h, w) to LDS and turns
// the sums round once eight entries are there: lane (entry e, pixel row r) adds up its row's eight
// pixels with plain multiply-adds, and one exchange over the rows leaves lane (sum q, entry e) with
// sum q of entry e.  The record's nine partials are consecutive floats, so the eight entries' sums
// go to memory as two atomic instructions over 36-byte spans.
// Measured: 16 training views of 2M Gaussians (23M steps of a wave) 2.98 -> 2.55 ms, one view of 1M
// 173 -> 139 us.  About 0.25 ms of the former are the atomics (29M requests; sums of a tile's four
// waves merged in LDS first are 11.5M, but the barriers and the LDS they need cost more: 2.95 ms),
// the rest is vector issue at some 70 % of its slots.
// With kCount, each wave adds to the tile's (zeroed) partials the (pixel, entry) lanes its walk
// visits, the pairs whose exponential it evaluates (blended in the forward, power in range) and
// the pairs that contribute to the gradients.
constexpr uint32_t kGradGroup = 8;           // entries per reduction
struct BwdLds {
  float4 s0[64], s1[64], s2[64];   // (u, v, -A/2, -B), (-C/2, alpha'', r, g), (b, cut, list position, record)
  float4 hw[kGradGroup][32];       // (h, w) of the pixels 2 k, 2 k + 1 of entry e at [e][k ^ e]: neither
                                   // the rows' writes nor the columns' reads meet in a bank
  float gl[3][64];                 // the pixels' colour gradients
};
// Records that cover many tiles are added to from every quadrant under them, and the additions to one
// address come one after the other: where the pairs' records are large on average, the four waves of a
// tile walk the list in common windows of 256 entries instead and add their sums (reduced over the
// wave entry by entry) up in LDS first, a quarter of the additions to memory.  The size is that of a
// pair's record: sum of squared tiles over sum of tiles.  Backward of one view, us, by that size, waves
// on their own and merged: 24 tiles (250,000 Gaussians) 163 and 192, 51 tiles (250,000) 432 and 571, 87
// tiles (64,000) 236 and 277, 102 tiles (64,000, 256 x 256) 198 and 227; 132 tiles (64,000) 220 and
// 171, 245 tiles (16,000) 213 and 139, 498 tiles (250,000) 368 and 244, 1,836 tiles (4,000) 836 and 320.
// Between 100 and 300 either may win by a little.  That mean alone also takes in batches of many small
// records and a few splats beside a camera, which waves on their own walk faster: their flushes seldom
// meet.  So, besides, either the records are large throughout (24 tiles on average), or two pairs drawn
// at random belong to one record once in 8,192 times (sum t^2 against D^2): 16 views of 2M, 656,000
// records of 17 tiles, mean 302, once in 38,000, 2,018 and 2,167 us; one view of 1M, 66,000 records of 16
// tiles, mean 157, once in 6,700, 370 and 325; 16 views, 458,000 records of 22 tiles, 2,203 and 2,245;
// one view of 250,000, 79,560 records of 79 tiles, mean 305, once in 21,000, 425 and 331.
struct MergedLds {
  float4 s0[kBlock], s1[kBlock], s2[kBlock];   // (u, v, -A/2, -B), (-C/2, alpha'', r, g), (b, cut, -, record)
  float acc[kBlock * kGscreen];                // [entry][9]: odd stride, conflict-free
  unsigned long long qmask[4][4];              // [staging wave][quadrant]: entries that may reach it
  uint32_t smax[4];
};
union BwdBlockLds {
  BwdLds wave[4];
  MergedLds merged;
};
static_assert(sizeof(BwdBlockLds) <= 160 * 1024 / 5, "five workgroups per CU");
constexpr unsigned long long kMergeTiles = 112, kMergeMean = 24;
constexpr int kMergeMeetLog = 13;
__device__ __forceinline__ bool merge_tiles(const unsigned long long* hdr) {
  const unsigned long long D = hdr[kHdrDup], squares = hdr[kHdrSquares];   // D <= 2^32 - 2: no product wraps
  return squares >= kMergeTiles * D && (D >= kMergeMean * hdr[kHdrRend] || squares >= (D >> kMergeMeetLog) * D);
}
template <bool kCount>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_blend_bwd(
    const DevView* __restrict__ views, int V, uint32_t tiles_total, int64_t VN,
    const float4* __restrict__ rec, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ svals, const unsigned long long* __restrict__ hdr,
    float bg0, float bg1, float bg2, const float* __restrict__ Tin,
    const uint32_t* __restrict__ lastin, const float* __restrict__ dL_drgb,
    float* __restrict__ gscreen, const uint32_t* __restrict__ order,
    unsigned long long* __restrict__ pair_part) {
  __shared__ BwdBlockLds lds;
  const int quad = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // the wave's quadrant
  BwdLds& S = lds.wave[quad];
  const uint32_t opos = xcd_tile_pos(blockIdx.x);
  if (opos >= tiles_total) return;
  const int tile_i = (int)order[opos];
  if (hdr[kHdrOverflow]) return;
  const int v = view_of_tile(views, V, (uint32_t)tile_i);
  const DevView& Vw = views[v];
  const int local = tile_i - (int)Vw.tile_base;
  const int tx = local % Vw.tiles_x, ty = local / Vw.tiles_x;
  const uint32_t lane = lane_id();
  const int qx0 = tx * kTile + (quad & 1) * 8, qy0 = ty * kTile + (quad >> 1) * 8;
  const int px = qx0 + (int)(lane & 7), py = qy0 + (int)(lane >> 3);
  const bool inside = px < Vw.width && py < Vw.height;
  const float fqx = (float)(qx0 + Vw.vx), fqy = (float)(qy0 + Vw.vy);
  const float pcx = (float)(px + Vw.vx) + 0.5f, pcy = (float)(py + Vw.vy) + 0.5f;
  const uint2 rg = ranges[tile_i];
  const float kSkip = 0.0039215688593685627f;
  const int64_t P = (int64_t)Vw.pix_base;
  const int64_t HW = (int64_t)Vw.width * Vw.height;
  const int64_t p = (int64_t)py * Vw.width + px;
  uint32_t last = 0;
  float T = 1.0f, g0c = 0.f, g1c = 0.f, g2c = 0.f;
  if (inside) {
    last = lastin[P + p];
    T = Tin[P + p];
    g0c = dL_drgb[3 * P + p];
    g1c = dL_drgb[3 * P + HW + p];
    g2c = dL_drgb[3 * P + 2 * HW + p];
  }
  // g . R: the pixel's colour gradient dotted with the normalised colour behind the current
  // entry (R starts as the background), kept as one scalar through the same recurrence.
  float gR = fmaf_(g0c, bg0, fmaf_(g1c, bg1, g2c * bg2));
  // The entries to walk: up to the largest last of the quadrant.
  uint32_t m = last;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { const uint32_t q = __shfl_xor(m, o, 64); m = q > m ? q : m; }
  m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
  unsigned long long n_walk = 0, n_live = 0, n_contrib = 0;   // wave-uniform (kCount)
  if (merge_tiles(hdr)) {
    MergedLds& M = lds.merged;
    if (lane == 0) M.smax[quad] = m;
    __syncthreads();
    m = max(max(M.smax[0], M.smax[1]), max(M.smax[2], M.smax[3]));
    if (m > rg.y - rg.x) m = rg.y - rg.x;
    const float tx0 = (float)(tx * kTile + Vw.vx), ty0 = (float)(ty * kTile + Vw.vy);
    const uint32_t t = threadIdx.x;
    for (uint32_t hi = m; hi > 0u;) {   // list positions [lo, hi) of this window
      const uint32_t lo = hi > (uint32_t)kBlock ? hi - kBlock : 0u;
      const uint32_t cnt = hi - lo;
      __syncthreads();
      uint32_t qm = 0;
      if (t < cnt) {
        uint32_t f = svals[rg.x + lo + t];
        if ((int64_t)f >= VN) f = 0u;   // defensive: the sort only emits indices < V*n
        const float4 g0 = rec[kRecQuads * (int64_t)f], g1 = rec[kRecQuads * (int64_t)f + 1], g2 = rec[kRecQuads * (int64_t)f + 2];
        const float cut = entry_cut(g0.z);
        M.s0[t] = make_float4(g0.x, g0.y, -0.5f * g1.x, -g1.y);
        M.s1[t] = make_float4(-0.5f * g1.z, g0.z, g2.x, g2.y);
        M.s2[t] = make_float4(g2.z, cut, 0.0f, __uint_as_float(f));
#pragma unroll
        for (int q = 0; q < 4; ++q)
          qm |= block_reached<8>(g0.x, g0.y, g1.x, g1.y, g1.z, g0.w, cut, tx0 + (float)((q & 1) * 8), ty0 + (float)((q >> 1) * 8)) << q;
      }
#pragma unroll
      for (int q = 0; q < kGscreen; ++q) M.acc[q * kBlock + t] = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t b = ballot64((qm >> q) & 1u);
        if (lane == 0) M.qmask[quad][q] = b;
      }
      __syncthreads();
      for (int c = 3; c >= 0; --c) {
        const unsigned long long mv = M.qmask[c][quad];
        uint64_t mk = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mv >> 32)) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mv);
        if (kCount) n_walk += 64ull * (unsigned)__popcll(mk);
        while (mk != 0ull) {
          const int e = 63 - __builtin_clzll(mk);
          mk &= ~(1ull << e);
          const int k = c * 64 + e;
          const float4 a = M.s0[k], c4 = M.s1[k], bc = M.s2[k];
          const float dx = a.x - pcx, dy = a.y - pcy;
          const float power = fmaf_(a.z * dx, dx, fmaf_(c4.x * dy, dy, (a.w * dx) * dy));
          const uint64_t lm = ballot64(__builtin_amdgcn_fmed3f(power, bc.y, 0.0f) == power) & ballot64(lo + (uint32_t)k < last);
          if (kCount) n_live += (unsigned long long)__popcll(lm);
          if (lm == 0ull) continue;
          const float G = cexp_core(power);
          const float prod = c4.y * G;
          const float al = fminf(0.99f, prod);
          const uint64_t cm = ballot64(al >= kSkip) & lm;
          if (kCount) n_contrib += (unsigned long long)__popcll(cm);
          if (cm == 0ull) continue;
          const uint64_t gm = ballot64(prod <= 0.99f) & cm;
          const float oma = 1.0f - al;
          const float r0 = __builtin_amdgcn_rcpf(oma);
          const float Tk = T * fmaf_(fmaf_(-oma, r0, 1.0f), r0, r0);
          const float gc = fmaf_(g0c, c4.z, fmaf_(g1c, c4.w, g2c * bc.x));
          const float dLda = Tk * (gc - gR);
          const float h = __builtin_amdgcn_inverse_ballot_w64(gm) ? dLda * G : 0.f;
          const float w = __builtin_amdgcn_inverse_ballot_w64(cm) ? al * Tk : 0.f;
          const float hx = h * dx, hy = h * dy;
          const float v8[8] = {hx, hy, hx * dx, hx * dy, hy * dy, h, g0c * w, g1c * w};
          float u = row_sum8(v8);         // lane 8 g + e: sum g over the rows; then over the columns
          u += dpp_read<0x141, 0xF>(u);   // row_half_mirror
          u += dpp_read<0x4E, 0xF>(u);    // quad_perm (2, 3, 0, 1)
          u += dpp_read<0xB1, 0xF>(u);    // quad_perm (1, 0, 3, 2)
          const float b = wave_total63(g2c * w);
          if ((lane & 7u) == 0u || lane == 63u) atomicAdd(&M.acc[k * kGscreen + (lane == 63u ? 8 : (int)(lane >> 3))], lane == 63u ? b : u);
          if (__builtin_amdgcn_inverse_ballot_w64(cm)) {
            gR = fmaf_(al, gc, oma * gR);
            T = Tk;
          }
        }
      }
      __syncthreads();
      // Consecutive threads take consecutive floats of an entry's nine; the partials from the sums as below.
      for (uint32_t it = t; it < cnt * kGscreen; it += kBlock) {
        const uint32_t k = it / kGscreen, q = it - k * kGscreen;
        float val = M.acc[it];
        if (q < 5u) {
          const float4 a = M.s0[k];
          const float4 c4 = M.s1[k];
          const float m0 = M.acc[k * kGscreen], m1 = M.acc[k * kGscreen + 1];
          val = q == 0u ? c4.y * fmaf_(2.f * a.z, m0, a.w * m1)
              : q == 1u ? c4.y * fmaf_(2.f * c4.x, m1, a.w * m0)
              : c4.y * (q == 3u ? -val : -0.5f * val);
        }
        if (val != 0.0f) atomicAdd(gscreen + (int64_t)__float_as_uint(M.s2[k].w) * kGscreen + q, val);
      }
      hi = lo;
    }
    if (kCount && lane == 0) {
      atomicAdd(pair_part + 3 * (int64_t)tile_i, n_walk);
      atomicAdd(pair_part + 3 * (int64_t)tile_i + 1, n_live);
      atomicAdd(pair_part + 3 * (int64_t)tile_i + 2, n_contrib);
    }
    return;
  }
  if (m > rg.y - rg.x) m = rg.y - rg.x;   // (a last of this list never is)
  if (m == 0u) return;
  S.gl[0][lane] = g0c;
  S.gl[1][lane] = g1c;
  S.gl[2][lane] = g2c;
  auto lds_fence = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // The sums of the group's first n entries, added to the accumulator.  Lane: entry e = lane % 8,
  // pixel row lane / 8 (its own pixel's row, so pcy is the row's), then sum lane / 8.
  uint32_t ng = 0;      // entries in the group
  uint64_t slots = 0;   // byte e: staged slot of the group's entry e
  auto reduce = [&](const uint32_t n) {
    lds_fence();
    // (Opaque copies: formed ahead of the walk, the addresses and pixel centres below take thirty
    // registers from it.)
    uint32_t ln = lane;
    float pc0 = fqx + 0.5f;
    asm volatile("" : "+v"(ln), "+v"(pc0));
    const uint32_t e = ln & 7u, r = ln >> 3;
    const uint32_t slot = (uint32_t)(slots >> (8u * e)) & 63u;
    const float4 ea = S.s0[slot];
    const float2 eb = *reinterpret_cast<const float2*>(&S.s1[slot]);
    float H = 0.f, HX = 0.f, HXX = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {   // two pixels at a time (all eight at once spill, or cost a third of the waves)
      const float4 hw = S.hw[e][(4u * r + k) ^ e];
      const float2 ga = *reinterpret_cast<const float2*>(&S.gl[0][8u * r + 2u * k]);
      const float2 gb = *reinterpret_cast<const float2*>(&S.gl[1][8u * r + 2u * k]);
      const float2 gc = *reinterpret_cast<const float2*>(&S.gl[2][8u * r + 2u * k]);
      auto one = [&](uint32_t c, float h, float w, float x0, float x1, float x2) {
        const float dx = ea.x - (pc0 + (float)c), t = h * dx;
        H += h;
        HX += t;
        HXX = fmaf_(t, dx, HXX);
        c0 = fmaf_(w, x0, c0);
        c1 = fmaf_(w, x1, c1);
        c2 = fmaf_(w, x2, c2);
      };
      one(2 * k, hw.x, hw.y, ga.x, gb.x, gc.x);
      one(2 * k + 1, hw.z, hw.w, ga.y, gb.y, gc.y);
      __builtin_amdgcn_sched_barrier(0);
    }
    const float dy = ea.y - pcy, HY = H * dy;
    const float v8[8] = {HX, HY, HXX, HX * dy, HY * dy, H, c0, c1};
    float u = row_sum8(v8);   // lane: sum lane / 8 of entry e
    // The ninth sum, over the rows (lanes of equal lane % 8).
    float b = c2 + dpp_read<0x128, 0xF>(c2);   // row_ror:8
    const auto b16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(b), __float_as_uint(b), false, false);
    b = __uint_as_float(b16[0]) + __uint_as_float(b16[1]);
    const auto b32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(b), __float_as_uint(b), false, false);
    b = __uint_as_float(b32[0]) + __uint_as_float(b32[1]);
    // du = -a'' (A m0 + B m1), dv = -a'' (C m1 + B m0), dA = -a'' m2 / 2, dB = -a'' m3,
    // dC = -a'' m4 / 2 (ea.z = -A/2, ea.w = -B, eb.x = -C/2), then sum h and the colours.
    const float a2 = eb.y, other = dpp_read<0x128, 0xF>(u);   // sum 1 for lane of sum 0, and back
    const float own = r == 0u ? 2.f * ea.z : r == 1u ? 2.f * eb.x : r == 3u ? -1.0f : -0.5f;
    float val = u;
    if (r < 5u) val = a2 * (own * u);
    if (r < 2u) val = a2 * fmaf_(own, u, ea.w * other);
    // To memory: consecutive lanes take consecutive floats of an entry's nine (the entries side by
    // side instead made every lane a request of its own), turned round through the group's (h, w),
    // which are used up.
    lds_fence();
    float* turn = reinterpret_cast<float*>(S.hw);   // [entry][9]
    turn[e * kGscreen + r] = val;
    if (r == 0u) turn[e * kGscreen + 8] = b;
    lds_fence();
#pragma unroll
    for (uint32_t it = 0; it < kGradGroup * kGscreen; it += 64) {
      const uint32_t item = it + ln;
      if (item < n * kGscreen) {
        const uint32_t te = item / kGscreen, q = item - te * kGscreen;
        const uint32_t f = __float_as_uint(S.s2[(uint32_t)(slots >> (8u * te)) & 63u].w);
        const float x = turn[item];
        if (x != 0.0f) atomicAdd(gscreen + (int64_t)f * kGscreen + q, x);
      }
    }
    lds_fence();
  };

  // One entry: (u, v, -A/2, -B), (-C/2, alpha'', r, g), (b, cut, position, record).
  auto pair = [&](const uint32_t k, const float4& a, const float4& c, const float4& bc) {
    const float dx = a.x - pcx, dy = a.y - pcy;
    const float power = fmaf_(a.z * dx, dx, fmaf_(c.x * dy, dy, (a.w * dx) * dy));
    // Live: blended in the forward (position < last) with power in [cut, 0] (one test, as in the
    // forward).  Other lanes compute discarded values.
    const uint64_t lm = ballot64(__builtin_amdgcn_fmed3f(power, bc.y, 0.0f) == power) &
                        ballot64(__float_as_uint(bc.z) < last);
    if (kCount) n_live += (unsigned long long)__popcll(lm);
    if (lm == 0ull) return;
    const float G = cexp_core(power);
    const float prod = c.y * G;
    const float al = fminf(0.99f, prod);
    const uint64_t cm = ballot64(al >= kSkip) & lm;       // contributing lanes
    if (kCount) n_contrib += (unsigned long long)__popcll(cm);
    if (cm == 0ull) return;
    const uint64_t gm = ballot64(prod <= 0.99f) & cm;     // ... below the clamp
    const float oma = 1.0f - al;
    // T before the entry, T / (1 - a): only gradients use it, so a hardware reciprocal with
    // one Newton step (within an ulp) replaces the correctly rounded division.
    const float r0 = __builtin_amdgcn_rcpf(oma);
    const float Tk = T * fmaf_(fmaf_(-oma, r0, 1.0f), r0, r0);
    const float gc = fmaf_(g0c, c.z, fmaf_(g1c, c.w, g2c * bc.x));   // g . c_k
    const float dLda = Tk * (gc - gR);
    const float h = dLda * G, w = al * Tk;
    reinterpret_cast<float2*>(&S.hw[ng][(lane >> 1) ^ ng])[lane & 1u] =
        make_float2(__builtin_amdgcn_inverse_ballot_w64(gm) ? h : 0.f, __builtin_amdgcn_inverse_ballot_w64(cm) ? w : 0.f);
    slots |= (uint64_t)k << (8u * ng);
    ++ng;
    if (__builtin_amdgcn_inverse_ballot_w64(cm)) {
      gR = fmaf_(al, gc, oma * gR);   // R_{k-1} = c_k a_k + (1 - a_k) R_k, dotted with g
      T = Tk;
    }
  };

  // Batches of up to 64 entries, back to front: lane l's is the (d + 1)-th from the end, d = d0 + l.
  // One register set: a batch's records are staged, the next one's requested (their indices are
  // there already) and the staged entries walked while they arrive.
  const uint32_t end = rg.x + m;
  auto index_at = [&](uint32_t d) {
    const uint32_t f = svals[end - 1u - (d < m ? d : m - 1u)];
    return (int64_t)f < VN ? f : 0u;   // defensive: the sort only emits indices < V*n
  };
  uint32_t f = index_at(lane), fn = index_at(64u + lane);
  float4 g0 = rec[kRecQuads * (int64_t)f], g1 = rec[kRecQuads * (int64_t)f + 1], g2 = rec[kRecQuads * (int64_t)f + 2];
  for (uint32_t d0 = 0; d0 < m; d0 += 64) {
    const uint32_t d = d0 + lane;
    bool rel = false;
    float cut = 0.0f;
    if (d < m) {
      cut = entry_cut(g0.z);
      rel = block_reached<8>(g0.x, g0.y, g1.x, g1.y, g1.z, g0.w, cut, fqx, fqy) != 0u;
    }
    const uint64_t mask = ballot64(rel);
    const uint32_t n = (uint32_t)__builtin_popcountll(mask);
    if (kCount) n_walk += 64ull * n;
    if (rel) {
      const uint32_t slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      S.s0[slot] = make_float4(g0.x, g0.y, -0.5f * g1.x, -g1.y);
      S.s1[slot] = make_float4(-0.5f * g1.z, g0.z, g2.x, g2.y);
      S.s2[slot] = make_float4(g2.z, cut, __uint_as_float(m - 1u - d), __uint_as_float(f));
    }
    if ((n & 1u) && lane == 63u) {   // the walk takes two at a time: an entry no pixel is live for
      S.s0[n] = make_float4(__builtin_nanf(""), __builtin_nanf(""), 0.0f, 0.0f);
      S.s2[n] = make_float4(0.0f, __builtin_inff(), 0.0f, 0.0f);
    }
    lds_fence();
    f = fn;
    g0 = rec[kRecQuads * (int64_t)f];
    g1 = rec[kRecQuads * (int64_t)f + 1];
    g2 = rec[kRecQuads * (int64_t)f + 2];
    fn = index_at(d + 128u);
    float4 a0 = S.s0[0], c0 = S.s1[0], b0 = S.s2[0];
    for (uint32_t k = 0; k < n; k += 2) {
      const float4 a1 = S.s0[k + 1u], c1 = S.s1[k + 1u], b1 = S.s2[k + 1u];
      pair(k, a0, c0, b0);
      const uint32_t k2 = k + 2u < 63u ? k + 2u : 63u;
      a0 = S.s0[k2]; c0 = S.s1[k2]; b0 = S.s2[k2];
      pair(k + 1u, a1, c1, b1);
      if (ng >= kGradGroup - 1u || (k + 2u >= n && ng > 0u)) {   // no room for two more, or the slots end
        reduce(ng);
        ng = 0;
        slots = 0;
      }
    }
    lds_fence();
  }
  if (kCount && lane == 0) {
    atomicAdd(pair_part + 3 * (int64_t)tile_i, n_walk);
    atomicAdd(pair_part + 3 * (int64_t)tile_i + 1, n_live);
    atomicAdd(pair_part + 3 * (int64_t)tile_i + 2, n_contrib);
  }
}

hipError_t launch_blend_bwd(const Layout& L, void* ws, const uint32_t* sorted_vals, clod_params prm,
                            const float* T, const uint32_t* last, const float* dL_drgb, int64_t* pairs,
                            hipStream_t s) {
  if (L.tiles_total == 0) return hipSuccess;
  char* w = (char*)ws;
  const uint32_t nb = xcd_grid(L.tiles_total);
  unsigned long long* part = pairs ? (unsigned long long*)(w + L.pair_part) : nullptr;
  if (part) {
    hipError_t e = launch_fill_u32((uint32_t*)part, 0u, 6 * (int64_t)L.tiles_total, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(part ? k_blend_bwd<true> : k_blend_bwd<false>, dim3(nb), dim3(kBlock), 0, s,
                     (const DevView*)(w + L.vinfo), L.V, L.tiles_total, L.VN, (const float4*)(w + L.rec),
                     (const uint2*)(w + L.ranges), sorted_vals, (const unsigned long long*)(w + L.hdr), prm.bg[0],
                     prm.bg[1], prm.bg[2], T, last, dL_drgb, (float*)(w + L.gscreen), (const uint32_t*)(w + L.order),
                     part);
  if (part)
    hipLaunchKernelGGL(k_reduce_pairs, dim3(1), dim3(kBlock), 0, s,
                       ReducePairsArgs{(const unsigned long long*)part, L.tiles_total, (unsigned long long*)pairs});
  return hipGetLastError();
}

}  // namespace clod
