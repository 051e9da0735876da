// Binning of frames of ordinary size (Sec. 3.1, splats sorted by depth per tile), and the depth
// sort that every binning starts with.
//
//   depth sort   the rendered (view, Gaussian) records, compacted from the flag plane in index
//                order and sorted stably by bits(depth) in three radix passes; the compaction also
//                sums the tile pairs D, so an overflow of the pair buffer is known before the sort;
//   rows         in depth order, one (record, tile row) pair per row of the record's rectangle,
//                partitioned stably by tile row of the batch (one radix pass fused with the
//                expansion);
//   columns      per tile row, each pair's tiles partitioned stably by column (again fused with
//                the expansion), straight into the final lists.
//
// Splitting the tile id into (row, column) moves D / (tiles per row of a rectangle) elements
// through the first pass instead of D, and the pairs themselves are written once, in place.  The
// result is the stable order of the keys (tile << 32 | bits(depth)) emitted per record in index
// order, as that of the general path in sort.hip, which takes over behind the depth sort for
// batches of more than kRowBinsMax tile rows or frames beyond 256 x 256 tiles.
//
// Radix passes.  Each wave owns a contiguous chunk of the input and works on its own: it counts
// its digits in a row of LDS counters (up), and ranks and scatters its elements behind running
// positions of its own (down), 64 at a time, without a block barrier inside the loop.  A pass is
// two launches: the up kernel stores one row of counts per wave and adds its block's counts to a
// sum per group of kGroup blocks; every down block adds up the groups before it and the rows
// before it in its group, so no scan kernel runs between the two.  The passes are bound by
// launch latency and by the scatter's transactions, not by bandwidth: consecutive chunks are
// placed on one XCD, so that the neighbouring short writes of a digit meet in one L2.
//
// Measured on one MI355X, kernel time of the whole binning per pass, against compaction, a depth
// sort of four 8-bit reduce-then-scan passes, emission of all pairs and two or three such passes
// over them (23 to 26 launches; now 13):
//   one 256 x 256 view, 10k Gaussians (3.3k records, 15k pairs)        118 -> 68 us
//   one 1080p view, 3M (158k records, 2.4M pairs)                      220 -> 110 us
//   five 1080p LoD frames, 3M (301k records, 4.7M pairs)               280 -> 155 us
//   six views of 720p to 4K, 3M (1.1M records, 9.9M pairs)             480 -> 275 us
//   16 training views, 2M (1.5M records, 20.9M pairs)                 1020 -> 450 us
// What bounds it now is the latency of a dozen dependent launches on the small ones, and the
// row and column scatters on the large ones.
#include "clod_internal.h"

namespace clod {

// ------------------------------------------------------------------------------- wave helpers
// Inclusive scan over the 64 lanes (DPP shifts within rows, then the two row broadcasts).
__device__ __forceinline__ uint32_t wave_scan_inc(uint32_t v) {
  auto step = [&](uint32_t moved) { v += moved; };
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true));   // row_shr:1
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true));   // row_shr:2
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true));   // row_shr:4
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true));   // row_shr:8
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return v;
}
__device__ __forceinline__ uint32_t wave_last(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

// LDS written by some lanes of this wave is read by others next.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lanes of `active` whose digit (its low kBits bits; higher bits are zero) equals this lane's.
template <int kBits>
__device__ __forceinline__ uint64_t match_bits(uint32_t d, uint64_t active) {
  uint64_t m = active;
#pragma unroll
  for (int b = 0; b < kBits; ++b) {
    const uint64_t bal = ballot64((d >> b) & 1u);
    m &= ((d >> b) & 1u) ? bal : ~bal;
  }
  return m;
}

// Position of this lane's element among the elements of its digit: the running position of the
// digit (LDS, owned by the wave) plus the lower lanes with the same digit; the running position
// moves on.  Inactive lanes return an unspecified value.
template <int kBits>
__device__ __forceinline__ uint32_t wave_rank(uint32_t* running, uint32_t d, bool valid, uint64_t lt) {
  const uint64_t m = match_bits<kBits>(d, ballot64(valid));
  uint32_t before = 0;
  if (valid) {
    before = running[d];
    const uint32_t r = (uint32_t)__popcll(m & lt);
    if (r == 0u) running[d] = before + (uint32_t)__popcll(m);
    before += r;
  }
  __builtin_amdgcn_wave_barrier();
  return before;
}

// Expansion of the wave's items into consecutive outputs: lane l's item has `len` outputs (valid
// items have at least one and come first).  body(p, ok, o) is called for 64 outputs at a time,
// lane-parallel: p is the lane's output among the wave's, ok whether it exists, o the lane that
// owns it.  The owners come from one bit per output in LDS (set where an item starts): the items
// before an output are the start bits up to it.  bits: 2 * ceil(total / 64) words of the wave's.
template <class F>
__device__ __forceinline__ void wave_expand(uint32_t off, uint32_t len, uint32_t total, uint32_t* bits, F&& body) {
  const uint32_t lane = lane_id();
  const uint32_t words = 2u * ((total + 63u) >> 6);
  for (uint32_t i = lane; i < words; i += 64) bits[i] = 0u;
  wave_lds_fence();
  if (len) atomicOr(&bits[off >> 5], 1u << (off & 31u));
  wave_lds_fence();
  uint32_t cnt = 0;
  for (uint32_t p0 = 0; p0 < total; p0 += 64) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)bits[p0 >> 5]);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)bits[(p0 >> 5) + 1]);
    // Start bits of the outputs up to and including the lane's, less one.
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    const uint32_t own = lane < 32u ? (lo >> lane) & 1u : (hi >> (lane - 32u)) & 1u;
    const uint32_t p = p0 + lane;
    body(p, p < total, (int)((cnt + below + own - 1u) & 63u));
    cnt += (uint32_t)__popc(lo) + (uint32_t)__popc(hi);
  }
  wave_lds_fence();
}

// ------------------------------------------------------------------------------ radix geometry
// Chunk of a block: consecutive chunks lie on one XCD (blocks go round-robin to the eight XCDs).
// A block without one gets an index of nb or more.
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t b, uint32_t nb) {
  const uint32_t per = (nb + 7u) / 8u, j = b / 8u;
  const uint32_t c = (b % 8u) * per + j;
  return j < per ? c : nb;
}

// Stores the counts of chunk c's waves, summed up over the waves (row w: waves 0 .. w), and adds
// the block's counts to its group's.
__device__ __forceinline__ void store_counts(const uint32_t* cnt, uint32_t stride, uint32_t bins, uint32_t c,
                                             uint32_t* __restrict__ hist, uint32_t* __restrict__ gsum) {
  uint32_t* row = hist + (size_t)c * 4 * bins;
  uint32_t* g = gsum + (size_t)(c / kGroup) * bins;
  for (uint32_t d = threadIdx.x; d < bins; d += kBlock) {
    uint32_t s = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      s += cnt[w * stride + d];
      row[w * bins + d] = s;
    }
    if (s) atomicAdd(&g[d], s);
  }
}

template <int kPer>
struct Digits {
  uint32_t v[kPer];
};
template <int kPer>
__device__ __forceinline__ Digits<kPer> load_digits(const uint32_t* __restrict__ row) {
  Digits<kPer> r;
  if constexpr (kPer == 1) {
    r.v[0] = row[0];
  } else if constexpr (kPer == 2) {
    const uint2 q = *reinterpret_cast<const uint2*>(row);
    r.v[0] = q.x; r.v[1] = q.y;
  } else {
#pragma unroll
    for (int k = 0; k < kPer; k += 4) {
      const uint4 q = *reinterpret_cast<const uint4*>(row + k);
      r.v[k] = q.x; r.v[k + 1] = q.y; r.v[k + 2] = q.z; r.v[k + 3] = q.w;
    }
  }
  return r;
}

// First output position of every digit for each of chunk c's four waves, into running[w * bins +
// d], with bins = 256 kPer.  Thread t takes the kPer digits from t kPer: their totals (tot) and
// first positions (base); returns the number of elements.  The rows are read eight at a time
// (the last one again past the end, not added), so that a block waits for a few loads in a row
// and not for every group and row before it.
template <int kPer>
__device__ __forceinline__ uint32_t load_starts(uint32_t* running, uint32_t c, uint32_t nb,
                                                const uint32_t* __restrict__ hist, const uint32_t* __restrict__ gsum,
                                                uint32_t* sm, uint32_t (&tot)[kPer], uint32_t (&base)[kPer]) {
  constexpr uint32_t bins = kPer * kBlock;
  constexpr uint32_t kRows = 8;
  const uint32_t d0 = threadIdx.x * kPer;
  const uint32_t ng = (nb + kGroup - 1) / kGroup, mg = c / kGroup;
  uint32_t pre[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) tot[k] = pre[k] = 0u;
  for (uint32_t g0 = 0; g0 < ng; g0 += kRows) {
    Digits<kPer> q[kRows];
#pragma unroll
    for (uint32_t j = 0; j < kRows; ++j) q[j] = load_digits<kPer>(gsum + (size_t)min(g0 + j, ng - 1u) * bins + d0);
#pragma unroll
    for (uint32_t j = 0; j < kRows; ++j)
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        tot[k] += g0 + j < ng ? q[j].v[k] : 0u;
        pre[k] += g0 + j < mg ? q[j].v[k] : 0u;
      }
  }
  // Blocks of the group before this one (the last row of each), and the waves of this block.
  const uint32_t b0 = mg * kGroup;
  for (uint32_t r0 = b0; r0 < c; r0 += kRows) {
    Digits<kPer> q[kRows];
#pragma unroll
    for (uint32_t j = 0; j < kRows; ++j) q[j] = load_digits<kPer>(hist + ((size_t)min(r0 + j, c - 1u) * 4 + 3) * bins + d0);
#pragma unroll
    for (uint32_t j = 0; j < kRows; ++j)
#pragma unroll
      for (int k = 0; k < kPer; ++k) pre[k] += r0 + j < c ? q[j].v[k] : 0u;
  }
  Digits<kPer> own[3];
#pragma unroll
  for (int w = 0; w < 3; ++w) own[w] = load_digits<kPer>(hist + ((size_t)c * 4 + w) * bins + d0);
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) s += tot[k];
  uint32_t total;
  uint32_t ex = block_exclusive_scan(s, sm, total);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    base[k] = ex;
    const uint32_t at = ex + pre[k];
    running[d0 + k] = at;
#pragma unroll
    for (int w = 0; w < 3; ++w) running[(w + 1) * bins + d0 + k] = at + own[w].v[k];
    ex += tot[k];
  }
  __syncthreads();
  return total;
}

// ---------------------------------------------------------------------------------- depth sort
// The rendered records are the (view, Gaussian) pairs whose flag byte has bit 2 set (the
// projection sets it exactly where it writes a record).  A lane takes 16 consecutive flags in one
// 16-byte load; the result is a mask, bit k = record j0 + k is rendered.
__device__ __forceinline__ uint32_t rendered_mask(const uint8_t* __restrict__ flags, int64_t count, int64_t j0) {
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  if (j0 + 16 <= count) {
    const uint4 q = *reinterpret_cast<const uint4*>(flags + j0);
    w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
  } else {
    for (int k = 0; k < 16 && j0 + k < count; ++k) w[k >> 2] |= (uint32_t)flags[j0 + k] << (8 * (k & 3));
  }
  uint32_t m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t b = (w[q] >> 2) & 0x01010101u;   // bit 2 of each byte, at bits 0, 8, 16, 24
    m |= ((b | (b >> 7) | (b >> 14) | (b >> 21)) & 0xFu) << (4 * q);
  }
  return m;
}

// Per chunk of kRecChunk flags: the rendered records, also added up per group of kRecGroup chunks
// (each sum on a line of its own: with the sums side by side the chunks' additions to the few
// shared lines took 34 us for 7,800 chunks).
// Clears the sums of the first radix pass and, for the general path, the tile ranges.
__device__ __forceinline__ void rec_count_body(const DepthArgs& a, Blk b) {
  __shared__ uint32_t sm[4];
  for (int64_t q = (int64_t)b.id * kBlock + threadIdx.x; q < a.range_words; q += (int64_t)b.n * kBlock) a.ranges[q] = 0u;
  zero_words(a.gnext, a.sums * kDepthBins0, b);
  const int64_t j0 = (int64_t)b.id * kRecChunk + 16 * (int64_t)threadIdx.x;
  const uint32_t r = wave_sum((uint32_t)__popc(rendered_mask(a.flags, a.VN, j0)));
  if (lane_id() == 0) sm[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t c = sm[0] + sm[1] + sm[2] + sm[3];
    a.part[b.id] = c;
    if (c) atomicAdd(&a.gcount[(b.id / kRecGroup) * kLineWords], c);
  }
}
__global__ __launch_bounds__(kBlock) void k_rec_count(DepthArgs a) { rec_count_body(a, grid_blk()); }

// The rendered records of a chunk, in index order, behind those of the chunks before it: key
// bits(depth) - bits(near), and the record.  Sums the chunk's tile pairs and finds its largest key.
// Records past the pair capacity are counted, not stored.
struct RecLds {
  uint32_t queue[kRecChunk];
};
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t x = __shfl_xor(v, o, 64);
    v = x > v ? x : v;
  }
  return v;
}
__device__ __forceinline__ void rec_compact_body(const DepthArgs& a, Blk b, RecLds& S) {
  __shared__ uint32_t sm[4];
  __shared__ unsigned long long sd[4];
  __shared__ float sq[4];
  const uint32_t t = threadIdx.x, w = t >> 6, lane = lane_id();
  const int64_t j0 = (int64_t)b.id * kRecChunk + 16 * (int64_t)t;
  uint32_t m = rendered_mask(a.flags, a.VN, j0);
  // Records of the groups, and of the chunks of this group, before this chunk.
  const uint32_t g = b.id / kRecGroup;
  uint32_t before = 0;
  for (uint32_t q = t; q < g; q += kBlock) before += a.gcount[q * kLineWords];
  for (uint32_t q = g * kRecGroup + t; q < b.id; q += kBlock) before += a.part[q];
  uint32_t out0, total;
  block_exclusive_scan(before, sm, out0);
  uint32_t o = block_exclusive_scan((uint32_t)__popc(m), sm, total);
  while (m) {
    S.queue[o++] = (uint32_t)j0 + (uint32_t)__builtin_ctz(m);
    m &= m - 1u;
  }
  __syncthreads();
  const uint32_t base = (uint32_t)a.hdr[kHdrKeyBase];
  unsigned long long pairs = 0;
  uint32_t kmax = 0;
  float squares = 0.f;
  for (uint32_t q0 = t; q0 < total; q0 += 4 * kBlock) {
    uint32_t f[4];
    float4 q3[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (q0 + j * kBlock < total) {
        f[j] = S.queue[q0 + j * kBlock];
        q3[j] = a.rec[kRecQuads * (int64_t)f[j] + 3];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t q = q0 + j * kBlock;
      if (q < total) {
        const uint32_t k = __float_as_uint(q3[j].x) - base;
        kmax = k > kmax ? k : kmax;
        const uint32_t tiles = __float_as_uint(q3[j].w);
        pairs += tiles;
        squares = fmaf_((float)tiles, (float)tiles, squares);
        if ((int64_t)out0 + q < a.cap) a.out[(size_t)out0 + q] = make_uint2(k, f[j]);
      }
    }
  }
  // One partial per chunk, summed up by the next stage: adding to a few shared words from every
  // chunk (7,800 of them for 16 views of 2M Gaussians) took 170 us instead of the time given above.
  pairs = wave_sum(pairs);
  kmax = wave_max(kmax);
  squares = wave_sum(squares);
  if (lane == 0) { sd[w] = pairs; sm[w] = kmax; sq[w] = squares; }
  __syncthreads();
  if (t == 0)
    a.stat[b.id] = DepthStat{sd[0] + sd[1] + sd[2] + sd[3], max(max(sm[0], sm[1]), max(sm[2], sm[3])),
                             sq[0] + sq[1] + sq[2] + sq[3]};
}
__global__ __launch_bounds__(kBlock) void k_rec_compact(DepthArgs a) {
  __shared__ RecLds S;
  rec_compact_body(a, grid_blk(), S);
}

struct RadixLds {
  uint32_t cnt[4 * kRowBinsMax];   // counts, then running positions
};

__device__ __forceinline__ int bit_length(uint32_t x) { return x ? 32 - __clz(x) : 0; }
// Width of a pass's digit for keys of `nbits` bits: the first takes kDepthBits0, the others share
// the rest (at least eight bits, the least number of bins a pass is made for, each).
__device__ __forceinline__ int depth_bits(int pass, int nbits) {
  if (pass == 0) return kDepthBits0;
  const int rem = nbits > kDepthBits0 ? nbits - kDepthBits0 : 0;
  const int w1 = (rem + 1) / 2 > 8 ? (rem + 1) / 2 : 8;
  if (pass == 1) return w1;
  return rem - w1 > 8 ? rem - w1 : 8;
}

// What a depth pass works on.  The first up kernel counts the records from the groups' sums, and
// its block 0 stores the header (pairs, overflow, records, key bits) that the kernels behind it
// read.
struct DepthState {
  uint32_t N;
  int nbits, bits, shift;
  bool over;
};
__device__ __forceinline__ DepthState depth_first(const DepthArgs& a, Blk b) {
  __shared__ unsigned long long sd[4];
  __shared__ uint32_t sk[4];
  __shared__ float sq[4];
  const uint32_t t = threadIdx.x, lane = lane_id();
  uint32_t R = 0;
  for (uint32_t g = lane; g < a.groups; g += 64) R += a.gcount[g * kLineWords];
  R = wave_sum(R);
  if (b.id == 0u) {
    unsigned long long D = 0;
    uint32_t kmax = 0;
    float squares = 0.f;
    for (uint32_t q0 = t; q0 < a.chunks; q0 += 4 * kBlock) {
      DepthStat q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j] = a.stat[min(q0 + j * kBlock, a.chunks - 1u)];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        D += q0 + j * kBlock < a.chunks ? q[j].pairs : 0ull;
        squares += q0 + j * kBlock < a.chunks ? q[j].squares : 0.f;
        kmax = q[j].kmax > kmax ? q[j].kmax : kmax;
      }
    }
    D = wave_sum(D);
    kmax = wave_max(kmax);
    squares = wave_sum(squares);
    if (lane == 0) { sd[t >> 6] = D; sk[t >> 6] = kmax; sq[t >> 6] = squares; }
    __syncthreads();
    if (t == 0) {
      D = sd[0] + sd[1] + sd[2] + sd[3];
      a.hdr[kHdrDup] = D;
      a.hdr[kHdrOverflow] = (int64_t)D > a.cap ? 1ull : 0ull;   // else R <= D <= cap: a record has a pair
      a.hdr[kHdrRend] = R;
      a.hdr[kHdrSquares] = (unsigned long long)((sq[0] + sq[1]) + (sq[2] + sq[3]));   // (R 2^40 at most)
      a.hdr[kHdrKeyBits] = (unsigned long long)bit_length(max(max(sk[0], sk[1]), max(sk[2], sk[3])));
    }
    zero_words(a.tord, a.tord_words, Blk{0u, 1u});
  }
  return DepthState{R, 0, kDepthBits0, 0, (int64_t)R > a.cap};
}
__device__ __forceinline__ DepthState depth_state(const DepthArgs& a) {
  DepthState s;
  s.over = a.hdr[kHdrOverflow] != 0ull;
  s.N = (uint32_t)a.hdr[kHdrRend];
  s.nbits = (int)a.hdr[kHdrKeyBits];
  s.bits = depth_bits(a.pass, s.nbits);
  s.shift = a.pass == 0 ? 0 : a.pass == 1 ? kDepthBits0 : kDepthBits0 + depth_bits(1, s.nbits);
  return s;
}

__device__ __forceinline__ void depth_up_body(const DepthArgs& a, Blk b, RadixLds& S) {
  const DepthState D = a.pass == 0 ? depth_first(a, b) : depth_state(a);
  if (D.over) return;
  const uint32_t bins = 1u << D.bits, N = D.N;
  const RadixGeom G = radix_geom(N, bins);
  const uint32_t c = xcd_chunk(b.id, G.nb);
  if (c >= G.nb) return;
  for (uint32_t i = threadIdx.x; i < 4 * bins; i += kBlock) S.cnt[i] = 0u;
  __syncthreads();
  const uint32_t w = threadIdx.x >> 6, lane = lane_id();
  const uint64_t lo = ((uint64_t)c * 4 + w) * G.kw, hi = lo + G.kw < N ? lo + G.kw : N;
  uint32_t* cnt = S.cnt + w * bins;
  for (uint64_t e0 = lo; e0 < hi; e0 += 256) {
    uint32_t k[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t e = e0 + 64u * j + lane;
      k[j] = e < hi ? a.in[e].x : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (e0 + 64u * j + lane < hi) atomicAdd(&cnt[(k[j] >> D.shift) & (bins - 1u)], 1u);
  }
  __syncthreads();
  store_counts(S.cnt, bins, bins, c, a.hist, a.gsum);
}
__global__ __launch_bounds__(kBlock) void k_depth_up(DepthArgs a) {
  __shared__ RadixLds S;
  depth_up_body(a, grid_blk(), S);
}

// The third pass stores the records in depth order with their tile rectangle packed in the key
// plane (x0 | x1 - 1 << 8 | y0 << 16 | y1 - 1 << 24), where the row path reads it.
template <int kBits>
__device__ __forceinline__ void depth_scatter(const DepthArgs& a, const DepthState& D, uint64_t lo, uint64_t hi,
                                              uint32_t* running) {
  const uint32_t lane = lane_id(), dm = (1u << D.bits) - 1u;
  const uint64_t lt = lanemask_lt();
  for (uint64_t e0 = lo; e0 < hi; e0 += 256) {
    uint2 e[4];
    uint32_t r[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t q = e0 + 64u * j + lane;
      e[j] = q < hi ? a.in[q] : make_uint2(0u, 0u);
    }
    if (a.pass == 2 && a.row_bins) {
      float4 q3[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) q3[j] = a.rec[kRecQuads * (int64_t)e[j].y + 3];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t rx = __float_as_uint(q3[j].y), ry = __float_as_uint(q3[j].z);
        r[j] = (rx & 0xFFu) | (((rx >> 16) - 1u) & 0xFFu) << 8 | (ry & 0xFFu) << 16 | (((ry >> 16) - 1u) & 0xFFu) << 24;
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool valid = e0 + 64u * j + lane < hi;
      const uint32_t pos = wave_rank<kBits>(running, (e[j].x >> D.shift) & dm, valid, lt);
      if (valid && pos < D.N) {
        if (a.pass < 2) {
          a.out[pos] = e[j];
        } else {
          a.kout[pos] = r[j];
          a.vout[pos] = e[j].y;
        }
      }
    }
  }
}

__device__ __forceinline__ void depth_down_body(const DepthArgs& a, Blk b, RadixLds& S) {
  __shared__ uint32_t sm[4];
  const DepthState D = depth_state(a);
  if (D.over) return;
  if (a.gnext) zero_words(a.gnext, a.sums * (a.pass == 2 ? a.row_bins : 1u << depth_bits(a.pass + 1, D.nbits)), b);
  const uint32_t bins = 1u << D.bits, N = D.N;
  const RadixGeom G = radix_geom(N, bins);
  const uint32_t c = xcd_chunk(b.id, G.nb);
  if (c >= G.nb) return;
  uint32_t t1[1], b1[1], t2[2], b2[2], t4[4], b4[4], t8[8], b8[8];
  switch (D.bits) {
    case 8: load_starts<1>(S.cnt, c, G.nb, a.hist, a.gsum, sm, t1, b1); break;
    case 9: load_starts<2>(S.cnt, c, G.nb, a.hist, a.gsum, sm, t2, b2); break;
    case 10: load_starts<4>(S.cnt, c, G.nb, a.hist, a.gsum, sm, t4, b4); break;
    default: load_starts<8>(S.cnt, c, G.nb, a.hist, a.gsum, sm, t8, b8); break;
  }
  const uint32_t w = threadIdx.x >> 6;
  const uint64_t lo = ((uint64_t)c * 4 + w) * G.kw, hi = lo + G.kw < N ? lo + G.kw : N;
  if (D.bits <= 9) depth_scatter<9>(a, D, lo, hi, S.cnt + w * bins);
  else depth_scatter<11>(a, D, lo, hi, S.cnt + w * bins);
}
__global__ __launch_bounds__(kBlock) void k_depth_down(DepthArgs a) {
  __shared__ RadixLds S;
  depth_down_body(a, grid_blk(), S);
}

// -------------------------------------------------------------------------------------- rows
// Tile rows are numbered through the batch (row_base of the view + row of the view).
// Dynamic LDS of the row kernels: the waves' counts or running positions (4 (bins + 1) words),
// then each wave's expansion start bits (64 records x 256 rows); sized by the batch's rows, so that
// an ordinary batch keeps many blocks on a CU.
constexpr uint32_t kRowBitWords = 64 * kColsMax / 32;
__host__ __device__ constexpr uint32_t row_lds_words(uint32_t bins) { return 4 * (bins + 1) + 4 * kRowBitWords; }

// A depth-sorted record: its first tile row, rows and columns.
struct RowRec {
  uint32_t row0, rows, xx;   // xx: x0 | x1 - 1 << 8
};
__device__ __forceinline__ RowRec row_rec(const RowArgs& a, uint32_t rect, uint32_t f) {
  // The view f / n, from the reciprocal (off by at most one: fewer than 2^11 views) and corrected.
  const uint32_t n = (uint32_t)a.n;
  uint32_t v = 0;
  if (a.V > 1) {
    v = (uint32_t)((float)f * a.inv_n);
    const int64_t rem = (int64_t)f - (int64_t)v * n;
    v = rem < 0 ? v - 1u : rem >= (int64_t)n ? v + 1u : v;
  }
  const uint32_t y0 = (rect >> 16) & 0xFFu, y1 = rect >> 24;
  return RowRec{a.views[v].row_base + y0, y1 - y0 + 1u, rect & 0xFFFFu};
}

// Records per wave of the row kernels.  (3,000 records of 68 rows each were twelve waves' work: 111 us
// for k_row_down, now 32; 200,000 of 13 rows 71 us, now 30.)
__device__ __forceinline__ RadixGeom row_geom(const RowArgs& a, uint32_t N) {
  return radix_geom(N, a.bins, a.hdr[kHdrDup] >= (uint64_t)kWideTiles * N ? kWaveMinWide : kWaveMin);
}

// First record of wave k of the row kernels.  The work is a record's rows, and the records come by
// depth: the nearest cover tens of rows each, the others two or three, and of equal shares the first
// set the time of the scatter.  So in large batches wave k of K starts at N f(k / K), in steps of 64,
// with f(x) = x (1 + 3 x) / 4, a quarter of the records for the first waves and 1.75 times as many
// for the last: 16 training views (1.5M records of 14 tiles on average) 163 -> 79 us, six views of
// 720p to 4K (1.1M of 9) 47 -> 36 us.  (x (1 + x) / 2: 107 and 36, x^2: 66 and 38 us.)  Where the
// records are small their rows are even, and the longer last shares only cost (five LoD frames, 1.15M
// of 6 tiles: 32 -> 38 us); so do they where shares are no longer than kWaveMin, which leaves the
// chip waves to spare (a far frame of 6M 25 -> 31 us, one training view 16 -> 18): equal shares.
__device__ __forceinline__ uint64_t row_chunk(const RowArgs& a, uint32_t N, const RadixGeom& G, uint32_t k) {
  const uint64_t K = 4u * G.nb;
  if (k >= K) return N;
  const bool uneven = G.kw > kWaveMin && a.hdr[kHdrDup] >= 8ull * N;
  const uint64_t at = uneven ? ((uint64_t)N * (k * (K + 3u * k)) / (4u * K * K)) & ~63ull : (uint64_t)G.kw * k;
  return at < N ? at : N;
}

// Pairs per row: a record adds one to every row of its rectangle, as +1 at the first and -1 past
// the last, summed up over the rows afterwards.
__device__ __forceinline__ void row_up_body(const RowArgs& a, Blk b, uint32_t* lds) {
  if (a.hdr[kHdrOverflow]) return;
  const uint32_t N = (uint32_t)a.hdr[kHdrRend], bins = a.bins;
  const RadixGeom G = row_geom(a, N);
  const uint32_t c = xcd_chunk(b.id, G.nb);
  if (c >= G.nb) return;
  const uint32_t stride = bins + 1u;
  for (uint32_t i = threadIdx.x; i < 4 * stride; i += kBlock) lds[i] = 0u;
  __syncthreads();
  const uint32_t w = threadIdx.x >> 6, lane = lane_id();
  const uint64_t lo = row_chunk(a, N, G, 4 * c + w), hi = row_chunk(a, N, G, 4 * c + w + 1);
  uint32_t* cnt = lds + w * stride;
  for (uint64_t e0 = lo; e0 < hi; e0 += 256) {
    uint32_t q[4], f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t e = min(e0 + 64u * j + lane, hi - 1);
      q[j] = a.rect[e];
      f[j] = a.f[e];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (e0 + 64u * j + lane < hi) {
        const RowRec r = row_rec(a, q[j], f[j]);
        atomicAdd(&cnt[r.row0], 1u);
        atomicAdd(&cnt[r.row0 + r.rows], 0xFFFFFFFFu);
      }
    }
  }
  wave_lds_fence();
  uint32_t carry = 0;
  for (uint32_t d = lane; d < bins; d += 64) {
    const uint32_t inc = wave_scan_inc(cnt[d]) + carry;
    cnt[d] = inc;
    carry = wave_last(inc);
  }
  __syncthreads();
  store_counts(lds, stride, bins, c, a.hist, a.gsum);
}
__global__ __launch_bounds__(kBlock) void k_row_up(RowArgs a) {
  extern __shared__ uint32_t row_lds[];
  row_up_body(a, grid_blk(), row_lds);
}

// Starting positions of the block, and (the first block) the row tables: per row its first pair,
// its first tile and its column units (kUnit pairs or a multiple).  Returns the number of pairs.
template <int kPer>
__device__ __forceinline__ uint32_t row_starts(const RowArgs& a, uint32_t c, uint32_t nb, uint32_t* lds, uint32_t* sm) {
  uint32_t tot[kPer], first[kPer];
  const uint32_t total = load_starts<kPer>(lds, c, nb, a.hist, a.gsum, sm, tot, first);
  if (c != 0u) return total;
  const uint32_t rows = a.rows, d0 = threadIdx.x * kPer;
  const uint32_t room = a.units_max - rows;   // units of full length that fit
  const uint32_t unit = unit_pairs(total, room);
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) s += ceil_div(tot[k], unit);
  uint32_t units;
  uint32_t u = block_exclusive_scan(s, sm, units);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t r = d0 + k;
    if (r < rows) {
      int lo = 0, hi = a.V - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.views[mid].row_base <= r) lo = mid; else hi = mid - 1;
      }
      const DevView& Vw = a.views[lo];
      a.tab.tile[r] = Vw.tile_base + (r - Vw.row_base) * (uint32_t)Vw.tiles_x;
      a.tab.start[r] = first[k];
      a.tab.ustart[r] = u;
      a.tab.pairs[r] = 0u;
      // (The sum of the units fits units_max.  The bound stands outside the loop: one in it, which
      // kept the stores from being unrolled, cost a far frame of 6M 19 us.)
      const uint32_t nu = min(ceil_div(tot[k], unit), a.units_max - min(u, a.units_max));
      for (uint32_t j = 0; j < nu; ++j) a.tab.urow[u + j] = r;
      u += nu;
    }
  }
  if (threadIdx.x == 0) {
    a.tab.tile[rows] = a.tiles_total;
    a.tab.start[rows] = total;
    a.tab.ustart[rows] = units;
    a.hdr[kHdrUnit] = unit;
    a.hdr[kHdrUnits] = units;
  }
  return total;
}

// Scatters the wave's (record, row) pairs to their rows.
template <int kBits>
__device__ __forceinline__ void row_scatter(const RowArgs& a, uint64_t lo, uint64_t hi, uint32_t total,
                                            uint32_t* running, uint32_t* bits) {
  const uint32_t lane = lane_id();
  const uint64_t lt = lanemask_lt();
  if (lo >= hi) return;
  // The records of the next step are read before this step's pairs are made.
  uint32_t q = a.rect[min(lo + lane, hi - 1)], f = a.f[min(lo + lane, hi - 1)];
  for (uint64_t e0 = lo; e0 < hi; e0 += 64) {
    const uint32_t cq = q, cf = f;
    q = a.rect[min(e0 + 64 + lane, hi - 1)];
    f = a.f[min(e0 + 64 + lane, hi - 1)];
    const RowRec r = row_rec(a, cq, cf);
    const uint32_t len = e0 + lane < hi ? r.rows : 0u;
    const uint32_t inc = wave_scan_inc(len), off = inc - len;
    const uint32_t rel = r.row0 - off;
    wave_expand(off, len, wave_last(inc), bits, [&](uint32_t p, bool ok, int o) {
      const uint32_t row = (uint32_t)__shfl((int)rel, o, 64) + p;
      const uint32_t of = (uint32_t)__shfl((int)cf, o, 64), ox = (uint32_t)__shfl((int)r.xx, o, 64);
      const uint32_t pos = wave_rank<kBits>(running, row, ok, lt);
      if (ok && pos < total) a.out[pos] = make_uint2(of, ox);
    });
  }
}

__device__ __forceinline__ void row_down_body(const RowArgs& a, Blk b, uint32_t* lds) {
  __shared__ uint32_t sm[4];
  if (a.hdr[kHdrOverflow]) return;
  const uint32_t N = (uint32_t)a.hdr[kHdrRend], bins = a.bins;
  const RadixGeom G = row_geom(a, N);
  const uint32_t c = xcd_chunk(b.id, G.nb > 0u ? G.nb : 1u);
  if (c >= G.nb && c != 0u) return;
  uint32_t total;
  if (bins == kBlock) total = row_starts<1>(a, c, G.nb, lds, sm);
  else if (bins == 2 * kBlock) total = row_starts<2>(a, c, G.nb, lds, sm);
  else if (bins == 4 * kBlock) total = row_starts<4>(a, c, G.nb, lds, sm);
  else total = row_starts<8>(a, c, G.nb, lds, sm);
  const uint32_t w = threadIdx.x >> 6;
  const uint64_t lo = row_chunk(a, N, G, 4 * c + w), hi = row_chunk(a, N, G, 4 * c + w + 1);
  uint32_t* bits = lds + 4 * (bins + 1) + w * kRowBitWords;
  if (bins <= 2 * kBlock) row_scatter<9>(a, lo, hi, total, lds + w * bins, bits);
  else row_scatter<11>(a, lo, hi, total, lds + w * bins, bits);
}
__global__ __launch_bounds__(kBlock) void k_row_down(RowArgs a) {
  extern __shared__ uint32_t row_lds[];
  row_down_body(a, grid_blk(), row_lds);
}

// ----------------------------------------------------------------------------------- columns
// A unit is a run of `count` consecutive pairs of one tile row.  (The loops below count from its first
// pair: positions near 2^32 would wrap past the run's end.)
struct Unit {
  uint32_t row, lo, count;
  bool first;   // of its row
};
__device__ __forceinline__ Unit unit_of(const ColArgs& a, uint32_t u) {
  const uint32_t row = a.tab.urow[u], len = (uint32_t)a.hdr[kHdrUnit];
  const uint32_t j = u - a.tab.ustart[row], s = a.tab.start[row], e = a.tab.start[row + 1];
  const uint32_t lo = s + j * len;   // (below e)
  return Unit{row, lo, min(e - lo, len), j == 0u};
}

// Per unit: pairs per column (+1 at the first column, -1 past the last, summed up).
__device__ __forceinline__ void col_up_body(const ColArgs& a, Blk b) {
  __shared__ uint32_t cnt[kColsMax + 1];
  __shared__ uint32_t sm[4];
  if (a.hdr[kHdrOverflow] || b.id >= (uint32_t)a.hdr[kHdrUnits]) return;
  const Unit U = unit_of(a, b.id);
  cnt[threadIdx.x] = 0u;
  if (threadIdx.x == 0) cnt[kColsMax] = 0u;
  __syncthreads();
  for (uint32_t o0 = 0; o0 < U.count; o0 += 2 * kBlock) {
    uint32_t x[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t o = o0 + j * kBlock + threadIdx.x;
      x[j] = o < U.count ? a.in[U.lo + o].y : 0u;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (o0 + j * kBlock + threadIdx.x < U.count) {
        atomicAdd(&cnt[x[j] & 0xFFu], 1u);
        atomicAdd(&cnt[(x[j] >> 8) + 1u], 0xFFFFFFFFu);
      }
    }
  }
  __syncthreads();
  const uint32_t v = cnt[threadIdx.x];
  uint32_t total;
  const uint32_t ex = block_exclusive_scan(v, sm, total);
  if (threadIdx.x < a.cols) a.hist[(size_t)b.id * a.cols + threadIdx.x] = ex + v;
}
__global__ __launch_bounds__(kBlock) void k_col_up(ColArgs a) { col_up_body(a, grid_blk()); }

// Block (row, 64 columns): the units' counts become exclusive prefixes over the row's units, one
// wave per quarter of them; the tile totals go to tcount, empty tiles get an empty range, and
// the totals' length classes are counted for the tile order (one copy of the counters per
// kOrderCopies blocks: the blocks finish together and would queue on one line).
__device__ __forceinline__ void col_scan_body(const ColArgs& a, Blk b) {
  __shared__ uint32_t sums[4][64];
  __shared__ uint32_t buckets[kTileBuckets];
  const uint32_t w = threadIdx.x >> 6, lane = lane_id();
  if (a.hdr[kHdrOverflow]) {
    for (uint32_t t = b.id * kBlock + threadIdx.x; t < a.tiles_total; t += b.n * kBlock) {
      a.tcount[t] = 0u;
      a.ranges[t] = make_uint2(0u, 0u);
    }
    if (b.id == 0 && threadIdx.x == 0) a.tordc[0] = a.tiles_total;
    return;
  }
  const uint32_t groups = a.cols / 64u;
  const uint32_t row = b.id / groups, col = (b.id % groups) * 64u + lane;
  const uint32_t t0 = a.tab.tile[row], width = a.tab.tile[row + 1] - t0;
  if ((b.id % groups) * 64u >= width) return;
  if (threadIdx.x < kTileBuckets) buckets[threadIdx.x] = 0u;
  const uint32_t u0 = a.tab.ustart[row], nu = a.tab.ustart[row + 1] - u0;
  const uint32_t q0 = u0 + (uint32_t)((uint64_t)nu * w / 4u), q1 = u0 + (uint32_t)((uint64_t)nu * (w + 1u) / 4u);
  uint32_t* __restrict__ h = a.hist + col;
  uint32_t s = 0;
#pragma unroll 8
  for (uint32_t u = q0; u < q1; ++u) s += h[(size_t)u * a.cols];
  sums[w][lane] = s;
  __syncthreads();
  uint32_t pre = 0, total = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) {
    pre += j < w ? sums[j][lane] : 0u;
    total += sums[j][lane];
  }
  for (uint32_t u = q0; u < q1; u += 8) {
    uint32_t v[8];
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) v[j] = u + j < q1 ? h[(size_t)(u + j) * a.cols] : 0u;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      if (u + j < q1) h[(size_t)(u + j) * a.cols] = pre;
      pre += v[j];
    }
  }
  if (w == 0u) {
    const bool in = col < width;
    if (in) {
      a.tcount[t0 + col] = total;
      if (total == 0u) a.ranges[t0 + col] = make_uint2(0u, 0u);
      atomicAdd(&buckets[bit_length(total)], 1u);
    }
    const uint32_t all = wave_sum(in ? total : 0u);
    if (lane == 0 && all) atomicAdd(&a.tab.pairs[row], all);
  }
  __syncthreads();
  if (threadIdx.x < kTileBuckets && buckets[threadIdx.x])
    atomicAdd(&a.tordc[(b.id % kOrderCopies) * kTileBuckets + threadIdx.x], buckets[threadIdx.x]);
}
__global__ __launch_bounds__(kBlock) void k_col_scan(ColArgs a) { col_scan_body(a, grid_blk()); }

// Sub-unit of 512 row pairs: each wave owns 128 of them, counts its columns, and places its tile
// pairs (record, column) in LDS ordered by column; the block then stores each column's run to its
// list, so that a store instruction covers a few runs instead of 64 separate words.  A sub-unit
// of more than kStagePairs tile pairs (wide rectangles) is taken in parts that fit, down to
// kLeastPart row pairs (which always do); the next sub-units start with parts of that size and
// go back to larger ones where a part is less than half full.  (Stored from the ranks directly, word
// by word, 3,000 Gaussians over the whole of a 1080p frame took 338 us instead of 185, and 200,000
// of 209 tiles each 366 instead of 217.)
constexpr uint32_t kSubUnit = 512, kStagePairs = 4096, kLeastPart = kStagePairs / kColsMax;
struct ColLds {
  uint32_t base[kColsMax];              // next output position per column
  uint32_t lstart[kColsMax];            // first place in the stage per column
  uint32_t cnt[4][kColsMax + 1];        // per wave: counts, then places
  uint32_t bits[4][512];
  uint32_t sf[kStagePairs];
  uint8_t scol[kStagePairs];
};
__device__ __forceinline__ void col_down_unit(const ColArgs& a, uint32_t u, ColLds& S) {
  __shared__ uint32_t sm[4];
  const Unit U = unit_of(a, u);
  const uint32_t t = threadIdx.x, w = t >> 6, lane = lane_id();
  const uint32_t tile0 = a.tab.tile[U.row], width = a.tab.tile[U.row + 1] - tile0;
  // First position of the row: the pairs of the rows before it.
  uint32_t before = 0;
  for (uint32_t r = t; r < U.row; r += kBlock) before += a.tab.pairs[r];
  uint32_t row0;
  block_exclusive_scan(before, sm, row0);
  const uint32_t mine = t < width ? a.tcount[tile0 + t] : 0u;
  const uint32_t pre = t < a.cols ? a.hist[(size_t)u * a.cols + t] : 0u;
  uint32_t all;
  const uint32_t at = row0 + block_exclusive_scan(mine, sm, all);
  S.base[t] = at + pre;
  if (U.first && t < width && mine) a.ranges[tile0 + t] = make_uint2(at, at + mine);
  const uint32_t D = (uint32_t)a.hdr[kHdrDup];
  const uint64_t lt = lanemask_lt();
  uint32_t part = kSubUnit;
  for (uint32_t o0 = 0; o0 < U.count;) {
    // The part's pairs: wave w the part / 4 from o0 + part / 4 w.
    const uint32_t wo = o0 + part / 4u * w, wn = min(part / 4u, U.count > wo ? U.count - wo : 0u);
    uint2 rp[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) rp[j] = 64u * j + lane < wn ? a.in[U.lo + wo + 64u * j + lane] : make_uint2(0u, 0u);
    uint32_t* cnt = S.cnt[w];
    for (uint32_t i = lane; i <= kColsMax; i += 64) cnt[i] = 0u;
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (64u * j + lane < wn) {
        atomicAdd(&cnt[rp[j].y & 0xFFu], 1u);
        atomicAdd(&cnt[(rp[j].y >> 8) + 1u], 0xFFFFFFFFu);
      }
    }
    wave_lds_fence();
    uint32_t carry = 0;
    for (uint32_t d = lane; d < a.cols; d += 64) {
      const uint32_t inc = wave_scan_inc(cnt[d]) + carry;
      cnt[d] = inc;
      carry = wave_last(inc);
    }
    __syncthreads();
    uint32_t c4[4], run = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c4[q] = t < a.cols ? S.cnt[q][t] : 0u;
      run += c4[q];
    }
    uint32_t total;
    uint32_t place = block_exclusive_scan(run, sm, total);
    if (total > kStagePairs && part > kLeastPart) {   // (the block scan ends with a barrier)
      while (part > kLeastPart && total > kStagePairs) { part /= 2u; total /= 2u; }
      continue;
    }
    S.lstart[t] = place;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      S.cnt[q][t] = place;
      place += c4[q];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bool in = 64u * j + lane < wn;
      const uint32_t x0 = rp[j].y & 0xFFu, len = in ? (rp[j].y >> 8) - x0 + 1u : 0u;
      const uint32_t inc = wave_scan_inc(len), off = inc - len;
      const uint32_t rel = x0 - off;
      wave_expand(off, len, wave_last(inc), S.bits[w], [&](uint32_t p, bool ok, int o) {
        const uint32_t col = (uint32_t)__shfl((int)rel, o, 64) + p;   // (of lanes with an output)
        const uint32_t f = (uint32_t)__shfl((int)rp[j].x, o, 64);
        const uint32_t q = wave_rank<8>(cnt, col, ok, lt);
        if (ok && q < kStagePairs) {
          S.sf[q] = f;
          S.scol[q] = (uint8_t)col;
        }
      });
    }
    __syncthreads();
    for (uint32_t q = t; q < total; q += kBlock) {
      const uint32_t col = S.scol[q], g = S.base[col] + (q - S.lstart[col]);
      if (g < D) { a.kout[g] = tile0 + col; a.vout[g] = S.sf[q]; }
    }
    __syncthreads();
    S.base[t] += run;
    o0 += part;
    if (part < kSubUnit && total < kStagePairs / 2u) part *= 2u;
  }
}

// Blocks past the units place the tiles in the longest-list-first order (see tile_scatter_body in
// sort.hip), from the tile totals, and clear the counters that the next binning starts with.
__device__ __forceinline__ void col_order(const ColArgs& a, uint32_t blk, uint32_t nblk) {
  __shared__ uint32_t cnt[kTileBuckets], cur[kTileBuckets], all[kTileBuckets];
  zero_words(a.clear, a.clear_words, Blk{blk, nblk});
  const uint32_t t = threadIdx.x, tiles = a.tiles_total;
  if (t < kTileBuckets) {
    cnt[t] = 0u;
    uint32_t s = 0;
    for (uint32_t k = 0; k < kOrderCopies; ++k) s += a.tordc[k * kTileBuckets + t];
    all[t] = s;
  }
  __syncthreads();
  const uint32_t t0 = blk * kTileOrderChunk;
  for (uint32_t i = t0 + t; i < tiles && i < t0 + kTileOrderChunk; i += kBlock) atomicAdd(&cnt[bit_length(a.tcount[i])], 1u);
  __syncthreads();
  if (t < kTileBuckets) {
    uint32_t start = 0;
    for (uint32_t c = t + 1; c < (uint32_t)kTileBuckets; ++c) start += all[c];
    cur[t] = cnt[t] ? start + atomicAdd(&a.tord[kTileBuckets + t], cnt[t]) : 0u;
    if (t == 0 && blk == 0) store_long_tiles(all, a.tord);
  }
  __syncthreads();
  for (uint32_t i = t0 + t; i < tiles && i < t0 + kTileOrderChunk; i += kBlock) {
    const uint32_t pos = atomicAdd(&cur[bit_length(a.tcount[i])], 1u);
    if (pos < tiles) a.order[pos] = i;
  }
}

// Items 0 .. order_blocks - 1 order the tiles, the others take a unit each.
__device__ __forceinline__ void col_down_body(const ColArgs& a, Blk b, ColLds& S) {
  const uint32_t nord = (a.tiles_total + kTileOrderChunk - 1) / kTileOrderChunk;
  if (b.id < nord) {
    col_order(a, b.id, nord);
    return;
  }
  const uint32_t u = b.id - nord;
  if (a.hdr[kHdrOverflow] || u >= (uint32_t)a.hdr[kHdrUnits]) return;
  col_down_unit(a, u, S);
}
__global__ __launch_bounds__(kBlock) void k_col_down(ColArgs a) {
  __shared__ ColLds S;
  col_down_body(a, grid_blk(), S);
}

// One kernel per stage kind of this file.
hipError_t launch_bin_stage(const Stage& st, hipStream_t s) {
  const dim3 g(st.items), blk(st.block);
  switch (st.kind) {
    case kStRecCount: hipLaunchKernelGGL(k_rec_count, g, blk, 0, s, st.a.depth); break;
    case kStRecCompact: hipLaunchKernelGGL(k_rec_compact, g, blk, 0, s, st.a.depth); break;
    case kStDepthUp: hipLaunchKernelGGL(k_depth_up, g, blk, 0, s, st.a.depth); break;
    case kStDepthDown: hipLaunchKernelGGL(k_depth_down, g, blk, 0, s, st.a.depth); break;
    case kStRowUp: hipLaunchKernelGGL(k_row_up, g, blk, st.lds, s, st.a.row); break;
    case kStRowDown: hipLaunchKernelGGL(k_row_down, g, blk, st.lds, s, st.a.row); break;
    case kStColUp: hipLaunchKernelGGL(k_col_up, g, blk, 0, s, st.a.col); break;
    case kStColScan: hipLaunchKernelGGL(k_col_scan, g, blk, 0, s, st.a.col); break;
    case kStColDown: hipLaunchKernelGGL(k_col_down, g, blk, 0, s, st.a.col); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace clod
