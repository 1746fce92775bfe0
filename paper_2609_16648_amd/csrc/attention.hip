// Verify attention (Sec. 3.1, Eq. verification-context): the query at block
// position i of sequence b attends causally to cache positions 0 .. m_b + i.
//
// bf16 path.  Work partition: the 16-token tiles of all sequences, laid end
// to end, are cut into P equal ranges, P = the number of workgroups the chip
// holds at once; workgroup (p, head group) takes range p for its heads, so
// every wave streams the same number of tiles whatever the length mix, and a
// range that crosses sequences streams on from one to the next without draining.
// A sequence inside one range is written as it is; a range that holds part of one
// yields a partial, and a combine kernel merges the partials of each such
// sequence.  One 64-lane wave per KV head and
// one or two 16-row query tiles (two: the k = 7 block, 32 rows, streams each KV
// tile once for both):
//  * GQA packing: the (n_heads / n_kv_heads) query heads of one KV head times
//    the block rows form the rows of 16-row matrix-core tiles, so each K/V
//    byte streamed from HBM serves every query that reads it;
//  * S^T = K Q^T on v_mfma_f32_16x16x32_bf16; the score tile comes out in the
//    operand layout of the P V product, so P never leaves registers;
//  * P is split into bf16 hi + lo parts that ride in the two halves of the
//    32-deep reduction of one v_mfma_f32_16x16x32_bf16 (V repeated), so the
//    weights keep ~16 mantissa bits at the cost of a single product;
//  * the KV pages are stored pre-swizzled (gm.h), so every 16-byte-per-lane
//    load reads 1 KiB contiguous straight into operand registers;
//  * K/V tiles stream through a ring of register buffers, every load
//    unconditional, so kAttnRing - 1 tiles are always in flight;
//  * tiles wholly inside every query's causal window skip the mask; the
//    online softmax (exp2 domain) rescales only when a running max grows by
//    more than 2^kLazyLog2, so most tiles need no rescale.
// float32 path: a workgroup per (row, head), its four waves splitting the tokens.
#include <atomic>

#include "common.h"
#include "forward.h"

namespace gm {

namespace {
constexpr int kAttnWavesPerGroup = 4;   // waves per workgroup (KV heads x query row tiles)
// Dynamic LDS a workgroup reserves so that a CU holds one at a time: with two
// per CU the older one wins the SIMD arbitration, finishes early and leaves the
// CU half idle for the rest of the launch (measured); one per CU keeps all ranges
// in step.  Each wave uses a slice of 16 rows of kAttnRowPad floats of it.
constexpr int kAttnLdsReserve = 84 * 1024;
constexpr int kAttnRowPad = 132;        // floats between rows of an output tile in LDS (128 + 4: distinct banks)
static_assert(kAttnWavesPerGroup * 16 * kAttnRowPad * 4 <= kAttnLdsReserve, "the waves' slices fit the reservation");
constexpr int kAttnRing = 3;            // K/V register buffers per wave
constexpr float kLazyLog2 = 8.f;        // rescale threshold of the running max (log2 units)
// Ranges of this many tiles store the partials of cut sequences through the caches, shorter and longer
// ones past them (attention and combine, us, past the caches -> through them, by tiles per range:
// 0.6: 18.4 -> 19.2 and 18.3 -> 20.1; 2.5: 22.1 -> 24.4 and 17.6 -> 19.8; 3.9: 24.5 -> 25.9; 4.2: 20.1 -> 21.5;
// 4.4: 27.3 -> 26.2; 5: 25.8 -> 23.9; 6.5: 21.4 -> 20.5; 10.5: 42.4 -> 38.1;
// 16: 36.7 -> 35.5; 80: 120.9 -> 118.6; 94: 133.2 -> 131.9; 117: 168.2 -> 168.2; 384: 496.5 -> 499.9;
// 576: 750 -> 775).
constexpr int kPartCachedTiles = 5, kPartStreamTiles = 128;

struct AttnK {
  const uint16_t *kp, *vp;
  const int32_t *bt, *base, *blen;
  const uint16_t *q;
  uint16_t *out;
  float *part_o;        // [P + B slots][n_kv][rows_pad][128]
  float2 *part_ml;      // [P + B slots][n_kv][rows_pad]
  int32_t *cum;         // [B + 1] tiles before sequence b (written by workgroup (0, 0))
  int32_t *dev_err;
  int B, base_off, blen_add, R, G, n_heads, n_kv, page_size, max_pages, num_pages, rows_pad;
  int parts, heads_per_group, row_tiles, waves_per_head;
  float scale_log2;
};

__device__ __forceinline__ int block_rows(const int32_t *blen, int add, int b, int R) {
  if (!blen) return R;
  const int n = blen[b] + add;
  return n < 0 ? 0 : (n > R ? R : n);
}

// 16-token tiles of sequence b: its context is its block's start m0 plus its valid block rows
__device__ __forceinline__ int seq_tiles(const AttnK &a, int b, int &m0, int &rows) {
  m0 = a.base[b] + a.base_off;
  rows = block_rows(a.blen, a.blen_add, b, a.R);
  const int L = m0 + rows;
  return L > 0 ? (L + 15) >> 4 : 0;
}

// a / b for a quotient below 2^31, in 32 bits where a fits (a 64-bit division is some 150 instructions: with
// every one of them in 64 bits 8 sequences of 64 tokens took 14.8 us, 13.9 so, combine included)
__device__ __forceinline__ int div_u(unsigned long long a, int b) {
  return a >> 32 ? (int)(a / (unsigned)b) : (int)((unsigned)a / (unsigned)b);
}
// first tile of range p when TT tiles are cut into P ranges
__device__ __forceinline__ int part_begin(int p, int TT, int P) { return div_u((unsigned long long)p * TT, P); }

// exclusive block-wide prefix sum (blockDim.x a multiple of 64, <= 1024); *total gets the sum
__device__ __forceinline__ int block_excl_scan(int v, int *sh, int *total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  int off = 0, t = 0;
  for (int i = 0; i < nw; ++i) {
    const int u = sh[i];
    off += i < wid ? u : 0;
    t += u;
  }
  *total = t;
  return off + x - v;
}

__device__ __forceinline__ uint32_t zero_half(uint32_t v, int hi) { return hi ? (v & 0x0000ffffu) : (v & 0xffff0000u); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {   // round to nearest even
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2_t{a, b}, bf16x2_t));
}

template <bool STREAM>
__device__ __forceinline__ uint4 load_kv(const uint16_t *p) {
  if (STREAM) return load_nt(p);
  return *reinterpret_cast<const uint4 *>(p);
}

struct TileBuf {
  uint4 k[4], v[4];
  int slot;   // the tile's place in the pool, -1: none
};

// One 16-token tile for the RT 16-row query tiles of a wave: S^T = K Q^T, online softmax,
// O^T += V^T (P_hi + P_lo).  MASK: apply the causal window (token < vis) and keep tokens
// past the context (t >= L, whose slots may hold anything) out of P V.  Each step runs
// for every query tile before the next, so the tiles' dependency chains interleave and
// the V operands of P V are formed once for all of them; each tile's arithmetic is the
// same as on its own.
template <bool MASK, int RT>
__device__ __forceinline__ void attn_tiles(int tb, int L, int g, float scale_log2, TileBuf &t,
                                           const bf16x8_t (&qf)[RT][4], const int (&vis)[RT], float (&m)[RT],
                                           float (&l)[RT], floatx4_t (&O)[RT][8]) {
  if (MASK) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (tb + 4 * g + e >= L) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if (e < 2) { t.v[p].x = zero_half(t.v[p].x, e); t.v[p].z = zero_half(t.v[p].z, e); }
          else { t.v[p].y = zero_half(t.v[p].y, e - 2); t.v[p].w = zero_half(t.v[p].w, e - 2); }
        }
      }
    }
  }
  floatx4_t S[RT];
#pragma unroll
  for (int u = 0; u < RT; ++u) S[u] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ii = 0; ii < 4; ++ii)
#pragma unroll
    for (int u = 0; u < RT; ++u)
      S[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t.k[ii]), qf[u][ii], S[u], 0, 0, 0);
  float s[RT][4], tmax[RT];
#pragma unroll
  for (int u = 0; u < RT; ++u) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[u][r] = S[u][r] * scale_log2;
      if (MASK && tb + 4 * g + r >= vis[u]) s[u][r] = -INFINITY;
    }
    tmax[u] = fmaxf(fmaxf(s[u][0], s[u][1]), fmaxf(s[u][2], s[u][3]));
  }
#pragma unroll
  for (int u = 0; u < RT; ++u) tmax[u] = fmaxf(tmax[u], __shfl_xor(tmax[u], 16, kWave));
#pragma unroll
  for (int u = 0; u < RT; ++u) tmax[u] = fmaxf(tmax[u], __shfl_xor(tmax[u], 32, kWave));
  // Each row decides for itself (m = -inf and a finite score also count as growth);
  // rows that did not grow keep alpha = 1 exactly, so a row's result never depends
  // on the other rows of the tile.  The branch only skips tiles where no row grew.
#pragma unroll
  for (int u = 0; u < RT; ++u) {
    const bool up = tmax[u] > m[u] + kLazyLog2;
    if (__any(up)) {
      const float mn = up ? fmaxf(m[u], tmax[u]) : m[u];
      const float alpha = (!up || mn == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m[u] - mn);
      l[u] *= alpha;
#pragma unroll
      for (int mm = 0; mm < 8; ++mm) O[u][mm] *= alpha;
      m[u] = mn;
    }
  }
  // s <= m + kLazyLog2 here, so p <= 2^kLazyLog2
  bf16x8_t pb[RT];
#pragma unroll
  for (int u = 0; u < RT; ++u) {
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(s[u][r] - m[u]);
      if (MASK && s[u][r] == -INFINITY) p[r] = 0.f;
      l[u] += p[r];
    }
    const uint32_t h01 = pack_bf16(p[0], p[1]), h23 = pack_bf16(p[2], p[3]);
    const uint32_t l01 = pack_bf16(p[0] - __uint_as_float(h01 << 16), p[1] - __uint_as_float(h01 & 0xffff0000u));
    const uint32_t l23 = pack_bf16(p[2] - __uint_as_float(h23 << 16), p[3] - __uint_as_float(h23 & 0xffff0000u));
    pb[u] = as_bf16x8(make_uint4(h01, h23, l01, l23));
  }
#pragma unroll
  for (int mm = 0; mm < 8; ++mm) {
    const uint4 &v4 = t.v[mm >> 1];
    const uint4 va = (mm & 1) ? make_uint4(v4.z, v4.w, v4.z, v4.w) : make_uint4(v4.x, v4.y, v4.x, v4.y);
#pragma unroll
    for (int u = 0; u < RT; ++u) O[u][mm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), pb[u], O[u][mm], 0, 0, 0);
  }
}

// RT: 16-row query tiles per wave.  A wave streams the KV tiles of its head once and
// runs the score / softmax / PV products of its RT query tiles on each of them; the
// waves_per_head = row_tiles / RT waves of one head split its query tiles.
// STREAM: every KV tile has exactly one reader (one wave per KV head), so its loads are
// marked non-temporal and do not displace the lines other waves re-read; where two waves
// read the same tiles the second read is meant to hit the cache (measured: non-temporal
// loads there cost 20%).
template <bool STREAM, int RT>
__global__ __launch_bounds__(64 * kAttnWavesPerGroup) void attn_mfma_kernel(AttnK a) {
  const int part = blockIdx.x, grp = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, uniform per wave
  const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
  const int kvh = grp * a.heads_per_group + w / a.waves_per_head, rt0 = (w % a.waves_per_head) * RT;
  const bool wave_ok = kvh < a.n_kv;
  const int rows = a.G * a.R;

  // Sequences come in chunks of blockDim.x, one per thread; the tiles of a chunk that fall in
  // the range stream in windows of kAttnWinTiles.
  __shared__ int scan_sh[16];
  __shared__ int cum_sh[64 * kAttnWavesPerGroup + 1];                        // tiles before each sequence of the chunk
  __shared__ int m0_sh[64 * kAttnWavesPerGroup], bl_sh[64 * kAttnWavesPerGroup];   // block start and valid block rows
  __shared__ int slot_sh[kAttnWinTiles], seq_sh[kAttnWinTiles];              // per tile: place in the pool, sequence

  // Total tiles TT over all sequences; every workgroup computes the same sums, and workgroup
  // (0, 0) also stores the prefix sums for the combine.
  const int tid = threadIdx.x, nthr = blockDim.x;
  const bool one_chunk = a.B <= nthr;   // a batch that fits one block needs a single scan
  const bool writer = part == 0 && grp == 0;
  int TT = 0, T1 = 0, cb1 = 0, m1 = 0, r1 = 0;   // this thread's sequence of the chunk
  if (one_chunk) {
    T1 = tid < a.B ? seq_tiles(a, tid, m1, r1) : 0;
    cb1 = block_excl_scan(T1, scan_sh, &TT);
    if (writer && tid < a.B) a.cum[tid] = cb1;
  } else {
    for (int c = 0; c < a.B; c += nthr) {
      const int T = c + tid < a.B ? seq_tiles(a, c + tid, m1, r1) : 0;
      int tot;
      const int cb = TT + block_excl_scan(T, scan_sh, &tot);
      if (writer && c + tid < a.B) a.cum[c + tid] = cb;
      TT += tot;
    }
  }
  if (writer && tid == 0) a.cum[a.B] = TT;
  const int s = part_begin(part, TT, a.parts), e = part_begin(part + 1, TT, a.parts);
  if (s >= e) return;   // an empty range (fewer tiles than workgroups)
  const int tpp = a.page_size >> 4;                        // tiles per page
  const long head_off = (long)kvh * a.page_size * 128;

  // this lane's query rows: row (rt0 + u) * 16 + j of the head's G x R rows
  int qrow[RT], qi[RT];
#pragma unroll
  for (int u = 0; u < RT; ++u) {
    const int r = (rt0 + u) * 16 + j;
    qi[u] = r < rows && wave_ok ? r % a.R : -1;
    qrow[u] = qi[u] >= 0 ? (qi[u] * a.n_heads + kvh * a.G + r / a.R) * 128 + 8 * g : 0;
  }
  auto load_q = [&](int b, bf16x8_t (&q)[RT][4]) {
    const uint16_t *qb = a.q + (long)b * a.R * a.n_heads * 128;
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
      for (int ii = 0; ii < 4; ++ii)
        q[u][ii] = as_bf16x8(qi[u] >= 0 ? *reinterpret_cast<const uint4 *>(qb + qrow[u] + 32 * ii) : make_uint4(0, 0, 0, 0));
  };

  // The segment (the tiles of one sequence in this range) being streamed: sequence, block
  // start, context, tiles before the sequence and up to its end, end of the segment; the queries, the softmax state, and the
  // queries of the next segment, loaded one segment ahead.
  int b = -1, m0 = 0, L = 0, cb = 0, seq_end = 0, seg_end = s;
  bool dead = false;
  bf16x8_t qf[RT][4], qn[RT][4];
  int vis[RT];
  float m[RT], l[RT];
  floatx4_t O[RT][8];
  // The end of a segment.  A sequence that lies wholly in this range is normalised and written
  // as it is (the combine skips it), its rows through this wave's slice of LDS so that a store
  // covers whole lines; a part of one goes to the partials (kPartCachedTiles).  Storing the
  // partials of every sequence, padding rows too, held the KV stream up by 25 us per segment
  // (1024 sequences of 2560 tokens: 1784 us so, 1598 us with whole sequences written directly);
  // the partials through LDS as well cost short ranges 1.5 us and long ones as much as they saved.
  extern __shared__ __attribute__((aligned(16))) float attn_sh[];   // kAttnLdsReserve bytes
  float *const rows_sh = attn_sh + w * 16 * kAttnRowPad;
  auto finish = [&]() __attribute__((always_inline)) {
    const bool cached = e - s >= kPartCachedTiles && e - s < kPartStreamTiles;
    const bool whole = cb >= s && seq_end <= e;
#pragma unroll
    for (int u = 0; u < RT; ++u) {
      float lu = l[u];
      lu += __shfl_xor(lu, 16, kWave);
      lu += __shfl_xor(lu, 32, kWave);
      if (!whole) {
        const long prow = ((long)(part + b) * a.n_kv + kvh) * a.rows_pad + (rt0 + u) * 16 + j;
        if (g == 0) a.part_ml[prow] = make_float2(m[u], lu);
        if ((rt0 + u) * 16 + j < rows) {
          floatx4_t *const dst = reinterpret_cast<floatx4_t *>(a.part_o + prow * 128 + 4 * g);
          if (cached) {
            asm volatile("" ::: "memory");   // (stores that differ in the hint alone would be merged)
#pragma unroll
            for (int mm = 0; mm < 8; ++mm) dst[4 * mm] = O[u][mm];
            asm volatile("" ::: "memory");
          } else {
#pragma unroll
            for (int mm = 0; mm < 8; ++mm) __builtin_nontemporal_store(O[u][mm], dst + 4 * mm);
          }
        }
        continue;
      }
      // rows with no visible token (past the block, or none readable) give 0
      const bool live = vis[u] > 0 && m[u] != -INFINITY;
      const float inv = 1.f / lu;
      wave_lds_sync();
#pragma unroll
      for (int mm = 0; mm < 8; ++mm)
        *reinterpret_cast<floatx4_t *>(rows_sh + j * kAttnRowPad + 16 * mm + 4 * g) =
            live ? O[u][mm] * inv : floatx4_t{0.f, 0.f, 0.f, 0.f};
      wave_lds_sync();
      const int nr = min(16, rows - (rt0 + u) * 16);   // rows of this tile that exist
#pragma unroll 1   // (the segment's end is inlined at every ring position: short code counts here)
      for (int q = 0; q < 4; ++q) {
        const int rl = 4 * q + g, r = (rt0 + u) * 16 + rl;
        if (rl >= nr) continue;
        const float *src = rows_sh + rl * kAttnRowPad + 8 * j;
        uint32_t pk[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          pk[c] = f32_to_bf16(src[2 * c]) | (uint32_t(f32_to_bf16(src[2 * c + 1])) << 16);
        const long o = (((long)b * a.R + r % a.R) * a.n_heads + kvh * a.G + r / a.R) * 128 + 8 * j;
        *reinterpret_cast<uint4 *>(a.out + o) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
      }
    }
  };

  int run = 0;
  for (int c = 0; c < a.B; c += nthr) {
    int T, cbt, tot;
    if (one_chunk) {
      T = T1;
      cbt = cb1;
      tot = TT;
    } else {
      T = c + tid < a.B ? seq_tiles(a, c + tid, m1, r1) : 0;
      cbt = run + block_excl_scan(T, scan_sh, &tot);
    }
    const int cbeg = run, cend = run + tot;
    run = cend;
    if (cend <= s) continue;
    if (cbeg >= e) break;
    __syncthreads();   // the previous chunk's tables are read
    cum_sh[tid] = cbt;
    if (tid == 0) cum_sh[nthr] = cend;
    m0_sh[tid] = m1;
    bl_sh[tid] = r1;
    const int xe = min(e, cend);
    for (int x0 = max(s, cbeg); x0 < xe; x0 += kAttnWinTiles) {
      const int nt = min(kAttnWinTiles, xe - x0);
      // The window's tiles, looked up once into LDS: in the loop a lookup is then an LDS read,
      // whose counter is separate from the KV loads', so no wait drains the prefetch.  A page
      // outside the pool is reported; it ends its segment before its first token.
      __syncthreads();
      for (int i = tid; i < nt; i += nthr) {
        int lo = 0, hi = min(nthr, a.B - c);   // the last sequence with at most x0 + i tiles before it
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (cum_sh[mid] <= x0 + i) lo = mid;
          else hi = mid;
        }
        const int t = x0 + i - cum_sh[lo], pi = t / tpp;
        const int page = pi < a.max_pages ? a.bt[(long)(c + lo) * a.max_pages + pi] : -1;
        const bool ok = page >= 0 && page < a.num_pages;
        if (!ok) raise_dev_err(a.dev_err, GM_DEVERR_PAGE);
        seq_sh[i] = lo;
        slot_sh[i] = ok ? page * a.n_kv * tpp + t % tpp : -1;   // 16 x 128 elements each, of the first head
      }
      __syncthreads();
      if (!wave_ok) continue;   // spare waves of the last head group (they only join the barriers)

      // A bad tile loads the pool's first tile instead; its segment is not consumed further.
      auto load_tile = [&](int i, TileBuf &t) {
        t.slot = __builtin_amdgcn_readfirstlane(slot_sh[i]);
        const long off = head_off + (long)max(t.slot, 0) * 2048;
#pragma unroll
        for (int q = 0; q < 4; ++q) t.k[q] = load_kv<STREAM>(a.kp + off + q * 512 + lane * 8);
#pragma unroll
        for (int q = 0; q < 4; ++q) t.v[q] = load_kv<STREAM>(a.vp + off + q * 512 + lane * 8);
      };
      auto step = [&](int i, TileBuf &t) __attribute__((always_inline)) {
        if (i >= nt) return;
        const int x = x0 + i;
        if (x == seg_end) {   // the first tile of a segment
          if (b >= 0) finish();
          const int q = __builtin_amdgcn_readfirstlane(seq_sh[i]);
          b = c + q;
          m0 = __builtin_amdgcn_readfirstlane(m0_sh[q]);
          const int blen = __builtin_amdgcn_readfirstlane(bl_sh[q]);
          L = m0 + blen;
          cb = __builtin_amdgcn_readfirstlane(cum_sh[q]);
          seq_end = __builtin_amdgcn_readfirstlane(cum_sh[q + 1]);
          seg_end = min(e, seq_end);
          dead = false;
#pragma unroll
          for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) qf[u][ii] = qn[u][ii];
          // the queries have arrived before the paths join, or every tile's products would wait
          // for all loads in flight
#pragma unroll
          for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) asm volatile("" : "+v"(qf[u][ii]));
          if (seg_end < x0 + nt) load_q(c + __builtin_amdgcn_readfirstlane(seq_sh[seg_end - x0]), qn);
#pragma unroll
          for (int u = 0; u < RT; ++u) {
            vis[u] = qi[u] >= 0 && qi[u] < blen ? m0 + qi[u] + 1 : 0;
            m[u] = -INFINITY;
            l[u] = 0.f;
#pragma unroll
            for (int mm = 0; mm < 8; ++mm) O[u][mm] = floatx4_t{0.f, 0.f, 0.f, 0.f};
          }
        }
        dead = dead || t.slot < 0;
        if (dead) return;
        // A tile below position m0 + 1 is inside the window of every valid query row and inside
        // the context: no mask.  The rest (the causal diagonal and the partial tile at the end of
        // the context) take the mask, which zeroes the V entries past the context in place.  Rows
        // that are not valid queries (past the block, or padding) compute finite values nobody reads.
        const int tb = 16 * (x - cb);
        if (tb + 16 <= m0 + 1) attn_tiles<false, RT>(tb, L, g, a.scale_log2, t, qf, vis, m, l, O);
        else attn_tiles<true, RT>(tb, L, g, a.scale_log2, t, qf, vis, m, l, O);
      };
      // The ring runs across segments: the loads of the next sequence's tiles are in flight while
      // this one's last tiles are consumed.  The loads run unguarded in whole turns of the ring
      // (one straight path, so every wait counts exactly the loads still in flight), as long as
      // every refill is a tile of the window; the last two to four tiles (one, in a window of one)
      // run behind the loop.  Re-reads of the last tile in their place were waited for at the end
      // of the range: 63 sequences of 67 tokens at k = 5 and k = 3 24.3 and 18.9 us with them, 22.2
      // and 17.6 without; 256 of 512-8704 tokens 749 and 746.
      TileBuf ring[kAttnRing];
      // the queries of the first segment that begins in this window
      if (seg_end < x0 + nt) load_q(c + __builtin_amdgcn_readfirstlane(seq_sh[seg_end - x0]), qn);
#pragma unroll
      for (int d = 0; d < kAttnRing - 1; ++d) load_tile(min(d, nt - 1), ring[d]);
      static_assert(kAttnRing == 3, "the tiles behind the loop are written out for a ring of three");
      int i = 0;
      for (; i + 2 * kAttnRing - 2 < nt; i += kAttnRing) {
#pragma unroll
        for (int d = 0; d < kAttnRing; ++d) {
          // refill the buffer consumed last step; the scheduling barriers keep each refill after
          // the step that frees its buffer, so the ring keeps fixed registers and no copy waits
          // on a load in flight
          __builtin_amdgcn_sched_barrier(0);
          load_tile(i + d + kAttnRing - 1, ring[(d + kAttnRing - 1) % kAttnRing]);
          __builtin_amdgcn_sched_barrier(0);
          step(i + d, ring[d]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (i + 2 < nt) load_tile(i + 2, ring[2]);
      __builtin_amdgcn_sched_barrier(0);
      step(i, ring[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (i + 3 < nt) load_tile(i + 3, ring[0]);
      __builtin_amdgcn_sched_barrier(0);
      step(i + 1, ring[1]);
      step(i + 2, ring[2]);
      step(i + 3, ring[0]);
    }
  }
  if (wave_ok) finish();   // the last segment
}

// Merge the partials of sequence b: the ranges that hold its tiles are parts
// p_first .. p_last (empty ranges among them wrote nothing and are skipped);
// the partial of (part p, sequence b) sits in slot p + b.  A thread per (KV head,
// row, four channels) reads partials kCombineBatch at a time with every load issued
// before the first use, and merges them in one pass.  SP groups of 32 threads share a
// row, group i taking batches i, i + SP, ..; their results meet in LDS in group order.
// SP = 16 where few sequences are cut into many partials each: the pass is a chain of
// load round trips (one sequence in 126 partials: 42 us with one group, 8.5 with sixteen).
constexpr int kCombineBatch = 8;

template <int SP>
__global__ __launch_bounds__(SP > 1 ? 32 * SP : 256) void attn_combine_kernel(AttnK a) {
  const int b = blockIdx.y;
  const int rows = a.G * a.R;
  const int tid = threadIdx.x, sp = SP > 1 ? tid >> 5 : 0;
  const int idx = SP > 1 ? blockIdx.x * 32 + (tid & 31) : blockIdx.x * blockDim.x + tid;
  if (idx >= a.n_kv * rows * 32) return;   // (SP > 1: a block per row, never taken)
  const int d = (idx & 31) * 4, r = (idx >> 5) % rows, kvh = (idx >> 5) / rows;
  const int hl = r / a.R, i = r % a.R;
  const int TT = a.cum[a.B], cb = a.cum[b], T = a.cum[b + 1] - cb, P = a.parts;
  int pf = 0, pl = 0;
  if (T > 0) {
    pf = min(div_u((unsigned long long)(cb + 1) * P - 1, TT), P - 1);
    pl = min(div_u((unsigned long long)(cb + T) * P - 1, TT), P - 1);
    if (pf == pl) return;   // wholly in range pf, which has written its rows
  }
  const int blen = block_rows(a.blen, a.blen_add, b, a.R);
  float M = -INFINITY, den = 0.f;
  float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
  auto merge = [&](float m2, float l2, float4 o2) {
    const float mn = fmaxf(M, m2);
    const float sc = __builtin_amdgcn_exp2f(M - mn), w = __builtin_amdgcn_exp2f(m2 - mn);   // M = -inf: sc = 0
    den = den * sc + l2 * w;
    num.x = num.x * sc + o2.x * w;
    num.y = num.y * sc + o2.y * w;
    num.z = num.z * sc + o2.z * w;
    num.w = num.w * sc + o2.w * w;
    M = mn;
  };
  if (i < blen && T > 0) {
    for (int p0 = pf + kCombineBatch * sp; p0 <= pl; p0 += kCombineBatch * SP) {
      float2 ml[kCombineBatch];
      float4 o[kCombineBatch];
#pragma unroll
      for (int u = 0; u < kCombineBatch; ++u) {
        const int p = min(p0 + u, pl);
        const long pr = ((long)(p + b) * a.n_kv + kvh) * a.rows_pad + r;
        ml[u] = a.part_ml[pr];
        o[u] = *reinterpret_cast<const float4 *>(a.part_o + pr * 128 + d);
      }
#pragma unroll
      for (int u = 0; u < kCombineBatch; ++u) {
        const int p = p0 + u;
        if (p > pl || ml[u].x == -INFINITY) continue;
        // ranges are empty only where there are more of them than tiles (asked first: two 64-bit
        // divisions per partial cost 3 sequences in 45 partials each 4 us of 31)
        if (TT < P && part_begin(p, TT, P) == part_begin(p + 1, TT, P)) continue;
        merge(ml[u].x, ml[u].y, o[u]);
      }
    }
  }
  if constexpr (SP > 1) {
    __shared__ float sh[SP][6][32];
    const int c = tid & 31;
    sh[sp][0][c] = M;
    sh[sp][1][c] = den;
    sh[sp][2][c] = num.x;
    sh[sp][3][c] = num.y;
    sh[sp][4][c] = num.z;
    sh[sp][5][c] = num.w;
    __syncthreads();
    if (sp) return;
#pragma unroll
    for (int u = 1; u < SP; ++u)
      if (sh[u][0][c] != -INFINITY) merge(sh[u][0][c], sh[u][1][c], make_float4(sh[u][2][c], sh[u][3][c], sh[u][4][c], sh[u][5][c]));
  }
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (M != -INFINITY) {
    const float inv = 1.f / den;
    v = make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv);
  }
  const uint2 packed = make_uint2(f32_to_bf16(v.x) | (uint32_t(f32_to_bf16(v.y)) << 16),
                                  f32_to_bf16(v.z) | (uint32_t(f32_to_bf16(v.w)) << 16));
  *reinterpret_cast<uint2 *>(a.out + (((long)b * a.R + i) * a.n_heads + kvh * a.G + hl) * 128 + d) = packed;
}

// ------------------------------------------------------------------ float32 path
struct AttnF {
  const float *kp, *vp, *q;
  float *out;
  const int32_t *bt, *base, *blen;
  int32_t *dev_err;
  int base_off, blen_add, R, G, n_heads, n_kv, page_size, max_pages, num_pages;
  float scale;
};

// One workgroup of four waves per (block row, head, sequence).  A wave takes every fourth
// chunk of 64 tokens with an online softmax of its own.  Scores: lane = token (8 channels
// are contiguous in the K tile).  P V: lane = channel, D / 64 of them, and the chunk's
// weights come back from LDS, so a lane's 16-byte load holds four tokens of its channel
// and a wave's loads cover whole V tiles.  The wave partials are merged in wave order.
// Bound by the chain of dependent loads, not by bytes (16 rows x 4 heads of 128 tokens:
// 18 us with one wave per row whose lanes each walked the channels of their own tokens,
// 6.8 us here).
template <int D>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnF a) {
  constexpr int C = D / 64;        // channels per lane in P V
  __shared__ float sh_q[D];
  __shared__ __attribute__((aligned(16))) float sh_p[4][64];
  __shared__ float sh_m[4], sh_l[4], sh_o[4][D];
  const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blen = block_rows(a.blen, a.blen_add, b, a.R);
  float *orow = a.out + (((long)b * a.R + i) * a.n_heads + h) * D;
  if (i >= blen) {
    for (int c = tid; c < D; c += 256) orow[c] = 0.f;
    return;
  }
  const int vis = a.base[b] + a.base_off + i + 1;
  const int kvh = h / a.G;
  for (int c = tid; c < D; c += 256) sh_q[c] = a.q[(((long)b * a.R + i) * a.n_heads + h) * D + c];
  __syncthreads();
  // the pool offset of tile tb (16 tokens, all in one page), or -1 for a page outside the pool
  auto tile_base = [&](int tb) -> long {
    const int pi = tb / a.page_size;
    const int page = pi < a.max_pages ? a.bt[(long)b * a.max_pages + pi] : -1;
    if (page < 0 || page >= a.num_pages) return -1;
    return (((long)page * a.n_kv + kvh) * a.page_size + tb % a.page_size) * D;
  };
  float m = -INFINITY, l = 0.f, o[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o[c] = 0.f;
  for (int c0 = 64 * w; c0 < vis; c0 += 256) {
    const int tok = c0 + lane;
    float sc = -INFINITY;
    if (tok < vis) {
      const long tile = tile_base(tok & ~15);
      if (tile < 0) {
        raise_dev_err(a.dev_err, GM_DEVERR_PAGE);
      } else {
        const float *kt = a.kp + tile + (tok & 15) * 8;
        sc = 0.f;
#pragma unroll
        for (int c = 0; c < D; c += 8) {
          const floatx4u_t k0 = *reinterpret_cast<const floatx4u_t *>(kt + k_tile_off(0, c));
          const floatx4u_t k1 = *reinterpret_cast<const floatx4u_t *>(kt + k_tile_off(0, c) + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) sc += sh_q[c + e] * k0[e];
#pragma unroll
          for (int e = 0; e < 4; ++e) sc += sh_q[c + 4 + e] * k1[e];
        }
        sc *= a.scale;
      }
    }
    const float mn = fmaxf(m, wave_max(sc));
    // no readable token in the chunk (the maximum passes NaN scores over: they have to reach the row)
    if (mn == -INFINITY && !__any(sc != sc)) continue;
    const float p = expf(sc - mn), al = expf(m - mn);
    l = l * al + wave_sum(p);
    m = mn;
    wave_lds_sync();                 // the last chunk's weights are read
    sh_p[w][lane] = p;
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] *= al;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int tb = c0 + 16 * t;
      if (tb >= vis) break;
      const long tile = tile_base(tb);
      if (tile < 0) continue;
#pragma unroll
      for (int s = 0; s < 16; s += 4) {
        const float4 pv = *reinterpret_cast<const float4 *>(&sh_p[w][16 * t + s]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const floatx4u_t v = *reinterpret_cast<const floatx4u_t *>(a.vp + tile + v_tile_off(s, lane + 64 * c));
          // slots past the visible tokens may hold anything
          o[c] += pv.x * (tb + s < vis ? v[0] : 0.f);
          o[c] += pv.y * (tb + s + 1 < vis ? v[1] : 0.f);
          o[c] += pv.z * (tb + s + 2 < vis ? v[2] : 0.f);
          o[c] += pv.w * (tb + s + 3 < vis ? v[3] : 0.f);
        }
      }
    }
  }
  if (lane == 0) {
    sh_m[w] = m;
    sh_l[w] = l;
  }
#pragma unroll
  for (int c = 0; c < C; ++c) sh_o[w][lane + 64 * c] = o[c];
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int u = 0; u < 4; ++u) M = fmaxf(M, sh_m[u]);
  if (tid < D) {
    float den = 0.f, num = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (sh_l[u] == 0.f) continue;   // the wave read no token
      const float f = expf(sh_m[u] - M);
      den += sh_l[u] * f;
      num += sh_o[u][tid] * f;
    }
    orow[tid] = num / den;
  }
}

// Geometry of the bf16 launch: row tiles per KV head, heads per workgroup, groups.
struct AttnGeom {
  int row_tiles, rt_per_wave, waves_per_head, heads_per_group, groups, block;
};
AttnGeom attn_geom(const gm_model_config &cfg, int rows_pad) {
  AttnGeom g;
  g.row_tiles = rows_pad / 16;
  g.rt_per_wave = g.row_tiles >= 2 ? 2 : 1;
  g.waves_per_head = g.row_tiles / g.rt_per_wave;
  g.heads_per_group = kAttnWavesPerGroup / g.waves_per_head;
  if (g.heads_per_group > cfg.n_kv_heads) g.heads_per_group = cfg.n_kv_heads;
  if (g.heads_per_group < 1) g.heads_per_group = 1;
  g.groups = (cfg.n_kv_heads + g.heads_per_group - 1) / g.heads_per_group;
  g.block = 64 * g.heads_per_group * g.waves_per_head;
  return g;
}

// Workgroups of `block` threads that one device holds at once (queried once per
// block size and device; a fixed guess when no device answers).  The LDS
// reservation makes this one per CU.
int resident_groups(int block) {
  static std::atomic<int> cache[16][kAttnWavesPerGroup + 1];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 256;
  const int wv = block / 64;
  int v = cache[dev][wv].load();
  if (v > 0) return v;
  int per_cu = 0, cus = 0;
  const void *kernels[] = {(const void *)attn_mfma_kernel<true, 1>, (const void *)attn_mfma_kernel<true, 2>,
                           (const void *)attn_mfma_kernel<false, 2>};
  bool ok = true;
  for (const void *f : kernels)
    ok = ok && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnLdsReserve) == hipSuccess;
  if (!ok || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_mfma_kernel<true, 2>, block, kAttnLdsReserve) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 || cus < 1) {
    (void)hipGetLastError();
    return 256;
  }
  v = per_cu * cus;
  cache[dev][wv].store(v);
  return v;
}
}  // namespace

AttnPlan plan_attention(const gm_model_config &cfg, int B, int R) {
  AttnPlan p{};
  const int G = cfg.n_heads / cfg.n_kv_heads;
  const int rows = G * R;
  const int nt = rows <= 16 ? 1 : (rows <= 32 ? 2 : 4);
  p.rows_pad = nt * 16;
  if (cfg.dtype != GM_BF16) return p;
  const AttnGeom g = attn_geom(cfg, p.rows_pad);
  long parts = resident_groups(g.block) / g.groups;
  // One range per workgroup that the chip holds, however long: every further round of workgroups
  // fills its rings again, writes more partials, and the last one leaves CUs idle (256 sequences
  // of 512-8704 tokens: 840 us with one round, 898 us in 4.25 rounds of at most 4096 tokens;
  // 32 sequences of 16-32K tokens: 500 us with one round, 530 with two, 577 with four).
  if (parts < 1) parts = 1;
  p.parts = (int)parts;
  // the partial of (range p, sequence b) is in slot p + b
  Carve c;
  const size_t n = (size_t)(parts + B) * cfg.n_kv_heads * p.rows_pad;
  p.part_o = c.take(n * 128 * sizeof(float));
  p.part_ml = c.take(n * sizeof(float2));
  p.cum = c.take((size_t)(B + 1) * sizeof(int32_t));
  p.total = c.off;
  return p;
}

AttnArgs attn_args(const gm_model_config &cfg, const gm_kv_cache &c, int layer, int B, int R,
                   const int32_t *base_lens, int base_off, const int32_t *blk_len) {
  AttnArgs a{};
  a.dtype = cfg.dtype;
  a.B = B;
  a.R = R;
  a.n_heads = cfg.n_heads;
  a.n_kv = cfg.n_kv_heads;
  a.head_dim = cfg.head_dim;
  a.page_size = c.page_size;
  a.max_pages = c.max_pages_per_seq;
  a.num_pages = c.num_pages;
  a.k_pages = c.k_pages[layer];
  a.v_pages = c.v_pages[layer];
  a.block_table = c.block_table;
  a.base_lens = base_lens;
  a.base_off = base_off;
  a.blk_len = blk_len;
  a.blk_len_add = 0;
  a.scale = 1.0f / sqrtf((float)cfg.head_dim);
  a.trace = "attn";
  a.trace_combine = "attn_combine";
  return a;
}

void run_attention(const AttnArgs &a, const AttnPlan &p, char *ws, hipStream_t s) {
  if (a.B == 0) return;
  const int G = a.n_heads / a.n_kv;
  if (a.dtype == GM_BF16) {
    gm_model_config cfg{};
    cfg.n_kv_heads = a.n_kv;
    const AttnGeom geo = attn_geom(cfg, p.rows_pad);
    AttnK k{};
    k.kp = (const uint16_t *)a.k_pages;
    k.vp = (const uint16_t *)a.v_pages;
    k.bt = a.block_table;
    k.base = a.base_lens;
    k.blen = a.blk_len;
    k.q = (const uint16_t *)a.q;
    k.out = (uint16_t *)a.out;
    k.part_o = (float *)(ws + p.part_o);
    k.part_ml = (float2 *)(ws + p.part_ml);
    k.cum = (int32_t *)(ws + p.cum);
    k.dev_err = a.dev_err;
    k.B = a.B;
    k.base_off = a.base_off;
    k.blen_add = a.blk_len_add;
    k.R = a.R;
    k.G = G;
    k.n_heads = a.n_heads;
    k.n_kv = a.n_kv;
    k.page_size = a.page_size;
    k.max_pages = a.max_pages;
    k.num_pages = a.num_pages;
    k.rows_pad = p.rows_pad;
    k.parts = p.parts;
    k.heads_per_group = geo.heads_per_group;
    k.row_tiles = geo.row_tiles;
    k.waves_per_head = geo.waves_per_head;
    k.scale_log2 = a.scale * 1.4426950408889634f;
    {
      TraceScope ts(a.trace, s);
      const dim3 grid(p.parts, geo.groups), block(geo.block);
      if (geo.rt_per_wave == 1)
        hipLaunchKernelGGL((attn_mfma_kernel<true, 1>), grid, block, kAttnLdsReserve, s, k);
      else if (geo.waves_per_head == 1)
        hipLaunchKernelGGL((attn_mfma_kernel<true, 2>), grid, block, kAttnLdsReserve, s, k);
      else
        hipLaunchKernelGGL((attn_mfma_kernel<false, 2>), grid, block, kAttnLdsReserve, s, k);
    }
    TraceScope ts(a.trace_combine, s);
    const int out_rows = a.n_kv * G * a.R;
    // Sixteen groups per row save a round trip per eight partials of a sequence and cost a workgroup per
    // row: taken where a sequence has more than a batch of partials and the launch at most 32 rows per
    // partial of a sequence.  (Rows, partials: attention and combine with one group -> sixteen, us.
    // 512, 32: 20.0 -> 16.3; 672, 43: 27.1 -> 21.8; 800, 26: 44.1 -> 42.5; 1024, 32: 28.0 -> 26.9;
    // 672, 18: 18.6 -> 18.8; 1024, 16: 18.6 -> 20.1; 1344, 18: 23.1 -> 26.4; 2048, 8: 21.0 -> 30.5.)
    if (p.parts >= 8 * a.B && (long)out_rows * a.B * a.B <= 32L * p.parts)
      hipLaunchKernelGGL(attn_combine_kernel<16>, dim3(out_rows, a.B), dim3(512), 0, s, k);
    else
      hipLaunchKernelGGL(attn_combine_kernel<1>, dim3((out_rows + 7) / 8, a.B), dim3(256), 0, s, k);
  } else {
    AttnF f{};
    f.kp = (const float *)a.k_pages;
    f.vp = (const float *)a.v_pages;
    f.q = (const float *)a.q;
    f.out = (float *)a.out;
    f.bt = a.block_table;
    f.base = a.base_lens;
    f.blen = a.blk_len;
    f.dev_err = a.dev_err;
    f.base_off = a.base_off;
    f.blen_add = a.blk_len_add;
    f.R = a.R;
    f.G = G;
    f.n_heads = a.n_heads;
    f.n_kv = a.n_kv;
    f.page_size = a.page_size;
    f.max_pages = a.max_pages;
    f.num_pages = a.num_pages;
    f.scale = a.scale;
    dim3 grid(a.R, a.n_heads, a.B);
    TraceScope ts(a.trace, s);
    if (a.head_dim == 64) hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(256), 0, s, f);
    else hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(256), 0, s, f);
  }
}

}  // namespace gm
