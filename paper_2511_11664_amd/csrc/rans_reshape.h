// rans_reshape.h -- reshape search (Sec. 3.2, Algorithm 1)
//
// Part of the one translation unit rans_if.hip (included there, in this order); not a stand-alone header.
#pragma once

#include "rans_common.h"

namespace {

// ------------------------------------------------------------------ kernels: reshape search (Sec. 3.2)

// The quantised tensor is fixed over all reshapes [N, K]: so are the nonzero values v and their number.  Only the
// histograms of the column indices (position mod K) and of the row counts change, and both follow from the zero mask
// alone.  Three launches: k_rs_mask reads the tensor once (mask, histogram of v), k_rs_count makes every histogram
// from the mask, an eighth of the tensor, and k_rs_cost sums the entropies and walks the candidates.
// Measured, the former seven launches (mask, scan of its tile counts, columns by an LDS addition per nonzero, rows by
// look-ups in a prefix array, costs) against these: 25.7 M symbols with 18 candidates 142 -> 38 us of kernels
// (10 + 19 + 9), 100 352 symbols with 12 candidates 37 -> 25 us.
constexpr uint32_t kRsTile = kWG * 16;       // symbols of a step of k_rs_mask
constexpr uint32_t kRsMaskBlocks = 1024;    // its work-groups at most: 16 waves on a compute unit
constexpr uint32_t kRsWG = 1024;             // threads of k_rs_count and k_rs_cost
constexpr uint32_t kRsColRows = 16;          // rows a thread of the column counts adds up bit by bit (5 planes)
constexpr uint32_t kRsColBlock = (kRsWG / 32) * kRsColRows;  // rows of a work-group of the column counts
constexpr uint32_t kRsHalo = 9;              // words behind a piece: a row that starts in it ends at most 255 positions on
constexpr uint32_t kRsPiece = 4 * kRsWG - 12;  // mask words of a piece of the row counts (a multiple of 4)
static_assert(kRsPiece + kRsHalo <= 4 * kRsWG && kRsPiece % 4 == 0, "four words a thread");
struct RsCands {
  uint32_t n;
  uint16_t K[RANS_RESHAPE_MAX_CAND];
};
struct RsOffsets {  // first bin of each candidate's row-count histogram; entry n = total
  uint32_t hr[RANS_RESHAPE_MAX_CAND + 1];
  uint32_t rep_stride, n_rep;  // partial histograms: work-group b of the row counts adds to copy b % n_rep
};
// Candidates are grouped so that the members of a group have a common multiple L of at most kRsLcmMax: one
// histogram of the nonzero positions modulo L then serves every member, whose own column histogram
// (positions modulo K) is that one folded K-periodically.
constexpr uint32_t kRsLcmMax = 32768;
struct RsGroups {
  uint32_t n;
  uint32_t L[RANS_RESHAPE_MAX_CAND];        // residues of group g: a multiple of every K in it
  uint32_t off[RANS_RESHAPE_MAX_CAND + 1];  // first word of its histogram in hl; entry n = total
  uint32_t wg0[RANS_RESHAPE_MAX_CAND + 1];  // its first work-group among the column counts' ones; entry n = their number
  uint8_t of[RANS_RESHAPE_MAX_CAND];        // group of candidate k
};
struct RsGrid {  // shares of the grid of k_rs_count, in this order: row counts, column counts, sums of hv_part
  uint32_t n_rows, n_cols, n_sum;
  uint32_t n_part;      // partial histograms of v
  uint32_t wg_words;    // mask words of a work-group of the row counts (a multiple of 4), its pieces' size below
  uint32_t piece;
  // copies of a bin in the row counts' LDS histogram: one per lane for the first n_wide candidates, the ones with the
  // most rows and the fewest bins, 1 << rep_log2 for the others
  uint32_t n_wide, rep_log2;
};

// Zero mask and histogram of v.  Bound by the LDS additions of the nonzeros (one each), so the grid fills the chip with
// waves.  A work-group stores its histogram whole: a thousand work-groups' additions to the same 256
// addresses take 12 us at the end of the kernel.  25.7 M symbols, 30 % nonzeros: 31 us with 512 work-groups, a branch
// per symbol and a scan per tile, now 10 us (2.8 TB/s).
__global__ __launch_bounds__(kWG) void k_rs_mask(const uint8_t *sym, uint32_t n, int aligned, uint32_t n_tiles,
                                                 uint16_t *mask16, uint32_t *hv_part, uint32_t *zero, uint32_t zero_words) {
  // eight counters per value, one per lane residue: activations have a few very frequent values, and a wave's
  // additions to one LDS address are performed one after the other
  __shared__ uint32_t h[256 * 8];
  for (uint32_t i = threadIdx.x; i < 256 * 8; i += kWG) h[i] = 0;
  // what the next kernel adds to
  for (uint32_t i = blockIdx.x * kWG + threadIdx.x; i < zero_words; i += gridDim.x * kWG) zero[i] = 0;
  const uint32_t rep = threadIdx.x & 7u;
  __syncthreads();
  const uint32_t n_entries = 2 * ((n + 31) / 32);  // whole words
  uint32_t w[4];
  load16w(sym, (uint64_t)blockIdx.x * kRsTile + threadIdx.x * 16, n, aligned, w);  // the grid has at most n_tiles work-groups
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const uint64_t e0 = (uint64_t)tile * kRsTile + threadIdx.x * 16;
    uint32_t nw[4] = {0, 0, 0, 0};  // the next tile's symbols are on their way while this one is looked at
    if (tile + gridDim.x < n_tiles) load16w(sym, e0 + (uint64_t)gridDim.x * kRsTile, n, aligned, nw);
    if ((e0 >> 4) < n_entries) mask16[e0 >> 4] = (uint16_t)nonzero_mask16(w);
#pragma unroll
    for (int k = 0; k < 16; k++) {
      const uint32_t b = (w[k >> 2] >> (8 * (k & 3))) & 0xffu;
      if (b) atomicAdd(&h[b * 8u + rep], 1u);
    }
#pragma unroll
    for (int j = 0; j < 4; j++) w[j] = nw[j];
  }
  __syncthreads();
  uint32_t t = 0;  // kWG == 256: a thread per value
#pragma unroll
  for (int r = 0; r < 8; r++) t += h[threadIdx.x * 8 + r];
  hv_part[(size_t)blockIdx.x * 256 + threadIdx.x] = t;
}

// Histogram of the nonzero positions modulo L (one group of candidates; see RsGroups), bit-sliced: a thread takes the
// 32 residues 32 w .. 32 w + 31, reads their bits in one row of L positions after the other - a 32-bit window at any
// bit position - and adds them up in 32 vertical counters, five bit planes for up to kRsColRows rows: about 20
// instructions per 32 positions whatever the density, where a walk over the set bits with an LDS addition each took
// 25 us on 25.7 M symbols with 30 % nonzeros.  A work-group is 32 windows by 32 interleaved rows.  Turning the planes into
// counts is the part that small tensors wait for: one counter at a time it made searches of 20 000 to 10^6 symbols with
// few divisors and 10 % nonzeros slower than the walk (111 479 symbols, 2 candidates 18.7 -> 22.8 us; four at a time 20.2, 99 999
// symbols, 4 candidates 21.5 / 21.6 / 19.6).  A tensor without any nonzero still takes up to 5 us longer than with the walk.
__device__ __forceinline__ void rs_count_cols(const uint32_t *mask, uint32_t n, uint32_t L, uint32_t bx, uint32_t *hl,
                                              uint32_t *s_c /* 16 * 33 words */) {
  const uint32_t n_words = (n + 31) / 32;
  const uint32_t W = (L + 31) / 32, n_wb = (W + 31) / 32, R = (n + L - 1) / L;
  const uint32_t wx = bx % n_wb, rb = bx / n_wb;
  const uint32_t wl = threadIdx.x & 31u, w = wx * 32 + wl;
  const uint32_t r0 = rb * kRsColBlock + (threadIdx.x >> 5);
  for (uint32_t i = threadIdx.x; i < 16 * 33; i += kRsWG) s_c[i] = 0;
  __syncthreads();
  if (w < W && r0 < R) {
    const uint32_t keep = L - 32 * w >= 32 ? ~0u : (1u << (L - 32 * w)) - 1u;  // the next row's bits are not this window's
    uint32_t p[5] = {0, 0, 0, 0, 0};
    // two rounds of eight rows, the loads of a round in flight together (n <= 2^30: no overflow)
#pragma unroll 1
    for (uint32_t r1 = r0; r1 < r0 + kRsColRows * (kRsWG / 32) && r1 < R; r1 += 8 * (kRsWG / 32)) {
      uint32_t lo[8], hi[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; u++) {
        const uint32_t r = r1 + u * (kRsWG / 32), at = (r * L + 32 * w) >> 5;
        const bool a = r < R && at < n_words, b = r < R && at + 1 < n_words;
        lo[u] = mask[a ? at : 0];  // always a load, so that none hides behind a branch
        hi[u] = mask[b ? at + 1 : 0];
        lo[u] = a ? lo[u] : 0u;
        hi[u] = b ? hi[u] : 0u;
      }
#pragma unroll
      for (uint32_t u = 0; u < 8; u++) {
        uint32_t x = __builtin_amdgcn_alignbit(hi[u], lo[u], ((r1 + u * (kRsWG / 32)) * L) & 31u) & keep;
#pragma unroll
        for (int j = 0; j < 5; j++) {
          const uint32_t c = p[j] & x;
          p[j] ^= x;
          x = c;
        }
      }
    }
    // four residues' counters at a time as the bytes of a word (at most kRsColRows each), added up as two pairs of 16-bit
    // fields: the work-group's 32 rows of counters make at most 32 * kRsColRows
    static_assert(kRsColRows < 256 && 32 * kRsColRows < 65536, "fields");
#pragma unroll 2  // short code: straight-line code that runs once is waited for line by line
    for (uint32_t b = 0; b < 8; b++) {
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < 5; j++) c |= ((p[j] >> b) & 0x01010101u) << j;
      atomicAdd(&s_c[(2 * b) * 33 + wl], c & 0x00ff00ffu);             // residues b, b + 16
      atomicAdd(&s_c[(2 * b + 1) * 33 + wl], (c >> 8) & 0x00ff00ffu);  // b + 8, b + 24
    }
  }
  __syncthreads();
  {
    const uint32_t i = threadIdx.x;  // kRsWG == 32 * 32
    const uint32_t r = i & 31u, two = s_c[(2 * (r & 7u) + ((r >> 3) & 1u)) * 33 + (i >> 5)];
    const uint32_t t = r & 16u ? two >> 16 : two & 0xffffu, at = wx * 1024 + i;
    if (t && at < L) atomicAdd(&hl[at], t);
  }
}

// Row-count histograms of all candidates over one range of mask words, every row counted where it starts.  The range
// is taken in pieces of up to kRsPiece words, which go to LDS with the number of nonzeros before each word, so a row's
// count is a population count of one window (K <= 32) or the difference of two look-ups: no pass over memory per
// candidate, no prefix array, no scan over the tensor.  K = 2 and 4 - the most rows - are counted for the whole word at
// a time in registers, 8 and 16 as fields of a word.  K = 1 is left out: its row counts are the zero mask itself.
// One work-group per compute unit: every work-group ends with additions to some hundred addresses, and they cost more
// than the counting when there are a thousand work-groups.  A short row's count takes few values, so the
// additions of a wave meet in one bin: the candidates with short rows have a counter per lane, summed by a wave scan
// before neighbouring bins leave together (a lone lane's addition per bin instead: 14 us more on 25.7 M symbols).
__device__ __forceinline__ void rs_count_rows(const uint32_t *mask, uint32_t n, const RsCands &cands, const RsOffsets &offs,
                                              const RsGrid &gr, uint32_t bx, uint32_t *hr, uint2 *s_wp /* 4 kRsWG */,
                                              uint32_t *s_h, uint32_t *sh, uint4 *s_cand) {
  const uint32_t n_words = (n + 31) / 32;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t bins = offs.hr[cands.n], wide = offs.hr[gr.n_wide], rl = gr.rep_log2;
  uint32_t *s_n = s_h + (wide << 6) - (wide << rl);  // bin b >= wide has its copies at s_n[b << rl]
  for (uint32_t i = threadIdx.x; i < (wide << 6) + ((bins - wide) << rl); i += kRsWG) s_h[i] = 0;
  uint32_t at2 = ~0u, at4 = ~0u, at8 = ~0u, at16 = ~0u;  // first bins of K = 2, 4, 8, 16 where they are candidates
  for (uint32_t k = 0; k < cands.n && cands.K[k] <= 16; k++) {
    const uint32_t K = cands.K[k];
    if (K == 2) at2 = offs.hr[k];
    if (K == 4) at4 = offs.hr[k];
    if (K == 8) at8 = offs.hr[k];
    if (K == 16) at16 = offs.hr[k];
  }
  auto slot = [&](uint32_t bin) {  // uniform choice: `bin` is any bin of one candidate
    return bin < wide ? s_h + (bin << 6) + lane : s_n + (bin << rl) + (lane & ((1u << rl) - 1u));
  };
  uint32_t *const s8 = slot(at8 == ~0u ? 0 : at8), *const s16 = slot(at16 == ~0u ? 0 : at16);
  const uint32_t l8 = at8 < wide ? 6 : rl, l16 = at16 < wide ? 6 : rl;
  uint32_t c2[3] = {0, 0, 0}, c4[5] = {0, 0, 0, 0, 0};
  const uint32_t g0 = bx * gr.wg_words, g1 = g0 + gr.wg_words < n_words ? g0 + gr.wg_words : n_words;
  for (uint32_t w0 = g0; w0 < g1; w0 += gr.piece) {
    const uint32_t w1 = w0 + gr.piece < g1 ? w0 + gr.piece : g1;
    const uint32_t at = w0 + 4 * threadIdx.x;
    uint32_t w[4] = {0, 0, 0, 0};
    if (at < w1 + kRsHalo) {
      if (at + 4 <= n_words) {  // the mask starts 256-byte aligned, `at` is a multiple of 4
        const uint4 q = *(const uint4 *)(mask + at);
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
      } else {
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) w[j] = at + j < n_words ? mask[at + j] : 0u;
      }
    }
    // every candidate's rows of this piece - their number, the first one's position, K, the first bin - by a thread each:
    // with the two divisions made by every wave for every candidate the kernel took 4 us more (25.7 M symbols)
    if (threadIdx.x < cands.n) {
      const uint32_t K = cands.K[threadIdx.x], s = w0 * 32, e = w1 * 32 < n ? w1 * 32 : n;
      const uint32_t i0 = (s + K - 1) / K, i1 = (e + K - 1) / K;
      const bool other = K <= 16 && (K & (K - 1)) == 0;  // K = 1, 2, 4, 8, 16
      s_cand[threadIdx.x] = make_uint4(other ? 0u : i1 - i0, i0 * K - s, K, offs.hr[threadIdx.x]);
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan<kRsWG>(__popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]), sh, &tot);
#pragma unroll
    for (uint32_t j = 0; j < 4; j++) {
      s_wp[4 * threadIdx.x + j] = make_uint2(w[j], ex);
      ex += __popc(w[j]);
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t j = 0; j < 4; j++) {
      if (at + j >= w1) continue;
      const uint32_t p0 = (at + j) * 32, m = s_wp[4 * threadIdx.x + j].x;
      if (p0 + 32 <= n) {  // all of the word's rows exist (n is a multiple of every K here)
        const uint32_t x = m & 0x55555555u, y = (m >> 1) & 0x55555555u;
        const uint32_t two = (uint32_t)__popc(x & y), one = (uint32_t)__popc(x ^ y);
        c2[2] += two; c2[1] += one; c2[0] += 16u - two - one;
        uint32_t t = m - ((m >> 1) & 0x55555555u);
        t = (t & 0x33333333u) + ((t >> 2) & 0x33333333u);  // eight fields of four bits: their population counts (0 .. 4)
        if (at4 != ~0u) {
          uint32_t rest = 8;
#pragma unroll
          for (uint32_t v = 1; v <= 4; v++) {
            const uint32_t z = t ^ (v * 0x11111111u);
            const uint32_t ne = (z | (z >> 1) | (z >> 2)) & 0x11111111u;  // bit 3 of a field is never set
            const uint32_t eq = 8u - (uint32_t)__popc(ne);
            c4[v] += eq;
            rest -= eq;
          }
          c4[0] += rest;
        }
        if (at8 != ~0u) {
          const uint32_t b = (t + (t >> 4)) & 0x0f0f0f0fu;  // four fields of eight bits
#pragma unroll
          for (int f = 0; f < 4; f++) atomicAdd(s8 + (((b >> (8 * f)) & 0xffu) << l8), 1u);
        }
        if (at16 != ~0u) {
          atomicAdd(s16 + ((uint32_t)__popc(m & 0xffffu) << l16), 1u);
          atomicAdd(s16 + ((uint32_t)__popc(m >> 16) << l16), 1u);
        }
      } else {  // the word with the end of the tensor: row by row
#pragma unroll 1
        for (uint32_t i = 0; i < 4; i++) {
          const uint32_t first = i == 0 ? at2 : i == 1 ? at4 : i == 2 ? at8 : at16, K = 2u << i;
          if (first == ~0u) continue;
          for (uint32_t q = 0; q < 32 && p0 + q < n; q += K)
            atomicAdd(slot(first + (uint32_t)__popc((m >> q) & ((1u << K) - 1u))), 1u);
        }
      }
    }
    for (uint32_t k = 0; k < cands.n; k++) {
      const uint4 c = s_cand[k];
      const uint32_t cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.x), first = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.y);
      const uint32_t K = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.z), bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.w);
      // many rows: the work-group takes them together; few: one wave, while the others take other candidates
      const bool all = cnt >= kRsWG / 2;
      if (!all && wave != k % (kRsWG / 64)) continue;
      const uint32_t step = all ? kRsWG : 64;
      uint32_t *const h = slot(bin);
      const uint32_t hs = bin < wide ? 6 : rl;
      if (K <= 32) {
        const uint32_t keep = K == 32 ? ~0u : (1u << K) - 1u;
        for (uint32_t i = all ? threadIdx.x : lane; i < cnt; i += step) {
          const uint32_t g = first + __umul24(i, K);
          const uint32_t r = (uint32_t)__popc(__builtin_amdgcn_alignbit(s_wp[(g >> 5) + 1].x, s_wp[g >> 5].x, g & 31u) & keep);
          atomicAdd(h + (r << hs), 1u);
        }
      } else {
        for (uint32_t i = all ? threadIdx.x : lane; i < cnt; i += step) {
          const uint32_t g = first + __umul24(i, K), f = g + K;
          const uint2 a = s_wp[g >> 5], b = s_wp[f >> 5];
          const uint32_t r = (b.y + (uint32_t)__popc(b.x & ((1u << (f & 31u)) - 1u))) -
                             (a.y + (uint32_t)__popc(a.x & ((1u << (g & 31u)) - 1u)));
          atomicAdd(h + (r << hs), 1u);
        }
      }
    }
    __syncthreads();  // the words make room for the next piece
  }
  // the register counts: one addition per wave and value
#pragma unroll
  for (uint32_t v = 0; v < 3; v++) {
    const uint32_t t = wave_incl_sum_scan(c2[v]);
    if (lane == 63 && at2 != ~0u) atomicAdd(slot(at2 + v), t);
  }
#pragma unroll
  for (uint32_t v = 0; v < 5; v++) {
    const uint32_t t = wave_incl_sum_scan(c4[v]);
    if (lane == 63 && at4 != ~0u) atomicAdd(slot(at4 + v), t);
  }
  __syncthreads();
  for (uint32_t i = wave; i < wide; i += kRsWG / 64) {
    const uint32_t t = wave_incl_sum_scan(s_h[(i << 6) + lane]);
    if (lane == 63) s_h[i << 6] = t;
  }
  __syncthreads();
  uint32_t *out = hr + (size_t)(bx % offs.n_rep) * offs.rep_stride;
  for (uint32_t i = threadIdx.x; i < bins; i += kRsWG) {  // neighbours together: a lone lane's addition costs as much as a wave's
    uint32_t t = 0;
    if (i < wide) t = s_h[i << 6];
    else
      for (uint32_t r = 0; r < 1u << rl; r++) t += s_n[(i << rl) + r];
    if (t) atomicAdd(&out[i], t);
  }
}

// All histograms that depend on the reshape, and the sum of the partial histograms of v, side by side in one grid:
// none of the three fills the chip for long.
__global__ __launch_bounds__(kRsWG) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_rs_count(const uint32_t *mask, uint32_t n, RsCands cands, RsOffsets offs,
                                                  RsGroups grps, RsGrid gr, const uint32_t *hv_part, uint32_t *hv,
                                                  uint32_t *hl, uint32_t *hr) {
  extern __shared__ uint32_t s_dyn[];
  __shared__ uint32_t sh[kRsWG / 64];
  __shared__ uint4 s_cand[RANS_RESHAPE_MAX_CAND];
  uint32_t b = blockIdx.x;
  if (b < gr.n_rows) {
    rs_count_rows(mask, n, cands, offs, gr, b, hr, (uint2 *)s_dyn, s_dyn + 8 * kRsWG, sh, s_cand);
    return;
  }
  b -= gr.n_rows;
  if (b < gr.n_cols) {
    uint32_t g = 0;
    while (grps.wg0[g + 1] <= b) g++;  // uniform; entry n is n_cols
    rs_count_cols(mask, n, grps.L[g], b - grps.wg0[g], hl + grps.off[g], s_dyn);
    return;
  }
  b -= gr.n_cols;  // up to 64 of the partial histograms, a quarter of the threads each
  if (threadIdx.x < 256) s_dyn[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t v = threadIdx.x & 255u;
  uint32_t t = 0;
#pragma unroll 8
  for (uint32_t u = 0; u < 16; u++) {
    const uint32_t i = b * 64 + u * 4 + (threadIdx.x >> 8);
    const uint32_t x = hv_part[(size_t)(i < gr.n_part ? i : 0) * 256 + v];
    t += i < gr.n_part ? x : 0u;
  }
  atomicAdd(&s_dyn[v], t);
  __syncthreads();
  if (threadIdx.x < 256 && s_dyn[v]) atomicAdd(&hv[v], s_dyn[v]);
}

// Costs and the walk of Algorithm 1.  One work-group per candidate sums its entropy terms in binary64
// (a fixed tree: lanes, then waves); the work-group that finishes last walks the candidates from the
// largest N down.  costs[] and the ticket live in the zeroed part of the workspace.
__global__ __launch_bounds__(kRsWG) void k_rs_cost(RsCands cands, uint32_t n, uint32_t q_bits, const uint32_t *hv,
                                                 const uint32_t *hl, const uint32_t *hr, RsOffsets offs, RsGroups grps,
                                                 double *costs, uint32_t *ticket, rans_reshape_result *res) {
  __shared__ double s_part[kWG / 64];
  __shared__ uint64_t s_sum[kRsWG / 64];
  __shared__ uint32_t s_ticket;
  __shared__ uint32_t s_cnt[257];  // the candidate's histogram of c and r (K <= 2^8)
  __shared__ uint32_t s_v[256];
  __shared__ double s_cost[RANS_RESHAPE_MAX_CAND];
  const uint32_t k = blockIdx.x, two_q = 1u << q_bits;
  const uint32_t K = cands.K[k], N = n / K;
  // every load of the work-group is under way before the first is waited for: hv, the row counts' copies (K = 1 has
  // none: its row counts are the zero mask itself) and the group's histogram of positions modulo L.  That one is
  // folded K-periodically (K divides L): a thread stays on one column, as the threads' stride is a multiple of K
  const uint32_t my_v = threadIdx.x < 256 ? hv[threadIdx.x] : 0u;
  const uint32_t n_r = K == 1 ? 0u : (K + 1) * offs.n_rep;
  // i / d = i (2^21 / d + 1) >> 21 for the i < 2056 and d <= 257 here (i d < 2^21): two divisions in all instead of one per index
  const uint32_t inv_r = (1u << 21) / (K + 1) + 1u, inv_c = (1u << 21) / K + 1u;
  const uint32_t col = threadIdx.x - ((threadIdx.x * inv_c) >> 21) * K;  // threadIdx.x % K
  uint32_t my_r[3], my_a[3];
  static_assert(257 * 8 <= 3 * kRsWG, "eight copies at most");
#pragma unroll
  for (uint32_t u = 0; u < 3; u++) {
    const uint32_t i = threadIdx.x + u * kRsWG, q = (i * inv_r) >> 21;
    my_a[u] = i - q * (K + 1);
    my_r[u] = u * kRsWG < n_r && i < n_r ? hr[(size_t)q * offs.rep_stride + offs.hr[k] + my_a[u]] : 0u;
  }
  if (threadIdx.x < 257) s_cnt[threadIdx.x] = 0;
  uint32_t my_c = 0;
  if (K > 1) {  // K = 1: all nonzeros are in the one column
    const uint32_t g = grps.of[k], L = grps.L[g], step = ((kRsWG * inv_c) >> 21) * K;
    const uint32_t *hg = hl + grps.off[g];
    if (threadIdx.x < step)
      for (uint32_t i0 = threadIdx.x; i0 < L; i0 += 16 * step) {
        uint32_t t[16];
#pragma unroll
        for (uint32_t u = 0; u < 16; u++) t[u] = hg[i0 + u * step < L ? i0 + u * step : 0];
#pragma unroll
        for (uint32_t u = 0; u < 16; u++) my_c += i0 + u * step < L ? t[u] : 0u;
      }
  }
  const uint32_t nnz = (uint32_t)block_sum64<kRsWG>(threadIdx.x ? my_v : 0u, s_sum);
  const bool bad = __syncthreads_or(threadIdx.x < 256 && threadIdx.x >= two_q && my_v != 0) != 0;  // not symbols of this bit width
  {
    if (threadIdx.x < 256) s_v[threadIdx.x] = threadIdx.x ? my_v : 0u;
    if (my_c) atomicAdd(&s_cnt[col], my_c);
    if (K == 1 && threadIdx.x == 0) s_cnt[0] = nnz;
#pragma unroll
    for (uint32_t u = 0; u < 3; u++)
      if (my_r[u]) atomicAdd(&s_cnt[my_a[u]], my_r[u]);
    __syncthreads();
    const uint32_t A = K + 1 > two_q ? K + 1 : two_q;
    const uint64_t len = 2ull * nnz + N;
    double h = 0.0;
    for (uint32_t a = threadIdx.x; a < A && threadIdx.x < kWG; a += kWG) {
      uint64_t c = 0;
      if (a < two_q) c += s_v[a];
      if (a <= K) c += s_cnt[a];
      if (K == 1 && a <= 1) c += a ? nnz : n - nnz;
      if (c) {
        const double p = (double)c / (double)len;
        h -= p * log2(p);
      }
    }
    const uint64_t bits = wave_incl_scan64((uint64_t)__double_as_longlong(h), [](uint64_t x, uint64_t y) {
      return (uint64_t)__double_as_longlong(__longlong_as_double((long long)x) + __longlong_as_double((long long)y));
    });
    if ((threadIdx.x & 63) == 63 && threadIdx.x < kWG) s_part[threadIdx.x >> 6] = __longlong_as_double((long long)bits);
    __syncthreads();
    if (threadIdx.x == 0) {
      double H = 0.0;
      for (int w = 0; w < kWG / 64; w++) H += s_part[w];
      // device-scope store, then the ticket: the last work-group reads every cost with device-scope loads
      __hip_atomic_store(costs + k, (double)len * H, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_ticket = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
  if (s_ticket != gridDim.x - 1) return;
  __atomic_thread_fence(__ATOMIC_ACQUIRE);
  // a thread per candidate, then the walk: one trip to memory for all costs
  static_assert(RANS_RESHAPE_MAX_CAND <= kRsWG, "a thread per candidate");
  if (threadIdx.x < cands.n) {
    const double cost = __hip_atomic_load(costs + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_cost[threadIdx.x] = cost;
    res->cand_rows[threadIdx.x] = n / cands.K[threadIdx.x];
    res->cand_cost[threadIdx.x] = cost;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double best = INFINITY, prev = INFINITY;
  uint64_t n_tilde = n;
  uint32_t evaluated = 0;
  for (uint32_t i = 0; i < cands.n; i++) {
    const double cost = s_cost[i];
    evaluated++;
    if (cost < best) {
      best = cost;
      n_tilde = n / cands.K[i];
    }
    if (cost > prev) break;  // the walk stops after this one
    prev = cost;
  }
  if (bad) {  // a symbol outside {0 .. 2^Q - 1}: no meaningful result
    best = __longlong_as_double(0x7ff8000000000000ll);
    n_tilde = n;
    evaluated = 0;
  }
  res->rows = n_tilde;
  res->cols = n / n_tilde;
  res->cost_bits = best;
  res->n_evaluated = evaluated;
  res->n_candidates = cands.n;
}

// an empty domain: rows = T, cols = 1, cost +inf
__global__ __launch_bounds__(kWG) void k_rs_empty(uint32_t n, uint32_t q_bits, const uint32_t *hv, rans_reshape_result *res) {
  const bool bad = __syncthreads_or((threadIdx.x >> q_bits) != 0 && hv[threadIdx.x] != 0) != 0;
  if (threadIdx.x != 0) return;
  res->rows = n;
  res->cols = 1;
  res->cost_bits = bad ? __longlong_as_double(0x7ff8000000000000ll) : INFINITY;
  res->n_evaluated = 0;
  res->n_candidates = 0;
}

}  // namespace
