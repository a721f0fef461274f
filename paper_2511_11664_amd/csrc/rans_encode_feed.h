// rans_encode_feed.h -- rANS encoder for few streams: one coding wave per work-group, three waves that feed it
//
// Part of the one translation unit rans_if.hip (included there, in this order); not a stand-alone header.
#pragma once

#include "rans_encode.h"

namespace {

// What bounds a coder with few streams (S up to a few hundred in all the chunks' groups of a compute unit) is the
// instruction stream of one wave: nothing else runs on its SIMD, so every instruction between two rows is time.
// k_encode spends about 30 on a row (symbol address and load or stage, table address and look-up, entry unpacking,
// bookkeeping).  Here the work-group's first wave only codes, and the other three hand it ready table entries:
//
//   feeders   symbol of (row, stream) -> table entry -> a slot of an LDS tile [row][lane], 16 bytes a slot; the
//             symbols of the tiles ahead wait in registers
//   coder     one 16-byte LDS read at a constant offset per row, then the nine vector instructions of Eq. 2 and the
//             word's store
//
// Tiles of kFeedRows rows alternate between two buffers with one barrier a tile.  Rows past the chunk's start,
// absent streams of the ragged last row and lanes without a stream get an entry that leaves the state alone, so the
// coder has no cases.
//
// The entry as fed: exact tables {lim, mx, F, 2^M - f | sh << 24} (the 24-bit multiply-add ignores the shift count on
// top of its operand), else {floor(2^32/f), f, F, 2^M - f} with a correction step.
//
// Measured, k_encode before against this: one chunk of 32 streams 946 -> 271 us in CSR form (6211 rows, 44 ns each), 235 us
// dense (6272 rows, 37 ns); 25 chunks of 64 x 64 symbols 15.0 -> 9.9 us; where the line to k_encode lies: encoder_is_fed.
// Who waits (cycles of a tile of 24 rows, stamped around the barrier in a copy): the coder works 2235 and waits 75 in CSR form,
// 2050 and 50 dense; the feeders work 1705 to 1855 and 1130 to 1285 of that.  So the coder is what a row waits for: its eleven
// instructions are about 72 cycles, of which the two LDS accesses are 32, and take 93 and 85 beside the feeders.
// Dense symbols requested two tiles at a time instead of one, entries laid out by the table build: the compress call of those
// 198 chunks 25.9 -> 24.5 us, of the 25 chunks 16.8 -> 16.7.
//
// When a stream's word area runs full, all streams of the wave move their complete blocks to scratch: a spill costs
// the wave the same whether one lane or all of them take part, and streams of one tensor fill up at about the same rate.
constexpr uint32_t kFeedWaves = kWG / 64 - 1;      // feeding waves
constexpr uint32_t kFeedPer = 8;                   // rows of a tile per feeding wave
constexpr uint32_t kFeedRows = kFeedWaves * kFeedPer;
constexpr uint32_t kFeedTileBytes = kFeedRows * kFeedSpw * 16;

// LDS_TAB: the 16-byte entries are staged in LDS (built there when build_tab), else read from global memory.
template <class Src, bool LDS_TAB, bool MUL24>
__global__ __launch_bounds__(kWG) void k_encode_feed(Src src, const uint2 *g_tab, const uint4 *g_tab4, uint32_t A, uint32_t M,
                                                     uint32_t S, uint32_t cs, CtlRef ctl, uint16_t *scratch, uint32_t capw,
                                                     uint32_t groups, uint32_t *wg_pub, unsigned long long *chunk_acc,
                                                     uint8_t *out, uint64_t cap, uint64_t *d_stream_bytes, uint32_t rw,
                                                     int build_tab, NormArgs na) {
  extern __shared__ __align__(16) uint32_t l_mem[];  // the only LDS of this kernel: the word areas start at offset kEncGuard
  const uint32_t k = blockIdx.x / groups, g = blockIdx.x % groups;
  const uint32_t lane = threadIdx.x & 63, wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto bail = [&]() {  // every exit publishes a total, see k_encode
    if (threadIdx.x == 0) {
      __hip_atomic_store(wg_pub + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(chunk_acc + k, 1ull << 40, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  const bool builds = LDS_TAB && build_tab;  // the table build looks at the status itself
  EncCounts counts{};
  if (builds) counts = enc_request_counts(ctl, na, A);
  const bool failed = !builds && group_has_status(ctl, l_mem);
  // l_D is known already: the tensor's size, or what the CSR kernels stored
  const uint64_t len = std::is_same<Src, SrcDense>::value ? na.n_elems : ctl->len_d;
  const uint32_t nc = enc_chunks(len, cs);
  auto give_up = [&]() {  // the size of a container that there is not, see k_encode
    if (threadIdx.x == 0 && d_stream_bytes && (blockIdx.x == 0 || (k == nc - 1 && g == groups - 1))) *d_stream_bytes = 0;
    bail();
  };
  if (failed) {
    give_up();
    return;
  }
  if (k >= nc) {  // the grid is sized for the longest D (an empty one never gets here: k_normalize and k_gather write it)
    bail();
    return;
  }
  const uint32_t totalM = 1u << M;
  // LDS: [guard][word areas of 64 streams][table][16 words][two tiles, before and after the coding small tables]
  const uint32_t stride = enc_area_stride(rw);
  uint32_t *l_tab = l_mem + (kEncGuard + stride * kFeedSpw) / 4;  // stride * 64 is a multiple of 16
  uint32_t *sh = l_tab + (LDS_TAB ? A * 4 : 0);
  uint32_t *l_tile = sh + 16;
  src.init(ctl);
  const uint64_t chunk_len = cs ? cs : len;
  const uint64_t base = (uint64_t)k * chunk_len;
  const uint64_t n_here = len - base < chunk_len ? len - base : chunk_len;
  const uint32_t j0 = g * kFeedSpw + lane;
  const uint32_t rows_full = (uint32_t)n_here / S, rem_row = (uint32_t)n_here - rows_full * S;  // l_D < 2^32
  const uint32_t rows = rows_full + (rem_row ? 1u : 0u);
  const uint32_t n_tiles = (rows + kFeedRows - 1) / kFeedRows;
  // Coding step p takes row rows - 1 - p; step kFeedRows i + 8 (wv - 1) + u of tile i is feeder wv's u-th.  Lanes
  // without a stream code another one's symbols to no effect; where a row does not reach a stream or there is no row
  // any more, the load goes to a valid place and the entry fed is the neutral one.  fetch() only loads, with no use
  // of what arrives, so that all of a wave's loads of two tiles are in flight together.
  const uint32_t jc = j0 < S ? j0 : S - 1;
  const uint32_t nnz = (uint32_t)src.nnz_of();
  // The part of D = v (+) c (+) r that the eight steps from p on lie in: 0, 1, 2, or 3 where they straddle two parts
  // or are not all there.
  auto part_of = [&](uint32_t p) -> uint32_t {
    if ((p == 0 && rem_row) || p + kFeedPer > rows) return 3u;
    if constexpr (std::is_same<Src, SrcDense>::value) return 0u;
    const uint32_t hi = (uint32_t)base + (rows - 1 - p) * S + (g * kFeedSpw + kFeedSpw < S ? g * kFeedSpw + kFeedSpw - 1 : S - 1);
    const uint32_t lo = (uint32_t)base + (rows - kFeedPer - p) * S + g * kFeedSpw;
    return hi < nnz ? 0u : (lo >= 2 * nnz ? 2u : (lo >= nnz && hi < 2 * nnz ? 1u : 3u));
  };
  auto index_of = [&](uint32_t p) {  // in D, for any step (CSR)
    const uint32_t i = (uint32_t)base + (p < rows ? rows - 1 - p : 0u) * S + jc, last = (uint32_t)(len - 1);
    return i < last ? i : last;
  };
  typedef const __attribute__((address_space(1))) uint8_t *gptr;
  struct __attribute__((packed, aligned(1))) U32 { uint32_t x; };
  typedef const __attribute__((address_space(1))) U32 *gptr32;
  auto fetch = [&](uint32_t *d, uint32_t tile) __attribute__((always_inline)) {
    const uint32_t p = tile * kFeedRows + (wv - 1) * kFeedPer;
    if constexpr (std::is_same<Src, SrcDense>::value) {  // a chunk has at most 2^30 symbols here
      const int32_t i0 = ((int32_t)rows - 1 - (int32_t)p) * (int32_t)S + (int32_t)jc, last = (int32_t)n_here - 1;
      const gptr col = (gptr)(uintptr_t)(src.bytes() + base);
#pragma unroll
      for (uint32_t u = 0; u < kFeedPer; u++) {
        int32_t i = i0 - (int32_t)(u * S);
        i = i < 0 ? 0 : i;
        d[u] = col[i < last ? i : last];
      }
    } else {
      // a symbol's four bytes from its address on, whatever part it is in (c and row_end follow v and r in the workspace)
      const uint32_t part = part_of(p);
      if (part != 3) {
        const uint32_t wide = part ? 1u : 0u;
        const uint64_t i0 = base + (uint64_t)(rows - 1 - p) * S;
        uint64_t a = part == 0 ? (uint64_t)(uintptr_t)src.v_ptr() + i0
                   : part == 1 ? (uint64_t)(uintptr_t)src.c_ptr() + 2 * (i0 - nnz)
                               : (uint64_t)(uintptr_t)src.r_ptr() + 2 * (i0 - 2ull * nnz);
        const uint32_t o = jc << wide;
#pragma unroll
        for (uint32_t u = 0; u < kFeedPer; u++) {
          d[u] = ((gptr32)((gptr)(uintptr_t)a + o))->x;
          a -= (uint64_t)S << wide;
        }
      } else {
#pragma unroll
        for (uint32_t u = 0; u < kFeedPer; u++) {
          const uint32_t i = index_of(p + u);
          const uint64_t a = i < nnz ? (uint64_t)(uintptr_t)src.v_ptr() + i
                           : i < 2ull * nnz ? (uint64_t)(uintptr_t)src.c_ptr() + 2ull * (i - nnz)
                                            : (uint64_t)(uintptr_t)src.r_ptr() + 2 * (i - 2ull * nnz);
          d[u] = ((gptr32)(uintptr_t)a)->x;
        }
      }
    }
  };
  // Two tiles' symbols are requested at a time, when the two before have arrived: across the branches of fetch() and feed() the
  // compiler cannot tell how old a request is, so a wave that waits for one waits for all of them.  Requested a tile at a time,
  // every tile of a dense tensor took a trip to memory.  CSR: a tile at a time, two in turn; its fetch() and feed() are long and
  // two more copies of each cost more than the trips (one chunk of 32 streams 307 us, 321 with two tiles at a time).
  constexpr bool DENSE = std::is_same<Src, SrcDense>::value;
  uint32_t w0[kFeedPer], wa[2][kFeedPer], wb[2][kFeedPer];
  // Not past the end of the chunk, where a wave would wait for symbols that nobody takes: compress calls of 4 to 200 rows took 0.3 to
  // 0.4 % longer so, in the mean.  The first three tiles are requested whatever there is: with conditions around them too, 0.6 % longer.
  auto fetch_two = [&](uint32_t (&w)[2][kFeedPer], uint32_t tile) __attribute__((always_inline)) {  // tile + 1 past the end: valid addresses, never fed
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    fetch(w[0], tile);
    fetch(w[1], tile + 1);
  };
  if (wv) {  // on their way while the table is built
    fetch(w0, 0);
    fetch(wa[0], 1);
    if (DENSE) fetch(wa[1], 2);
  }
  uint32_t exact_tab;
  uint64_t dir_off, payload_off;
  if (builds) {
    const EncTable t = enc_build_table<true>(ctl, na, counts, A, (uint32_t)len, nc, l_tab, l_tile, sh + 15);
    if (!t.ok) {
      give_up();
      return;
    }
    dir_off = t.dir_off; payload_off = t.payload_off;
    exact_tab = t.exact;
  } else {
    dir_off = ctl->dir_off; payload_off = ctl->payload_off;
    exact_tab = ctl->enc_exact;
    if (LDS_TAB) {
      for (uint32_t a = threadIdx.x; a < A; a += kWG) {
        if (exact_tab) {
          ((uint4 *)l_tab)[a] = enc_fed_form(g_tab4[a]);
        } else {
          const uint2 q = g_tab[a];
          ((uint4 *)l_tab)[a] = make_uint4(q.x, q.y & 0xffffu, q.y >> 16, totalM - (q.y & 0xffffu));
        }
      }
      __syncthreads();
    }
  }
  typedef __attribute__((address_space(3))) uint16_t lds_u16;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  if ((uint32_t)(uintptr_t)(lds_u16 *)l_mem != 0) {  // cannot happen without static LDS; the slot arithmetic relies on it
    if (threadIdx.x == 0) set_status(ctl, RANS_ERR_HIP);
    give_up();
    return;
  }
  const bool live = threadIdx.x < kFeedSpw && j0 < S;
  uint32_t s = kL;
  const uint32_t colb = kEncGuard + stride * lane;  // the stream's area: slots colb, colb + 2, ..., top - 2
  const uint32_t top = colb + 2 * rw;
  uint32_t wp = top - 2;                            // LDS address of the slot of the next word
  uint16_t *const g0 = scratch + (uint64_t)blockIdx.x * kFeedSpw * capw + lane * 8;  // block-major, as in k_encode
  uint16_t *gp = g0;
  auto words_in_area = [&]() { return (top - 2 - wp) >> 1; };
  auto spill = [&]() {  // complete 8-word blocks, oldest first, to scratch; the rest to the top of the area
    const uint32_t n_used = words_in_area();
    const uint32_t nblk = n_used >> 3, r = n_used & 7;
    for (uint32_t b = 0; b < nblk; b++) {
      const lds_u32 *q = (const lds_u32 *)(uintptr_t)(top - 16 * (b + 1));
      *(uint4 *)gp = make_uint4(q[0], q[1], q[2], q[3]);
      gp += kFeedSpw * 8;
    }
    if (r && nblk) {
      for (uint32_t i = 0; i < r; i++)
        *(lds_u16 *)(uintptr_t)(top - 2 * r + 2 * i) = *(const lds_u16 *)(uintptr_t)(wp + 2 + 2 * i);
    }
    wp = top - 2 - 2 * r;
  };
  auto entry_of = [&](uint32_t a, bool exact) -> uint4 {  // in the form the coder takes
    if (LDS_TAB) return ((const uint4 *)l_tab)[a];
    if (exact) return enc_fed_form(g_tab4[a]);
    const uint2 q = g_tab[a];
    return make_uint4(q.x, q.y & 0xffffu, q.y >> 16, totalM - (q.y & 0xffffu));
  };
  auto feed = [&](const uint32_t *d, uint32_t tile, auto exact_tag) __attribute__((always_inline)) {
    constexpr bool EXACT = decltype(exact_tag)::value;
    const uint32_t p = tile * kFeedRows + (wv - 1) * kFeedPer;
    uint4 *to = (uint4 *)l_tile + (tile & 1) * (kFeedRows * kFeedSpw) + ((wv - 1) * kFeedPer) * kFeedSpw + lane;
    const uint32_t part = part_of(p);
    if (part != 3) {
      const uint32_t mask = part ? 0xffffu : 0xffu;
      uint4 e[kFeedPer];
#pragma unroll
      for (uint32_t u = 0; u < kFeedPer; u++) e[u] = entry_of(d[u] & mask, EXACT);
#pragma unroll
      for (uint32_t u = 0; u < kFeedPer; u++) to[u * kFeedSpw] = e[u];
    } else {
#pragma unroll
      for (uint32_t u = 0; u < kFeedPer; u++) {
        const uint32_t a = d[u] & (std::is_same<Src, SrcDense>::value || index_of(p + u) < nnz ? 0xffu : 0xffffu);
        const bool none = p + u >= rows || (p + u == 0 && rem_row && j0 >= rem_row);
        to[u * kFeedSpw] = none ? (EXACT ? make_uint4(0xffffffffu, 0, 0, 0) : make_uint4(0, totalM, 0, 0)) : entry_of(a, EXACT);
      }
    }
  };
  auto run = [&](auto exact_tag) {
    constexpr bool EXACT = decltype(exact_tag)::value;
    const uint32_t sh_lim = 32 - M;
    auto row = [&](const uint4 &e) {
      const bool c = EXACT ? s > e.x : (s >> sh_lim) >= e.y;  // too large for this symbol: emit 16 bits
      *(lds_u16 *)(uintptr_t)wp = (uint16_t)s;                // speculative: the slot counts only if c
      s = c ? s >> 16 : s;
      wp = c ? wp - 2 : wp;
      if constexpr (EXACT) {
        const uint32_t q = __umulhi(s, e.y) >> (e.w >> 24);
        s = (MUL24 ? __umul24(q, e.w) : q * (e.w & 0xffffffu)) + (s + e.z);
      } else {
        uint32_t q = __umulhi(s, e.x);
        const uint32_t rem = s - (MUL24 ? __umul24(q, e.y) : q * e.y);
        q += rem >= e.y ? 1u : 0u;
        s = s + e.z + (MUL24 ? __umul24(q, e.w) : q * e.w);
      }
    };
    auto code_tile = [&](uint32_t tile) __attribute__((always_inline)) {
      const uint4 *tp = (const uint4 *)l_tile + (tile & 1) * (kFeedRows * kFeedSpw) + lane;
      uint4 e[2][8];
#pragma unroll
      for (uint32_t u = 0; u < 8; u++) e[0][u] = tp[u * kFeedSpw];
#pragma unroll
      for (uint32_t b = 0; b < kFeedRows / 8; b++) {
        if (b + 1 < kFeedRows / 8) {
#pragma unroll
          for (uint32_t u = 0; u < 8; u++) e[(b + 1) & 1][u] = tp[((b + 1) * 8 + u) * kFeedSpw];
        }
#pragma unroll
        for (uint32_t u = 0; u < 8; u++) row(e[b & 1][u]);
        if (__any(wp < colb + 2 * 7)) spill();  // at least eight free slots at the start of every batch
      }
    };
    if (wv) feed(w0, 0, exact_tag);
    else __builtin_amdgcn_s_setprio(3);  // nothing may delay the one wave that everything waits for
    lds_barrier();
    // two or four tiles a turn, so that the waiting symbols never move between registers
    auto step = [&](uint32_t t, const uint32_t *w) __attribute__((always_inline)) {
      if (wv == 0) code_tile(t);
      else if (t + 1 < n_tiles) feed(w, t + 1, exact_tag);
      lds_barrier();
      return t + 1 < n_tiles;
    };
    if constexpr (DENSE) {
      for (uint32_t t = 0;; t += 4) {
        if (wv && t + 3 < n_tiles) fetch_two(wb, t + 3);
        if (!step(t, wa[0]) || !step(t + 1, wa[1])) break;
        if (wv && t + 5 < n_tiles) fetch_two(wa, t + 5);
        if (!step(t + 2, wb[0]) || !step(t + 3, wb[1])) break;
      }
    } else {
      for (uint32_t t = 0;; t += 2) {
        if (wv) fetch(w0, t + 2);  // past the end: valid addresses, never fed
        if (!step(t, wa[0])) break;
        if (wv) fetch(wa[0], t + 3);
        if (!step(t + 1, w0)) break;
      }
    }
    if (wv == 0) __builtin_amdgcn_s_setprio(0);
  };
  if (exact_tab) run(std::true_type{});
  else run(std::false_type{});
  const uint32_t n_lds = live ? words_in_area() : 0;
  const uint32_t nbg = live ? (uint32_t)((gp - g0) / (kFeedSpw * 8)) : 0;
  const uint32_t nw = 8 * nbg + n_lds;
  uint32_t tot;
  const uint32_t ex = block_excl_scan<kWG>(nw, sh, &tot);
  if (threadIdx.x == 0) {
    __hip_atomic_store(wg_pub + blockIdx.x, tot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(chunk_acc + k, (1ull << 40) | tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (builds && blockIdx.x == 0 && threadIdx.x == kWG - 64) {  // the header, see k_encode
    if (na.dense) ctl->len_d = len;
    write_header(ctl, na, len, nc, dir_off, payload_off);
  }
  // what the whole work-group needs of each stream to move its words
  uint32_t *t_n = l_tile, *t_ex = t_n + kFeedSpw, *t_at = t_ex + kFeedSpw, *t_bex = t_at + kFeedSpw, *t_nbg = t_bex + kFeedSpw;
  uint32_t n_spilled;
  const uint32_t bex = block_excl_scan<kWG>(nbg, sh, &n_spilled);
  if (threadIdx.x < kFeedSpw) {
    t_n[lane] = n_lds;
    t_ex[lane] = ex;
    t_at[lane] = (wp + 2) >> 1;
    t_bex[lane] = bex;
    t_nbg[lane] = nbg;
  }
  __syncthreads();
  const EncBefore before = enc_look_back(ctl, k, g, groups, S, chunk_acc, wg_pub, sh);
  const uint64_t off = before.off, pre = before.pre;
  if (before.failed) {  // uniform
    if (threadIdx.x == 0) {
      if (get_status(ctl) == 0) set_status(ctl, RANS_ERR_HIP);
      if (k == nc - 1 && g == groups - 1 && d_stream_bytes) *d_stream_bytes = 0;
    }
    return;
  }
  if (!enc_directory(ctl, EncPlace{off, pre, dir_off, payload_off, cap, k, g, groups, nc, S, tot}, out, d_stream_bytes)) return;
  uint8_t *ck = out + payload_off + off;
  if (live) {
    st32(ck + 4ull * j0, s);
    st32(ck + 4ull * S + 4ull * j0, nw);
  }
  uint16_t *dst = (uint16_t *)(ck + 8ull * S) + pre;  // first word of this group
  for (uint32_t L0 = threadIdx.x >> 3; L0 < kFeedSpw; L0 += kWG / 8)
    enc_copy_words((const uint16_t *)l_mem, t_at[L0], dst + t_ex[L0], t_n[L0], lane & 7);
  // the spilled blocks of the work-group as one list in stream order, inside a stream the last written first
  constexpr int kU = 8;
  for (uint32_t i0 = threadIdx.x; i0 < n_spilled; i0 += kU * kWG) {
    uint4 q[kU];
    uint32_t d_off[kU];
#pragma unroll
    for (int u = 0; u < kU; u++) {
      const uint32_t i = i0 + u * kWG;
      d_off[u] = ~0u;
      if (i < n_spilled) {
        uint32_t o = 0;  // the last stream whose first block is at or before i
#pragma unroll
        for (uint32_t step = kFeedSpw / 2; step; step >>= 1) o = t_bex[o + step] <= i ? o + step : o;
        const uint32_t bi = i - t_bex[o];
        d_off[u] = t_ex[o] + t_n[o] + 8 * bi;
        q[u] = *(const uint4 *)(scratch + (uint64_t)blockIdx.x * kFeedSpw * capw + ((uint64_t)(t_nbg[o] - 1 - bi) * kFeedSpw + o) * 8);
      }
    }
#pragma unroll
    for (int u = 0; u < kU; u++)
      if (d_off[u] != ~0u) *(Block16 *)(dst + d_off[u]) = Block16{q[u].x, q[u].y, q[u].z, q[u].w};
  }
  if (g == groups - 1 && live && j0 == S - 1 && ((pre + tot) & 1)) dst[tot] = 0;  // pad the chunk to 4 bytes
}

}  // namespace
