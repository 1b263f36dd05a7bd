// Device side of the row-sorted order that other translation units' kernels carry along in workgroups of their own (gfx950).
#pragma once
#include "mar_common.h"

// ------------------------------------------------------------ occurrence numbering -----
// Occurrence k of a batch with n edges and cn = chunks*N negatives per side (roles = 3, or 2 for
// the relation-free Dot score, which has no relation occurrences):
//   [0,n) source of edge k | [n,2n) destination | [2n,3n) relation (roles = 3 only) |
//   [roles*n, +cn) destination-replacing negatives | then cn source-replacing negatives
__device__ __forceinline__ int32_t occ_unified_id(const OccArgs& a, int64_t k) {
  const int64_t n = a.n;
  if (k < n) return a.src[k];
  if (k < 2 * n) return a.dst[k - n];
  if (k < a.roles * n) return a.num_nodes + a.rel[k - 2 * n];
  k -= a.roles * n;
  if (k < a.cn) return a.neg_dst[k];
  return a.neg_src[k - a.cn];
}

// Block-wide exclusive scan of one value per thread (BT threads); returns the exclusive
// prefix and the block total through `total`.
// wave_tot: LDS, a word per wave.
template <int BT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total, uint32_t* wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  __syncthreads();                    // protects wave_tot across successive calls
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < BT / 64; ++w) {
    const uint32_t t = wave_tot[w];
    if (w < wave) base += t;
    tot += t;
  }
  *total = tot;
  return base + inc - v;
}

// Lanes of the wave that hold the same digit as this lane (valid lanes only).
__device__ __forceinline__ uint64_t match_digit(uint32_t digit, int bits, bool valid) {
  uint64_t mask = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const bool bit = (digit >> b) & 1u;
    const uint64_t bal = __ballot(bit);
    mask &= bit ? bal : ~bal;
  }
  return mask;
}

// FIRST: computes the keys from the batch's ids and stores them; also resets the owner list's counter.
// h: LDS, a word per digit.
template <int FIRST, int ITEMS>
__device__ __forceinline__ void sort_hist_tile(int tile, uint32_t* h, const OccArgs& a, int64_t n_pos, int sy2, const uint32_t* __restrict__ keys_in,
                                               uint32_t* __restrict__ keys_out, int shift, int bits, int tpad, uint32_t* __restrict__ hist,
                                               int32_t* __restrict__ scalars) {
  const int bins = 1 << bits;
  const int lane = threadIdx.x & 63;
  const int64_t base = (int64_t)tile * (256 * ITEMS);
  const int64_t n3 = a.roles * (int64_t)a.n;
  uint32_t key[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int64_t gr = base + j * 256 + threadIdx.x;
    const int64_t grc = gr < n_pos ? gr : n_pos - 1;
    key[j] = FIRST ? (uint32_t)occ_unified_id(a, grc < n3 ? grc : n3 + (grc - n3) / sy2) : keys_in[grc];
  }
  for (int i = threadIdx.x; i < bins; i += 256) h[i] = 0u;
  if (FIRST && tile == 0 && threadIdx.x == 0) scalars[2] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int64_t gr = base + j * 256 + threadIdx.x;
    const bool valid = gr < n_pos;
    if (FIRST && valid) keys_out[gr] = key[j];
    // one LDS atomic per distinct digit of the wave (a hot row fills whole waves with one key)
    const uint32_t digit = (key[j] >> shift) & (uint32_t)(bins - 1);
    const uint64_t same = match_digit(digit, bits, valid);
    if (valid && (same & ((1ull << lane) - 1ull)) == 0ull) atomicAdd(&h[digit], (uint32_t)__popcll(same));
  }
  __syncthreads();
  for (int i = threadIdx.x; i < bins; i += 256) hist[(size_t)i * tpad + tile] = h[i];
}

// Scatters the tile's elements to their places in digit order.  Global place of an element =
// (elements with a smaller digit anywhere) + (same digit in earlier tiles) + (same digit earlier in this
// tile).  Inside the tile wave w owns a contiguous quarter and walks it 64 consecutive elements at a time,
// so "earlier in this tile" = same digit in earlier waves + earlier rounds of this wave + lower lanes.
// vals_in == NULL: the values are the element indices (first pass).  next_hist: the next pass's counts, digit by digit and tile by
// tile of the places that the elements go to, added to here (whole numbers: the same whatever the order), so that it needs no
// counting pass of its own; it must hold zeros.  lds: SORT_LDS_BYTES.
template <int ITEMS>
__device__ __forceinline__ void sort_scatter_tile(int tile, uint32_t* lds, const uint32_t* __restrict__ keys_in, const int32_t* __restrict__ vals_in,
                                                  uint32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out, const uint32_t* __restrict__ hist,
                                                  uint32_t* __restrict__ next_hist, int64_t n, int shift, int bits, int ntiles, int tpad) {
  typedef uint32_t Digits[1 << MAR_SORT_MAX_BITS];
  Digits* const wcnt = reinterpret_cast<Digits*>(lds);      // [4]: per wave, elements per digit, then their exclusive prefix over waves
  uint32_t* const gbase = lds + (4 << MAR_SORT_MAX_BITS);   // global place of the tile's first element of each digit
  uint32_t* const wave_tot = lds + (5 << MAR_SORT_MAX_BITS);
  const int bins = 1 << bits;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < 4 * bins; i += 256) wcnt[i >> bits][i & (bins - 1)] = 0u;

  // keys and values of this wave's quarter, round r = 64 consecutive elements
  const int64_t q0 = (int64_t)tile * (256 * ITEMS) + (int64_t)wave * (64 * ITEMS) + lane;
  uint32_t key[ITEMS];
  int32_t val[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t idx = q0 + 64 * r;
    key[r] = idx < n ? keys_in[idx] : 0u;
    val[r] = (vals_in && idx < n) ? vals_in[idx] : (int32_t)idx;
  }

  // digit offsets: thread t owns digits [t*per, (t+1)*per), per = 1 or 2; a digit's counts beyond the last tile are not used
  const int per = (bins + 255) / 256;
  uint32_t before[2] = {0u, 0u}, total[2] = {0u, 0u};
  const int d0 = threadIdx.x * per;
  for (int b0 = 0; b0 < ntiles; b0 += 32) {                 // 32 tiles' counts in flight per digit
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j < per && d0 + j < bins) {
        uint4 v[8];
        const uint4* hrow = reinterpret_cast<const uint4*>(hist + (size_t)(d0 + j) * tpad + b0);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = b0 + 4 * i < tpad ? hrow[i] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t c[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int other = b0 + 4 * i + k;
            if (other < ntiles) total[j] += c[k];
            if (other < tile) before[j] += c[k];
          }
        }
      }
    }
  }
  uint32_t tot_all;
  uint32_t run = block_exclusive_scan<256>(total[0] + total[1], &tot_all, wave_tot);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j < per && d0 + j < bins) { gbase[d0 + j] = run + before[j]; run += total[j]; }
  }
  __syncthreads();                                          // counters cleared, gbase written

  uint32_t loc[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = q0 + 64 * r < n;
    const uint32_t digit = (key[r] >> shift) & (uint32_t)(bins - 1);
    const uint64_t same = match_digit(digit, bits, valid);
    const uint32_t lower = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    loc[r] = 0u;
    if (valid) {
      // every lane of a group reads the wave's counter before the group's first lane advances it: one wave
      // executes both accesses in program order
      const uint32_t old = wcnt[wave][digit];
      loc[r] = old + lower;
      if (lower == 0u) wcnt[wave][digit] = old + (uint32_t)__popcll(same);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < bins; d += 256) {
    const uint32_t c0 = wcnt[0][d], c1 = wcnt[1][d], c2 = wcnt[2][d];
    wcnt[0][d] = 0u; wcnt[1][d] = c0; wcnt[2][d] = c0 + c1; wcnt[3][d] = c0 + c1 + c2;
  }
  __syncthreads();
  const int tile_bits = ntiles > 1 ? 32 - __clz(ntiles - 1) : 0;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = q0 + 64 * r < n;
    uint32_t p = 0u;
    if (valid) {
      const uint32_t digit = (key[r] >> shift) & (uint32_t)(bins - 1);
      p = gbase[digit] + wcnt[wave][digit] + loc[r];
      keys_out[p] = key[r];
      vals_out[p] = val[r];
    }
    // uniform; one atomic per distinct (digit, tile) of the wave.  A row that many waves hold makes them queue (48,000 rows, power
    // law 1.2: 20 us, uniform 12, without counts 9; 90,000: 36, 15, 10); gathered over the workgroup in LDS first: 18 and 25, but
    // 2 us more where no row is hot, and beside a pass no faster.
    if (next_hist) {
      const uint32_t digit = (key[r] >> (shift + bits)) & (uint32_t)(bins - 1), to = p / (256 * ITEMS);
      const uint64_t same = match_digit(digit | to << bits, bits + tile_bits, valid);
      if (valid && (same & ((1ull << lane) - 1ull)) == 0ull) atomicAdd(&next_hist[(size_t)digit * tpad + to], (uint32_t)__popcll(same));
    }
  }
}

// Heads of segments: positions whose id differs from their predecessor's.
__device__ __forceinline__ bool is_head(const uint32_t* __restrict__ ids, int64_t p, int64_t n) { return p < n && (p == 0 || ids[p - 1] != ids[p]); }

// Ranks in one launch: each of j.blocks workgroups takes `per` neighbouring tiles of MAR_RANK_TILE positions, counts the heads before
// them itself (at most 98,304 ids from the cache, beside a pass; 16 loads a thread in flight, or it would outlast the pass), and
// writes what k_rank_count, k_rank_apply and k_debug_uniq do.
__device__ __forceinline__ void sort_rank_tiles(int first, int last, uint32_t* lds, const MarSortJob& j) {
  static_assert(MAR_RANK_TILE == 1024, "16 bytes of ids a thread");
  const uint32_t* __restrict__ ids = j.keys_in;
  const int n = j.n_pos, lane = threadIdx.x & 63;
  const uint32_t nodes = (uint32_t)j.occ.num_nodes;
  auto count = [&](uint4 v, uint32_t before, int p, uint32_t& all, uint32_t& of_nodes) {   // heads among positions p .. p + 3, all below n
    const uint32_t up = __shfl_up(v.w, 1);
    const uint32_t prev = lane ? up : before;
    const bool h0 = p == 0 || prev != v.x, h1 = v.x != v.y, h2 = v.y != v.z, h3 = v.z != v.w;
    all += (h0 ? 1u : 0u) + (h1 ? 1u : 0u) + (h2 ? 1u : 0u) + (h3 ? 1u : 0u);
    of_nodes += (h0 && v.x < nodes ? 1u : 0u) + (h1 && v.y < nodes ? 1u : 0u) + (h2 && v.z < nodes ? 1u : 0u) + (h3 && v.w < nodes ? 1u : 0u);
  };
  uint32_t all = 0u, of_nodes = 0u, tot;                    // heads before these tiles, and those of nodes
  constexpr int UN = 16;
  for (int t = 0; t < first; t += UN) {                     // uniform
    uint4 v[UN];
    uint32_t before[UN];
#pragma unroll
    for (int k = 0; k < UN; ++k) {
      const int p = (min(t + k, first - 1)) * MAR_RANK_TILE + 4 * (int)threadIdx.x;
      v[k] = *reinterpret_cast<const uint4*>(ids + p);
      before[k] = lane == 0 && p > 0 ? ids[p - 1] : 0u;
    }
#pragma unroll
    for (int k = 0; k < UN; ++k) if (t + k < first) count(v[k], before[k], (t + k) * MAR_RANK_TILE + 4 * (int)threadIdx.x, all, of_nodes);
  }
  uint32_t base, base_n;
  block_exclusive_scan<256>(all, &base, lds);
  block_exclusive_scan<256>(of_nodes, &base_n, lds);
  for (int t = first; t < last; ++t) {
    const int p0 = t * MAR_RANK_TILE + 4 * (int)threadIdx.x;
    uint32_t id[4], prev = p0 > 0 && p0 <= n ? ids[p0 - 1] : 0u, c = 0u, cn = 0u;
    bool head[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      id[k] = p0 + k < n ? ids[p0 + k] : 0u;
      head[k] = p0 + k < n && (p0 + k == 0 || prev != id[k]);
      prev = id[k];
      c += head[k] ? 1u : 0u; cn += head[k] && id[k] < nodes ? 1u : 0u;
    }
    uint32_t heads = base + block_exclusive_scan<256>(c, &tot, lds);
    base += tot;
    uint32_t heads_n = base_n + block_exclusive_scan<256>(cn, &tot, lds);
    base_n += tot;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int p = p0 + k;
      if (p < n) {
        const bool node = id[k] < nodes;
        heads += head[k] ? 1u : 0u;
        heads_n += head[k] && node ? 1u : 0u;
        j.rank_sorted[p] = (int32_t)heads - 1;
        if (head[k]) {
          if (node) { if (j.uniq_nodes) j.uniq_nodes[heads - 1u] = (int32_t)id[k]; }
          else if (j.uniq_rels) j.uniq_rels[heads - heads_n - 1u] = (int32_t)(id[k] - nodes);   // every node's head lies before
        }
        if (p == n - 1 && j.num_uniq) { j.num_uniq[0] = (int32_t)heads_n; j.num_uniq[1] = (int32_t)(heads - heads_n); }
      }
    }
  }
}

// What a workgroup with blockIdx.x < j.blocks does in place of its kernel's own work (256 threads; lds: SORT_LDS_BYTES).
template <int KINDS> __device__ __forceinline__ void sort_job(const MarSortJob& j, uint32_t* lds) {
  const int block = (int)blockIdx.x;
  if ((KINDS & MAR_SORT_HIST) && (j.kind & MAR_SORT_HIST)) {
    if (block >= j.tiles) return;                           // (a workgroup a tile: mar_sort_slot)
    sort_hist_tile<1, MAR_SORT_RIDE_ITEMS>(block, lds, j.occ, j.n_pos, j.sy2, nullptr, j.keys_out, 0, j.bits, j.tpad, j.hist, j.scalars);
    for (int i = block * 256 + threadIdx.x; i < j.zero_words; i += 256 * j.tiles) j.next_hist[i] = 0u;
  }
  if ((KINDS & MAR_SORT_SCATTER) && (j.kind & MAR_SORT_SCATTER)) {
    for (int tile = block; tile < j.tiles; tile += j.blocks) {
      if (tile != block) __syncthreads();                   // the counters of the tile before have been read
      sort_scatter_tile<MAR_SORT_RIDE_ITEMS>(tile, lds, j.keys_in, j.vals_in, j.keys_out, j.vals_out, j.hist, j.next_hist, j.n_pos, j.shift, j.bits, j.tiles, j.tpad);
    }
  }
  if ((KINDS & MAR_SORT_RANKS) && (j.kind & MAR_SORT_RANKS)) {
    const int per = (j.tiles + j.blocks - 1) / j.blocks;
    if (block * per < j.tiles) sort_rank_tiles(block * per, min(j.tiles, (block + 1) * per), lds, j);
  }
}
