// Integer side of the training step: counter-based sampling and table fill, and the row-sorted order of the batch's
// gradient rows (gfx950).
//
// The gradient rows (one per occurrence of a table row in the batch, and per part of a negative's) are put in order of
// their "unified id" (a node id, or num_nodes + relation id) by a stable radix sort, so that every table row owns a
// contiguous segment of positions whose order -- the occurrence order -- is the same in every run: the per-row sums that
// follow are bit-reproducible.  The reduce reads segment borders off the sorted ids; ranks of the rows among the unique
// rows and the ascending unique list are formed only where a caller asks for them.
#include "mar_common.h"
#include "mar_sort_dev.h"

// ---------------------------------------------------------------- Philox4x32-10 -----
// Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy as 1, 2, 3" (SC'11).
__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3,
                                              uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
}

// Negative sampling (Sec. 2.1; degree-based fraction of Table 1).  One thread per pair of
// slots: counter = (slot >> 1, 2*chunk + side, step lo, step hi), key = seed; even slot takes
// output words 0,1 and odd slot words 2,3 as a 64-bit value x; id = mulhi64(x, range).
__global__ void __launch_bounds__(256)
k_sample(uint64_t seed, uint64_t step, int64_t num_nodes, const int32_t* __restrict__ es,
         const int32_t* __restrict__ ed, int64_t num_edges, int C, int N, int Ndeg,
         int32_t* __restrict__ neg_src, int32_t* __restrict__ neg_dst) {
  const int pairs = (N + 1) >> 1;
  const int64_t total = (int64_t)2 * C * pairs;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int pr = (int)(i % pairs);
  const int cs = (int)(i / pairs);            // 2*chunk + side
  const int side = cs & 1, chunk = cs >> 1;
  uint32_t c0 = (uint32_t)pr, c1 = (uint32_t)cs, c2 = (uint32_t)step, c3 = (uint32_t)(step >> 32);
  philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t x[2] = {(uint64_t)c0 | ((uint64_t)c1 << 32), (uint64_t)c2 | ((uint64_t)c3 << 32)};
  int32_t* out = (side == MAR_SIDE_SRC ? neg_src : neg_dst) + (size_t)chunk * N;
  const int32_t* endpoint = side == MAR_SIDE_SRC ? es : ed;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int slot = 2 * pr + h;
    if (slot >= N) break;
    int32_t id;
    if (slot < Ndeg) id = endpoint[__umul64hi(x[h], (uint64_t)num_edges)];
    else id = (int32_t)__umul64hi(x[h], (uint64_t)num_nodes);
    out[slot] = id;
  }
}

// N(0, std^2) fill: counter = (block lo, block hi, 0, 0x80000000 | table) gives elements
// 4*block .. 4*block+3 by two Box-Muller pairs on 24-bit uniforms.
__global__ void __launch_bounds__(256)
k_init_normal(float* __restrict__ tab, int64_t n, uint64_t seed, uint32_t table, float std) {
  const int64_t nblocks = (n + 3) >> 2;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nblocks; b += (int64_t)gridDim.x * blockDim.x) {
    uint32_t c0 = (uint32_t)b, c1 = (uint32_t)((uint64_t)b >> 32), c2 = 0u, c3 = 0x80000000u | table;
    philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint32_t o[4] = {c0, c1, c2, c3};
    float z[4];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float u1 = (float)((o[2 * p] >> 8) + 1u) * (1.0f / 16777216.0f);
      const float u2 = (float)(o[2 * p + 1] >> 8) * (1.0f / 16777216.0f);
      const float r = sqrtf(-2.0f * logf(u1));
      float sn, cs;
      sincospif(2.0f * u2, &sn, &cs);
      z[2 * p] = r * cs * std;
      z[2 * p + 1] = r * sn * std;
    }
    const int64_t e = b << 2;
    if (e + 3 < n) {
      *reinterpret_cast<float4*>(tab + e) = make_float4(z[0], z[1], z[2], z[3]);
    } else {
      for (int k = 0; k < 4 && e + k < n; ++k) tab[e + k] = z[k];
    }
  }
}

__global__ void __launch_bounds__(256) k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Blocks of the index kernels stay at 256 threads: they run beside the contraction kernels on a second stream and have
// to fit into the wave slots and registers those leave free on a CU.  (k_sort_one, 1,024 threads and 96 KB of LDS, stands alone in
// the pipeline, or ahead of or beside the gather of a small batch that does not carry the order.)

// ------------------------------------------------ row-sorted order of the gradient rows -----
// Gradient row gr belongs to occurrence k = gr (edge side, gr < roles*n) or to part (gr - roles*n) % sy2
// of negative occurrence roles*n + (gr - roles*n) / sy2; its sort key is the unified id of the occurrence's
// table row.  A least-significant-digit radix sort with digits of `bits` bits puts the gradient rows in key order;
// every pass is stable, so equal keys stay in gradient-row order.
// Small batches: the step's own launches carry the pieces along (MarSortJob, mar_sort_slot); in the pipeline k_sort_one up to
// mar_sort_one_limit.  Else one pass = k_sort_hist (digit counts per tile of 256 ITEMS elements)
// + k_sort_scatter (each tile derives its digits' global offsets from the counts of all tiles and scatters its elements).
// Counts are kept digit by digit, the tiles' counts of a digit side by side, so that the thread that owns a digit reads
// them 16 bytes at a time.
// Small batches take small tiles (few elements per thread, many workgroups: their time is latency), large ones tiles of
// 4096 (see sort_items).  Every tile reads bins x tiles counts, so that the reads grow with the square of the batch:
// 250,000 gradient rows and 27-bit ids (three passes of 9 bits) 62 tiles x 31,744 counts a pass, 8 MB of cached reads;
// sixteen times the batch 2 GB.

template <int FIRST, int ITEMS>
__global__ void __launch_bounds__(256)
k_sort_hist(OccArgs a, int64_t n_pos, int sy2, const uint32_t* __restrict__ keys_in, uint32_t* __restrict__ keys_out, int shift, int bits,
            int tpad, uint32_t* __restrict__ hist, int32_t* __restrict__ scalars) {
  __shared__ uint32_t h[1 << MAR_SORT_MAX_BITS];
  sort_hist_tile<FIRST, ITEMS>(blockIdx.x, h, a, n_pos, sy2, keys_in, keys_out, shift, bits, tpad, hist, scalars);
}

template <int ITEMS>
__global__ void __launch_bounds__(256)
k_sort_scatter(const uint32_t* __restrict__ keys_in, const int32_t* __restrict__ vals_in, uint32_t* __restrict__ keys_out,
               int32_t* __restrict__ vals_out, const uint32_t* __restrict__ hist, int64_t n, int shift, int bits, int ntiles, int tpad) {
  __shared__ uint32_t lds[SORT_LDS_BYTES / 4];
  sort_scatter_tile<ITEMS>(blockIdx.x, lds, keys_in, vals_in, keys_out, vals_out, hist, nullptr, n, shift, bits, ntiles, tpad);
}

// The whole sort of a small batch (at most MAR_SORT_ONE rows) in one workgroup: wave w owns 64 `rounds` consecutive elements,
// element `idx` = round r, lane l of it, in registers; between two passes keys and values change places through LDS.
// Bound by the latency of its own chain (16 waves on one CU; 2 to 3 passes of ballots and counters): 11,000 rows, two passes 27 us
// against 20 in four launches, but the host issues one launch for two a pass.
template <int ROUNDS>
__global__ void __launch_bounds__(1024)
k_sort_one(OccArgs a, int n, int sy2, int passes, int bits, uint32_t* __restrict__ ids_sorted, int32_t* __restrict__ perm, int32_t* __restrict__ scalars) {
  __shared__ uint32_t buf[1024 * ROUNDS], wave_tot[16];
  __shared__ uint32_t cnt[16][1 << MAR_SORT_MAX_BITS];      // per wave: elements per digit, then the place of its first of each digit
  const int bins = 1 << bits, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n3 = a.roles * a.n;
  const int rounds = (n + 1023) / 1024;                     // uniform, at most ROUNDS
  const int q0 = wave * 64 * rounds + lane;
  uint32_t key[ROUNDS];
  int32_t val[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int idx = q0 + 64 * r;
    key[r] = r < rounds && idx < n ? (uint32_t)occ_unified_id(a, idx < n3 ? idx : n3 + (idx - n3) / sy2) : 0u;
    val[r] = idx;
  }
  if (threadIdx.x == 0) scalars[2] = 0;
  for (int p = 0; p < passes; ++p) {
    const int shift = p * bits;
    for (int i = threadIdx.x; i < 16 << bits; i += 1024) cnt[i >> bits][i & (bins - 1)] = 0u;
    __syncthreads();
    uint32_t place[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      place[r] = 0u;
      if (r < rounds) {                                     // uniform
        const bool valid = q0 + 64 * r < n;
        const uint32_t digit = (key[r] >> shift) & (uint32_t)(bins - 1);
        const uint64_t same = match_digit(digit, bits, valid);
        const uint32_t lower = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        if (valid) {                                        // as in k_sort_scatter: read by all before the group's first lane writes
          const uint32_t old = cnt[wave][digit];
          place[r] = old + lower;
          if (lower == 0u) cnt[wave][digit] = old + (uint32_t)__popcll(same);
        }
      }
    }
    __syncthreads();
    uint32_t c[16], sum = 0u, all;
    const int d = threadIdx.x;
#pragma unroll
    for (int w = 0; w < 16; ++w) { c[w] = d < bins ? cnt[w][d] : 0u; sum += c[w]; }
    uint32_t first = block_exclusive_scan<1024>(sum, &all, wave_tot);
    if (d < bins) {
#pragma unroll
      for (int w = 0; w < 16; ++w) { cnt[w][d] = first; first += c[w]; }
    }
    __syncthreads();
    const bool last = p == passes - 1;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      if (r < rounds && q0 + 64 * r < n) {
        place[r] += cnt[wave][(key[r] >> shift) & (uint32_t)(bins - 1)];
        if (last) { ids_sorted[place[r]] = key[r]; perm[place[r]] = val[r]; }
        else buf[place[r]] = key[r];
      }
    }
    if (last) return;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) if (r < rounds && q0 + 64 * r < n) key[r] = buf[q0 + 64 * r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) if (r < rounds && q0 + 64 * r < n) buf[place[r]] = (uint32_t)val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) if (r < rounds && q0 + 64 * r < n) val[r] = (int32_t)buf[q0 + 64 * r];
  }
}

// Ranks (debug outputs, staged pipeline): a position whose id differs from its predecessor's heads a segment; a row's rank
// is the number of heads before it.  k_rank_count counts the heads of MAR_RANK_TILE positions each; k_rank_apply adds
// up the counts of the tiles before its own and writes the rank of every position and of every gradient row, the
// ascending unique list and, into scalars, the number of unique rows and of unique nodes.
__global__ void __launch_bounds__(256) k_rank_count(const uint32_t* __restrict__ ids, int64_t n, uint32_t* __restrict__ counts) {
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < MAR_RANK_TILE / 256; ++j) c += is_head(ids, (int64_t)blockIdx.x * MAR_RANK_TILE + threadIdx.x * (MAR_RANK_TILE / 256) + j, n) ? 1u : 0u;
  uint32_t tot;
  __shared__ uint32_t wave_tot[4];
  block_exclusive_scan<256>(c, &tot, wave_tot);
  if (threadIdx.x == 0) counts[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(256)
k_rank_apply(const uint32_t* __restrict__ ids, const int32_t* __restrict__ perm, int64_t n, const uint32_t* __restrict__ counts, int32_t num_nodes,
             int32_t* __restrict__ rank_sorted, uint32_t* __restrict__ rank_of_row, int32_t* __restrict__ uniq, int32_t* __restrict__ scalars) {
  constexpr int PER = MAR_RANK_TILE / 256;
  uint32_t before = 0;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) before += counts[i];
  uint32_t base, c = 0, tot;
  __shared__ uint32_t wave_tot[4];
  block_exclusive_scan<256>(before, &base, wave_tot);
  const int64_t p0 = (int64_t)blockIdx.x * MAR_RANK_TILE + threadIdx.x * PER;
  bool head[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) { head[j] = is_head(ids, p0 + j, n); c += head[j] ? 1u : 0u; }
  uint32_t heads = base + block_exclusive_scan<256>(c, &tot, wave_tot);   // heads before this thread's positions
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int64_t p = p0 + j;
    if (p >= n) break;
    heads += head[j] ? 1u : 0u;
    const uint32_t id = ids[p];
    rank_sorted[p] = (int32_t)heads - 1;
    rank_of_row[perm[p]] = heads - 1u;
    if (head[j]) {
      uniq[heads - 1u] = (int32_t)id;
      // the first relation's rank is the number of unique nodes
      if (id >= (uint32_t)num_nodes && (p == 0 || ids[p - 1] < (uint32_t)num_nodes)) scalars[1] = (int32_t)heads - 1;
    }
    if (p == n - 1) { scalars[0] = (int32_t)heads; if (id < (uint32_t)num_nodes) scalars[1] = (int32_t)heads; }
  }
}

// Copies the unique id lists into the caller's debug buffers.
__global__ void __launch_bounds__(256)
k_debug_uniq(const int32_t* __restrict__ uniq, const int32_t* __restrict__ scalars, int32_t num_nodes,
             int32_t* __restrict__ num_uniq, int32_t* __restrict__ uniq_nodes, int32_t* __restrict__ uniq_rels) {
  const int total = scalars[0], un = scalars[1];
  if (blockIdx.x == 0 && threadIdx.x == 0 && num_uniq) { num_uniq[0] = un; num_uniq[1] = total - un; }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    if (i < un) { if (uniq_nodes) uniq_nodes[i] = uniq[i]; }
    else if (uniq_rels) uniq_rels[i - un] = uniq[i] - num_nodes;
  }
}

// ------------------------------------------------------------------- launchers -----
static inline unsigned grid_for(int64_t n, int threads, unsigned cap) {
  int64_t g = (n + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

hipError_t mar_launch_init(const mar_ctx* c, int fill, hipStream_t st) {
  const MarDims& d = c->dm;
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, (uint32_t*)c->L.scalars, (int64_t)16, 0u);
  if (fill) {
    const int64_t nn = d.num_nodes * d.dim, nr = (int64_t)d.num_rels * d.dim;
    hipLaunchKernelGGL(k_init_normal, dim3(grid_for((nn + 3) / 4, 256, 1 << 16)), dim3(256), 0, st,
                       c->node_emb, nn, c->cfg.seed, 0u, c->cfg.init_std);
    hipLaunchKernelGGL(k_init_normal, dim3(grid_for((nr + 3) / 4, 256, 1 << 16)), dim3(256), 0, st,
                       c->rel_emb, nr, c->cfg.seed, 1u, c->cfg.init_std);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nn, 256, 1 << 16)), dim3(256), 0, st, (uint32_t*)c->node_state, nn, 0u);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nr, 256, 1 << 16)), dim3(256), 0, st, (uint32_t*)c->rel_state, nr, 0u);
  }
  return hipGetLastError();
}

hipError_t mar_launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 256, 4096)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t mar_launch_sample(const mar_ctx* c, uint64_t step, const int32_t* es, const int32_t* ed,
                             int64_t num_edges, int32_t* neg_src, int32_t* neg_dst, hipStream_t st) {
  const MarDims& d = c->dm;
  const int64_t total = (int64_t)2 * d.C * ((d.N + 1) / 2);
  hipLaunchKernelGGL(k_sample, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, c->cfg.seed, step,
                     d.num_nodes, es, ed, num_edges, d.C, d.N, d.Ndeg, neg_src, neg_dst);
  return hipGetLastError();
}

template <int ITEMS>
static void launch_sort(const mar_ctx* c, const MarBatch& b, const OccArgs& a, hipStream_t st) {
  const MarDims& d = c->dm;
  const MarLayout& L = c->L;
  const int ntiles = (int)((b.n_pos + 256 * ITEMS - 1) / (256 * ITEMS)), tpad = (ntiles + 3) & ~3;
  const uint32_t* kin = L.keys0;
  const int32_t* vin = nullptr;
  for (int p = 0; p < d.sort_passes; ++p) {
    const bool last = p == d.sort_passes - 1;
    uint32_t* kout = last ? L.ids_sorted : L.kbuf[p & 1];
    int32_t* vout = last ? L.perm : L.vbuf[p & 1];
    const int shift = p * d.sort_bits;
    if (p == 0) hipLaunchKernelGGL((k_sort_hist<1, ITEMS>), dim3(ntiles), dim3(256), 0, st, a, b.n_pos, (int)d.sy2, nullptr, L.keys0, shift, (int)d.sort_bits, tpad, L.hist, L.scalars);
    else hipLaunchKernelGGL((k_sort_hist<0, ITEMS>), dim3(ntiles), dim3(256), 0, st, a, b.n_pos, (int)d.sy2, kin, nullptr, shift, (int)d.sort_bits, tpad, L.hist, L.scalars);
    hipLaunchKernelGGL((k_sort_scatter<ITEMS>), dim3(ntiles), dim3(256), 0, st, kin, vin, kout, vout, L.hist, b.n_pos, shift, (int)d.sort_bits, ntiles, tpad);
    kin = kout; vin = vout;
  }
}

// Slots of a step that carry the order along: 0 the gather (counts of the first digit), 1 pass 1 (first scatter), 2 the chain rule
// (the second of three, or of two before the ranks), 3 pass 2 (the last, or the ranks).
MarSortJob mar_sort_slot(const mar_ctx* c, const MarBatch& b, int slot, bool ranks, const mar_debug_out* dbg) {
  const MarDims& d = c->dm;
  const MarLayout& L = c->L;
  MarSortJob j = {};
  const int tile = 256 * MAR_SORT_RIDE_ITEMS;
  const bool rank = ranks && slot == 3 && d.sort_passes < 3, early = ranks || d.sort_passes > 2;
  const int p = early || slot < 2 ? slot - 1 : slot - 2;    // scatter pass of the slot
  if ((p >= d.sort_passes || (!early && slot == 2)) && !rank) return j;
  j.occ = OccArgs{b.src, b.rel, b.dst, b.neg_src, b.neg_dst, b.n, b.cn, (int32_t)d.num_nodes, d.roles};
  j.n_pos = (int32_t)b.n_pos; j.sy2 = d.sy2; j.bits = d.sort_bits; j.scalars = L.scalars;
  j.tiles = (j.n_pos + (rank ? MAR_RANK_TILE : tile) - 1) / (rank ? MAR_RANK_TILE : tile);
  j.blocks = (j.tiles + 7) & ~7;
  j.tpad = (j.tiles + 3) & ~3;
  const int words = j.tpad << d.sort_bits;                  // of one pass's counts
  if (rank) {
    j.kind = MAR_SORT_RANKS;
    j.keys_in = L.ids_sorted; j.rank_sorted = L.rank_sorted;
    j.num_uniq = dbg->num_uniq; j.uniq_nodes = dbg->uniq_nodes; j.uniq_rels = dbg->uniq_rels;
  } else if (slot == 0) {
    j.kind = MAR_SORT_HIST;
    j.keys_out = L.keys0; j.hist = L.hist; j.next_hist = L.hist + words; j.zero_words = (d.sort_passes - 1) * words;
  } else {
    const bool last = p == d.sort_passes - 1;
    j.kind = MAR_SORT_SCATTER;
    j.keys_in = p == 0 ? L.keys0 : L.kbuf[(p - 1) & 1]; j.vals_in = p == 0 ? nullptr : L.vbuf[(p - 1) & 1];
    j.keys_out = last ? L.ids_sorted : L.kbuf[p & 1]; j.vals_out = last ? L.perm : L.vbuf[p & 1];
    j.hist = L.hist + (size_t)p * words; j.next_hist = last ? nullptr : j.hist + words; j.shift = p * d.sort_bits;
  }
  return j;
}

hipError_t mar_launch_ranks(const mar_ctx* c, const MarBatch& b, hipStream_t st) {
  const MarDims& d = c->dm;
  const MarLayout& L = c->L;
  const unsigned nt = (unsigned)((b.n_pos + MAR_RANK_TILE - 1) / MAR_RANK_TILE);
  hipLaunchKernelGGL(k_rank_count, dim3(nt), dim3(256), 0, st, L.ids_sorted, b.n_pos, L.hist);
  hipLaunchKernelGGL(k_rank_apply, dim3(nt), dim3(256), 0, st, L.ids_sorted, L.perm, b.n_pos, L.hist, (int32_t)d.num_nodes, L.rank_sorted, L.keys0, L.uniq, L.scalars);
  return hipGetLastError();
}

hipError_t mar_launch_index(const mar_ctx* c, const MarBatch& b, int ranks, hipStream_t st) {
  const MarDims& d = c->dm;
  const MarLayout& L = c->L;
  OccArgs a{b.src, b.rel, b.dst, b.neg_src, b.neg_dst, b.n, b.cn, (int32_t)d.num_nodes, d.roles};
  if (b.n_pos <= 8 * 1024 && b.n_pos <= d.sort_one) hipLaunchKernelGGL((k_sort_one<8>), dim3(1), dim3(1024), 0, st, a, (int)b.n_pos, (int)d.sy2, (int)d.sort_passes, (int)d.sort_bits, L.ids_sorted, L.perm, L.scalars);
  else if (b.n_pos <= d.sort_one) hipLaunchKernelGGL((k_sort_one<16>), dim3(1), dim3(1024), 0, st, a, (int)b.n_pos, (int)d.sy2, (int)d.sort_passes, (int)d.sort_bits, L.ids_sorted, L.perm, L.scalars);
  else if (d.sort_items == 4) launch_sort<4>(c, b, a, st); else launch_sort<16>(c, b, a, st);
  if (ranks) return mar_launch_ranks(c, b, st);
  return hipGetLastError();
}

hipError_t mar_launch_debug_copy(const mar_ctx* c, const MarBatch& b, const mar_debug_out* dbg, hipStream_t st) {
  (void)b;
  if (dbg->num_uniq || dbg->uniq_nodes || dbg->uniq_rels)
    hipLaunchKernelGGL(k_debug_uniq, dim3(64), dim3(256), 0, st, c->L.uniq, c->L.scalars, (int32_t)c->dm.num_nodes,
                       dbg->num_uniq, dbg->uniq_nodes, dbg->uniq_rels);
  return hipGetLastError();
}
