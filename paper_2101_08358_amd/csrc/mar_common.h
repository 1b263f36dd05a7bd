// Internal declarations shared by the library's translation units (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/marius_hip.h"

// Side index of a corrupted endpoint; also the generator's "side" counter bit.
#define MAR_SIDE_SRC 0   // negatives replace the source
#define MAR_SIDE_DST 1   // negatives replace the destination

// Workspace carve-up (device pointers).
struct MarLayout {
  int32_t*  scalars;      // [16]: 0 = unique rows (nodes + relations), 1 = unique nodes, 2 = number of entries in `owners`
  int32_t*  uniq;         // ascending unified ids of the touched rows
  uint32_t* keys0;        // [n_pos] gradient row -> unified id of its table row (sort keys); -> its rank, once ranks have been formed
  uint32_t* kbuf[2];      // [n_pos] each: keys between two passes of the radix sort
  int32_t*  vbuf[2];      // [n_pos] each: gradient row numbers between two passes
  uint32_t* hist;         // [bins][sort tiles] digit counts of the current pass; heads per tile of the rank kernels
  int32_t*  perm;         // position in row-sorted order -> gradient row
  uint32_t* ids_sorted;   // position -> unified id (node id, or num_nodes + relation id)
  int32_t*  rank_sorted;  // position -> rank among the unique rows (where a caller asks for ranks)
  int32_t*  owners;       // [reduce blocks] workgroups of the reduce in which a segment begins that continues into later ones
  float*    Q;            // TransE: [2][batch][dk] edge-side operands (side-major)
  float*    Km;           // TransE on dense operands: [2][chunks][N][dk] gathered negative rows
  float*    qq;           // [2][batch] squared norms of Q rows (TransE)
  float*    kk;           // [2][chunks*N] squared norms of Km rows (TransE)
  float*    pos;          // [batch] positive scores
  float*    gQ;           // [sy1][2][batch][dk] per-part unnormalised gradient w.r.t. Q rows; bilinear models' evaluation: fp32 operands
  float*    ml;           // [sy1][2][batch][2] per-part softmax reference (bilinear models: in log2 units) and sum
  float*    gQx;          // [rem1.k - 1][rem1.rows][dk] parts 1.. of the stripes that are split to fill the last round
  float*    mlx;          // [rem1.k - 1][rem1.rows][2]
  float*    T;            // TransE: [2*chunks][S rounded up to 64][N rounded up to 128] softmax weights exp(score - reference)
                          // divided by the distance, pass 1 -> pass 2
  float*    R;            // TransE: [2*chunks][N rounded up to 128, / 16][S rounded up to 64] the reference each 16-negative block of T was written with
  char*     Kimg;         // bilinear models: [2*chunks][N / 32 rounded up][image] hi/lo planes of the negatives' rows (mar_split.h)
  char*     Qimg;         // bilinear models: [2*chunks][S / 32 rounded up][image] the same of the edge-side operands
  float*    Kexp;         // exponents of the images' 16-row blocks, [2*chunks][2 * image tiles]
  float*    Qexp;
  float*    Knorm;        // evaluation: bounds of the norms of Kimg's scaled rows, per 16-row block and per row
  float*    shift;        // TransE on images: [512] what k_prep takes off every operand
  float*    Gx;           // [rem2.k - 1][rem2.rows][dk] parts 1.. of pass 2's split stripes (bilinear models)
  float*    G;            // [roles*n + 2*cn*sy2][dk] gradient rows: edge-side occurrence k < roles*n at row k, part i
                          // of negative occurrence k at row roles*n + (k - roles*n)*sy2 + i
                          // (bilinear models' evaluation: the negatives' fp32 rows, or the images' exponents and norms)
  float*    carry;        // [reduce blocks][2][dk] partial sums of segments that cross workgroup borders
  float*    loss_part;    // per-block partial loss sums
  void*     metric_part;  // [MAR_METRIC_MAX_PARTS] partial records of the rank metrics
};

// A full batch's (chunk-side, stripe) units beyond the last whole round of the chip's workgroup slots: units from
// whole_units on are each split into k parts of tps streamed tiles, which a small kernel merges.
struct MarRem {
  int32_t whole_units, k, tps;
  int64_t rows;                    // stripe rows of all split units
};

struct MarDims {
  int32_t dim, dk;                 // row width and its multiple-of-4 padding
  int32_t B, C, S, N, Ndeg;
  int32_t roles;                   // edge-side occurrences per edge: source, destination and (unless Dot) relation
  int64_t num_nodes; int32_t num_rels;
  int64_t n_occ_max;               // roles*B + 2CN
  int64_t n_pos_max;               // roles*B + 2CN*sy2: gradient rows per step
  int32_t sy1, sy2;                // how many workgroups share the streamed rows of one stripe (pass 1 / 2)
  int32_t tps1, tps2;              // streamed tiles per workgroup
  MarRem rem1, rem2;               // split stripes of pass 1; of pass 2 (bilinear models): parts 1.. are added by a small kernel
  int64_t u_max;                   // min(num_nodes + num_rels, n_occ_max)
  int32_t sort_passes, sort_bits, sort_items;  // radix sort of the gradient rows by unified id: passes, bits per pass, elements per thread
  int32_t bilinear;                // DistMult, ComplEx, Dot: the passes of mar_split.hip; TransE: those of mar_flash.hip
  int32_t dist_img;                // TransE whose training passes are those of mar_split.hip too (mar_dist_images)
  int32_t reduce_small;            // positions that the reduce gives a lane group (8, or 4 in the smallest batches); 0: one per lane
  int32_t split_bf16;              // training passes on bf16 hi + lo operands (precision SPLIT_BF16)
  int32_t sort_one;                // most gradient rows that one workgroup sorts by itself
  int32_t long_passes;             // a contraction pass takes some 25 us or more
  int32_t order_rides;             // the row order is carried along by the step's own launches (MarSortJob)
  int32_t one_stream;              // everything on the caller's stream: the order carried along, or (smallest batches) ahead of the gather
  int32_t index_after_gather;      // launch order of a step: gather first, index build behind it (large batches)
};

#define MAR_LN2 0.69314718055994531f
#define MAR_MAX_PARTS 8                   // most parts a stripe of pass 1 is split into
#define MAR_MAX_PROFILE_STEPS 4096

struct mar_ctx {
  mar_config cfg;
  MarDims dm;
  float *node_emb, *node_state, *rel_emb, *rel_state;
  void* workspace; size_t workspace_bytes;
  MarLayout L;
  // second stream for work that is independent of the contraction passes, and its fork/join events
  hipStream_t aux;
  hipEvent_t ev_fork, ev_index, ev_pass1, ev_chain;
  // profiling
  int32_t prof_max, prof_steps;
  uint32_t prof_mask;
  hipEvent_t* prof_events;         // 2 * MAR_NUM_PHASES per step (begin, end of each phase)
};

void mar_set_error(const char* fmt, ...);

// Radix sort of the gradient rows by unified id: the widest digit.
#define MAR_SORT_MAX_BITS 9
#define MAR_SORT_ONE (16 * 1024)  // most elements k_sort_one can hold
// Most gradient rows that one workgroup sorts by itself (the pipeline; steps whose order is not carried along): one launch in place of
// two a pass, which the host cannot issue as fast as a small step runs.  Half as many where the
// sort's own time counts (11,000 rows 27 us, in four launches 20): above 256 floats, where the kernels take longer than the host,
// and in the pipeline, where it stands alone ahead of the staging (us a batch, one workgroup / launches: 4,000 rows of 100 floats
// 94 / 101, 8,000 125 / 129, 9,300 171 / 167, 11,000 177 / 171, 15,600 176 / 163).
static inline int32_t mar_sort_one_limit(int dk, bool alone) { return alone || dk > 256 ? MAR_SORT_ONE / 2 : MAR_SORT_ONE; }
#define MAR_RANK_TILE 1024        // positions per workgroup of the rank kernels

// Rank metrics: ranks per partial record, records a scratch area holds, bytes per record.
#define MAR_METRIC_TILE 4096
#define MAR_METRIC_MAX_PARTS 4096
#define MAR_METRIC_PART_BYTES 72


// Lanes that move one table row as float4s.
static inline int mar_lane_group(int dk) { return dk <= 64 ? 16 : (dk <= 128 ? 32 : 64); }
// Positions of the row-sorted order per workgroup of the reduce.
static inline int mar_reduce_block(const MarDims& d) { return d.reduce_small ? 256 / mar_lane_group(d.dk) * d.reduce_small : 256; }

// Occurrences of a batch (mar_sort_dev.h).
struct OccArgs {
  const int32_t *src, *rel, *dst, *neg_src, *neg_dst;
  int32_t n, cn;
  int32_t num_nodes;
  int32_t roles;
};
// A piece of the row-sorted order that a kernel of the step carries along: its first `blocks` workgroups do it and nothing else.
// Small batches are bound by the host and by the order's own chain of launches on a second stream (1,000 edges of 50 floats,
// 100 negatives: 78 us a step of which 55 were kernels); carried along, it takes no launch, no event and no second stream.
#define MAR_SORT_HIST 1
#define MAR_SORT_SCATTER 2
#define MAR_SORT_RANKS 4
#define MAR_SORT_RIDE_ITEMS 4     // elements a thread: tiles of 1,024
#define SORT_LDS_BYTES ((5 << MAR_SORT_MAX_BITS) * 4 + 16)
struct MarSortJob {
  int32_t kind, blocks, tiles;     // blocks: a multiple of 8, 0 for none; tiles of the work that they share
  int32_t n_pos, sy2, shift, bits, tpad, zero_words;
  OccArgs occ;
  const uint32_t* keys_in; const int32_t* vals_in;
  uint32_t* keys_out; int32_t* vals_out;
  uint32_t *hist, *next_hist;      // counts of this pass; of the next (of all later ones, zeroed, in MAR_SORT_HIST)
  int32_t* scalars;
  int32_t *rank_sorted, *num_uniq, *uniq_nodes, *uniq_rels;
};

// ---- launchers (each returns a hipError_t from the launch) --------------------------
hipError_t mar_launch_init(const mar_ctx* c, int fill, hipStream_t st);
hipError_t mar_launch_sample(const mar_ctx* c, uint64_t step, const int32_t* es, const int32_t* ed,
                             int64_t num_edges, int32_t* neg_src, int32_t* neg_dst, hipStream_t st);
hipError_t mar_launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st);

struct MarBatch {
  const int32_t *src, *rel, *dst, *neg_src, *neg_dst;
  int32_t n;        // edges
  int32_t nchunks;  // ceil(n / S)
  int32_t cn;       // nchunks * N
  int64_t n_occ;    // roles*n + 2cn
  int64_t n_pos;    // roles*n + 2cn*sy2 gradient rows
};

// ranks != 0: also the rows' ranks, the unique list and the counts in scalars
hipError_t mar_launch_index(const mar_ctx* c, const MarBatch& b, int ranks, hipStream_t st);
hipError_t mar_launch_ranks(const mar_ctx* c, const MarBatch& b, hipStream_t st);
MarSortJob mar_sort_slot(const mar_ctx* c, const MarBatch& b, int slot, bool ranks, const mar_debug_out* dbg);
// bf16 != 0 (SPLIT_BF16 training): the operand images hold bf16 instead of scaled f16 parts
// rank_dst / rank_src (evaluation): set to 1
hipError_t mar_launch_prep(const mar_ctx* c, const MarBatch& b, float* pos_out, int bf16, int32_t* rank_dst, int32_t* rank_src,
                           hipStream_t st, const MarSortJob* job = nullptr);
// Small evaluations of the bilinear models run on dense fp32 operands and fp32 matrix instructions (see mar_api.hip).
bool mar_eval_dense(const MarDims& d, const MarBatch& b);
hipError_t mar_launch_flash(const mar_ctx* c, const MarBatch& b, int pass, int32_t* rank_dst, int32_t* rank_src,
                            hipStream_t st, const MarSortJob* job = nullptr);
// dbg: where the log-sum-exps go if a caller asks for them
hipError_t mar_launch_chain(const mar_ctx* c, const MarBatch& b, const mar_debug_out* dbg, hipStream_t st, const MarSortJob* job = nullptr);
hipError_t mar_launch_filter(const mar_ctx* c, const MarBatch& b, const int64_t* dst_off, const int32_t* dst_ids,
                             const int64_t* src_off, const int32_t* src_ids, const float* pos, int32_t* rank_dst,
                             int32_t* rank_src, hipStream_t st);
hipError_t mar_launch_reduce(const mar_ctx* c, const MarBatch& b, float* loss_out, float* dbg_grad, float* defer_grad, hipStream_t st);

#define MAR_STAGE_PREV 8
// Staging buffers of one batch of out-of-memory training (see mar_rows.hip).
struct MarStage {
  float *host_emb, *host_state;                      // node table and accumulators in pinned host memory
  float *compact, *gsum;                             // [unique rows][dim] staged rows, [unique rows][dk] summed gradients
  int32_t *c_src, *c_dst, *c_neg_dst, *c_neg_src;    // the batch's node ids replaced by ranks
  // batches whose updates may still change the host rows after they have been staged: their unique lists and counts
  const int32_t* prev_uniq[MAR_STAGE_PREV]; const int32_t* prev_scalars[MAR_STAGE_PREV];
  int32_t num_prev;                                  // -1: more than MAR_STAGE_PREV, every row counts as shared
  uint8_t* shared;                                   // [unique rows] 1: the row is in one of those batches
};
hipError_t mar_launch_stage_in(const mar_ctx* c, const MarBatch& b, const MarStage& sg, hipStream_t st);
hipError_t mar_launch_stage_out(const mar_ctx* c, const MarBatch& b, const MarStage& sg, hipStream_t st);
hipError_t mar_launch_debug_copy(const mar_ctx* c, const MarBatch& b, const mar_debug_out* dbg, hipStream_t st);
hipError_t mar_launch_rank_metrics(const int32_t* ranks, int64_t n, const int32_t* ks, int num_k, double* out, void* part,
                                   hipStream_t st);
int mar_flash_supported(int dk);
int mar_flash_tile_rows(int dk, int pass);
int mar_flash_stripe_rows(int dk, int pass);
hipError_t mar_flash_prepare(int dk);   // before the first contraction launch of a context (LDS size limits)
int mar_flash_wgs_per_cu(int dk, int pass);        // workgroups of a pass that a CU holds at once
hipError_t mar_launch_flash_merge(const mar_ctx* c, const MarBatch& b, hipStream_t st);   // after pass 1: merges split stripes
// Passes of the bilinear models (mar_split.hip): geometry for the planning of a configuration, and the launches.
int mar_split_supported(int dk);
int mar_split_wgs_per_cu(int dk, int pass);
#define MAR_SPLIT_STRIPE_ROWS 128
#define MAR_SPLIT_TILE_ROWS 32
#define MAR_SHARES 256            // workgroups of an evaluation cut into equal shares: one a CU
static inline bool mar_on_images(const MarDims& d) { return d.bilinear || d.dist_img; }
bool mar_dist_images(const MarDims& d);            // TransE's training: images and 16-bit products, or dense fp32 operands
static inline int mar_stripe_rows(const MarDims& d, int pass) { return mar_on_images(d) ? MAR_SPLIT_STRIPE_ROWS : mar_flash_stripe_rows(d.dk, pass); }
static inline int mar_tile_rows(const MarDims& d, int pass) { return mar_on_images(d) ? MAR_SPLIT_TILE_ROWS : mar_flash_tile_rows(d.dk, pass); }
// How many workgroups share one of `units` units of a pass, and the streamed tiles each takes (n_y streamed rows).
int mar_check_config(const mar_config* cfg, MarDims* d);   // refuses, or plans: every rule a context follows
void mar_plan_parts(const MarDims& d, int pass, long units, int n_y, int32_t* sy, int32_t* tps);
bool mar_split_shares(int dk);                     // an evaluation on images can cut all units' tiles into equal shares
bool mar_plan_shares(const MarDims& d, long units, int ntiles, int sy, int tps);   // and should, rather than `sy` parts a unit
size_t mar_split_image_bytes(int dk);
hipError_t mar_split_prepare(int dk);
