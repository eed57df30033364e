// Internal declarations shared by the host orchestration and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/flexprefill.h"

namespace fp {

// Longest key chunk owned by one workgroup of the representative-score kernels.  Short
// problems use chunks of 512 or 256 keys (SeqTable::ch_len) so that those kernels still
// get enough workgroups to fill the GPU.
constexpr int kScoreChunk = 1024;
constexpr int kScoreChunkMin = 256;
// workgroups of the line-sum kernel wanted before the chunk is shortened (4 per CU)
constexpr int kScoreWorkgroups = 1024;
constexpr int kHistBuckets = 2048;     // radix-select digit: 11 bits
constexpr int kHistCounts = 1024;      // last digit (10 bits), the only one with counts

// Per-call table of packed sequences, passed by value to every kernel.
struct SeqTable {
  int32_t n_seq;
  int32_t max_nb;
  int32_t cu[FP_MAX_BATCH + 1];       // token offsets
  int32_t nb_off[FP_MAX_BATCH + 1];   // prefix sums of nb_s = ceil(n_s / block)
  int32_t ch_len;                     // keys per score chunk: 1024, 512 or 256
  int32_t ch_off[FP_MAX_BATCH + 1];   // prefix sums of ceil(n_s / ch_len)
  int64_t tri_off[FP_MAX_BATCH + 1];  // prefix sums of nb_s (nb_s + 1) / 2
};

// Everything a kernel of the selection pipeline needs.
struct SelectArgs {
  SeqTable st;
  const uint16_t *q;       // [T][Hq][d] bf16
  const uint16_t *k;       // [T][Hkv][d] bf16
  int32_t hq, hkv, d, block;
  int32_t total_tokens;    // T
  int32_t nb_total;        // NB
  int64_t tri_total;       // TRI
  float scale;             // softmax scale
  float gamma, tau;
  int32_t min_budget;
  int32_t force_pattern;
  int32_t max_budget;      // 0 = no cap
  int32_t qa_mode;         // 0 flattened map (Algorithm 4), 1 per query block
  int32_t vs_granularity;  // 0 token lines (Algorithm 3), 1 block-pooled lines
  // set by the launcher: every selection problem in one workgroup (no histograms), and the
  // line marks made by convert_tiles itself (no vs_marks)
  int32_t small, marks_inline;
  // set by the launchers: the line pass merges the chunk statistics, pools Q, and the parts
  // it cuts a score chunk into
  int32_t merge_inline, pool_inline, line_parts;
  // workspace
  float2 *chunk_stats;     // [ch_total][Hq][block] (max, sum) in log2 units
  float2 *row_stats;       // [n_seq][Hq][block]
  float *kbar;             // [NB][Hkv][d]
  float *qbar;             // [NB][Hq][d]
  float *a_v;              // [Hq][T]
  float *a_s;              // [Hq][T]
  float *av_blk;           // [Hq][NB] a_v summed per key block (block-pooled lines)
  float *as_blk;           // [Hq][NB] a_s summed per offset block
  float *pat_logit;        // [Hq][NB] scale * q_bar . K_bar_J of the pattern search
  double *pat_ahat;        // [Hq][NB] a_hat[J] = a_v summed per key block
  uint8_t *vs_marks;       // [Hq][NB][4] per key block / diagonal: column, diagonal (full
                           // rows), diagonal (partial last row), diagonal + 1
  float *flat;             // [Hq][TRI]
  struct SelState *sel;    // [n_seq][Hq][2]
  uint32_t *hist_cnt;      // [n_seq][Hq][2][kHistCounts]
  unsigned long long *hist_mass;  // [n_seq][Hq][2][kHistBuckets]
  // outputs
  int32_t *kb_idx;
  int32_t *kb_cnt;
  uint8_t *pattern;
  float *js;
  int32_t *units;
};

// State of one cumulative-mass selection problem (one score vector).
struct SelState {
  unsigned long long total;       // fixed-point mass of all units
  unsigned long long thr;         // ceil(gamma * total)
  unsigned long long mass_above;  // mass of keys above the current digit range
  unsigned long long ticket;      // slices of the radix pass that are done, and (in the upper
                                  // 32 bits) the units that they counted above its range
  uint32_t cnt_above;             // number of keys above the current digit range
  uint32_t prefix;                // key bits fixed so far
  uint32_t key;                   // final threshold key
  int32_t idcut;                  // last id taken among key == `key`
  int32_t k;                      // units selected
  int32_t mode;                   // 0 active, 1 take all, 2 inactive (other pattern)
  int32_t n;                      // number of units
};

// The split grid is taken for at most this many tenths of a row per resident workgroup.
// Where the line lies (attention over selected lists, us, other grid -> split grid; single
// runs differ by 3-10%): block 128, head dim 128, 2.0 rows (32 heads, 4k tokens) 143 -> 121,
// 2.9 (6k) 251 -> 250, 3.4 (7k) 320 -> 318, 5.0 (10k) 516 -> 544; head dim 64, 3.0 rows (64
// heads, 4500) 208 -> 170, 3.6 (5500) 229 -> 194, 4.6 (7k) 375 -> 347, 6.2 (9500) 549 -> 549,
// so on the safe side there; block 64, head dim 128, 4.0 rows (32 heads, 8k) 282 -> 223, 4.8
// (9800) 460 -> 496; head dim 64, 4.6 (64 heads, 7k) 374 -> 293, 5.5 (8500) 517 -> 437, 6.9
// (10500) 586 -> 541.
constexpr int kSplitRows128 = 30;
constexpr int kSplitRows64 = 48;
// Shortest segment that a longer list is cut into: 3, 4 and 6 blocks measure the same within
// 3% (two heads of 64, 2k tokens: 29.9, 28.8, 28.4 us; 8 heads, 4k: 43.5, 44.6, 44.7).
constexpr int kSegBlocks = 4;
constexpr int kSplitUnits = 2816;   // units per KV group: 8 B of key slots (a power of two),
                                    // 32 B of records each in the sort's 128 KB of LDS

// Short attention problems: one workgroup per unit, a unit being a row's list or a segment
// of it (unit_cap = 0: not used).
struct SplitArgs {
  int4 *units;             // [Hkv][unit_cap] records {row, blocks, first block, second block}
  int4 *segs;              // [Hkv][unit_cap] {first list entry, first slot, segment, segments}
  int32_t *tickets;        // [slots] at a split row's first slot: its segments stored so far
  unsigned long long *partials;   // [slots] partial results of segments
  int32_t unit_cap;        // units per KV group, the unused last ones marked empty
  int32_t extra;           // units per KV group beyond its rows; 2 * extra slots
  int32_t all;             // `extra` covers every segment of kSegBlocks
  int32_t slots;           // resident workgroups of the chip
};

struct AttnArgs {
  SeqTable st;
  const uint16_t *q, *k, *v;
  uint16_t *o;
  const int32_t *kb_idx;
  const int32_t *kb_cnt;
  int32_t hq, hkv, d, block;
  int32_t nb_total;
  int64_t tri_total;
  float scale_log2;        // softmax scale * log2(e)
  int4 *items;             // [Hkv][G * NB] workspace: ordered item records per KV group
  int32_t *queue;          // [8] workspace: per-XCD work-queue counters
  int32_t mix;             // set by the launcher: an XCD's KV groups served interleaved
  uint16_t *vt;            // [Hkv][NB][B * d] workspace: V^T tiles per key block
  unsigned long long *sort_keys;  // [Hkv][G * NB] workspace: items' sort keys
  int4 *sort_recs;         // [Hkv][G * NB] workspace: item records in item-id order
  SplitArgs split;
};

// Device address of the current device's fixed scratch array (fp_noalloc.hip).
hipError_t noalloc_scratch(void **out);

// Launchers (each returns the hipError_t of its launch).
hipError_t launch_sparse_attn(const AttnArgs &a, hipStream_t s);
hipError_t launch_select_pipeline(const SelectArgs &a, hipStream_t s);
hipError_t launch_dense_lists(const SelectArgs &a, hipStream_t s);
hipError_t launch_qa_rows(const SelectArgs &a, hipStream_t s);

}  // namespace fp
