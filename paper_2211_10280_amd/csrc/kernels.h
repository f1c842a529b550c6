// Host-callable launchers of the HIP kernels (one per pipeline stage).  All of them only
// enqueue work on `st`; none synchronises.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint32_t u32;
typedef uint64_t u64;
typedef int64_t i64;

#define TN_MAX_SRC 32     // own + up to 31 peers
#define TN_SUB_MAX_DIM 128   // rows of at most this many elements (16 bytes for at most 32 lanes): several to a wave
#define TN_MAX_BLOCKS ((1 << 24) - 1)   // workgroups of 256 threads that one launch may have (2^32 threads in all)
// Sorted entries per wave in the segmented reduction, 2^tn_seg_shift: small problems get small tiles so that
// enough waves exist to hide the latency of the row loads, but every row of more than a tile is chained from partials.
// Tiles of 8 / 16 / 32 entries, step in us: 4 100 entries, D = 460 28.4 / 29.0 / 32.5; 6 900, D = 256 (gradient) 48.3 /
// 49.6 / 52.2; 12 200, D = 144 36.2 / 34.5 / 37.0; 21 000, D = 224 52.5 / 48.8 / 47.2; 32 500, D = 168, unannounced 69.6 /
// 67.0 / 68.7; 52 800, D = 216 73.6 / 66.3 / 63.8.  Rows of at most TN_SUB_MAX_DIM elements, of which a wave sums several
// side by side: 1 500 entries, D = 32 22.9 / 22.9 / 21.9; 61 400, D = 128 56.9 / 49.1 / 47.4; 63 700, D = 92 56.1 / 46.9 / 41.6.
#define TN_SEG_MAX_TILE 32
static inline int tn_seg_shift(i64 n, int D) { return D <= TN_SUB_MAX_DIM || n > 32768 ? 5 : n > 8192 ? 4 : 3; }
static inline i64 tn_seg_tiles(i64 n, int D) { return (n + (1 << tn_seg_shift(n, D)) - 1) >> tn_seg_shift(n, D); }
#define TN_RADIX_TILE 2048    // keys per workgroup in a pass of the sort
#define TN_RADIX_MAX_BITS 9   // widest digit of a pass
#define TN_RADIX_MAX_ND (1 << TN_RADIX_MAX_BITS)
#define TN_RADIX_MAX_PASSES_ND (3 * TN_RADIX_MAX_ND)   // digits of all passes together, at most (28 key bits: 4 x 128)
// Number of passes and digit width for keys of `key_bits` bits: the fewest passes.  A pass is bound by round trips to
// memory, and a digit's keys leave a tile as one run, so wider digits cost little; 9 bits are what a tile's counters
// and their chained scan take without slowing the pass down.
static inline void tn_radix_shape(int key_bits, int *passes, int *bits)
{
    if (key_bits < 1) key_bits = 1;
    *passes = (key_bits + TN_RADIX_MAX_BITS - 1) / TN_RADIX_MAX_BITS;
    *bits = (key_bits + *passes - 1) / *passes;
}
#define TN_SCAN_TILE 2048   // entries per workgroup in the segment scan
#define TN_SEG_XBLOCK 256    // tiles of the segmented reduction per block of partials
#define TN_SEG_CROSS_MIN 16384  // problems with more tiles than this get partials per block of tiles

// ---- stage 0: table initialisation
void tn_launch_init_tables(void *w_in, void *w_out, i64 V, int D, int stride, int dtype, u64 seed,
                           hipStream_t st);

// ---- stage 1: pair enumeration, negative sampling, sort keys
struct BatchDesc {
    const int *tok;   // DEVICE int32[T]
    i64 T;
    i64 begin;        // first center position
    int n_centers;
    int w, N;
    i64 pair_base;    // pairs_before(begin)
    i64 P;            // pairs in the batch
};

// ---- preparation of a mini-batch (prep_dev.h): one launch per phase -- keys, the passes of the sort, segments
#define PREP_KEYS_SLOTS 1024   // most slots per workgroup
// Slots per workgroup: few where there are few (a workgroup's time is that of one slot after the other), more where the
// workgroups' digit counts, added up in memory, would cost more (step, 1 024 / 512 / 256 slots: 1 536 slots in all 26.5 / 24.4 /
// 23.7 us, 6 000 - / 29.9 / 29.4, gradient of 12 000 - / 41.3 / 40.0; step, 61 000 56.3 / 54.6 / 55.4, 64 000 - / 43.0 / 45.0;
// 85 000 60.1 / 62.0, 143 000 64.5 / 66.1).
static inline int tn_prep_keys_slots(i64 slots) { return slots <= 16384 ? 256 : slots <= 65536 ? 512 : PREP_KEYS_SLOTS; }
// the negatives' draws: pure functions of the position, the offset and the negative's number
struct NoiseDraw {
    i64 V;
    const uint2 *draw;     // [V] alias table: threshold, alias
    u32 k0, k1, ctr3;
    int resample;          // a negative equal to the pair's center or context word is drawn once more
};
struct PrepKeys {
    BatchDesc b;
    NoiseDraw noise;
    int centers_only;      // the in-side list alone (in a launch of its own)
    u32 *out_keys, *in_keys;
    int *pair_center, *neg_dbg, *status;
    u32 *hist;             // [2 lists][passes][2^bits] digit counts, added to: zero before (NULL: not wanted)
    int passes, bits;
    int items;             // slots per thread of a workgroup of BLOCK threads
    u32 *clear;            // what the later phases publish into and their tickets: zeroed
    size_t n_clear;
};
struct PrepPassList {
    const u32 *kin, *vin;  // vin: not read by the first pass, whose values are the entries' places
    u32 *kout, *vout;
    u32 *state;            // [tiles][2^bits] published words (chained), digit counts (counted)
    u32 *hist;             // [2^bits] keys per digit (chained); [groups + 1][2^bits] per group of tiles (counted)
    int n, tiles;
};
struct PrepPass {
    PrepPassList p[2];     // out-side, in-side
    u32 *ticket;
    int shift, bits, first;
    int scanned;           // counted: hist holds the keys of the lower groups, in the row after the last all keys
};
struct PrepSegmentsList {
    const u32 *keys;       // sorted keys
    const u32 *vals;       // sorted values
    int n, tiles;
    u64 *state;            // [tiles] published words; in-side: [2][tiles], the second for the weights
    int *seg_of;           // [n] out: row index (0..U-1) of every sorted entry
    int *seg_start;        // [U+1] out: index of the first sorted entry of every row, then n
    int *long_cnt;         // [1] zeroed here: the segmented reduction counts its long rows in it
    int *row_ids;          // [capacity] out
    int *n_rows;           // [1] out
    int *seg_offsets;      // [U+1] out or NULL
    i64 capacity;
};
struct PrepSegments {
    PrepSegmentsList p[2];
    i64 begin, T;
    int w;
    u32 *hist;             // zeroed for the next mini-batch
    int n_hist;
    u32 *ticket;
    int *status;
};
// chained preparations: keys, passes, segments; counted ones: keys, (count, counted pass)..., heads, counted segments
enum { PREP_KEYS, PREP_PASS, PREP_SEGMENTS, PREP_COUNT, PREP_PASS_COUNTED, PREP_HEADS, PREP_SEGMENTS_COUNTED };
struct PrepPhase {
    int kind;
    int blocks;            // workgroups
    union {
        PrepKeys keys;
        PrepPass pass;
        PrepSegments seg;
    };
};
#define TN_PREP_GROUP 64       // tiles per group of a counted pass
// Most groups whose counts every tile of a counted pass adds up by itself.  With more of them that would be the pass
// (its reads grow with the square of the tiles), so a launch before it sums them once (262 000 words, each tile by
// itself / summed once: 4.2 M occurrences, 32 groups, gradient 0.769 / 0.774 ms; 6.3 M 1.16 / 1.13; 34 M 8.5 / 7.1;
// 134 M 48 / 21.6; at 2.1 M, 16 groups, no difference).
#define TN_PREP_GROUPS_OWN 40
static inline int tn_prep_groups(int tiles) { return (tiles + TN_PREP_GROUP - 1) / TN_PREP_GROUP; }
// Most tiles of a chained preparation: as launches of its own (longer ones are faster counted), and riding in other
// launches, where its latency is hidden.  Beyond 256 tiles the tickets alone hold those launches up, and a counted
// preparation on a stream of its own beside them is faster (step riding / beside: 222 tiles 131 / 146 us at 300 000
// words, D = 64, 315 / 318 at a million, D = 300; 260 tiles 155 / 146 and 369 / 366; 440 tiles 230 / 208 and 606 / 580).
// Under a table update that takes at least TN_PREP_RIDE_LONG_UPDATE times as long as the preparation it is the other way
// round up to 512 tiles (2 million words in bfloat16, D = 512, 440 tiles: 15 peers 3 665 / 3 700 us, 11 peers 2 946 / 2 953,
// 300 tiles 2 789 / 2 826 and 2 226 / 2 251; at a ratio of 11 to 14: 15 peers, D = 256, 1 680 / 1 664, D = 300 in fp32
// 2 304 / 2 287, 7 peers, D = 512, 2 191 / 2 190).
#define TN_PREP_CHAIN_OWN 128
#define TN_PREP_CHAIN_RIDE 256
#define TN_PREP_CHAIN_MAX 512
#define TN_PREP_RIDE_LONG_UPDATE 16.0
static inline int tn_prep_tiles(i64 n) { return (int)((n + TN_RADIX_TILE - 1) / TN_RADIX_TILE); }   // n: up to 2^31 - 1
static inline int tn_prep_seg_tiles(i64 n) { return (int)((n + TN_SCAN_TILE - 1) / TN_SCAN_TILE); }
void tn_launch_prep(const PrepPhase &x, hipStream_t st);   // the phase as a launch of its own
void tn_launch_prep_clear(u32 *hist, int n, hipStream_t st);

// row ids / row count / segment offsets of a prepared mini-batch -> the consuming call's buffers
struct RowIndexCopy {
    struct Side {
        const int *src_ids, *src_n, *src_off;   // src_off [U+1]
        int *dst_ids, *dst_n, *dst_off;         // dst_off may be NULL
    } side[2];
};

// ---- stage 4: forward pass and per-center partial of the W_in gradient
struct FwdArgs {
    const void *w_in, *w_out;
    i64 V;
    int dtype, D, stride;
    BatchDesc b;
    const u32 *out_keys;   // unsorted out-side keys [P][N+1]
    float *g;              // [P][N+1] out: (sigmoid - label)/P per occurrence
    float *center_part;    // [n_centers][D] out
    float *center_loss;    // [n_centers] out (sum of the loss terms, not yet divided by P)
    float inv_P;
    int repeats;           // a position's tasks are expected to name the same words many times over (and are at most
                           // TN_REPEAT_MAX_TASKS): a hint, rows of up to 320 elements heed it
};
#define TN_REPEAT_MAX_TASKS 512
struct AuxWork;
void tn_launch_forward(const FwdArgs &a, const AuxWork *aux, hipStream_t st);   // aux may be NULL
void tn_launch_forward_sub(const FwdArgs &a, const AuxWork &aux, hipStream_t st);

// ---- stage 5: segmented reduction of rows (duplicates summed in sorted order)
struct SegReduceArgs {
    int n;                 // sorted entries
    int shift;             // tiles of 2^shift entries (the launcher sets it: tn_seg_shift)
    const u32 *vals;       // sorted values
    const int *seg_of;     // row index per sorted entry
    const int *seg_start;  // first sorted entry of every row; [U] = n
    float *out_rows;       // [U][D]
    float *part;           // [ntiles][2][D] scratch for rows that cross tile borders
    float *cross;          // [ceil(ntiles / TN_SEG_XBLOCK)][D] scratch: partials of long rows per block of tiles
                           // (the launcher clears the pointer for problems of at most TN_SEG_CROSS_MIN tiles)
    int *long_cnt;         // [1] number of long rows found (zeroed by the segment scan)
    int4 *long_list;       // [ntiles] the long rows, in no particular order: the tile it begins in, the row, tiles after that one, word (where noted)
    int *xinfo;            // [ceil(ntiles / TN_SEG_XBLOCK)] scratch: does a long row cross the block's border
    const int *row_ids;    // [U] the rows' words, where the table update chains the long ones ...
    u64 *long_mask;        // ... which are noted here too, a bit per word (else NULL)
    int D;
    // source of the contribution of an entry:
    //  mode 0 (out-side): value = occurrence index o; row = g[o] * W_in[pair_center[o/(N+1)]]
    //  mode 1 (in-side):  value = center index i;     row = center_part[i]
    int mode;
    const float *g;
    const int *pair_center;
    int Np1;
    const void *table;
    int dtype, stride;
    const float *center_part;
};
// the W_out-side and the W_in-side problem of a mini-batch in one launch (either may be NULL); `rider` (may be NULL):
// rides with the launch that chains the long rows, if there is one (tn_seg_chains)
void tn_launch_segreduce(const SegReduceArgs *out, const SegReduceArgs *in, const AuxWork *aux, const PrepPhase *rider,
                         hipStream_t st);
// The W_out-side and the W_in-side reduction of a mini-batch are independent: one launch runs both
// (workgroups [0, blocks_in) take the in-side problem, the rest the out-side one), so that the small
// in-side problem costs no launch of its own and its few workgroups start first.
struct SegReducePair {
    SegReduceArgs out, in;
    int blocks_in;    // workgroups of the in-side problem at the front of the grid
};
void tn_launch_segreduce_sub(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st);
// The chaining of long rows left to the table update (tn_launch_apply_update): each is summed and applied by a workgroup at the
// front of its grid.
struct ChainWork {
    SegReducePair p;
    int blocks;       // workgroups; p.blocks_in of them take the in-side rows
};
#ifndef TN_CHAIN_UPDATE_MAX_OCC
// Occurrences up to which it is (chains_with_update).  Beyond, up to 520 000, 60 steps with the chaining in the update take 0.96 of the time
// with a launch of its own in the mean, from 0.83 to 1.02: the line could lie higher.
#define TN_CHAIN_UPDATE_MAX_OCC 131072
#endif
#define TN_CHAIN_UPDATE_MAX_V (1 << 2 * TN_RADIX_MAX_BITS)     // words up to which it is: their keys are sorted in two passes
void tn_chain_work(ChainWork &c, const SegReduceArgs &out, const SegReduceArgs &in);
// workgroups that chain long rows: they exist only where a problem has more than one tile
static inline int tn_seg_chains(i64 n, int D)
{
    const i64 tiles = tn_seg_tiles(n, D);
    return tiles > 1 ? (int)(tiles < 1024 ? tiles : 1024) : 0;
}

// ---- stages 4 and 5 of a very large mini-batch over a small vocabulary whose words repeat (group.hip)
// Up to so many words a counter and a bucket of the alias table per word fit a compute unit's LDS.  Step of 8 192 centers, 256 tasks
// each, 3 peers, D = 256, Zipf exponent 1.3, by occurrences / by pairs: 1 323 words 231 / 116 us, 2 000 239 / 120, 5 000 258 / 141, 10 000
// 273 / 170 (exponent 1.1 338 / 235, 1.45 235 / 140), 12 288 277 / 179.
#define TN_GROUP_MAX_VOCAB 12288
// Occurrences from which on it goes by pairs: an announced mini-batch of no more is sorted beside the call before it and goes by
// occurrences, and one that nobody announced has to give the same bits (step of 1 000 words, a million occurrences of 128 tasks
// each, by occurrences announced 98 us at D = 64, 138 at D = 256, not announced 121 and 151, by pairs 87 and 94).
#define TN_GROUP_MIN_OCC (1 << 20)
// Tasks per position, at least: where an earlier form, which took nearly twice as long, gained nothing.  Step of 1.2 million
// occurrences by occurrences / by pairs: 128 tasks, 700 words, D = 64 128 / 87 us, D = 256 in bfloat16 168 / 92, 4 000 words 154 / 111 and
// 195 / 115; 64 tasks, 700 words, D = 64 143 / 96, D = 256 189 / 104, 4 000 words 173 / 125 and 219 / 134: the line could lie lower.
#define TN_GROUP_MIN_TASKS 128
#define TN_GROUP_HOT 16        // frequent center words that a workgroup takes at a time
// A center word of more than so many positions is frequent: it is taken against the whole vocabulary, others against the list of
// the words they met.  A pair of a list takes three to four times as long as one of all pairs: from where two words in seven are
// met, nearly, as are of three tasks for every two words.  Step of 16 384 centers, 10 000 words, D = 256, 256 tasks: frequent from
// 16 / 32 / 64 positions on 199 / 193 / 194 us, from 177 217, from 255 237; 12 000 words, D = 1 024, 512 tasks, 2 355 centers from 5 / 36 / 108
// 661 / 559 / 616.
static inline i64 tn_group_rare(i64 V, int per_center, i64 n_centers)        // per_center <= TN_REPEAT_MAX_TASKS
{
    const i64 padded = (V + 63) / 64 * 64, least = (padded * 3 / 2 + per_center - 1) / per_center, few = (n_centers + 511) / 512;
    const i64 most = 65535 / per_center;                                     // a list's counts fit 16 bits
    const i64 n = least > few ? least : few;
    return n < 4 ? 4 : n < most ? n : most;
}
// Positions of a frequent center word that are counted together: their counts fit 16 bits.
static inline i64 tn_group_chunk(int per_center, i64 n_centers)
{
    const i64 few = (n_centers + 2047) / 2048, most = 65535 / per_center, least = per_center <= 256 ? 64 : 32;
    return few < least ? least : few < most ? few : most;
}
// Frequent center words and their chunks, at most, of any mini-batch of up to n_centers positions.
static inline i64 tn_group_frequent(i64 V, int per_center, i64 n_centers)
{
    const i64 least = n_centers / (tn_group_rare(V, per_center, 1) + 1), many = n_centers * per_center / 65535 + 1;
    const i64 n = least < 1024 ? least : many < 1024 ? 1024 : many < least ? many : least;
    return n < V ? n : V;
}
// A chunk is a 2 048th of the positions; where that is fewer than `least`, `least`; and never more than a whole number of positions whose
// counts fit.  On top of so many comes a chunk that is not full per frequent center word.
static inline i64 tn_group_chunks(i64 V, int per_center, i64 n_centers)
{
    const i64 many = n_centers / (65535 / per_center) + 1, n = n_centers / 32;
    return (n < 2048 ? n + 1 : many < 2048 ? 2048 : many) + tn_group_frequent(V, per_center, n_centers);
}
// Workgroups per 64 words of the vocabulary that share the frequent center words, and that share the rows' elements: several
// where the vocabulary alone would leave most of the chip idle (step of 2 355 centers, 512 tasks, 40 words, D = 1 024: 123 us with
// three workgroups in all, 86 with twelve).
static inline int tn_group_slices(i64 V, i64 frequent)
{
    const i64 some = 1024 / ((V + 63) / 64), all = (frequent + TN_GROUP_HOT - 1) / TN_GROUP_HOT;
    return (int)(all < 1 ? 1 : some < all ? (some < 1 ? 1 : some) : all);
}
static inline int tn_group_parts(i64 V, int slices, int D)
{
    const i64 some = 512 / ((V + 63) / 64 * slices), all = (D + 255) / 256;
    return (int)(some < 1 ? 1 : some < all ? some : all);
}
struct GroupArgs {
    FwdArgs f;               // g: scales of the rare center words' words, in the place of their list entries; center_part by sorted
                             // position; center_loss too, then a workgroup of the frequent ones each
    NoiseDraw noise;
    int *status;
    const u32 *vals;         // positions in the order of their center words
    const int *seg_of, *seg_start, *n_in, *in_ids;
    int words;               // 64-word groups of the vocabulary
    int rare, chunk;         // see tn_group_rare, tn_group_chunk
    int per_center;          // tasks of a position, at most
    int slices, parts, most_frequent;   // see tn_group_slices
    u32 *dense;              // [chunks][64 * words] counts of the chunks of frequent center words
    u32 *list, *counts;      // [positions in all][per_center] the rare center words' words, from their first position's place on
    u64 *any;                // [words] words that occur
    u64 *masks;              // [center words][words] words of a rare center word
    unsigned short *starts;  // [center words][words] words of its list before these
    u64 *turned;             // [center words / 64][64 * words] a word's rare center words
    int4 *meta;              // [center words] the word, first sorted position, words in the list (none if frequent), 1 + number if frequent
    int4 *frequent;          // the word, row, chunks, the first of them
    int *n_frequent;
    double *hot_rows;        // [slices][64 * words][D] what the frequent center words give a word's row
    double *hot_part;        // [frequent][words][D] what 64 words give a frequent center word's row
    float *in_rows, *out_rows;
    int *out_ids, *out_n;
    u64 *index_mask;         // [words] the table update's index of the out-side rows (NULL: not wanted)
    u32 *index_start;
};
struct AuxWork;
// what: the pairs and their rows, or one of the tables' sums or both; `aux` rides with the rows, with the sums
enum { GROUP_ROWS = 0, GROUP_SUMS_IN = 1, GROUP_SUMS_OUT = 2 };
void tn_launch_group(const GroupArgs &a, int what, const AuxWork &aux, hipStream_t st);

void tn_launch_loss(const float *center_loss, int n_centers, float inv_P, float *mean_loss,
                    hipStream_t st);
void tn_launch_empty_grad(int *n_in, int *n_out, float *mean_loss, int *seg_in, int *seg_out,
                          hipStream_t st);

// ---- stage 6/7: DASGD merge and table update
struct ApplySrc {
    const int *ids;
    const void *rows;        // [capacity][D] fp32; bfloat16 for the sources 1.. of a call with packed peers
    const int *n_rows;
    i64 capacity;
};
struct ApplyArgs {
    void *table[2];          // W_in, W_out
    int dtype, D, stride;
    i64 V;
    int n_src;               // own + peers actually passed
    ApplySrc src[2][TN_MAX_SRC];
    u32 *start[2];           // [words+1][n_src]
    u64 *mask[2];            // [words][n_src]
    const u64 *skip[2];      // [words] rows that the chaining of long rows updates, a bit each (NULL: none)
    float lr;
    int *status;
    int packed;              // 1: the peers' rows (sources 1..) are bfloat16 messages, the own gradient's fp32
    // packed peers only, optional (NULL to skip): the own gradient is also written out as a bfloat16 message
    // while its rows pass through the update (ids, count and rounded rows; capacity checked on the host)
    unsigned short *msg_rows[2];
    int *msg_ids[2], *msg_n[2];
    // stochastic rounding of bf16 tables (a variant): key and serial number of this update
    int sr;
    u32 sr_k0, sr_k1, sr_serial;
};
// Small jobs that ride at the front of the grid of the forward pass or of the segmented reduction
// (workgroups [0, total) of that launch): phases of a mini-batch's preparation, the mean loss, clearing the masks of
// the table update's index, copying a prepared mini-batch's row index to the caller's buffers, indexing the sources
// [k_begin, k_end) of the coming table update.  Clearing and indexing must not share a launch (the index needs
// cleared masks); of two phases neither may need the other's result.
struct AuxWork {
    int total;               // prep + loss + clear_blocks + 2 * copy_blocks + 2 * (k_end - k_begin) * index_blocks
    PrepPhase prep[2];
    const float *center_loss;   // mean loss: sum of [n_centers] terms times inv_P
    float *mean_loss;           // NULL: not wanted
    int n_centers;
    float inv_P;
    int clear_blocks;
    u64 *clear_mask[2];      // masks to zero (both tables), clear_n entries each -- not necessarily apply's
    size_t clear_n;
    int copy_blocks;         // per table
    RowIndexCopy copy;
    int index_blocks;        // per (source, table)
    int k_begin, k_end;
    ApplyArgs apply;
};
void tn_aux_none(AuxWork &x);
void tn_aux_add_prep(AuxWork &x, const PrepPhase &p);   // twice at most
void tn_aux_add_loss(AuxWork &x, const float *center_loss, int n_centers, float inv_P, float *mean_loss);
void tn_aux_add_clear(AuxWork &x, u64 *mask_in, u64 *mask_out, size_t n);
void tn_aux_add_copy(AuxWork &x, const RowIndexCopy &c, i64 max_rows);
void tn_aux_add_index(AuxWork &x, const ApplyArgs &a, int k_begin, int k_end);

void tn_launch_apply_clear(const ApplyArgs &a, hipStream_t st);
void tn_launch_apply_index(const ApplyArgs &a, int k_begin, int k_end, hipStream_t st);
// rows of W_out that an update's sources may have, by their capacities
static inline i64 tn_union_rows(const ApplyArgs &a)
{
    i64 cap = 0;
    for (int k = 0; k < a.n_src; ++k)
        if (a.src[1][k].ids != nullptr) cap += a.src[1][k].capacity;
    return cap;
}
// whether a phase can ride with the update: its workgroups come on top of those for the rows (of 16 vocabulary rows
// each, at least), and one launch has to hold them all
static inline bool tn_apply_carries(int D, i64 V) { return D <= 512 && (V + 15) / 16 + TN_PREP_CHAIN_MAX <= TN_MAX_BLOCKS; }
void tn_launch_apply_update(const ApplyArgs &a, const PrepPhase *rider, const ChainWork *chain, hipStream_t st);   // both may be NULL
void tn_launch_apply_update_riding(const ApplyArgs &a, const PrepPhase &rider, hipStream_t st);
void tn_launch_apply_update_chaining(const ApplyArgs &a, const PrepPhase *rider, const ChainWork &chain, hipStream_t st);   // not where tn_streams
static inline bool tn_streams(i64 V, int stride, int dtype) { return 2 * V * (i64)stride * (dtype == 0 ? 4 : 2) > ((i64)1 << 30); }

// ---- sum of sparse gradients: out = src_0 + src_1 + ... on the union of their rows
struct GradSumArgs {
    ApplyArgs a;             // sources, index arrays, V, D (tables, lr unused)
    int *out_ids[2];         // [capacity] ascending
    float *out_rows[2];      // [capacity][D]
    int *out_n[2];           // [1]
    i64 out_cap[2];
    u32 *wbase[2];           // [words] scratch: rows of the union before each 64-row word
    u32 *wblk[2];            // [ceil(words / TN_UNION_WORDS)] scratch: rows of the union per block of words
};
#define TN_UNION_WORDS 1024  // vocabulary words per workgroup in the union scan (256 threads x 4)
void tn_launch_grad_sum_index(const GradSumArgs &g, hipStream_t st);   // index + scan
void tn_launch_grad_sum_rows(const GradSumArgs &g, hipStream_t st);    // the rows themselves

// ---- a sparse gradient as a bfloat16 message: row counts and ids copied, rows rounded to nearest even
struct GradPackArgs {
    const int *n[2], *ids[2];
    const float *rows[2];
    int *out_n[2], *out_ids[2];
    unsigned short *out_rows[2];
    i64 cap[2], out_cap[2];
    int D;
    int *status;
};
void tn_launch_grad_pack(const GradPackArgs &a, hipStream_t st);

// ---- dense-model apply, embedding lookup, cosine difference between two tables
struct DenseApplyArgs {
    void *theta;                       // [n] f32 or bf16
    const float *grads[TN_MAX_SRC];    // n_grads blocks of [n] fp32
    i64 n;
    int n_grads, dtype;
    float lr;
};
void tn_launch_dense_apply(const DenseApplyArgs &a, hipStream_t st);
struct LookupArgs {
    const void *table;
    const int *ids;
    float *out;       // [n][D]
    i64 n, V;
    int D, stride, dtype;
    int *status;
};
void tn_launch_lookup(const LookupArgs &a, hipStream_t st);
struct CosineArgs {
    const void *a, *b;
    float *diff;      // [V]
    i64 V;
    int D, stride, dtype;
};
void tn_launch_cosine_diff(const CosineArgs &a, hipStream_t st);

// ---- measurement aid: plain copy of `bytes` (multiple of 16)
void tn_launch_copy_probe(void *dst, const void *src, size_t bytes, hipStream_t st);
// mode 0 plain copy, 1 copy around the caches, 2 read only, 3 three reads per write (src holds 3 * bytes)
void tn_launch_stream_probe(void *dst, const void *src, size_t bytes, int mode, hipStream_t st);

// ---- host-side helpers shared by the files that hold C-ABI entry points
// records the thread-local message of tensair_last_error and returns `code`
int tn_fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
