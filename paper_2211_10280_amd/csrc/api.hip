// C ABI of libtensair: argument checks, workspace carving, alias-table construction
// and the order in which the kernels of one DASGD worker step are enqueued.
// Call names follow the Model operator of TensAIR (arXiv 2211.10280), Algorithm 1.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/tensair.h"
#include "dev_common.h"
#include "kernels.h"

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(TENSAIR_EHIP, "%s: %s", #expr, hipGetErrorString(e_));             \
    } while (0)

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

struct Sizes {
    i64 Bmax, Pmax, Omax;
    int key_bits, passes, bits, nd;
    size_t pub_words;          // what the preparation's workgroups publish, and their tickets (prep_layout)
    int tiles_out, tiles_in;   // segmented-reduction tiles
    i64 words;
    bool group;                // mini-batches may be large enough to go by pairs of words (group.hip), as far as the sizes go
};

bool config_ok(const tensair_config *c, const char **why)
{
    *why = nullptr;
    if (!c) { *why = "cfg is NULL"; return false; }
    if (c->vocab < 1 || c->vocab > TENSAIR_MAX_VOCAB) { *why = "vocab outside 1..TENSAIR_MAX_VOCAB"; return false; }
    if (c->dim < 4 || c->dim > TENSAIR_MAX_DIM || c->dim % 4) { *why = "dim must be a multiple of 4 in 4..1024"; return false; }
    if (c->row_stride < c->dim || c->row_stride % 4) { *why = "row_stride must be >= dim and a multiple of 4"; return false; }
    if (c->dtype != TENSAIR_F32 && c->dtype != TENSAIR_BF16) { *why = "unknown dtype"; return false; }
    if (c->window < 1 || c->window > 1024) { *why = "window out of range"; return false; }
    if (c->negatives < 0 || c->negatives > 65535) { *why = "negatives out of range"; return false; }
    if (c->max_centers < 1) { *why = "max_centers must be positive"; return false; }
    if (c->max_peers < 0 || c->max_peers > TENSAIR_MAX_PEERS) { *why = "max_peers out of range"; return false; }
    if (c->worker_id >= 65536u) { *why = "worker_id must be below 65536"; return false; }
    if (c->flags & ~(TENSAIR_RESAMPLE_NEGATIVES | TENSAIR_STOCHASTIC_ROUNDING)) { *why = "unknown flag"; return false; }
    i64 omax = (i64)2 * c->window * c->max_centers * (c->negatives + 1);
    if (omax + c->max_centers >= 0x7FFFFFFFLL) { *why = "batch too large: occurrences must fit 31 bits"; return false; }
    return true;
}

// What the preparation of a mini-batch of O occurrences and n centers publishes between its workgroups, in 32-bit
// words from the start of the set's area: a ticket per phase, the segment scan's words (64 bits; in-side for row counts
// and weights, then out-side), then per pass of the sort the groups' counts (counted passes) of the in-side and the
// out-side list and the two lists' tiles' digit words.
#define PREP_TICKETS 8
struct PrepLayout {
    bool chained;
    size_t seg_in, seg_out, pass0;
    size_t groups, group_out;                // words of a pass's groups, the out-side ones among them
    size_t tile0, per_pass, tile_out;        // words of the tiles of pass i: from tile0 + i * per_pass
    size_t clear, words;                     // what the keys clear, from the start; all
};
PrepLayout prep_layout(const Sizes &s, int O, int n, bool chained)
{
    PrepLayout l;
    l.chained = chained;
    const size_t ti = (size_t)tn_prep_tiles(n), to = (size_t)tn_prep_tiles(O);
    l.seg_in = PREP_TICKETS;
    l.seg_out = l.seg_in + 2 * (2 * (size_t)tn_prep_seg_tiles(n));
    l.pass0 = l.seg_out + 2 * (size_t)tn_prep_seg_tiles(O);
    const size_t gi = l.chained ? 0 : (size_t)tn_prep_groups((int)ti) + 1;      // and a row for the sum of all
    const size_t go = l.chained ? 0 : (size_t)tn_prep_groups((int)to) + 1;
    l.groups = (gi + go) * s.nd;
    l.group_out = gi * s.nd;
    l.tile0 = l.pass0 + s.passes * l.groups;
    l.tile_out = ti * s.nd;
    l.per_pass = l.chained ? (ti + to) * s.nd : 0;      // counted: written and read within a pass, one set is enough
    l.words = l.tile0 + (l.chained ? s.passes : 1) * (ti + to) * s.nd;
    l.clear = l.chained ? l.words : l.tile0;
    return l;
}

Sizes sizes_of(const tensair_config &c)
{
    Sizes s;
    s.Bmax = c.max_centers;
    s.Pmax = (i64)2 * c.window * s.Bmax;
    s.Omax = s.Pmax * (c.negatives + 1);
    int kb = 1;
    while (((i64)1 << kb) < c.vocab) ++kb;
    s.key_bits = kb;
    tn_radix_shape(kb, &s.passes, &s.bits);
    s.nd = 1 << s.bits;
    {   // a mini-batch may be prepared either way as long as it has at most TN_PREP_CHAIN_MAX tiles
        const PrepLayout l = prep_layout(s, (int)s.Omax, (int)s.Bmax, false);
        i64 tiles = (i64)tn_prep_tiles((int)s.Omax) + tn_prep_tiles((int)s.Bmax);
        if (tiles > TN_PREP_CHAIN_MAX) tiles = TN_PREP_CHAIN_MAX;
        const size_t chained = l.pass0 + (size_t)s.passes * (size_t)tiles * s.nd;
        s.pub_words = l.words > chained ? l.words : chained;
    }
    auto seg_tiles = [&](i64 most) {   // worst case over n <= most: at most, and at the last n of every tile size
        i64 tiles = tn_seg_tiles(most, c.dim);
        for (i64 n : {(i64)8192, (i64)32768})
            if (n < most) tiles = std::max(tiles, tn_seg_tiles(n, c.dim));
        return (int)tiles;
    };
    s.tiles_out = seg_tiles(s.Omax);
    s.tiles_in = seg_tiles(s.Bmax);
    s.words = (c.vocab + 63) / 64;
    const i64 per_center = (i64)2 * c.window * (c.negatives + 1);
    s.group = c.vocab <= TN_GROUP_MAX_VOCAB && s.Omax > TN_GROUP_MIN_OCC && per_center >= TN_GROUP_MIN_TASKS && per_center <= TN_REPEAT_MAX_TASKS;
    return s;
}

}  // namespace

int tn_fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

// Everything about a mini-batch that does not depend on the tables: keys (pairs and negatives), their
// sorted order, segments, unique row ids.  There are two sets, used in turn, so that the set of the
// coming mini-batch can be filled (tensair_prefetch) while the kernels of the current one still read theirs.
struct BatchSet {
    u32 *keys[3], *vals[2];
    u32 *hist;             // digit counts of both key lists, all passes; zero between mini-batches ...
    bool hist_clean = false;   // ... once everything enqueued so far has run
    u32 *pub;              // see prep_layout
    int *seg_of, *seg_start;
    int *long_cnt;
    int *pair_center;
    // row index of a prefetched mini-batch, copied to the caller's buffers when it is consumed
    int *ids_in, *ids_out, *n_rows, *off_in, *off_out;
    int cur = 0, kb = 1;   // which vals / keys buffer holds the sorted order
};

// A mini-batch announced by tensair_prefetch.
struct Prefetched {
    bool valid = false;
    bool chained = false;      // how it is (to be) prepared: on the caller's stream, most often riding in the launches ...
    int phase = 0;             // ... of the call before; phases that are enqueued, the consuming call does the rest;
    bool on_side = false;      // or as a whole on the second stream (ev_prep),
    bool late = false;         // where it may still be running when it is consumed: its keys have an event of their own
    const int32_t *tokens = nullptr;
    i64 n_tokens = 0, begin = 0, P = 0;
    int n_centers = 0;
    u32 epoch = 0, worker_id = 0;
    bool is(const int32_t *t, i64 nt, i64 b, int n, u32 e, u32 w) const
    {
        return valid && tokens == t && n_tokens == nt && begin == b && n_centers == n && epoch == e &&
               worker_id == w;
    }
};

// What is expected of the words that a mini-batch meets, going by the unigram counts.
struct WordStats {
    double different = 1.0;    // share of a position's negatives that are different words
    double hottest = 0.0;      // share of the most frequent word among all negatives,
    double per_pair = 0.0;     // the same word's occurrences among the tasks of a pair
    double center = 0.0;       // and its share of the centers
};

// A bucket of the alias table; the two lie side by side, so that a draw reads both with one access.
struct Draw {
    uint32_t thr;
    int32_t alias;
};

struct tensair_model {
    tensair_config cfg;
    Sizes sz;
    void *w_in, *w_out;
    // carved from the caller's workspace
    uint2 *draw;               // alias table: threshold, alias
    int *status;
    BatchSet set[2];
    int4 *long_list;
    float *g, *center_part, *center_loss, *part_out, *part_in, *cross_out, *cross_in;
    int *xinfo_out, *xinfo_in;
    u32 *start[2];
    u64 *mask[2];              // masks of the update's index, per table (buffer 0)
    u64 *mask_alt[2];          // a second set (buffer 1): inside tensair_step the two are used in turn, so that
                               // the one the next step will index can be cleared while this step still reads its own
    bool mask_clean[2] = {false, false};   // buffer b is all zeros (or will be when everything enqueued so far has run)
    u64 *group_masks = nullptr, *group_any = nullptr, *group_turned = nullptr;    // see GroupArgs
    unsigned short *group_starts = nullptr;
    int4 *group_meta = nullptr, *group_frequent = nullptr;
    int *group_n = nullptr;
    double *group_hot_rows = nullptr, *group_hot_part = nullptr;
    u32 *group_dense = nullptr;
    u64 *long_mask[2];         // rows of a step's own gradient that the table update chains, per table
    u32 *wbase[2], *wblk[2];   // tensair_grad_add: place of every 64-row word in the summed gradient
    std::vector<Draw> h_draw;  // the same on the host
    WordStats words;
    // second stream, forked from and joined to the caller's stream with events: the forward pass beside the sort of a
    // large mini-batch that was not prepared, the preparation of an announced one that is too large to ride
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_fwd = nullptr;
    // mini-batch sets: `busy` is the one the most recent gradient call reads; announced mini-batches are
    // prepared into the other one, riding in the launches of that call or on the second stream (ev_prep recorded
    // behind them)
    int busy = 1;
    Prefetched pend;               // prepared, or being prepared, or to be prepared in set 1 - busy
    Prefetched next;               // announced after `pend`: prepared from when `pend` is consumed
    hipEvent_t ev_prep = nullptr, ev_keys = nullptr, ev_reduced = nullptr;
    bool side_follows = false;     // the second stream has waited for the start of the latest gradient call
    // every event recorded on the second stream takes a ticket; the caller's stream is behind all of
    // them up to main_ticket, so a prepared set with prep_ticket <= main_ticket needs no wait
    u64 side_ticket = 0, main_ticket = 0, prep_ticket = 0, keys_ticket = 0;
    // set by tensair_step: the index of the coming apply is built by extra workgroups at the front of the
    // forward pass (clearing) and of the segmented reduction (the id lists), on the caller's stream
    ApplyArgs *fused_apply = nullptr;
    bool fused_index_done = false;
    ChainWork chain = {};               // tensair_step: the chaining of long rows that its update takes along (no blocks: none)
    bool prepare_under_apply = false;   // tensair_step: the table update is long enough to hide a preparation ...
    bool ride_long_update = false;      // ... many times over
    Prefetched deferred;                // the mini-batch to prepare under that update (enqueued by tensair_step)
    bool captured = false;              // a call on this handle was recorded into a HIP graph (see note_capture)
    u32 apply_serial = 0;               // table updates enqueued so far (stochastic rounding draws from it)
    // stage timing (tensair_profile): events recorded on the caller's stream
    int prof_level = 0;
    std::vector<hipEvent_t> prof_pool;
    std::vector<std::pair<int, hipEvent_t>> prof_marks;
    size_t prof_used = 0;
};

namespace {

// Lays the workspace out; with m == nullptr only the size is computed.
size_t carve(const tensair_config &c, const Sizes &s, char *base, tensair_model *m)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> char * {
        char *p = base ? base + off : nullptr;
        off += align_up(bytes);
        return p;
    };
    const size_t V = (size_t)c.vocab, D = (size_t)c.dim;
    const size_t NE = (size_t)(s.Omax + s.Bmax);
    const size_t K1 = (size_t)(c.max_peers + 1 > 2 ? c.max_peers + 1 : 2);   // the gradient sum indexes two sources
    char *p;
    p = take(V * 8); if (m) m->draw = (uint2 *)p;
    p = take(256); if (m) m->status = (int *)p;
    const size_t cap_in = (size_t)(s.Bmax < (i64)V ? s.Bmax : (i64)V);
    const size_t cap_out = (size_t)(s.Omax < (i64)V ? s.Omax : (i64)V);
    for (int u = 0; u < 2; ++u) {
        BatchSet *b = m ? &m->set[u] : nullptr;
        for (int i = 0; i < 3; ++i) { p = take(NE * 4); if (b) b->keys[i] = (u32 *)p; }
        for (int i = 0; i < 2; ++i) { p = take(NE * 4); if (b) b->vals[i] = (u32 *)p; }
        p = take((size_t)2 * s.passes * s.nd * 4); if (b) b->hist = (u32 *)p;
        p = take(s.pub_words * 4); if (b) b->pub = (u32 *)p;
        p = take(NE * 4); if (b) b->seg_of = (int *)p;
        p = take((NE + 2) * 4); if (b) b->seg_start = (int *)p;   // out-side rows at 0, in-side at Omax+1
        p = take(256); if (b) b->long_cnt = (int *)p;
        p = take((size_t)s.Pmax * 4); if (b) b->pair_center = (int *)p;
        p = take(cap_in * 4); if (b) b->ids_in = (int *)p;
        p = take(cap_out * 4); if (b) b->ids_out = (int *)p;
        p = take(256); if (b) b->n_rows = (int *)p;
        p = take((cap_in + 1) * 4); if (b) b->off_in = (int *)p;
        p = take((cap_out + 1) * 4); if (b) b->off_out = (int *)p;
    }
    p = take((size_t)(s.tiles_out + s.tiles_in) * 16); if (m) m->long_list = (int4 *)p;
    p = take((size_t)s.Omax * 4); if (m) m->g = (float *)p;
    p = take((size_t)s.Bmax * D * 4); if (m) m->center_part = (float *)p;
    const int per_center = 2 * c.window * (c.negatives + 1);
    const i64 frequent = s.group ? tn_group_frequent(c.vocab, per_center, s.Bmax) : 0;
    const size_t hot_blocks = s.group ? (size_t)s.words * tn_group_slices(c.vocab, frequent) : 0;
    p = take(((size_t)s.Bmax + hot_blocks) * 4); if (m) m->center_loss = (float *)p;
    p = take((size_t)s.tiles_out * 2 * D * 4); if (m) m->part_out = (float *)p;
    p = take((size_t)s.tiles_in * 2 * D * 4); if (m) m->part_in = (float *)p;
    p = take((size_t)(s.tiles_out / TN_SEG_XBLOCK + 2) * D * 4); if (m) m->cross_out = (float *)p;
    p = take((size_t)(s.tiles_in / TN_SEG_XBLOCK + 2) * D * 4); if (m) m->cross_in = (float *)p;
    p = take((size_t)(s.tiles_out / TN_SEG_XBLOCK + 2) * 4); if (m) m->xinfo_out = (int *)p;
    p = take((size_t)(s.tiles_in / TN_SEG_XBLOCK + 2) * 4); if (m) m->xinfo_in = (int *)p;
    if (s.group) {
        const size_t words = (size_t)s.words, most = (size_t)frequent;
        p = take(words * 8); if (m) m->group_any = (u64 *)p;
        p = take(cap_in * words * 8); if (m) m->group_masks = (u64 *)p;
        p = take(cap_in * words * 2); if (m) m->group_starts = (unsigned short *)p;
        p = take((cap_in + 63) / 64 * 64 * words * 8); if (m) m->group_turned = (u64 *)p;
        p = take(cap_in * 16); if (m) m->group_meta = (int4 *)p;
        p = take(most * 16); if (m) m->group_frequent = (int4 *)p;
        p = take(256); if (m) m->group_n = (int *)p;
        p = take(hot_blocks * 64 * D * 8); if (m) m->group_hot_rows = (double *)p;
        p = take(most * words * D * 8); if (m) m->group_hot_part = (double *)p;
        p = take((size_t)tn_group_chunks(c.vocab, per_center, s.Bmax) * 64 * words * 4); if (m) m->group_dense = (u32 *)p;
    }
    for (int t = 0; t < 2; ++t) {
        p = take((size_t)(s.words + 1) * K1 * 4); if (m) m->start[t] = (u32 *)p;
        p = take((size_t)s.words * K1 * 8); if (m) m->mask[t] = (u64 *)p;
        p = take((size_t)s.words * K1 * 8); if (m) m->mask_alt[t] = (u64 *)p;
        p = take((size_t)s.words * 8); if (m) m->long_mask[t] = (u64 *)p;
        p = take((size_t)s.words * 4); if (m) m->wbase[t] = (u32 *)p;
        p = take((size_t)(s.words / TN_UNION_WORDS + 1) * 4); if (m) m->wblk[t] = (u32 *)p;
    }
    return off;
}

// Alias table (Vose) of the noise distribution count^0.75 / sum.  Buckets whose scaled
// probability is below 1 keep floor(p * 2^32) as acceptance threshold and hand the rest
// of their mass to a donor; work lists are filled in ascending id order and consumed
// from the back, so the table is a deterministic function of the counts.
// n: draws per position, N: per pair.
bool build_alias(const uint64_t *counts, i64 V, std::vector<Draw> &draw, double n, int N, WordStats &words)
{
    draw.resize((size_t)V);
    std::vector<double> prob((size_t)V);
    double total = 0.0, tokens = 0.0;
    i64 most = 0;
    for (i64 i = 0; i < V; ++i) {
        prob[(size_t)i] = std::pow((double)counts[i], 0.75);
        total += prob[(size_t)i];
        tokens += (double)counts[i];
        if (counts[i] > counts[most]) most = i;
        draw[(size_t)i] = {0xFFFFFFFFu, (int32_t)i};
    }
    if (!(total > 0.0)) return false;
    words.hottest = prob[(size_t)most] / total;
    words.center = (double)counts[most] / tokens;
    words.per_pair = words.center + N * words.hottest;
    std::vector<int32_t> lo, hi;
    lo.reserve((size_t)V);
    hi.reserve((size_t)V);
    const double scale = (double)V;
    const double per_word = n / scale;
    double met = 0.0;
    for (i64 i = 0; i < V; ++i) {
        double q = prob[(size_t)i] * scale / total;
        prob[(size_t)i] = q;
        const double x = std::min(q * per_word, 1.0);   // 1 - exp(-x), nearly
        met += x - 0.37 * x * x;
        (q < 1.0 ? lo : hi).push_back((int32_t)i);
    }
    words.different = n > 0.0 ? met / n : 1.0;   // roughly
    const double two32 = 4294967296.0;
    while (!lo.empty() && !hi.empty()) {
        const int32_t poor = lo.back();
        lo.pop_back();
        const int32_t rich = hi.back();
        hi.pop_back();
        const double t = std::floor(prob[(size_t)poor] * two32);
        draw[(size_t)poor] = {t >= two32 ? 0xFFFFFFFFu : (uint32_t)t, rich};
        const double rest = (prob[(size_t)rich] + prob[(size_t)poor]) - 1.0;
        prob[(size_t)rich] = rest;
        (rest < 1.0 ? lo : hi).push_back(rich);
    }
    // whatever is left on either list keeps the full bucket (threshold max, alias = itself)
    return true;
}

// Share of different words among a position's negatives from which the forward pass works on the different ones only:
// measured at expected shares of 0.45 to 0.9, it gains below 0.9 (0.87: step 306 against 310 us) and loses nothing above
// but the table's cost (0.6 % at 0.9).
#define TN_REPEATS_BELOW 0.85
// The same for going by pairs of words (group.hip): rows of more than 128 elements gain wherever words repeat, narrow ones,
// whose gathers weigh less, less so.  Step over 12 000 words, 1.3 million occurrences of 256 tasks per position, by occurrences / by
// pairs, expected share 0.78, 0.82, 0.87, 0.92: D = 64 180 / 171, 191 / 186, 202 / 204, 220 / 235; D = 128 207 / 174, 219 / 189, 233 / 207,
// 252 / 240; D = 132 223 / 177, 237 / 191, 255 / 211, 273 / 245; 128 tasks, D = 64 192 / 163, 205 / 178, 214 / 199, 229 / 230.
static double pairs_below(int D) { return D <= TN_SUB_MAX_DIM ? 0.8 : TN_REPEATS_BELOW; }
// ... and only where no word is most of the negatives: an earlier form counted a word's occurrences by additions one after the other
// and was slower there (4 200 centers of 256 tasks, one word 103 by occurrences / 185 us by pairs then, a share of 0.63 96 / 110).  This
// one is not (step, D = 32, by occurrences / by pairs: one word, 4 200 centers 103 / 62, 65 536 centers 809 / 154; a share of 0.63
// 96 / 59 and 717 / 147; of 0.42 92 / 59 and 673 / 151): the line could go.
#define TN_GROUP_MAX_SHARE 0.5
// Stage tags of tensair_profile_read.  A tag's duration runs from the previous mark to its own.
enum { PF_BEGIN_GRAD = 0, PF_KEYS, PF_FORWARD, PF_SORT, PF_SEGMENTS, PF_REDUCE_IN, PF_REDUCE_OUT,
       PF_BEGIN_APPLY, PF_APPLY_INDEX, PF_APPLY_UPDATE, PF_BEGIN_ADD, PF_ADD_INDEX, PF_ADD_ROWS,
       PF_BEGIN_PACK, PF_PACK };

// records a timing event on `st` if stage timing asks for this tag; returns it (another stream may wait on
// it, which saves that stream's fork an event of its own) or nullptr
hipEvent_t mark(tensair_model *m, int tag, hipStream_t st)
{
    if (m->prof_level == 0) return nullptr;
    if (m->prof_level == 1 && tag != PF_APPLY_INDEX && tag != PF_APPLY_UPDATE && tag != PF_ADD_INDEX &&
        tag != PF_ADD_ROWS && tag != PF_BEGIN_PACK && tag != PF_PACK)
        return nullptr;
    if (m->prof_marks.size() >= 65536) return nullptr;
    hipEvent_t ev;
    if (m->prof_used < m->prof_pool.size()) {
        ev = m->prof_pool[m->prof_used];
    } else {
        if (hipEventCreate(&ev) != hipSuccess) return nullptr;
        m->prof_pool.push_back(ev);
    }
    ++m->prof_used;
    if (hipEventRecord(ev, st) != hipSuccess) return nullptr;
    m->prof_marks.emplace_back(tag, ev);
    return ev;
}

// A call that is being recorded into a HIP graph does not run now, and may run again at any time later: what it leaves
// in the workspace (zeroed digit counts and masks, a mini-batch that is prepared, wholly or in part) is not there when
// the host says so, and what other calls left there is gone after a replay.  From the first such call on, every call on
// the handle therefore starts from nothing: it prepares its own mini-batch and clears what it needs cleared.
bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) != hipSuccess) {   // another thread's capture: this stream takes no part in it
        (void)hipGetLastError();
        return false;
    }
    return s == hipStreamCaptureStatusActive;
}
void note_capture(tensair_model *m, hipStream_t st)
{
    if (!m->captured && !capturing(st)) return;
    m->captured = true;
    m->pend.valid = m->next.valid = m->deferred.valid = false;
    m->mask_clean[0] = m->mask_clean[1] = false;
    m->set[0].hist_clean = m->set[1].hist_clean = false;
}

i64 pair_count(const tensair_config &c, i64 T, i64 begin, int n)
{
    return pairs_before(begin + n, T, c.window) - pairs_before(begin, T, c.window);
}

int check_rows(const tensair_sparse_rows &r, i64 need, const char *what)
{
    if (!r.n_rows || !r.row_ids || !r.row_grads) return fail(TENSAIR_EINVAL, "%s: NULL pointer", what);
    if (r.capacity < need)
        return fail(TENSAIR_ECAPACITY, "%s: capacity %lld < %lld rows required", what,
                    (long long)r.capacity, (long long)need);
    if (r.capacity > 0x7FFFFFFFLL) return fail(TENSAIR_EINVAL, "%s: capacity too large", what);
    return TENSAIR_OK;
}

// One source of the table update: the two tables' rows of a gradient (fp32) or of a bfloat16 message.
template <typename Grad>
int fill_apply_src(ApplyArgs &a, int k, const Grad *g, const char *what)
{
    for (int t = 0; t < 2; ++t) {
        const auto &r = t ? g->out : g->in;
        if (!r.n_rows || !r.row_ids || !r.row_grads) return fail(TENSAIR_EINVAL, "%s: NULL pointer", what);
        if (r.capacity < 0 || r.capacity > 0x7FFFFFFFLL) return fail(TENSAIR_EINVAL, "%s: bad capacity", what);
        if (((uintptr_t)r.row_grads & 15) || ((uintptr_t)r.row_ids & 3) || ((uintptr_t)r.n_rows & 3))
            return fail(TENSAIR_EINVAL, "%s: rows must be 16-byte aligned, ids and counts 4-byte aligned", what);
        a.src[t][k].ids = r.row_ids;
        a.src[t][k].rows = r.row_grads;
        a.src[t][k].n_rows = r.n_rows;
        a.src[t][k].capacity = r.capacity;
    }
    return TENSAIR_OK;
}

}  // namespace

extern "C" {

const char *tensair_last_error(void) { return g_err; }

int32_t tensair_aligned_row_stride(int32_t dim, int32_t dtype)
{
    if (dim < 1 || dim > TENSAIR_MAX_DIM || (dtype != TENSAIR_F32 && dtype != TENSAIR_BF16)) return -1;
    const int per_line = dtype == TENSAIR_F32 ? 32 : 64;   // elements in 128 bytes
    return (dim + per_line - 1) / per_line * per_line;
}

size_t tensair_workspace_bytes(const tensair_config *cfg)
{
    const char *why;
    if (!config_ok(cfg, &why)) { fail(TENSAIR_EINVAL, "%s", why); return 0; }
    return carve(*cfg, sizes_of(*cfg), nullptr, nullptr);
}

int64_t tensair_capacity_in(const tensair_config *cfg, int32_t n_centers)
{
    if (!cfg || n_centers < 0) return -1;
    i64 n = n_centers;
    return n < cfg->vocab ? n : cfg->vocab;
}

int64_t tensair_capacity_out(const tensair_config *cfg, int32_t n_centers)
{
    if (!cfg || n_centers < 0) return -1;
    i64 n = (i64)2 * cfg->window * n_centers * (cfg->negatives + 1);
    return n < cfg->vocab ? n : cfg->vocab;
}

int tensair_model_init(tensair_model **out, const tensair_config *cfg, void *w_in, void *w_out,
                       int fill_tables, const uint64_t *unigram_counts, void *workspace,
                       size_t workspace_bytes, void *stream)
{
    const char *why;
    if (!out) return fail(TENSAIR_EINVAL, "out is NULL");
    *out = nullptr;
    if (!config_ok(cfg, &why)) return fail(TENSAIR_EINVAL, "%s", why);
    if (!w_in || !w_out || !unigram_counts || !workspace) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (((uintptr_t)w_in | (uintptr_t)w_out) & 15) return fail(TENSAIR_EINVAL, "tables must be 16-byte aligned");
    if ((uintptr_t)workspace & 255) return fail(TENSAIR_EINVAL, "workspace must be 256-byte aligned");
    Sizes sz = sizes_of(*cfg);
    size_t need = carve(*cfg, sz, nullptr, nullptr);
    if (workspace_bytes < need)
        return fail(TENSAIR_ECAPACITY, "workspace has %zu bytes, %zu needed", workspace_bytes, need);
    tensair_model *m = new (std::nothrow) tensair_model();
    if (!m) return fail(TENSAIR_EINVAL, "out of host memory");
    m->cfg = *cfg;
    m->sz = sz;
    m->w_in = w_in;
    m->w_out = w_out;
    carve(*cfg, sz, (char *)workspace, m);
    if (!build_alias(unigram_counts, cfg->vocab, m->h_draw, 2.0 * cfg->window * cfg->negatives, cfg->negatives, m->words)) {
        delete m;
        return fail(TENSAIR_EINVAL, "unigram_counts has no positive entry");
    }
    hipStream_t st = (hipStream_t)stream;
    // in pieces of 4 MB: longer copies from pageable memory take another, slower way (8 MB: 7 ms more)
    hipError_t e = hipSuccess;
    for (size_t at = 0, n = (size_t)cfg->vocab; at < n && e == hipSuccess; at += (size_t)1 << 19) {
        const size_t k = n - at < ((size_t)1 << 19) ? n - at : (size_t)1 << 19;
        e = hipMemcpyAsync(m->draw + at, m->h_draw.data() + at, k * sizeof(Draw), hipMemcpyHostToDevice, st);
    }
    int zero[4] = {0, 0, 0, 0};
    if (e == hipSuccess) e = hipMemcpyAsync(m->status, zero, sizeof(zero), hipMemcpyHostToDevice, st);
    if (e == hipSuccess && fill_tables) {
        tn_launch_init_tables(w_in, w_out, cfg->vocab, cfg->dim, cfg->row_stride, cfg->dtype, cfg->seed, st);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        delete m;
        return fail(TENSAIR_EHIP, "model_init: %s", hipGetErrorString(e));
    }
    if (hipStreamCreateWithFlags(&m->side, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m->ev_fwd, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m->ev_prep, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m->ev_keys, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&m->ev_reduced, hipEventDisableTiming) != hipSuccess) {
        tensair_model_destroy(m);
        return fail(TENSAIR_EHIP, "model_init: cannot create the side stream");
    }
    *out = m;
    return TENSAIR_OK;
}

int tensair_model_rebind(tensair_model *m, void *w_in, void *w_out, uint32_t worker_id)
{
    if (!m || !w_in || !w_out) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (((uintptr_t)w_in | (uintptr_t)w_out) & 15) return fail(TENSAIR_EINVAL, "tables must be 16-byte aligned");
    if (worker_id >= 65536u) return fail(TENSAIR_EINVAL, "worker_id must be below 65536");
    m->w_in = w_in;
    m->w_out = w_out;
    m->cfg.worker_id = worker_id;
    return TENSAIR_OK;
}

int tensair_model_alias(const tensair_model *m, uint32_t *thr, int32_t *alias)
{
    if (!m || !thr || !alias) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    for (size_t i = 0; i < (size_t)m->cfg.vocab; ++i) {
        thr[i] = m->h_draw[i].thr;
        alias[i] = m->h_draw[i].alias;
    }
    return TENSAIR_OK;
}

int64_t tensair_pair_count(const tensair_model *m, int64_t n_tokens, int64_t center_begin, int32_t n_centers)
{
    if (!m || n_tokens < 1 || center_begin < 0 || n_centers < 0 || center_begin + n_centers > n_tokens) {
        fail(TENSAIR_EINVAL, "pair_count: bad range");
        return -1;
    }
    return pair_count(m->cfg, n_tokens, center_begin, n_centers);
}

// A mini-batch as its preparation and its gradient calculation take it.
struct BatchWork {
    BatchDesc b;
    i64 P, O;
    u32 epoch, worker_id;
    bool centers_only;     // the occurrences are not listed
};

static BatchWork batch_work(const tensair_config &c, const int32_t *tokens, i64 n_tokens, i64 center_begin,
                            int n_centers, u32 epoch, i64 P)
{
    BatchWork w;
    w.b.tok = tokens;
    w.b.T = n_tokens;
    w.b.begin = center_begin;
    w.b.n_centers = n_centers;
    w.b.w = c.window;
    w.b.N = c.negatives;
    w.b.pair_base = pairs_before(center_begin, n_tokens, c.window);
    w.b.P = P;
    w.P = P;
    w.O = P * (c.negatives + 1);
    w.epoch = epoch;
    w.worker_id = c.worker_id;
    w.centers_only = false;
    return w;
}

// Tiles of a mini-batch's two key lists together, and the phases of its preparation: the keys, the sort (per pass one, or a
// count and a pass), the segments (one, or the heads and the segments).
static int prep_tiles(const tensair_config &c, i64 P, int n_centers) { return tn_prep_tiles((int)(P * (c.negatives + 1))) + tn_prep_tiles(n_centers); }
static int prep_phases(const Sizes &s, bool chained) { return chained ? s.passes + 2 : 2 * s.passes + 3; }
static int prep_sort_end(const Sizes &s, bool chained) { return prep_phases(s, chained) - (chained ? 1 : 2); }

struct RowIndexDst {
    int *ids, *n_rows, *offsets;
    i64 capacity;
};

// A key list in sorted order and its segments (side 0: W_out, 1: W_in)
struct SortedSide {
    const u32 *keys, *vals;
    int *seg_of, *seg_start, *long_cnt;
};

static SortedSide sorted_side(const tensair_model *m, const BatchSet &S, int side)
{
    const size_t at = side ? (size_t)m->sz.Omax : 0;
    return {S.keys[S.kb] + at, S.vals[S.cur] + at, S.seg_of + at, S.seg_start + (side ? (size_t)m->sz.Omax + 1 : 0),
            S.long_cnt + side};
}

static NoiseDraw noise_draw(const tensair_model *m, const BatchWork &w)
{
    const tensair_config &c = m->cfg;
    return {c.vocab, m->draw, (u32)(c.seed & 0xFFFFFFFFu), (u32)(c.seed >> 32), w.worker_id + 65536u * w.epoch,
            (c.flags & TENSAIR_RESAMPLE_NEGATIVES) != 0};
}

// One phase as it is launched.  Key lists: out-side occurrences at [0, O), in-side centers at [Omax, Omax + n_centers);
// the unsorted keys in keys[0] are never written again (the forward pass reads them); the passes go 0 -> 1 -> 2 -> 1.
static void make_prep_phase(tensair_model *m, BatchSet &S, const BatchWork &w, bool chained, int phase,
                            const RowIndexDst &in, const RowIndexDst &out, int32_t *negatives_dbg, PrepPhase &x)
{
    const tensair_config &c = m->cfg;
    const Sizes &s = m->sz;
    const PrepLayout l = prep_layout(s, (int)w.O, w.b.n_centers, chained);
    memset(&x, 0, sizeof(x));
    const int n[2] = {(int)w.O, w.b.n_centers};
    const size_t at[2] = {0, (size_t)s.Omax};
    if (phase == 0) {
        PrepKeys &k = x.keys;
        x.kind = PREP_KEYS;
        k.centers_only = w.centers_only;
        const i64 slots = k.centers_only ? (i64)w.b.n_centers : (i64)w.b.n_centers * 2 * c.window * (c.negatives + 1);
        const int per_block = tn_prep_keys_slots(slots);
        x.blocks = (int)((slots + per_block - 1) / per_block);
        k.items = per_block / BLOCK;
        k.b = w.b;
        k.noise = noise_draw(m, w);
        k.out_keys = S.keys[0];
        k.in_keys = S.keys[0] + s.Omax;
        k.pair_center = S.pair_center;
        k.neg_dbg = negatives_dbg;
        k.status = m->status;
        k.hist = l.chained ? S.hist : nullptr;
        k.passes = s.passes;
        k.bits = s.bits;
        k.clear = S.pub;
        k.n_clear = l.clear;
    } else if (phase < prep_sort_end(s, l.chained)) {
        PrepPass &p = x.pass;
        const int i = l.chained ? phase - 1 : (phase - 1) / 2;
        x.kind = l.chained ? PREP_PASS : (phase & 1) ? PREP_COUNT : PREP_PASS_COUNTED;
        const int kin = i == 0 ? 0 : (i & 1) ? 1 : 2, kout = (i & 1) ? 2 : 1;
        for (int t = 0; t < 2; ++t) {
            PrepPassList &q = p.p[t];
            q.kin = S.keys[kin] + at[t];
            q.kout = S.keys[kout] + at[t];
            q.vin = S.vals[i & 1] + at[t];
            q.vout = S.vals[(i & 1) ^ 1] + at[t];
            q.n = n[t];
            q.tiles = tn_prep_tiles(n[t]);
            q.state = S.pub + l.tile0 + (size_t)i * l.per_pass + (t == 0 ? l.tile_out : 0);
            q.hist = l.chained ? S.hist + (size_t)(t * s.passes + i) * s.nd
                               : S.pub + l.pass0 + (size_t)i * l.groups + (t == 0 ? l.group_out : 0);
            x.blocks += q.tiles;
        }
        p.ticket = S.pub + i;
        p.shift = i * s.bits;
        p.bits = s.bits;
        p.scanned = !l.chained && std::max(tn_prep_groups(p.p[0].tiles), tn_prep_groups(p.p[1].tiles)) > TN_PREP_GROUPS_OWN;
        p.first = i == 0;
        S.kb = kout;
        S.cur = (i & 1) ^ 1;
    } else {
        PrepSegments &g = x.seg;
        x.kind = l.chained ? PREP_SEGMENTS : phase == prep_phases(s, false) - 1 ? PREP_SEGMENTS_COUNTED : PREP_HEADS;
        for (int t = 0; t < 2; ++t) {
            PrepSegmentsList &q = g.p[t];
            const RowIndexDst &d = t ? in : out;
            const SortedSide v = sorted_side(m, S, t);
            q.keys = v.keys;
            q.vals = v.vals;
            q.n = n[t];
            q.tiles = tn_prep_seg_tiles(n[t]);
            q.state = (u64 *)(S.pub + (t ? l.seg_in : l.seg_out));
            q.seg_of = v.seg_of;
            q.seg_start = v.seg_start;
            q.long_cnt = v.long_cnt;
            q.row_ids = d.ids;
            q.n_rows = d.n_rows;
            q.seg_offsets = d.offsets;
            q.capacity = d.capacity;
            x.blocks += q.tiles;
        }
        g.begin = w.b.begin;
        g.T = w.b.T;
        g.w = c.window;
        g.hist = S.hist;
        g.n_hist = 2 * s.passes * s.nd;
        g.ticket = S.pub + s.passes;
        g.status = m->status;
    }
}

// Notes that a phase is enqueued; the keys of a chained preparation add to digit counts that must be zero, which its
// segments leave behind -- unless it was left unfinished (an announcement dropped, a failed call): then they are
// cleared here.
static void before_prep_phase(tensair_model *m, BatchSet &S, int kind, hipStream_t st)
{
    if (kind == PREP_KEYS) {
        if (!S.hist_clean) tn_launch_prep_clear(S.hist, 2 * m->sz.passes * m->sz.nd, st);
        S.hist_clean = false;
    } else if (kind == PREP_SEGMENTS || kind == PREP_SEGMENTS_COUNTED) {
        S.hist_clean = true;
    }
}

// the phases [from, to) as launches of their own
static void enqueue_prep(tensair_model *m, BatchSet &S, const BatchWork &w, bool chained, int from, int to,
                         const RowIndexDst &in, const RowIndexDst &out, int32_t *negatives_dbg, hipStream_t st)
{
    for (int phase = from; phase < to; ++phase) {
        PrepPhase x;
        make_prep_phase(m, S, w, chained, phase, in, out, negatives_dbg, x);
        before_prep_phase(m, S, x.kind, st);
        tn_launch_prep(x, st);
    }
}

// where a mini-batch that is prepared ahead leaves its row index
static void set_row_index(const tensair_model *m, const BatchSet &S, RowIndexDst &in, RowIndexDst &out)
{
    const tensair_config &c = m->cfg;
    in = {S.ids_in, S.n_rows, S.off_in, tensair_capacity_in(&c, c.max_centers)};
    out = {S.ids_out, S.n_rows + 1, S.off_out, tensair_capacity_out(&c, c.max_centers)};
}

static int check_batch(const tensair_model *m, const int32_t *tokens, i64 n_tokens, i64 center_begin, int n_centers,
                       u32 epoch)
{
    if (!tokens) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (n_tokens < 1 || center_begin < 0 || n_centers < 0 || center_begin + n_centers > n_tokens)
        return fail(TENSAIR_EINVAL, "center range [%lld, +%d) outside the stream of %lld tokens",
                    (long long)center_begin, n_centers, (long long)n_tokens);
    if (n_centers > m->cfg.max_centers)
        return fail(TENSAIR_ECAPACITY, "n_centers %d > max_centers %d", n_centers, m->cfg.max_centers);
    if (epoch >= 65536u) return fail(TENSAIR_EINVAL, "epoch must be below 65536");
    return TENSAIR_OK;
}

// Where an announced mini-batch is prepared.
//   Riding: phase by phase at the front of the launches of the gradient call before the one that consumes it (forward
//     pass, reduction, chaining, table update), whose latencies hide it: no launch, event or stream of its own.  An
//     event between two streams costs the host 15 us and the waiting stream 4 to 7, a launch 3 to 5: steps of 60 000
//     occurrences took 80 us of host time with the preparation on the second stream and 65 us in all riding.  Up to
//     TN_PREP_CHAIN_RIDE tiles, TN_PREP_CHAIN_MAX where a very long table update follows.
//   On the second stream for larger ones: under a table update that is long enough (tensair_step decides), else beside
//     the forward pass and the reductions, up to TN_BESIDE_MAX_OCC occurrences.
//   At once, when it is announced with nothing before it: there is no call whose launches it could ride in, and the
//     GPU may have nothing else to do until it is consumed.  On the caller's stream up to TN_PREP_CHAIN_OWN tiles, all
//     but the segments, which ride with the consuming call's forward pass; on the second stream up to TN_BESIDE_MAX_OCC
//     occurrences, where the consuming call's forward pass waits for the keys alone and runs beside the sort.  Step
//     after a pause, announced before it / not announced: 31 tiles 68 / 110 us, 108 tiles 94 / 142, 160 tiles 111 / 191,
//     222 tiles 843 / 925; without a pause 91 / 89, 131 / 121, 179 / 160, 911 / 891 (all of the small ones' preparation
//     at once 99 and 137; waiting for the large ones' sort before the forward pass 198 and 935).
//   Else not ahead: beside a forward pass of cache-resident tables both fight for the caches (262 000 pairs per step
//     4 % slower).
#ifndef TN_BESIDE_MAX_OCC
#define TN_BESIDE_MAX_OCC (1 << 20)
#endif
static bool rides(const tensair_model *m, const Prefetched &d, bool long_update)
{
    return prep_tiles(m->cfg, d.P, d.n_centers) <= (long_update ? TN_PREP_CHAIN_MAX : TN_PREP_CHAIN_RIDE);
}

// The next phase of the announced mini-batch m->pend, if it is one that rides and is not done: the caller attaches it
// to the launch that it makes next on `st`.  The keys ride with a forward pass, the others with whatever follows it.
static bool next_rider(tensair_model *m, bool forward, PrepPhase &x, hipStream_t st)
{
    Prefetched &d = m->pend;
    if (!d.valid || !d.chained || d.on_side || (d.phase == 0) != forward || d.phase >= prep_phases(m->sz, true)) return false;
    BatchSet &S = m->set[1 - m->busy];
    BatchWork w = batch_work(m->cfg, d.tokens, d.n_tokens, d.begin, d.n_centers, d.epoch, d.P);
    w.worker_id = d.worker_id;     // the id it was announced under
    RowIndexDst in, out;
    set_row_index(m, S, in, out);
    make_prep_phase(m, S, w, true, d.phase, in, out, nullptr, x);
    before_prep_phase(m, S, x.kind, st);
    ++d.phase;
    return true;
}

// Enqueue the preparation of an announced mini-batch in launches of its own, into the set that the latest gradient call
// does not read: on the second stream, which must already be behind that set's last readers, or on the caller's.
// late: it may still be running when the mini-batch is consumed, so its keys are made available on their own.
static int enqueue_prepare(tensair_model *m, const Prefetched &d, bool on_side, bool late, hipStream_t st)
{
    BatchSet &S = m->set[1 - m->busy];
    BatchWork w = batch_work(m->cfg, d.tokens, d.n_tokens, d.begin, d.n_centers, d.epoch, d.P);
    w.worker_id = d.worker_id;     // the id it was announced under
    RowIndexDst in, out;
    set_row_index(m, S, in, out);
    const bool chained = !on_side;                       // what goes to the second stream is too long for chained passes
    const int phases = prep_phases(m->sz, chained) - (chained ? 1 : 0);   // the segments: with the consuming call's forward pass
    enqueue_prep(m, S, w, chained, 0, 1, in, out, nullptr, st);
    if (late) {
        HIP_TRY(hipEventRecord(m->ev_keys, st));
        m->keys_ticket = ++m->side_ticket;
    }
    enqueue_prep(m, S, w, chained, 1, phases, in, out, nullptr, st);
    HIP_TRY(hipGetLastError());
    if (on_side) {
        HIP_TRY(hipEventRecord(m->ev_prep, st));
        m->prep_ticket = ++m->side_ticket;
    }
    m->pend = d;
    m->pend.chained = chained;
    m->pend.phase = phases;
    m->pend.on_side = on_side;
    m->pend.late = late;
    return TENSAIR_OK;
}

// After a HIP call has failed in the middle of a call that had already forked work to the second stream, the
// two streams and the host's record of them may disagree.  Wait for the second stream (best effort), forget
// every announcement and count the caller's stream as behind everything, so that the next call on the handle
// starts from a known state instead of racing leftover work.
static void abandon_side_work(tensair_model *m)
{
    if (m->side) (void)hipStreamSynchronize(m->side);
    m->pend.valid = m->next.valid = m->deferred.valid = false;
    m->side_follows = false;
    m->main_ticket = m->side_ticket;
    m->fused_apply = nullptr;
    m->fused_index_done = false;
    m->mask_clean[0] = m->mask_clean[1] = false;
    m->set[0].hist_clean = m->set[1].hist_clean = false;
}

// Whether chaining the longest row that a mini-batch is expected to have takes as long as a phase of a preparation, which
// then rides with it for nothing.  A workgroup adds up 32 partials at a time (as many per group of lanes, where rows are
// narrow), 0.8 us each time.  After 16 times a phase is always hidden; after 4 it is better off there than under the update
// of small tables, which is as short itself, while that of larger ones hides it.  Step, us, phase under the update / riding
// here: after 16 times and more, D = 132, 6 000 centers, 1 000 words, Zipf exponent 1.0 92.9 / 86.0, 30 000 words, 1.2 109.6 /
// 107.4, D = 64, 1 000 words, 1.4 76.3 / 71.5; after 4 to 16, 300 words, D = 132 and 2 500 centers 54.9 / 50.2, 8 000 words
// and 6 000 centers 107.8 / 101.2; 8 000 words, D = 300 63.1 / 64.3, 16 000 67.6 / 71.9; 1 000 words, D = 64 50.2 / 52.2.
static bool long_chain(const tensair_model *m, i64 P, int n_centers)
{
    const int D = m->cfg.dim, side_by_side = D > TN_SUB_MAX_DIM ? 1 : D > 64 ? 2 : D > 32 ? 4 : 8;
    const int times = D > TN_SUB_MAX_DIM && m->cfg.vocab * D <= (i64)1 << 21 ? 4 : 16;
    const double out = m->words.per_pair * (double)P, in = m->words.center * n_centers;
    const i64 O = P * (m->cfg.negatives + 1);
    return std::max(out / (1 << tn_seg_shift(O, D)), in / (1 << tn_seg_shift(n_centers, D))) >= times * 32 * side_by_side;
}

// Whether the table update of a step chains the long rows itself, a workgroup each at the front of its grid (apply_kernels.h),
// instead of a launch before it: where the preparation of the mini-batch after it finds a launch for every phase without that
// one, and the longest row expected is chained as fast as the rest is updated (in rounds as in long_chain: up to 16; up to 4 and
// 8 where the update of wide rows of a small vocabulary is as short itself).  Step, us, a launch before it / the update: 1 000
// words, D = 32, 64 centers 21.9 / 18.6; 1 316 words, D = 136, 64 centers 25.4 / 18.8; 1 119 words, D = 120, 1 380 centers 49.0
// / 40.1; 6 433 words, D = 252, 2 160 centers 54.0 / 45.8; 50 000 words, D = 128, 1 024 centers 46.8 / 43.2; 50 000 words, D =
// 512, 1 000 centers, 5 peers 152 / 143; more rounds: 300 words, D = 300, 300 centers 36.7 / 40.8, 5 000 words 37.1 / 37.2, D =
// 200 35.2 / 30.9; 9 to 13 rounds, 3 576 words, D = 272, 788 centers, messages 44.4 / 47.5, 3 827 in bfloat16, D = 260, 309
// centers 40.8 / 43.1, without messages 3 221, D = 400, 491 centers 50.4 / 52.3 (tables of 2^19 to 2^21 elements of wide rows,
// as a share: 4 to 8 rounds 0.86 in the mean, none above 1.00; more 0.95, up to 1.07).  Not with packed peers of narrow rows,
// whose update of a large vocabulary makes use of the waves that the chaining's registers take: 260 000 words, D = 32, 1 000
// centers 89 / 92, D = 200 113 / 110; nor, with bfloat16 tables, of rows of up to 256 elements where few are touched (the update's
// sweeps): 240 802 words, D = 224, 73 centers, 5 peers 40.8 / 42.6, 21 such shapes 0.99 in the mean, 19 of up to 196 608 words 0.97.
static bool chains_with_update(const tensair_model *m, i64 P, int n_centers, const ApplyArgs &a)
{
    const tensair_config &c = m->cfg;
    const i64 O = P * (c.negatives + 1);
    const int side_by_side = c.dim > TN_SUB_MAX_DIM ? 1 : c.dim > 64 ? 2 : c.dim > 32 ? 4 : 8;
    const i64 elements = c.dim > TN_SUB_MAX_DIM ? c.vocab * c.dim : (i64)1 << 62;
    const int times = elements <= (i64)1 << 19 ? 4 : elements <= (i64)1 << 21 ? 8 : 16;
    const double out = m->words.per_pair * (double)P / (1 << tn_seg_shift(O, c.dim)), in = m->words.center * n_centers / (1 << tn_seg_shift(n_centers, c.dim));
    const bool slow = a.packed && (c.dim <= TN_SUB_MAX_DIM ? c.vocab > 131072
                                   : c.dim <= 256 && c.dtype == TENSAIR_BF16 && c.vocab > 196608 && 5 * tn_union_rows(a) < c.vocab);
    return O <= TN_CHAIN_UPDATE_MAX_OCC && c.vocab <= TN_CHAIN_UPDATE_MAX_V && tn_apply_carries(c.dim, c.vocab) &&
           !tn_streams(c.vocab, c.row_stride, c.dtype) && !slow && std::max(out, in) <= times * 32.0 * side_by_side;
}

// Whether the gradient of a mini-batch goes by pairs of words (group.hip).  Such a mini-batch is prepared by its own call.
// Counting a chunk and adding up a word look at every word and every chunk, whatever they hold: that has to be paid for by
// occurrences per word, the more of them the cheaper an occurrence is by itself -- narrow rows, positions that repeat words.
// The lines lie where an earlier form broke even, which took nearly twice as long: this one does from about 90 occurrences per word on, so
// nothing that goes by pairs is slower for it.  Step over 12 000 words, us, by occurrences / by pairs: expected share of different words
// 0.55, 128 tasks per position, D = 32, 94 occurrences per word 138 / 117, 160 185 / 129, 200 212 / 135; D = 128, 94 151 / 120,
// 160 212 / 132; D = 256, 94 164 / 127, 128 202 / 130, 160 237 / 138; 256 tasks, D = 32, 87 123 / 123, 94 132 / 118, 200 196 / 141; D = 256,
// 94 159 / 127, 160 225 / 144; share 0.72, 128 tasks, D = 32, 87 148 / 146, 94 159 / 140, 160 213 / 165; D = 132, 94 196 / 144, 128
// 239 / 159; 256 tasks, D = 32, 87 144 / 150, 94 150 / 149, 160 196 / 171; D = 132, 94 190 / 154; D = 320, 0.55, 87 occurrences 160 / 144, D = 512
// 220 / 165.
static bool goes_by_pairs(const tensair_model *m, i64 P)
{
    const tensair_config &c = m->cfg;
    const WordStats &x = m->words;
    const i64 O = P * (c.negatives + 1);
    if (!m->sz.group || x.different > pairs_below(c.dim) || x.hottest > TN_GROUP_MAX_SHARE || O <= TN_GROUP_MIN_OCC) return false;
    const bool repeat = x.different < 0.65;
    const int per_word = c.dim > 256 ? 0 : c.dim <= 64 ? (repeat ? 200 : 150) : c.dim <= TN_SUB_MAX_DIM ? (repeat ? 150 : 90)
                         : repeat ? 136 : 2 * c.window * (c.negatives + 1) < 256 ? 104 : 90;
    return O >= per_word * c.vocab;
}

int tensair_prefetch(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                     int32_t n_centers, uint32_t epoch, void *stream)
{
    if (!m) return fail(TENSAIR_EINVAL, "model is NULL");
    int rc = check_batch(m, tokens, n_tokens, center_begin, n_centers, epoch);
    if (rc) return rc;
    const tensair_config &c = m->cfg;
    Prefetched d;
    d.tokens = tokens;
    d.n_tokens = n_tokens;
    d.begin = center_begin;
    d.n_centers = n_centers;
    d.epoch = epoch;
    d.worker_id = c.worker_id;
    d.P = pair_count(c, n_tokens, center_begin, n_centers);
    if (d.P == 0) return TENSAIR_OK;   // nothing to prepare
    d.valid = true;
    note_capture(m, (hipStream_t)stream);
    if (m->captured) return TENSAIR_OK;
    if (m->pend.valid) {   // one mini-batch is waiting already: this one is prepared when that is consumed
        m->next = d;
        return TENSAIR_OK;
    }
    if (d.P * (c.negatives + 1) > TN_BESIDE_MAX_OCC) {
        m->pend = d;               // kept as an announcement: the consuming call prepares it itself
        return TENSAIR_OK;
    }
    hipStream_t st = (hipStream_t)stream;
    const bool on_side = prep_tiles(c, d.P, n_centers) > TN_PREP_CHAIN_OWN;
    // The set being filled was last read by the gradient call before the latest one.  If the second
    // stream has waited for the start of the latest call it is already behind those readers; if not,
    // it is put behind everything enqueued on the caller's stream so far.
    if (on_side && !m->side_follows) {
        HIP_TRY(hipEventRecord(m->ev_fork, st));
        HIP_TRY(hipStreamWaitEvent(m->side, m->ev_fork, 0));
        m->side_follows = true;
    }
    const int rc2 = enqueue_prepare(m, d, on_side, on_side, on_side ? m->side : st);
    if (rc2 == TENSAIR_EHIP) abandon_side_work(m);
    return rc2;
}

static int sgns_grad_impl(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                          int32_t n_centers, uint32_t epoch, tensair_sparse_grad *grad_out, float *mean_loss,
                          int32_t *negatives_dbg, int32_t *seg_offsets_in, int32_t *seg_offsets_out, void *stream)
{
    if (!m || !grad_out) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    const tensair_config &c = m->cfg;
    int rc = check_batch(m, tokens, n_tokens, center_begin, n_centers, epoch);
    if (rc) return rc;
    if ((rc = check_rows(grad_out->in, tensair_capacity_in(&c, n_centers), "grad_out.in"))) return rc;
    if ((rc = check_rows(grad_out->out, tensair_capacity_out(&c, n_centers), "grad_out.out"))) return rc;
    hipStream_t st = (hipStream_t)stream;
    const Sizes &s = m->sz;

    note_capture(m, st);
    const i64 P = pair_count(c, n_tokens, center_begin, n_centers);
    if (P == 0) {
        tn_launch_empty_grad(grad_out->in.n_rows, grad_out->out.n_rows, mean_loss, seg_offsets_in,
                             seg_offsets_out, st);
        HIP_TRY(hipGetLastError());
        return TENSAIR_OK;
    }
    const int Np1 = c.negatives + 1;
    const BatchWork w = batch_work(c, tokens, n_tokens, center_begin, n_centers, epoch, P);

    // Streams.  The sort and the segment scan only need the keys, the forward pass the keys and the
    // tables, the reductions both.  Everything runs on the caller's stream, with these exceptions: a large
    // mini-batch that nobody prepared has its forward pass on the library's second stream, next to its sort,
    // and an announced one that is too large to ride is prepared there.  What is small rides
    // at the front of other launches: the phases that are still missing of this mini-batch's preparation and
    // those of the announced one after it, the prepared row index to the caller's buffers, and inside
    // tensair_step the index of the coming table update.  An event between streams costs the host 15 us and
    // idles the waiting stream for microseconds, a launch of its own 3 to 5 us.  When every stage is being
    // timed (profile level 2) everything is serialised on the caller's stream in launches of its own.
    const bool overlap = m->prof_level < 2;
    const bool fuse = overlap && m->fused_apply != nullptr;
    const bool announced = overlap && negatives_dbg == nullptr &&
                           m->pend.is(tokens, n_tokens, center_begin, n_centers, epoch, c.worker_id);
    const Prefetched own = announced ? m->pend : Prefetched();
    // the announced mini-batch after this one is prepared during this call; announcements that this
    // call does not follow are dropped
    const Prefetched following = announced ? m->next : Prefetched();
    m->pend.valid = false;
    m->next.valid = false;
    m->deferred.valid = false;
    // this call takes the set that announced mini-batches are prepared into; one that does not match
    // is overwritten, after its preparation has finished
    const int u = 1 - m->busy;
    BatchSet &S = m->set[u];
    // its preparation may still be running: the forward pass waits for its keys only, the reductions for the rest
    const bool split = own.late && m->prep_ticket > m->main_ticket;
    if (split) {
        if (m->keys_ticket > m->main_ticket) {
            HIP_TRY(hipStreamWaitEvent(st, m->ev_keys, 0));
            m->main_ticket = m->keys_ticket;
        }
    } else if (m->prep_ticket > m->main_ticket) {
        HIP_TRY(hipStreamWaitEvent(st, m->ev_prep, 0));
        m->main_ticket = m->prep_ticket;
    }
    m->busy = u;
    m->side_follows = false;
    // how far this mini-batch is prepared, and how the rest is done
    int phase = own.phase;
    const bool by_pairs = phase == 0 && goes_by_pairs(m, P);
    const bool chained = phase > 0 ? own.chained : prep_tiles(c, P, n_centers) <= TN_PREP_CHAIN_OWN;
    const int phases = prep_phases(s, chained), sorted = prep_sort_end(s, chained);
    const bool prepared = phase == phases;
    // the one after it: riding, under a long table update that follows (tensair_step decides), beside this call's
    // forward pass, or left to its own call
    bool beside = false;
    if (following.valid) {
        if (rides(m, following, fuse && m->ride_long_update)) {
            m->pend = following;
            m->pend.chained = true;
        } else if (fuse && m->prepare_under_apply && !goes_by_pairs(m, following.P)) {
            m->deferred = following;
        } else if (following.P * Np1 <= TN_BESIDE_MAX_OCC) {
            beside = true;
        } else {
            m->pend = following;
        }
    }
    const bool chain_later = fuse && !by_pairs && chains_with_update(m, P, n_centers, *m->fused_apply);
    mark(m, PF_BEGIN_GRAD, st);

    FwdArgs f;
    f.w_in = m->w_in;
    f.w_out = m->w_out;
    f.V = c.vocab;
    f.dtype = c.dtype;
    f.D = c.dim;
    f.stride = c.row_stride;
    f.b = w.b;
    f.out_keys = S.keys[0];
    f.g = m->g;
    f.center_part = m->center_part;
    f.center_loss = mean_loss ? m->center_loss : nullptr;   // loss terms only on request
    f.inv_P = 1.0f / (float)P;
    f.repeats = m->words.different <= TN_REPEATS_BELOW && 2 * c.window * Np1 <= TN_REPEAT_MAX_TASKS;

    AuxWork aux_fwd, aux_red;     // what rides at the front of the forward pass / of the reduction
    tn_aux_none(aux_fwd);
    tn_aux_none(aux_red);
    if (fuse) {
        // The index of the coming table update.  Its masks must be zero before the id lists are indexed, and the
        // two cannot share a launch, so there are two sets of masks: this step indexes a clean one, with the
        // forward pass (hidden behind its row gathers) where the id lists are known by then -- the peers'
        // always, the own one if the mini-batch was prepared -- else with the reductions; the other set, which
        // the previous step used, is cleared with the reductions and is the clean one of the next step.
        ApplyArgs &fa = *m->fused_apply;
        int pick = m->mask_clean[0] ? 0 : (m->mask_clean[1] ? 1 : -1);
        if (pick < 0) {           // the first step, or other calls have used both sets since
            pick = 0;
            ApplyArgs full = fa;  // the whole buffer, whatever layout its last user had
            full.n_src = (c.max_peers + 1 > 2 ? c.max_peers + 1 : 2);
            tn_launch_apply_clear(full, st);
        }
        for (int t = 0; t < 2; ++t) fa.mask[t] = pick ? m->mask_alt[t] : m->mask[t];
        m->mask_clean[pick] = false;
        const bool own_early = prepared && !split;   // the own id lists exist when the forward pass starts
        tn_aux_add_index(aux_fwd, fa, own_early || by_pairs ? 0 : 1, fa.n_src);
        if (by_pairs) {           // the out-side ids come with the sums, which index them
            aux_fwd.apply.src[1][0].ids = nullptr;
        } else if (!own_early) {
            tn_aux_add_index(aux_red, fa, 0, 1);
        }
        if (!m->mask_clean[1 - pick]) {
            const size_t all = (size_t)s.words * (size_t)(c.max_peers + 1 > 2 ? c.max_peers + 1 : 2);
            tn_aux_add_clear(aux_red, pick ? m->mask[0] : m->mask_alt[0], pick ? m->mask[1] : m->mask_alt[1], all);
            m->mask_clean[1 - pick] = true;
        }
        m->fused_index_done = true;
        if (chain_later) {        // the update before this call is the last reader of the rows noted there
            tn_aux_add_clear(aux_fwd, m->long_mask[0], m->long_mask[1], (size_t)s.words);
            for (int t = 0; t < 2; ++t) fa.skip[t] = m->long_mask[t];
        }
    }

    const RowIndexDst in = {grad_out->in.row_ids, grad_out->in.n_rows, seg_offsets_in, grad_out->in.capacity};
    const RowIndexDst out = {grad_out->out.row_ids, grad_out->out.n_rows, seg_offsets_out, grad_out->out.capacity};
    PrepPhase x;
    if (by_pairs) {
        // the positions sorted by their center's word, then the gradient itself, whose counting draws the negatives by
        // itself.  Its sums take the same order whatever outputs are asked for; the occurrences are listed for the negatives
        // and sorted for their offsets alone.  Where every stage is being timed the count of the sort stays in a launch of its
        // own, as in long sorts.
        const bool list = seg_offsets_out || negatives_dbg;
        const bool chain = overlap && !list && prep_tiles(c, 0, n_centers) <= TN_PREP_CHAIN_OWN;
        BatchWork sorted_lists = w;
        sorted_lists.centers_only = !list;
        if (!seg_offsets_out) sorted_lists.O = 0;
        for (int i = 0; i < prep_phases(s, chain); ++i) {
            make_prep_phase(m, S, sorted_lists, chain, i, in, out, negatives_dbg, x);
            before_prep_phase(m, S, x.kind, st);
            tn_launch_prep(x, st);
            if (i == 0) mark(m, PF_KEYS, st);
            if (i + 1 == prep_sort_end(s, chain)) mark(m, PF_SORT, st);
        }
        mark(m, PF_SEGMENTS, st);
        if (beside) {
            HIP_TRY(hipEventRecord(m->ev_fork, st));
            HIP_TRY(hipStreamWaitEvent(m->side, m->ev_fork, 0));
            m->side_follows = true;
            if ((rc = enqueue_prepare(m, following, true, true, m->side))) return rc;
        }
        if (next_rider(m, true, x, st)) tn_launch_prep(x, st);
        const SortedSide si = sorted_side(m, S, 1);
        GroupArgs ga;
        memset(&ga, 0, sizeof(ga));
        ga.f = f;
        ga.noise = noise_draw(m, w);
        ga.status = m->status;
        ga.vals = si.vals;
        ga.seg_of = si.seg_of;
        ga.seg_start = si.seg_start;
        ga.n_in = grad_out->in.n_rows;
        ga.in_ids = grad_out->in.row_ids;
        ga.words = (int)s.words;
        ga.per_center = 2 * c.window * Np1;
        ga.rare = (int)tn_group_rare(c.vocab, ga.per_center, n_centers);
        ga.chunk = (int)tn_group_chunk(ga.per_center, n_centers);
        ga.most_frequent = (int)tn_group_frequent(c.vocab, ga.per_center, n_centers);
        ga.slices = tn_group_slices(c.vocab, ga.most_frequent);
        ga.parts = tn_group_parts(c.vocab, ga.slices, c.dim);
        ga.dense = m->group_dense;
        ga.list = S.keys[1];      // the out-side list's room: not sorted, or no longer needed
        ga.counts = S.keys[2];
        ga.any = m->group_any;
        ga.masks = m->group_masks;
        ga.starts = m->group_starts;
        ga.turned = m->group_turned;
        ga.meta = m->group_meta;
        ga.frequent = m->group_frequent;
        ga.n_frequent = m->group_n;
        ga.hot_rows = m->group_hot_rows;
        ga.hot_part = m->group_hot_part;
        ga.in_rows = grad_out->in.row_grads;
        ga.out_rows = grad_out->out.row_grads;
        ga.out_ids = grad_out->out.row_ids;
        ga.out_n = grad_out->out.n_rows;
        if (fuse) {
            ga.index_mask = m->fused_apply->mask[1] + idx_at(s.words, 0, 0);
            ga.index_start = m->fused_apply->start[1] + idx_at(s.words, 0, 0);
        }
        const int losses = n_centers + ga.words * ga.slices;
        tn_launch_group(ga, GROUP_ROWS, aux_fwd, st);
        mark(m, PF_FORWARD, st);
        if (overlap) {
            if (mean_loss) tn_aux_add_loss(aux_red, m->center_loss, losses, f.inv_P, mean_loss);
            tn_launch_group(ga, GROUP_SUMS_IN | GROUP_SUMS_OUT, aux_red, st);
        } else {         // one after the other, so that each can be timed
            if (mean_loss) tn_launch_loss(m->center_loss, losses, f.inv_P, mean_loss, st);
            tn_launch_group(ga, GROUP_SUMS_IN, aux_red, st);
            mark(m, PF_REDUCE_IN, st);
            tn_launch_group(ga, GROUP_SUMS_OUT, aux_red, st);
        }
        mark(m, PF_REDUCE_OUT, st);
        HIP_TRY(hipGetLastError());
        return TENSAIR_OK;
    }
    if (prepared) {
        // this mini-batch's row index goes to the caller's buffers with the forward pass -- with the reductions if the
        // forward pass starts on the keys alone
        AuxWork &with = split ? aux_red : aux_fwd;
        RowIndexCopy rc2;
        rc2.side[0] = {S.ids_in, S.n_rows, S.off_in, grad_out->in.row_ids, grad_out->in.n_rows, seg_offsets_in};
        rc2.side[1] = {S.ids_out, S.n_rows + 1, S.off_out, grad_out->out.row_ids, grad_out->out.n_rows,
                       seg_offsets_out};
        tn_aux_add_copy(with, rc2, tensair_capacity_out(&c, n_centers));
        if (fuse) {   // the own id lists are indexed where they are
            ApplySrc &o_in = with.apply.src[0][0], &o_out = with.apply.src[1][0];
            o_in.ids = S.ids_in;
            o_in.n_rows = S.n_rows;
            o_in.capacity = tensair_capacity_in(&c, c.max_centers);
            o_out.ids = S.ids_out;
            o_out.n_rows = S.n_rows + 1;
            o_out.capacity = tensair_capacity_out(&c, c.max_centers);
        }
    } else if (phase == 0) {
        // 1. keys
        enqueue_prep(m, S, w, chained, 0, 1, in, out, negatives_dbg, st);
        phase = 1;
    }
    mark(m, PF_KEYS, st);
    // 2. forward on the unsorted keys (the sort never writes their buffer): g per occurrence, per-center share of the
    //    W_in gradient, loss terms
    const bool aside = overlap && !chained && !prepared;
    if (aside || beside) {
        HIP_TRY(hipEventRecord(m->ev_fork, st));
        HIP_TRY(hipStreamWaitEvent(m->side, m->ev_fork, 0));
        m->side_follows = true;
    }
    if (overlap && !aside) {
        if (phase < phases) {
            make_prep_phase(m, S, w, chained, phase, in, out, nullptr, x);
            before_prep_phase(m, S, x.kind, st);
            ++phase;
            tn_aux_add_prep(aux_fwd, x);
        }
        if (next_rider(m, true, x, st)) tn_aux_add_prep(aux_fwd, x);
    }
    tn_launch_forward(f, &aux_fwd, aside ? m->side : st);
    mark(m, PF_FORWARD, st);
    u64 fwd_ticket = 0;
    if (aside) {
        HIP_TRY(hipEventRecord(m->ev_fwd, m->side));
        fwd_ticket = ++m->side_ticket;
    }
    if (split) {    // the rest of this mini-batch's preparation
        HIP_TRY(hipStreamWaitEvent(st, m->ev_prep, 0));
        m->main_ticket = m->prep_ticket;
    }
    if (beside && (rc = enqueue_prepare(m, following, true, true, m->side))) return rc;   // behind a forward pass aside
    // 3./4. what is missing of sort and segments, row index straight into the caller's buffers
    if (phase < sorted) {
        enqueue_prep(m, S, w, chained, phase, sorted, in, out, nullptr, st);
        phase = sorted;
    }
    mark(m, PF_SORT, st);
    enqueue_prep(m, S, w, chained, phase, phases, in, out, nullptr, st);
    mark(m, PF_SEGMENTS, st);
    if (aside) {
        // the keys of the announced mini-batch after this one, in a launch of their own: a forward pass on the second
        // stream carries none, and without them none of its other phases could ride with what follows (nor could any
        // mini-batch's after it: each would be left to its own call, with the forward pass aside again)
        if (next_rider(m, true, x, st)) tn_launch_prep(x, st);
        HIP_TRY(hipStreamWaitEvent(st, m->ev_fwd, 0));
        if (fwd_ticket > m->main_ticket) m->main_ticket = fwd_ticket;
    }

    // 5. segmented reductions: duplicates of a row summed in sorted (= occurrence) order
    const SortedSide so = sorted_side(m, S, 0), si = sorted_side(m, S, 1);
    SegReduceArgs r_in, r_out;
    memset(&r_in, 0, sizeof(r_in));
    r_in.D = c.dim;
    r_in.n = n_centers;
    r_in.vals = si.vals;
    r_in.seg_of = si.seg_of;
    r_in.seg_start = si.seg_start;
    r_in.long_cnt = si.long_cnt;
    r_in.long_list = m->long_list + s.tiles_out;
    r_in.out_rows = grad_out->in.row_grads;
    r_in.part = m->part_in;
    r_in.cross = m->cross_in;
    r_in.xinfo = m->xinfo_in;
    r_in.mode = 1;
    r_in.center_part = m->center_part;
    r_out = r_in;
    r_out.n = (int)w.O;
    r_out.vals = so.vals;
    r_out.seg_of = so.seg_of;
    r_out.seg_start = so.seg_start;
    r_out.long_cnt = so.long_cnt;
    r_out.long_list = m->long_list;
    r_out.out_rows = grad_out->out.row_grads;
    r_out.part = m->part_out;
    r_out.cross = m->cross_out;
    r_out.xinfo = m->xinfo_out;
    r_out.mode = 0;
    r_out.g = m->g;
    r_out.pair_center = S.pair_center;
    r_out.Np1 = Np1;
    r_out.table = m->w_in;
    r_out.dtype = c.dtype;
    r_out.stride = c.row_stride;
    if (chain_later) {
        r_in.row_ids = prepared ? S.ids_in : grad_out->in.row_ids;
        r_out.row_ids = prepared ? S.ids_out : grad_out->out.row_ids;
        r_in.long_mask = m->long_mask[0];
        r_out.long_mask = m->long_mask[1];
        tn_chain_work(m->chain, r_out, r_in);
    }
    if (overlap) {   // both sides in one launch
        if (mean_loss) tn_aux_add_loss(aux_red, m->center_loss, n_centers, f.inv_P, mean_loss);
        if (next_rider(m, false, x, st)) tn_aux_add_prep(aux_red, x);
        PrepPhase y;
        // where the chaining of long rows is short (4 us where a pass of the sort takes 9), a phase rides with it only if there
        // are more left than the table update and the next forward pass can take (1 024 centers, 50 000 words: step 54.6
        // -> 49.0 us with the second pass under the update instead)
        const int later = 1 + (fuse && tn_apply_carries(c.dim, c.vocab) ? 1 : 0);
        const bool rider = !chain_later && tn_seg_chains(r_out.n, c.dim) + tn_seg_chains(r_in.n, c.dim) > 0 &&
                           (long_chain(m, P, n_centers) || m->pend.phase + later < prep_phases(s, true)) &&
                           next_rider(m, false, y, st);
        tn_launch_segreduce(&r_out, &r_in, &aux_red, rider ? &y : nullptr, st);
    } else {         // one after the other, so that each can be timed
        if (mean_loss) tn_launch_loss(m->center_loss, n_centers, f.inv_P, mean_loss, st);
        tn_launch_segreduce(nullptr, &r_in, nullptr, nullptr, st);
        mark(m, PF_REDUCE_IN, st);
        tn_launch_segreduce(&r_out, nullptr, nullptr, nullptr, st);
    }
    mark(m, PF_REDUCE_OUT, st);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_sgns_grad(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                      int32_t n_centers, uint32_t epoch, tensair_sparse_grad *grad_out, float *mean_loss,
                      int32_t *negatives_dbg, int32_t *seg_offsets_in, int32_t *seg_offsets_out, void *stream)
{
    const int rc = sgns_grad_impl(m, tokens, n_tokens, center_begin, n_centers, epoch, grad_out, mean_loss,
                                  negatives_dbg, seg_offsets_in, seg_offsets_out, stream);
    if (rc == TENSAIR_EHIP && m) abandon_side_work(m);
    return rc;
}

// The preparation of the mini-batch that tensair_sgns_grad left in m->deferred: enqueued on the second
// stream behind everything that is on the caller's stream now (the reductions), so that it runs under the
// table update that the caller enqueues next.  `ev`: an event just recorded on the caller's stream, or
// nullptr to record one.
static int enqueue_deferred_prepare(tensair_model *m, hipEvent_t ev, hipStream_t st)
{
    if (!m->deferred.valid) return TENSAIR_OK;
    const Prefetched d = m->deferred;
    m->deferred.valid = false;
    if (!ev) {
        HIP_TRY(hipEventRecord(m->ev_reduced, st));
        ev = m->ev_reduced;
    }
    HIP_TRY(hipStreamWaitEvent(m->side, ev, 0));
    m->side_follows = true;
    return enqueue_prepare(m, d, true, false, m->side);
}

// peers are fp32 gradients (`peers`) or bfloat16 messages (`packed`), never both
static int make_apply_args(tensair_model *m, const tensair_sparse_grad *own, const tensair_sparse_grad *peers,
                           const tensair_packed_grad *packed, int32_t n_peers, float lr, ApplyArgs &a)
{
    const tensair_config &c = m->cfg;
    if (n_peers < 0 || n_peers > c.max_peers)
        return fail(TENSAIR_ECAPACITY, "n_peers %d outside 0..max_peers %d", n_peers, c.max_peers);
    if (n_peers > 0 && !peers && !packed) return fail(TENSAIR_EINVAL, "peers is NULL");
    if (!(lr == lr)) return fail(TENSAIR_EINVAL, "lr is NaN");
    memset(&a, 0, sizeof(a));
    a.table[0] = m->w_in;
    a.table[1] = m->w_out;
    a.dtype = c.dtype;
    a.D = c.dim;
    a.stride = c.row_stride;
    a.V = c.vocab;
    a.n_src = 1 + n_peers;
    a.lr = lr;
    a.status = m->status;
    a.packed = (packed != nullptr && n_peers > 0) ? 1 : 0;
    a.sr = ((c.flags & TENSAIR_STOCHASTIC_ROUNDING) && c.dtype == TENSAIR_BF16) ? 1 : 0;
    a.sr_k0 = (u32)(c.seed & 0xFFFFFFFFu);
    a.sr_k1 = (u32)(c.seed >> 32);
    a.sr_serial = m->apply_serial;
    for (int t = 0; t < 2; ++t) {
        a.start[t] = m->start[t];
        a.mask[t] = m->mask[t];
    }
    int rc;
    if (own && (rc = fill_apply_src(a, 0, own, "own"))) return rc;
    for (int k = 0; k < n_peers; ++k)
        if ((rc = packed ? fill_apply_src(a, 1 + k, &packed[k], "peer") : fill_apply_src(a, 1 + k, &peers[k], "peer")))
            return rc;
    return TENSAIR_OK;
}

static int apply_impl(tensair_model *m, const tensair_sparse_grad *own, const tensair_sparse_grad *peers,
                      const tensair_packed_grad *packed, int32_t n_peers, float lr, void *stream)
{
    if (!m) return fail(TENSAIR_EINVAL, "model is NULL");
    ApplyArgs a;
    int rc = make_apply_args(m, own, peers, packed, n_peers, lr, a);
    if (rc) return rc;
    if (!own && n_peers == 0) return TENSAIR_OK;
    hipStream_t st = (hipStream_t)stream;
    note_capture(m, st);
    mark(m, PF_BEGIN_APPLY, st);
    m->mask_clean[0] = false;
    tn_launch_apply_clear(a, st);
    tn_launch_apply_index(a, 0, a.n_src, st);
    mark(m, PF_APPLY_INDEX, st);
    tn_launch_apply_update(a, nullptr, nullptr, st);
    ++m->apply_serial;
    mark(m, PF_APPLY_UPDATE, st);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_dasgd_apply(tensair_model *m, const tensair_sparse_grad *own, const tensair_sparse_grad *peers,
                        int32_t n_peers, float lr, void *stream)
{
    return apply_impl(m, own, peers, nullptr, n_peers, lr, stream);
}

int tensair_dasgd_apply_packed(tensair_model *m, const tensair_sparse_grad *own, const tensair_packed_grad *peers,
                               int32_t n_peers, float lr, void *stream)
{
    if (n_peers > 0 && !peers) return fail(TENSAIR_EINVAL, "peers is NULL");
    return apply_impl(m, own, nullptr, peers, n_peers, lr, stream);
}

int tensair_grad_pack(tensair_model *m, const tensair_sparse_grad *g, tensair_packed_grad *out, void *stream)
{
    if (!m || !g || !out) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    GradPackArgs a;
    memset(&a, 0, sizeof(a));
    a.D = m->cfg.dim;
    a.status = m->status;
    const tensair_sparse_rows *src[2] = {&g->in, &g->out};
    const tensair_packed_rows *dst[2] = {&out->in, &out->out};
    for (int t = 0; t < 2; ++t) {
        const tensair_sparse_rows &r = *src[t];
        const tensair_packed_rows &d = *dst[t];
        if (!r.n_rows || !r.row_ids || !r.row_grads || !d.n_rows || !d.row_ids || !d.row_grads)
            return fail(TENSAIR_EINVAL, "grad_pack: NULL pointer");
        if (r.capacity < 0 || r.capacity > 0x7FFFFFFFLL || d.capacity < 0 || d.capacity > 0x7FFFFFFFLL)
            return fail(TENSAIR_EINVAL, "grad_pack: bad capacity");
        if (((uintptr_t)r.row_grads | (uintptr_t)d.row_grads) & 15)
            return fail(TENSAIR_EINVAL, "grad_pack: rows must be 16-byte aligned");
        if ((const void *)d.row_grads == (const void *)r.row_grads || d.row_ids == r.row_ids || d.n_rows == r.n_rows)
            return fail(TENSAIR_EINVAL, "grad_pack: out must not share buffers with g");
        a.n[t] = r.n_rows;
        a.ids[t] = r.row_ids;
        a.rows[t] = r.row_grads;
        a.cap[t] = r.capacity;
        a.out_n[t] = d.n_rows;
        a.out_ids[t] = d.row_ids;
        a.out_rows[t] = d.row_grads;
        a.out_cap[t] = d.capacity;
    }
    hipStream_t st = (hipStream_t)stream;
    mark(m, PF_BEGIN_PACK, st);
    tn_launch_grad_pack(a, st);
    mark(m, PF_PACK, st);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_grad_add(tensair_model *m, const tensair_sparse_grad *a, const tensair_sparse_grad *b,
                     tensair_sparse_grad *out, void *stream)
{
    if (!m || !a || !b || !out) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    const tensair_config &c = m->cfg;
    GradSumArgs g;
    memset(&g, 0, sizeof(g));
    ApplyArgs &ap = g.a;
    ap.dtype = c.dtype;
    ap.D = c.dim;
    ap.stride = c.row_stride;
    ap.V = c.vocab;
    ap.n_src = 2;
    ap.status = m->status;
    int rc;
    if ((rc = fill_apply_src(ap, 0, a, "a")) || (rc = fill_apply_src(ap, 1, b, "b"))) return rc;
    const tensair_sparse_rows *dst[2] = {&out->in, &out->out};
    const tensair_sparse_rows *src[2][2] = {{&a->in, &b->in}, {&a->out, &b->out}};
    for (int t = 0; t < 2; ++t) {
        const tensair_sparse_rows &r = *dst[t];
        if (!r.n_rows || !r.row_ids || !r.row_grads) return fail(TENSAIR_EINVAL, "out: NULL pointer");
        if (r.capacity < 0 || r.capacity > 0x7FFFFFFFLL) return fail(TENSAIR_EINVAL, "out: bad capacity");
        for (int k = 0; k < 2; ++k)
            if (r.row_grads == src[t][k]->row_grads || r.row_ids == src[t][k]->row_ids ||
                r.n_rows == src[t][k]->n_rows)
                return fail(TENSAIR_EINVAL, "out must not share buffers with a or b");
        ap.start[t] = m->start[t];
        ap.mask[t] = m->mask[t];
        g.out_ids[t] = r.row_ids;
        g.out_rows[t] = r.row_grads;
        g.out_n[t] = r.n_rows;
        g.out_cap[t] = r.capacity;
        g.wbase[t] = m->wbase[t];
        g.wblk[t] = m->wblk[t];
    }
    hipStream_t st = (hipStream_t)stream;
    note_capture(m, st);
    mark(m, PF_BEGIN_ADD, st);
    m->mask_clean[0] = false;
    tn_launch_grad_sum_index(g, st);
    mark(m, PF_ADD_INDEX, st);
    tn_launch_grad_sum_rows(g, st);
    mark(m, PF_ADD_ROWS, st);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

static int step_impl(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                     int32_t n_centers, uint32_t epoch, const tensair_sparse_grad *peers,
                     const tensair_packed_grad *packed, int32_t n_peers, float lr, tensair_sparse_grad *own_out,
                     tensair_packed_grad *own_msg, float *mean_loss, void *stream)
{
    if (!m || !own_out) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    // validate the apply arguments before anything is enqueued
    ApplyArgs a;
    int rc = make_apply_args(m, own_out, peers, packed, n_peers, lr, a);
    if (rc) return rc;
    if (own_msg) {   // the own gradient leaves the update as a bfloat16 message as well
        if (n_centers < 0) return fail(TENSAIR_EINVAL, "n_centers is negative");
        const tensair_packed_rows *d[2] = {&own_msg->in, &own_msg->out};
        const tensair_sparse_rows *o[2] = {&own_out->in, &own_out->out};
        const int64_t need[2] = {tensair_capacity_in(&m->cfg, n_centers), tensair_capacity_out(&m->cfg, n_centers)};
        for (int t = 0; t < 2; ++t) {
            if (!d[t]->n_rows || !d[t]->row_ids || !d[t]->row_grads) return fail(TENSAIR_EINVAL, "own_msg: NULL pointer");
            if ((uintptr_t)d[t]->row_grads & 15) return fail(TENSAIR_EINVAL, "own_msg: rows must be 16-byte aligned");
            if (d[t]->capacity < need[t])
                return fail(TENSAIR_ECAPACITY, "own_msg: capacity %lld < %lld rows required", (long long)d[t]->capacity,
                            (long long)need[t]);
            if ((const void *)d[t]->row_grads == (const void *)o[t]->row_grads || d[t]->row_ids == o[t]->row_ids ||
                d[t]->n_rows == o[t]->n_rows)
                return fail(TENSAIR_EINVAL, "own_msg must not share buffers with own_out");
            a.msg_rows[t] = d[t]->row_grads;
            a.msg_ids[t] = d[t]->row_ids;
            a.msg_n[t] = d[t]->n_rows;
        }
        a.packed = 1;   // the kernel that handles messages, also with no peer at all
    }
    m->fused_apply = &a;
    m->fused_index_done = false;
    m->chain.blocks = 0;
    m->deferred.valid = false;
    {   // rough times of the table update (bytes of the gradient blocks at their largest, at 5 TB/s) and of
        // the preparation of a mini-batch (0.2 ns per occurrence plus its launches)
        const tensair_config &c = m->cfg;
        const double occ = 2.0 * c.window * (double)n_centers * (c.negatives + 1);
        const double rows = occ < (double)c.vocab ? occ : (double)c.vocab;
        const double src_bytes = 4.0 + (a.packed ? 2.0 : 4.0) * (a.n_src - 1);
        const double t_apply = src_bytes * rows * c.dim / 5e12;
        const double t_prepare = occ * 0.2e-9 + 60e-6;
        m->prepare_under_apply = t_apply >= 2.0 * t_prepare;
        m->ride_long_update = t_apply >= TN_PREP_RIDE_LONG_UPDATE * t_prepare;
    }
    rc = sgns_grad_impl(m, tokens, n_tokens, center_begin, n_centers, epoch, own_out, mean_loss, nullptr,
                        nullptr, nullptr, stream);
    m->fused_apply = nullptr;
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    mark(m, PF_BEGIN_APPLY, st);
    if (!m->fused_index_done) {   // an empty mini-batch, or every stage in a launch of its own
        m->mask_clean[0] = false;
        tn_launch_apply_clear(a, st);
        tn_launch_apply_index(a, 0, a.n_src, st);
    }
    // the event that opens the timing of the table update also lets the second stream go
    const hipEvent_t ev = mark(m, PF_APPLY_INDEX, st);
    if ((rc = enqueue_deferred_prepare(m, ev, st))) return rc;
    PrepPhase x;
    const bool rider = m->prof_level < 2 && tn_apply_carries(a.D, a.V) && next_rider(m, false, x, st);
    tn_launch_apply_update(a, rider ? &x : nullptr, m->chain.blocks ? &m->chain : nullptr, st);
    m->chain.blocks = 0;
    ++m->apply_serial;
    mark(m, PF_APPLY_UPDATE, st);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_step(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                 int32_t n_centers, uint32_t epoch, const tensair_sparse_grad *peers, int32_t n_peers,
                 float lr, tensair_sparse_grad *own_out, float *mean_loss, void *stream)
{
    const int rc = step_impl(m, tokens, n_tokens, center_begin, n_centers, epoch, peers, nullptr, n_peers, lr,
                             own_out, nullptr, mean_loss, stream);
    if (rc == TENSAIR_EHIP && m) abandon_side_work(m);
    return rc;
}

int tensair_step_packed(tensair_model *m, const int32_t *tokens, int64_t n_tokens, int64_t center_begin,
                        int32_t n_centers, uint32_t epoch, const tensair_packed_grad *peers, int32_t n_peers,
                        float lr, tensair_sparse_grad *own_out, tensair_packed_grad *own_msg_out, float *mean_loss,
                        void *stream)
{
    if (n_peers > 0 && !peers) return fail(TENSAIR_EINVAL, "peers is NULL");
    const int rc = step_impl(m, tokens, n_tokens, center_begin, n_centers, epoch, nullptr, peers, n_peers, lr,
                             own_out, own_msg_out, mean_loss, stream);
    if (rc == TENSAIR_EHIP && m) abandon_side_work(m);
    return rc;
}

int tensair_dense_apply(void *theta, int32_t dtype, int64_t n, const float *const *grads, int32_t n_grads,
                        float lr, void *stream)
{
    if (!theta || (n_grads > 0 && !grads)) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (dtype != TENSAIR_F32 && dtype != TENSAIR_BF16) return fail(TENSAIR_EINVAL, "unknown dtype");
    if (n < 0 || n > TENSAIR_MAX_DENSE) return fail(TENSAIR_EINVAL, "n outside 0..TENSAIR_MAX_DENSE");
    if (n_grads < 0 || n_grads > TENSAIR_MAX_PEERS + 1)
        return fail(TENSAIR_ECAPACITY, "n_grads %d outside 0..%d", n_grads, TENSAIR_MAX_PEERS + 1);
    if (!(lr == lr)) return fail(TENSAIR_EINVAL, "lr is NaN");
    if ((uintptr_t)theta & 15) return fail(TENSAIR_EINVAL, "theta must be 16-byte aligned");
    DenseApplyArgs a;
    memset(&a, 0, sizeof(a));
    a.theta = theta;
    a.n = n;
    a.n_grads = n_grads;
    a.dtype = dtype;
    a.lr = lr;
    for (int k = 0; k < n_grads; ++k) {
        if (!grads[k]) return fail(TENSAIR_EINVAL, "grads[%d] is NULL", k);
        if ((uintptr_t)grads[k] & 15) return fail(TENSAIR_EINVAL, "grads[%d] must be 16-byte aligned", k);
        a.grads[k] = grads[k];
    }
    if (n == 0 || n_grads == 0) return TENSAIR_OK;
    tn_launch_dense_apply(a, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_lookup(tensair_model *m, int32_t table, const int32_t *ids, int64_t n, float *out, void *stream)
{
    if (!m || (n > 0 && (!ids || !out))) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (table != 0 && table != 1) return fail(TENSAIR_EINVAL, "table must be 0 (W_in) or 1 (W_out)");
    if (n < 0) return fail(TENSAIR_EINVAL, "n is negative");
    if ((uintptr_t)out & 15) return fail(TENSAIR_EINVAL, "out must be 16-byte aligned");
    const tensair_config &c = m->cfg;
    LookupArgs a;
    a.table = table ? m->w_out : m->w_in;
    a.ids = ids;
    a.out = out;
    a.n = n;
    a.V = c.vocab;
    a.D = c.dim;
    a.stride = c.row_stride;
    a.dtype = c.dtype;
    a.status = m->status;
    tn_launch_lookup(a, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_cosine_difference(const void *a, const void *b, int32_t dtype, int64_t vocab, int32_t dim,
                              int32_t row_stride, float *diff, void *stream)
{
    if (!a || !b || !diff) return fail(TENSAIR_EINVAL, "NULL pointer argument");
    if (dtype != TENSAIR_F32 && dtype != TENSAIR_BF16) return fail(TENSAIR_EINVAL, "unknown dtype");
    if (vocab < 0 || vocab > 0x7FFFFFFFLL) return fail(TENSAIR_EINVAL, "vocab out of range");
    if (dim < 4 || dim > TENSAIR_MAX_DIM || dim % 4) return fail(TENSAIR_EINVAL, "dim must be a multiple of 4 in 4..1024");
    if (row_stride < dim || row_stride % 4) return fail(TENSAIR_EINVAL, "row_stride must be >= dim and a multiple of 4");
    if (((uintptr_t)a | (uintptr_t)b) & 15) return fail(TENSAIR_EINVAL, "tables must be 16-byte aligned");
    CosineArgs c;
    c.a = a;
    c.b = b;
    c.diff = diff;
    c.V = vocab;
    c.D = dim;
    c.stride = row_stride;
    c.dtype = dtype;
    tn_launch_cosine_diff(c, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_status(tensair_model *m, void *stream)
{
    if (!m) return fail(TENSAIR_EINVAL, "model is NULL");
    hipStream_t st = (hipStream_t)stream;
    int word = 0;
    HIP_TRY(hipMemcpyAsync(&word, m->status, sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (word != 0) {
        int zero = 0;
        HIP_TRY(hipMemcpyAsync(m->status, &zero, sizeof(int), hipMemcpyHostToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        return fail(TENSAIR_EDATA, "kernels met invalid data:%s%s%s", (word & ST_BAD_ID) ? " id out of range" : "",
                    (word & ST_BAD_ORDER) ? " ids not strictly ascending" : "",
                    (word & ST_OVERFLOW) ? " row count above capacity" : "");
    }
    return TENSAIR_OK;
}

int tensair_copy_probe(void *dst, const void *src, size_t bytes, void *stream)
{
    if (!dst || !src || (bytes & 15) || (((uintptr_t)dst | (uintptr_t)src) & 15))
        return fail(TENSAIR_EINVAL, "copy_probe: pointers and size must be multiples of 16");
    tn_launch_copy_probe(dst, src, bytes, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_stream_probe(void *dst, const void *src, size_t bytes, int32_t mode, void *stream)
{
    if (!dst || !src || (bytes & 15) || (((uintptr_t)dst | (uintptr_t)src) & 15))
        return fail(TENSAIR_EINVAL, "stream_probe: pointers and size must be multiples of 16");
    if (mode < 0 || mode > 3) return fail(TENSAIR_EINVAL, "stream_probe: mode must be 0..3");
    tn_launch_stream_probe(dst, src, bytes, mode, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return TENSAIR_OK;
}

int tensair_profile(tensair_model *m, int level)
{
    if (!m || level < 0 || level > 2) return fail(TENSAIR_EINVAL, "profile: bad argument");
    m->prof_level = level;
    return TENSAIR_OK;
}

int tensair_profile_read(tensair_model *m, int32_t *tags, float *ms, int32_t max_records)
{
    if (!m || !tags || !ms || max_records < 0) return fail(TENSAIR_EINVAL, "profile_read: bad argument");
    int n = 0;
    if (!m->prof_marks.empty()) {
        hipError_t e = hipEventSynchronize(m->prof_marks.back().second);
        if (e != hipSuccess) return fail(TENSAIR_EHIP, "profile_read: %s", hipGetErrorString(e));
    }
    for (size_t i = 1; i < m->prof_marks.size() && n < max_records; ++i) {
        const int tag = m->prof_marks[i].first;
        if (tag == PF_BEGIN_GRAD || tag == PF_BEGIN_APPLY || tag == PF_BEGIN_ADD || tag == PF_BEGIN_PACK) continue;
        if (m->prof_level == 1 && tag != PF_APPLY_UPDATE && tag != PF_ADD_ROWS && tag != PF_PACK) continue;
        float t = 0.f;
        if (hipEventElapsedTime(&t, m->prof_marks[i - 1].second, m->prof_marks[i].second) != hipSuccess) continue;
        tags[n] = tag;
        ms[n] = t;
        ++n;
    }
    m->prof_marks.clear();
    m->prof_used = 0;
    return n;
}

int tensair_model_destroy(tensair_model *m)
{
    if (m) {
        for (hipEvent_t ev : m->prof_pool) (void)hipEventDestroy(ev);
        if (m->ev_fork) (void)hipEventDestroy(m->ev_fork);
        if (m->ev_fwd) (void)hipEventDestroy(m->ev_fwd);
        if (m->ev_prep) (void)hipEventDestroy(m->ev_prep);
        if (m->ev_keys) (void)hipEventDestroy(m->ev_keys);
        if (m->ev_reduced) (void)hipEventDestroy(m->ev_reduced);
        if (m->side) {
            (void)hipStreamSynchronize(m->side);   // a pending prefetch still writes the workspace
            (void)hipStreamDestroy(m->side);
        }
    }
    delete m;
    return TENSAIR_OK;
}

}  // extern "C"
