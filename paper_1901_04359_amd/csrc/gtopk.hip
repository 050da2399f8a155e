// gTop-k S-SGD data-parallel hot path for MI355X (gfx950, wave64): the C ABI.
//
// Pipeline of one iteration (paper: Algorithm 4; Definition 1; Algorithm 3; Eq. 3):
//
//   local select   sample histogram -> speculative threshold -> ONE streaming pass
//                  (acc = residual + grad, written back; entries at or above the
//                  speculative threshold are compacted into a short candidate list)
//                  -> exact select of the k-th key among the candidates
//                  -> index-ordered emit of the k selected entries.
//                  The speculative threshold only decides how much work the exact
//                  part has; if it left a worker fewer than k candidates or more than
//                  the list holds, that worker's exact part reads its dense row
//                  instead (same kernels, decided on the device).
//   tree           per round: index-ordered union of the two k-sets of each pair
//                  (values at shared indices added) -> the same exact select
//                  -> ordered emit; the last round divides by P.  Very large sets are
//                  merged through a speculative threshold of their own (a sample of
//                  the union; only the slots that reach it are kept), with the
//                  complete union standing by for a pair whose threshold misses.
//   large densities  (an eighth and more, large rows) go another way behind the
//                  sample: see grouped.hip.h.
//   restore        membership test of each local entry in the global index set.
//
// Nothing here is a dense contraction, so there is no MFMA; the streaming pass is
// bound by HBM bandwidth and everything after it by launch latency.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "gtopk.h"
#include "common.hip.h"
#include "stream_pass.hip.h"
#include "select.hip.h"
#include "merge.hip.h"
#include "merge_block.hip.h"
#include "apply.hip.h"
#include "aggregate.hip.h"
#include "small.hip.h"
#include "grouped.hip.h"

using namespace gtopk;

namespace {

// ---------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
inline uint32_t ceil_div(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }
inline bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

struct Carver {
    char* base;
    size_t off = 0;
    template <class T> T* take(size_t n) {
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off = align_up(off + n * sizeof(T));
        return p;
    }
};

// hist .. hist_dense are carved back to back so that one clear covers them
// with_finish: the select may be finished by k_finish, which needs the groups' offsets
SelState carve_select(Carver& c, size_t sets, uint32_t list_cap, uint32_t maxgroups,
                      bool with_dense_hist = false, bool with_finish = true) {
    SelState s;
    s.hist = c.take<uint32_t>(sets * kHistBins);
    s.list_cnt = c.take<uint32_t>(sets);
    s.grp_gt = c.take<uint32_t>(sets * maxgroups);
    s.grp_in = c.take<uint32_t>(sets * maxgroups);
    s.bin_hi = c.take<uint32_t>(sets);
    s.bin_lo_inv = c.take<uint32_t>(sets);
    s.hist_dense = with_dense_hist ? c.take<uint32_t>(sets * kHistBins) : nullptr;   // cleared as well
    s.d1 = c.take<uint32_t>(sets);
    s.krem = c.take<uint32_t>(sets);
    s.T = c.take<uint32_t>(sets);
    s.need = c.take<uint32_t>(sets);
    s.T_out = nullptr;
    s.list = c.take<uint2>(sets * list_cap);
    s.off_gt = with_finish ? c.take<uint32_t>(sets * maxgroups) : nullptr;
    s.off_eq = with_finish ? c.take<uint32_t>(sets * maxgroups) : nullptr;
    s.list_cap = list_cap;
    s.maxgroups = maxgroups;
    s.seg_list = 0u;
    return s;
}
// words from s.hist to the end of s.bin_lo_inv / s.hist_dense (padding included)
inline size_t select_clear_words(const SelState& s) { return (size_t)(s.d1 - s.hist); }

// A second copy of the arrays that must be zero when a select starts; everything
// else is shared with `base`.  Two such states alternate between the rounds of the tree,
// so that one can be cleared while the other is in use.
SelState carve_select_alt(Carver& c, const SelState& base, size_t sets, size_t* clear_words) {
    SelState s = base;
    s.hist = c.take<uint32_t>(sets * kHistBins);
    s.list_cnt = c.take<uint32_t>(sets);
    s.grp_gt = c.take<uint32_t>(sets * base.maxgroups);
    s.grp_in = c.take<uint32_t>(sets * base.maxgroups);
    s.bin_hi = c.take<uint32_t>(sets);
    s.bin_lo_inv = c.take<uint32_t>(sets);
    uint32_t* end = c.take<uint32_t>(1);
    *clear_words = base.hist ? (size_t)(end - s.hist) : 0;
    return s;
}

// slots per group of an array of n slots: a multiple of 256, at least min_slots, and large
// enough that there are at most max_groups (<= kMaxGroups) groups
uint32_t group_slots_for(uint64_t n, uint32_t max_groups, uint32_t min_slots = 1024) {
    uint32_t L = ceil_div(n, max_groups);
    L = (L + 255u) & ~255u;
    return L < min_slots ? min_slots : L;
}
constexpr uint32_t kMergeMinSlots = 512;        // merged sets: one round of a block (swept 512 / 1024)

// Groups per set when `sets` sets are selected from side by side.  Every block of k_bucket
// and k_emit pays a fixed price (it reads the set's 4096-bin histogram, or the list of
// in-bin keys), so a batch gets about kTargetBlocks blocks in total and no more (swept: 512 .. 4096;
// a tree of 32 sets of 255,570 entries: 268 / 291 / 307 us at 1024 / 2048 / 4096).
constexpr uint32_t kTargetBlocks = 1024;
constexpr uint32_t kLocalTargetBlocks = 8192;   // the same for the local selection's P sets
uint32_t groups_for(uint32_t sets) {
    const uint32_t g = kTargetBlocks / (sets ? sets : 1);
    return g < 32 ? 32 : (g > (uint32_t)kMaxGroups ? (uint32_t)kMaxGroups : g);
}

constexpr uint64_t kInlineFinishMax = 1u << 20;  // sets up to this many slots: no k_finish
// Which union: one entry per thread with a search of its own (k_union: short chains, latency) or eight
// slots per thread cut by output position (k_union_path: less work per slot, throughput).  Sets above
// kUnionPathMinK take the latter; smaller ones do once the launch holds enough entries to be bound
// by throughput.  A merge call in us, k_union / k_union_path, for batches of 1, 4 and 16 pairs:
//   k = 100,000   28.5 / 29.6   41.0 / 39.2   73.6 / 58.2
//   k =  50,000   26.3 / 28.0   32.2 / 33.2   58.0 / 52.0
//   k =  25,000        -        29.0 / 31.0   43.2 / 42.6
constexpr uint32_t kUnionPathMinK = 131072;
constexpr uint64_t kUnionPathMinEntries = 3u << 17;      // of one operand, all pairs together
constexpr uint32_t kUnionPathFewK = 16384;               // at least four tiles per pair
inline bool union_by_path(uint32_t k, uint32_t batch) {
    return k > kUnionPathMinK || (k >= kUnionPathFewK && (uint64_t)k * batch >= kUnionPathMinEntries);
}
constexpr int kUnionPathEpt = 8;
constexpr int kUnionHistBlock = 1024;           // threads per block of the union that also histograms
constexpr uint32_t kUnionCutsMinK = 1u << 19;   // sets above this size: cut points in a kernel of their own

struct MergeWs {
    SelState sel;      // state of even rounds
    SelState sel_alt;  // state of odd rounds (own hist / list_cnt / grp_gt)
    size_t alt_clear_words;
    uint32_t* m_idx;   // [pairs][m_stride]: the 2k slots of a pair, padded to a multiple of 8
    float* m_val;
    uint32_t m_stride;
    uint32_t* tmin[2]; // [pairs] smallest key of each output set, alternating between rounds
    uint32_t* inv_min; // [2*pairs] 0x7fffffff - smallest key of each caller-supplied operand
    uint32_t* cuts;    // [pairs][tiles + 1] cut points of k_union_path's blocks (large sets)
    // the largest sets are merged through a speculative threshold (FiltSrc); all NULL otherwise
    uint32_t* f_samp_hist;  // [pairs][16384]  } cleared together at the start of every round
    uint32_t* f_set_cnt;    // [pairs]         }
    size_t f_clear_words;
    uint32_t* f_tspec;      // [pairs]
    uint32_t* f_tile_cnt;   // [pairs][tiles]
    SelState sel_rep;       // select state of the pairs that fall back to their complete union
    size_t rep_clear_words;
    uint32_t L;
    size_t bytes;
};

// Sets of more than 2^22 entries whose 8192-slot union tiles fit the select's group tables
// are merged through a speculative threshold.  Measured at C4 size: at k = 6.4 M the rounds of
// the tree take 3.4 instead of 3.6 ms; at k = 1.85 M the sample and the stand-by launches for a
// threshold that misses (about 65 us per round) cost more than the smaller select saves.
constexpr uint32_t kMergeFilterMinK = 1u << 22;
inline bool merge_filtered(uint32_t k) {
    return k > kMergeFilterMinK &&
           ceil_div(2ull * k, (uint64_t)kUnionHistBlock * kUnionPathEpt) <= (uint32_t)kMaxGroups;
}

MergeWs carve_merge(Carver& c, uint32_t k, size_t pairs) {
    MergeWs w;
    w.L = group_slots_for(2ull * k, kMaxGroups, kMergeMinSlots);
    w.sel = carve_select(c, pairs, 2 * k, ceil_div(2ull * k, w.L));
    w.sel_alt = carve_select_alt(c, w.sel, pairs, &w.alt_clear_words);
    w.m_stride = (2 * k + 7u) & ~7u;
    w.m_idx = c.take<uint32_t>(pairs * w.m_stride);
    w.m_val = c.take<float>(pairs * w.m_stride);
    w.tmin[0] = c.take<uint32_t>(pairs);
    w.tmin[1] = c.take<uint32_t>(pairs);
    w.inv_min = c.take<uint32_t>(2 * pairs);
    w.cuts = c.take<uint32_t>(k > kUnionCutsMinK
                                  ? pairs * ((size_t)ceil_div(2ull * k, kUnionHistBlock * kUnionPathEpt) + 1)
                                  : 0);
    w.f_samp_hist = w.f_set_cnt = w.f_tspec = w.f_tile_cnt = nullptr;
    w.f_clear_words = w.rep_clear_words = 0;
    w.sel_rep = w.sel;
    if (merge_filtered(k)) {
        const size_t ntiles = ceil_div(2ull * k, kUnionHistBlock * kUnionPathEpt);
        w.f_samp_hist = c.take<uint32_t>(pairs * kSampleBins);
        w.f_set_cnt = c.take<uint32_t>(pairs);
        uint32_t* end = c.take<uint32_t>(1);
        w.f_clear_words = w.f_samp_hist ? (size_t)(end - w.f_samp_hist) : 0;
        w.f_tspec = c.take<uint32_t>(pairs);
        w.f_tile_cnt = c.take<uint32_t>(pairs * ntiles);
        w.sel_rep = carve_select_alt(c, w.sel, pairs, &w.rep_clear_words);
    }
    w.bytes = c.off;
    return w;
}

struct StepWs {
    // local select
    uint32_t* samp_hist;   // [P][16384] or NULL: not needed  } cleared before
    uint32_t* cand_count;  // [P]                             } every selection
    size_t samp_words;
    uint32_t* tspec;       // [P] speculative threshold of the streaming pass
    uint32_t* cand_idx;    // [P][cap] candidates as the streaming pass left them (runs)
    float* cand_val;
    uint2* run_table;      // [P][nchunks]
    uint32_t* run_off;     // [P][nchunks]
    uint32_t* ord_idx;     // [P][cap] candidates in index order
    float* ord_val;
    SelState sel;          // P sets
    uint32_t cap, nchunks, chunk_log2;
    uint32_t Lc, gcand;    // candidate list: slots per group, groups
    uint32_t Ld, gdense;   // dense row: slots per group, groups
    // tree
    MergeWs mrg;           // P/2 pairs
    uint32_t* x_idx;       // [P/2][k] ping
    float* x_val;
    uint32_t* y_idx;       // [P/4][k] pong
    float* y_val;
    // step
    uint32_t* gbits;       // [ceil(m/32)] one bit per gradient element: the global set
    size_t gbits_words;
    uint32_t* loc_idx;     // [P][k] when the caller does not want them
    float* loc_val;
    size_t bytes;
};

uint32_t cand_capacity(int64_t m, uint32_t k) {
    uint64_t cap = 3ull * k + 8192;
    if (cap > (uint64_t)m) cap = (uint64_t)m;
    return (uint32_t)cap;
}

// Small problems take the few-launch path: the local selection of a worker in one block,
// the whole tree with the average and the extra residual in one block.
static bool small_problem(int64_t m, int64_t k, int64_t P) {
    return P <= kSmallMaxP && k <= kSmallMaxK && P * k <= kSmallMaxEntries &&
           m + 3 <= (int64_t)kSmallMaxChunks * kSmallChunk;
}

struct SamplePlan { uint32_t tile_stride, n_tiles, target; uint64_t sampled; };

// Long candidate lists are selected where the streaming pass left them, one group per run
// (RunSrc): from about 256 expected candidates per 2^15 elements of the row on (k = 0.56 % of m),
// whatever the pass's chunks, and while the runs of a row are no more than the select's group tables hold.
// The line is that of chunks of 2^15.  gtopk_local_select in us, put into index order first / in place:
//   chunks of 2^15, m = 3 M  P = 32  k = 9000   260 / 262   k = 15,000   272 / 276   (2^14) k = 60,000  313 / 323
//   2^13 .. 2^14    m = 3 M  P = 8   k = 9000  97.5 / 94.5  k = 24,000  98.1 / 95.8  k = 750,000       177 / 171
//   2^12            m = 1 M  P = 8   k = 1000  54.8 / 49.0  k = 8000    63.6 / 58.0  k = 125,000      81.3 / 85.0
// so with short chunks it could lie lower, and rows of an eighth dense go either way.
static bool run_groups(int64_t m, uint32_t k) {
    const double per_chunk = 1.4 * (double)k * (double)kChunk / (double)m;     // of the largest chunk
    return per_chunk >= 256.0 && ceil_div((uint64_t)m + 3, kChunk) <= (uint64_t)kMaxGroups;
}
// (the few-launch path takes a smaller sample: one block per worker reads it)
constexpr double kSampleMean = 256.0, kSampleMinTiles = 4096.0;
constexpr double kSmallSampleMean = 16.0, kSmallSampleMin = 8192.0;
SamplePlan plan_sample(int64_t m, uint32_t k, uint32_t tile, double sample_mean, double min_elements);

// Medium problems: rows so short that the three launches in front of the pass (clear, k_sample,
// k_sample_pick) weigh as much as it does, and a sample that one block per worker reads in one or two
// rounds is enough: k_small_sample then does all three.  A step, three launches / one, in us:
//   m = 200,000  P = 8  k = 20,000   131 -> 99       m = 100,000  P = 2  k = 1000    60 -> 50
//   m = 1 M      P = 4  k = 1000      88 -> 77       m = 2 M      P = 32 k = 2000   277 -> 270
// (the first two include what their shorter chunks give, see pass_chunk_log2).  A larger sample in one
// block loses: 65,536 elements at m = 8 M, P = 4, k = 8000 take the step from 148 to 161 us.
constexpr uint64_t kMidElements = 1ull << 26;            // of all rows together
constexpr double kMidSampleMin = 16384.0, kMidSampleMax = 32768.0;
// Expected sample rank of the k-th key, at least.  At rank 16 the threshold keeps 2.5 k candidates on average
// with a spread of a sixth; a list of 3 k + 8192 entries has room for that only while k is in the
// thousands (k = 4096, the shortest list for it: 5 k, missed with a probability of some 1e-5 per worker, and
// then that worker is selected from its dense row).  At rank 64 it keeps 1.7 k +- an eighth.
// The step from one to the other leaves a gap: rows of 512 k .. 2048 k elements (2.1 to 8.4 M at the border)
// take the three launches from k = 4097 until rank 64 fits too.  With rank 16 up to k = 8192 in its place
// gtopk_local_select takes, m = 3 M, k = 6000, P = 4: 67.0 -> 61.5 us, P = 8: 107.5 -> 106.0, but lists are
// missed where they are shortest, m = 8 M, P = 2, k = 5600: 72.6 -> 138.
static double mid_sample_mean(uint32_t k) { return k <= 4096u ? 16.0 : 64.0; }
// Rows no longer than the few-launch path's smallest sample, which is all of them there too, always are.
static bool mid_problem(int64_t m, uint32_t k, uint64_t P) {
    if ((double)m <= kSmallSampleMin) return true;
    return (uint64_t)m * P <= kMidElements && mid_sample_mean(k) * (double)m <= kMidSampleMax * (double)k &&
           !merge_filtered(k) && !small_problem(m, k, (int64_t)P);
}
static SamplePlan plan_row_sample(int64_t m, uint32_t k, uint64_t P) {
    return mid_problem(m, k, P) ? plan_sample(m, k, kMidSampleTile, mid_sample_mean(k), kMidSampleMin)
                                : plan_sample(m, k, kSampleTile, kSampleMean, kSampleMinTiles * kSampleTile);
}

// Elements per block of the pass = per run of candidates: 2^15, less
//   - where that gives fewer than 1024 blocks: a block that has a CU to itself reads at some 60 GB/s;
//   - at densities from 0.6 % on (runs selected where they lie): a run is compacted, walked and
//     emitted by one block or wave, and hot layers make some runs ten times as long as others.
//     Shorter runs even that out until the blocks' fixed price in the emit outweighs it.
// Measured, a step in us with chunks of 2^15 / 2^14 / 2^13 elements:
//   m = 5 M   P = 8   k = 1 M      502 / 451 / 449      m = 2 M  P = 32  k = 400,000   780 / 675 / 661
//   m = 5 M   P = 8   k = 50,000   210 /  -  / 195      m = 5 M  P = 32  k = 50,000    550 / 538 /  -
//   m = 14 M  P = 16  k = 1.4 M   1282 / 1229 / 1245    m = 14 M P = 16  k = 140,000   645 / 688 /  -
//   m = 25.6 M P = 32 k = 1.85 M  3616 / 3950 /  -      (k = 6.4 M: 6607 / 6775)
static uint32_t pass_chunk_log2(int64_t m, uint32_t k, uint64_t P) {
    const bool few = (uint64_t)m * P <= kMidElements;
    const double rho = (double)k / (double)m;
    const uint64_t most = rho >= 0.05 ? 16384 : (rho >= 0.006 ? 10240 : 0);      // blocks, all workers
    uint32_t l = kChunkLog2;
    while (l > 12 && ceil_div((uint64_t)m + 3, 1u << (l - 1)) <= (uint32_t)kMaxGroups &&
           ((few && P * ceil_div((uint64_t)m + 3, 1u << l) < 1024) ||
            (l > 13 && P * ceil_div((uint64_t)m + 3, 1u << (l - 1)) <= most)))
        --l;
    return l;
}

StepWs carve_step(void* ws, int64_t m, uint32_t k, uint32_t P) {
    Carver c{reinterpret_cast<char*>(ws)};
    StepWs s;
    s.cap = cand_capacity(m, k);
    s.chunk_log2 = pass_chunk_log2(m, k, P);
    s.nchunks = ceil_div((uint64_t)m + 3, 1u << s.chunk_log2);      // a row may start up to 3 elements into a chunk
    {
        uint32_t g = kLocalTargetBlocks / P;
        g = g < 32 ? 32 : (g > (uint32_t)kMaxGroups ? (uint32_t)kMaxGroups : g);
        s.Lc = group_slots_for(s.cap, g);
        const uint32_t lmin = group_slots_for(s.cap, kMaxGroups);
        if (s.Lc > 8192u) s.Lc = lmin > 8192u ? lmin : 8192u;
        s.gcand = ceil_div(s.cap, s.Lc);
    }
    // dense rows (a worker whose candidate list cannot be used; the dense top-k)
    s.gdense = P == 1 ? (uint32_t)kMaxGroups : 1024u;
    s.Ld = group_slots_for((uint64_t)m, s.gdense);
    s.gdense = ceil_div((uint64_t)m, s.Ld);
    s.cand_count = c.take<uint32_t>(P);
    s.tspec = c.take<uint32_t>(P);
    s.cand_idx = c.take<uint32_t>((size_t)P * s.cap);
    s.cand_val = c.take<float>((size_t)P * s.cap);
    // The run tables are sized for the shortest chunks (the few-launch path's among them): how long the chunks
    // are changes in steps with m and k, and a workspace should serve smaller k too (a density that comes
    // down), and the tree, whose rows are m = k.  (The groups' tables still go up and down by some KB.)
    uint32_t table = ceil_div((uint64_t)m + 3, 4096);
    static_assert(kSmallChunk == 4096, "the shortest chunk");
    if (table > (uint32_t)kMaxGroups) table = (uint32_t)kMaxGroups;
    if (table < s.nchunks) table = s.nchunks;
    s.run_table = c.take<uint2>((size_t)P * table);
    s.run_off = c.take<uint32_t>((size_t)P * table);
    s.ord_idx = c.take<uint32_t>((size_t)P * s.cap);
    s.ord_val = c.take<float>((size_t)P * s.cap);
    {
        uint32_t g = s.gcand > s.gdense ? s.gcand : s.gdense;
        if (run_groups(m, k) && s.nchunks > g) g = s.nchunks;      // one group per run
        // (only the dense top-k, one row, is ever finished by k_finish: see local_grid)
        s.sel = carve_select(c, P, s.cap, g, /*with_dense_hist=*/true, /*with_finish=*/P == 1);
        // The sample histograms lie where the list of in-bin keys will: k_bucket writes that long after they
        // have been read.  (Rows that need one are longer than 8192, and so is their list.)
        static_assert(kSmallSampleMin >= 8192.0 && 8192 * sizeof(uint2) == kSampleBins * sizeof(uint32_t), "fits");
        s.samp_words = mid_problem(m, k, P) ? 0 : (size_t)P * kSampleBins;
        s.samp_hist = s.samp_words ? reinterpret_cast<uint32_t*>(s.sel.list) : nullptr;
    }
    const size_t pairs = P > 1 ? P / 2 : 1;
    s.mrg = carve_merge(c, k, pairs);
    s.x_idx = c.take<uint32_t>(pairs * k);
    s.x_val = c.take<float>(pairs * k);
    const size_t quarter = P > 3 ? P / 4 : 1;
    s.y_idx = c.take<uint32_t>(quarter * k);
    s.y_val = c.take<float>(quarter * k);
    s.gbits_words = (size_t)((m + 31) / 32);
    s.gbits = c.take<uint32_t>(s.gbits_words);
    s.loc_idx = c.take<uint32_t>((size_t)P * k);
    s.loc_val = c.take<float>((size_t)P * k);
    s.bytes = c.off;
    return s;
}

// The step at large densities (grouped.hip.h) lives in memory that the other path uses for the candidates in index
// order and for the merged pairs.
struct GroupWs {
    GroupSets gs;
    size_t clear_words;         // from gs.hist on
    uint64_t* bits;             // [P][ngroups * kGroup / 64] the workers' sets
    uint64_t* gbits;            // [ngroups * kGroup / 64] the global set
    uint32_t* samples;          // [P / 2][ngroups * per_group] of a round's unions; before them [P][row_samples] of the rows
    uint32_t per_group, row_samples;
    bool fits;
};
GroupWs carve_grouped(const StepWs& s, int64_t m, uint32_t k, uint32_t P) {
    GroupWs w;
    const size_t ng = ceil_div((uint64_t)m, kGroup), sets = 2 * (size_t)P;
    Carver c{reinterpret_cast<char*>(s.ord_idx)};
    GroupSets& gs = w.gs;
    gs.m = (uint32_t)m;
    gs.ngroups = (uint32_t)ng;
    gs.hist = c.take<uint32_t>(sets * kBrkBins);
    gs.hist_all = c.take<uint32_t>(sets * kAllBins);
    gs.list_cnt = c.take<uint32_t>(sets);
    gs.arrived = c.take<uint32_t>(sets);
    gs.brk_cnt = c.take<uint32_t>(P);
    const size_t clear_end = c.off;
    w.clear_words = clear_end / sizeof(uint32_t);
    gs.lo = c.take<uint32_t>(sets);
    gs.hi = c.take<uint32_t>(sets);
    gs.d1 = c.take<uint32_t>(sets);
    gs.krem = c.take<uint32_t>(sets);
    gs.T = c.take<uint32_t>(sets);
    gs.need = c.take<uint32_t>(sets);
    gs.run = c.take<uint4>(sets * ng);
    gs.grp_gt = c.take<uint32_t>(sets * ng);
    gs.off = c.take<uint2>(sets * (ng + 1));
    gs.tail = c.take<uint32_t>((size_t)P * ng * 3);
    gs.mask = c.take<uint64_t>((size_t)P * (ng + 1));
    w.bits = c.take<uint64_t>((size_t)P * ng * (kGroup / 64));
    w.gbits = c.take<uint64_t>(ng * (kGroup / 64));
    // about 2^16 sampled elements of a pair's union
    w.per_group = 2 * kGrpWaves;
    while (w.per_group < kGroup / kGrpPer && 2 * w.per_group * ng <= 65536) w.per_group *= 2;
    w.row_samples = plan_row_sample(m, k, P).n_tiles * kSampleKept;
    const size_t of_rows = (size_t)P * w.row_samples, of_pairs = (size_t)(P / 2) * ng * w.per_group;
    w.samples = c.take<uint32_t>(of_rows > of_pairs ? of_rows : of_pairs);
    w.fits = ng <= kMaxIndexGroups && c.off <= 2 * align_up((size_t)P * s.cap * sizeof(uint32_t));
    return w;
}

// Which steps take the grouped path: it reads the hot parts of the rows where the other one writes, walks and reads
// lists of their candidates, and pays per element there instead of per entry, so it wins from a density of an eighth
// on.  Its tree has no fewer launches, so short rows stay with the other one but for the highest densities (up to a
// third: above that a bracket has little room) and where all workers together have some 0.8 M entries per round of the tree,
// two added: with fewer, rows whose bracket's keys crowd into a few layers lose.  Those, in us, lists / groups, ten layers |
// 24 equal ones:  m = 1.05 M  P = 16  k = m/4  309 / 332 | 316 / 309   m = 2.1 M  P = 8  k = m/5  263 / 263 | 268 / 244 (left out)
// m = 1.05 M  P = 16  k = m/3  340 / 322 | 348 / 326   m = 1.9 M  P = 16  k = m/5  369 / 355 | 382 / 346 (taken).
// Lower lines in general; a step in us, lists / groups, rows of 20 layers | of one:
//   m = 25.6 M  P = 32  k = m/4   6434 / 4488 | 7199 / 5576     m/8  4813 / 3955 | 5129 / 4545     m/10  4293 / 3785 | 4482 / 4308
//   m = 25.6 M  P = 8   k = m/4   1856 / 1386 | 1933 / 1479     m/8  1280 / 1097 | 1306 / 1269     m/10  1129 / 1065 | 1175 / 1221
//   m = 17 M    P = 2   k = m/4    383 / 254  |  367 / 282      m/8   281 / 219  |  271 / 242      m/10   246 / 216  |  245 / 239
//   m = 5 M     P = 16  k = m/4    870 / 649  |  888 / 716      m/8   624 / 570  |  646 / 621      m/10   537 / 555  |  561 / 609
//   m = 2.1 M   P = 8   k = m/4    287 / 247  |  287 / 262      m/6   230 / 244  |  233 / 250
//   m = 1.05 M  P = 32  k = m/4    481 / 442  |  485 / 439      m/6   394 / 417  |  381 / 416
//   m = 0.5 M   P = 32  k = m/4    332 / 358  |  311 / 322
// (Masses of equal values besides: a row of zeros among ordinary ones at the first of these sizes 41.7 / 6.5 ms, all rows
// of one magnitude 188 / 4.7 ms, values rounded to integers 52.8 / 5.7 ms.)
static bool grouped_step(int64_t m, uint32_t k, uint32_t P, const StepWs& s) {
    const uint64_t n = (uint64_t)m;
    uint32_t rounds = 0;
    while (2u << rounds <= P) ++rounds;
    const bool entries = 5ull * P * k >= (uint64_t)(rounds + 2) << 22;
    const bool size = (n >= (1u << 22) && 8ull * k >= n) || (n >= (1u << 20) && 5ull * k >= n && entries);
    return P >= 2 && size && 3ull * k <= n && carve_grouped(s, m, k, P).fits;
}

constexpr int64_t kMaxMergeK = (int64_t)1 << 30;     // a merged pair has 2k slots, a uint32

bool sizes_ok(int64_t m, int64_t k, int64_t P) {
    return m >= 1 && m <= ((int64_t)1 << 31) && k >= 1 && k <= m && is_pow2(P) && P <= 65535 &&
           (P == 1 || k <= kMaxMergeK);
}

int launch_status() { return hipGetLastError() == hipSuccess ? GTOPK_OK : GTOPK_EHIP; }

// Instrumentation: the caller's events of one gtopk_step_timed call (NULL: none).
void mark_stage(int i, void* const* events, hipStream_t st) {
    if (events) (void)hipEventRecord((hipEvent_t)events[i], st);
}

ZeroJob zero_job(uint32_t* p0 = nullptr, size_t n0 = 0, uint32_t* p1 = nullptr, size_t n1 = 0,
                 uint32_t* p2 = nullptr, size_t n2 = 0, uint32_t* p3 = nullptr, size_t n3 = 0,
                 uint32_t* p4 = nullptr, size_t n4 = 0, uint32_t* p5 = nullptr, size_t n5 = 0) {
    return ZeroJob{{p0, p1, p2, p3, p4, p5}, {n0, n1, n2, n3, n4, n5}};
}

// blocks that clear the longest array of the job, `words` words each, at most 1024
uint32_t zero_blocks(const ZeroJob& job, uint32_t words) {
    size_t n = 0;
    for (int a = 0; a < kZeroSlots; ++a) n = job.n[a] > n ? job.n[a] : n;
    return (uint32_t)((n + words - 1) / words > 1024 ? 1024 : (n + words - 1) / words);
}

void zero_async(hipStream_t st, const ZeroJob& job) {
    const uint32_t blocks = zero_blocks(job, 1024);
    if (blocks) hipLaunchKernelGGL(k_zero_u32, dim3(blocks), dim3(256), 0, st, job);
}

inline uint32_t min_key_blocks(uint32_t k) {
    const uint32_t b = ceil_div(k, 8 * kMinKeyBlock);
    return b < 1 ? 1 : (b > 64 ? 64 : b);
}

// Smallest keys of `sets` sets (rows of v0, or of v0 and v1 in turn) into out; clears what `job` says.
// Sets up to kMinKeyWholeK (and longer than one block merges): in one launch, a block per set.  A merge call in us, clear and
// several blocks per set / one launch:  1 pair  k = 16,000: 23.6 / 21.7   k = 32,000: 26.6 / 26.8
// 16 pairs  k = 16,000: 31.6 / 29.7   k = 65,000: 52.8 / 65.9
constexpr uint32_t kMinKeyWholeK = 16384;
void find_min_keys(const float* v0, const float* v1, int64_t stride, uint32_t k, uint32_t sets, uint32_t* out,
                   ZeroJob job, hipStream_t st) {
    if (k <= kMinKeyWholeK && sets <= 32767u) {              // (at most 65535 rows of blocks)
        const uint32_t zblocks = zero_blocks(job, 4 * kMinKeyBlock);
        hipLaunchKernelGGL(k_set_min_key<true>, dim3(1, sets + zblocks), dim3(kMinKeyBlock), 0, st, v0, v1, stride, k,
                           sets, out, job);
    } else {
        job.p[kZeroSlots - 1] = out;
        job.n[kZeroSlots - 1] = sets;
        zero_async(st, job);
        hipLaunchKernelGGL(k_set_min_key<false>, dim3(min_key_blocks(k), sets), dim3(kMinKeyBlock), 0, st, v0, v1,
                           stride, k, sets, out, ZeroJob{});
    }
}

// how a batch of sets is walked and emitted
struct SelGrid {
    uint32_t sets;
    uint32_t walk_blocks;   // blocks per set of k_bucket
    uint32_t groups;        // blocks per set of k_emit (= emit groups, at most)
    uint64_t nphys_max;     // slots of a set's list, at most (sizes k_hist)
    bool own_finish;        // k_finish once per set instead of a finish in every emit block
};

// histogram + bucket + emit
template <class Src, bool DIVIDE>
void run_select(const Src& src, const SelState& ss0, const SelGrid& gr, uint32_t k, uint32_t* out_idx,
                float* out_val, int64_t out_stride, float divisor, uint32_t* gbits, hipStream_t st,
                bool with_hist = true) {
    // large merged sets, finished once per set: the in-bin keys stay with their groups (no shared counter)
    SelState ss = ss0;
    ss.seg_list = (Src::kSegList && gr.own_finish) ? 1u : 0u;
    // few blocks per set (a popular bin takes one same-address atomic per block): 4 slots per
    // thread up to 32 blocks, then 32 blocks with more slots per thread, then 32 slots per thread up to
    // 256 blocks, of which a list gets at most its share of the 1024 that fill the chip.  Every block flushes up
    // to 4096 bins by global atomics.  A step in us with 32 / 64 / 170 blocks per list: m = 25.6 M, P = 32, k = 1.85 M
    // 3636 / 3635 / 3665;  m = 14 M, P = 16, k = 1 M  1043 / 1045 / 1057;  m = 30 M, P = 2, k = 1.8 M  344 / 333 / 329.
    // A dense row among lists keeps them all: gtopk_local_select with one row of zeros at the first of these sizes
    // 3.93 / 3.54 ms with the list's 32 blocks / 170 (3.27 ms without such a row).
    uint32_t hb = ceil_div(gr.nphys_max, 4 * kHistBlock), dense_hb;
    if (hb > 32) {
        hb = ceil_div(gr.nphys_max, 32 * kHistBlock);
        hb = hb < 32 ? 32 : (hb > 256 ? 256 : hb);
        dense_hb = hb;
        const uint32_t most = 1024u / gr.sets;
        hb = hb > most ? most : hb;
        hb = hb < 32 ? 32 : hb;
    } else {
        dense_hb = hb = hb < 1 ? 1 : hb;
    }
    if (with_hist)
        hipLaunchKernelGGL((k_hist<Src>), dim3(dense_hb + (Src::kRunScan ? 1 : 0), gr.sets), dim3(kHistBlock), 0,
                           st, src, ss, hb, dense_hb);
    hipLaunchKernelGGL((k_bucket<Src>), dim3(gr.walk_blocks, gr.sets), dim3(kBlock), 0, st, src, ss, k);
    // small sets: every block of the emit finishes the select itself (the list of keys it
    // needs for that is short); large sets: once per set, in a kernel of its own
    if (!gr.own_finish) {
        hipLaunchKernelGGL((k_emit<Src, DIVIDE, true>), dim3(gr.groups, gr.sets), dim3(kBlock), 0, st,
                           src, ss, k, out_idx, out_val, out_stride, divisor, gbits);
    } else {
        hipLaunchKernelGGL((k_finish<Src>), dim3(gr.sets), dim3(1024), 0, st, src, ss);
        hipLaunchKernelGGL((k_emit<Src, DIVIDE, false>), dim3(gr.groups, gr.sets), dim3(kBlock), 0, st,
                           src, ss, k, out_idx, out_val, out_stride, divisor, gbits);
    }
}

// Sample plan for the speculative threshold: tiles of `tile` contiguous elements, evenly spaced, about
// sample_mean / rho elements per worker but at least min_elements (all elements if the row is short).
// `target` is the rank in the sample whose bucket edge is taken: the expected sample rank of the
// k-th key plus 5.5 standard deviations, so that the candidate list holds at least k entries except
// with probability ~1e-8 per worker (and then that worker is merely selected from its dense row;
// lists that come out too long are as rare, but for the small samples of medium rows, see
// mid_sample_mean).
// sample_mean: expected sample rank of the k-th key, at least.  min_elements: spread (a layer of 1 % of
// the row still gets ~40 of the 4096 tiles of 64 of long rows, ~10 of the 1024 tiles of 16 of medium ones).
SamplePlan plan_sample(int64_t m, uint32_t k, uint32_t tile, double sample_mean, double min_elements) {
    SamplePlan p;
    double want = sample_mean * (double)m / (double)k;
    if (want < min_elements) want = min_elements;
    if (want >= (double)m) {
        p.tile_stride = tile;
    } else {
        const uint64_t tiles = (uint64_t)(want / tile) + 1;
        const uint64_t ts = (uint64_t)m / tiles;
        p.tile_stride = (uint32_t)(ts < (uint64_t)tile ? tile : ts);
    }
    p.n_tiles = ceil_div((uint64_t)m, p.tile_stride);
    const uint64_t last = (uint64_t)m - (uint64_t)(p.n_tiles - 1) * p.tile_stride;
    const uint64_t sampled = (uint64_t)(p.n_tiles - 1) * tile + (last < tile ? last : tile);
    p.sampled = sampled < (uint64_t)m ? sampled : (uint64_t)m;
    if (sampled >= (uint64_t)m) {
        p.target = k;                        // the "sample" is the whole row: exact count
    } else {
        // 5.5 standard deviations of the count, plus 3 % for the tiles' placement error
        const double mean = (double)k * (double)sampled / (double)m;
        double t = 1.03 * mean + 5.5 * __builtin_sqrt(mean) + 2.0;
        if (t > (double)sampled) t = (double)sampled;
        p.target = (uint32_t)t;
        if (p.target < 1) p.target = 1;
    }
    return p;
}

// Rank in a sample, `mean` the expected sample rank of the k-th key, that at most `target_hi` keys of the sample
// reach at a key above the k-th: the counterpart of plan_sample's target (`placed`: 1 less its share for the
// tiles' placement).
uint32_t bracket_target_hi(double mean, double placed) {
    const double t = placed * mean - 5.5 * __builtin_sqrt(mean) - 2.0;
    return t > 0.0 ? (uint32_t)t : 0u;
}
// The ranks of the rows' brackets, and of the unions', whose samples are scattered.
uint32_t row_bracket_target_hi(int64_t m, uint32_t k, const SamplePlan& sp) {
    return bracket_target_hi((double)k * (double)sp.sampled / (double)m, 0.97);
}
uint32_t union_bracket_target_lo(double mean) { return (uint32_t)(1.02 * mean + 5.5 * __builtin_sqrt(mean) + 2.0); }
uint32_t union_bracket_target_hi(double mean) { return bracket_target_hi(mean, 0.98); }

// Entries per thread with which one block selects from a worker's candidate list (k_small_select), 0: the general
// kernels do, three of them.  A list is expected to hold 2.5 k entries (mid_sample_mean), a longer one than the threads hold
// takes the block some walks.  gtopk_step in us, three kernels and three per round of the tree / one and one:
//   m = 30,000  P = 8  k = 1000   86.5 / 45.1     m = 400,000  P = 4   k = 1000  74.2 / 43.8    k = 4000  73.0 / 60.1
//   m = 100,000 P = 8  k = 4000   92.7 / 73.4     m = 400,000  P = 16  k = 900  123.7 / 62.2
//   m = 100,000 P = 32 k = 2000  136.3 / 81.6     m = 524,288  P = 32  k = 4000  169 / 119
// One worker with more entries loses (k = 4000, m = 262,144 36.8 / 38.7; k = 1000 38.6 / 31.4).
// A row that cannot be filtered (its sample misled, or masses of equal values) is read by the one block, or by a few where
// few workers leave the chip idle (row_shares); the line in m keeps that within what the general kernels take.  Rows of zeros |
// of ones, whose residuals after 100 to 300 steps hold many equal values | whose sample misled, in us as above:
//   m = 200,000  P = 8   k = 2000   194 / 108 | 172 / 134 | 169 .. 175 / 111 .. 121
//   m = 524,288  P = 8   k = 2000   291 / 146 | 261 / 191 | 242 .. 260 / 169 .. 190
//   m = 524,288  P = 32  k = 4000   534 / 232 | 440 / 285 | 443 .. 489 / 238 .. 266
//   m = 524,288  P = 4   k = 1000   143 /  92 | 139 / 107 | 112 .. 212 / 82 .. 95
//   m = 262,144  P = 2   k = 1000   138 /  73 | 130 /  87 | 123 / 64 .. 70
//   m = 524,288  P = 2   k = 1000   101 /  79 |  91 /  95 |  78 .. 180 / 71 .. 81
// With one worker the general kernels have the whole chip for such rows (m = 524,288, k = 1000 70 / 72 | 64 / 87 |
// 54 .. 157 / 64 .. 72; m = 200,000, k = 520 60 / 63 | 56 / 72 | 44 .. 83 / 57 .. 62).
uint32_t select_in_block(int64_t m, uint32_t k, uint32_t P) {
    if (m > 1 << 19 || (P == 1 && k > 1984)) return 0;
    const uint32_t n = 4 * k + 256;
    return n <= 4096 ? 4 : (n <= 8192 ? 8 : (n <= 16384 ? 16 : 0));
}
// Blocks that share a row that cannot be filtered, where few workers leave the chip idle.  A step in us, one block / up to
// eight, rows of ones | misled samples:  m = 524,288, k = 1000  P = 4  167 / 107 | 151 .. 164 / 82 .. 95   P = 1  148 / 87 | 133 .. 142 /
// 64 .. 72.  (Rows of 2^17 elements and less gain little: their one block takes some 20 us.)
uint32_t row_shares(int64_t m, uint32_t k, uint32_t P) {
    if (P >= 8 || m <= 1 << 17) return 1;
    uint32_t most = cand_capacity(m, k) / k;                   // their entries lie where the ordered list would
    if (most > 1024u * kRowPart / k) most = 1024u * kRowPart / k;
    return most < 8 ? most : 8;
}
// What the select of a local selection needs cleared.
ZeroJob local_clear(const StepWs& w, int64_t m, uint32_t k, uint32_t P) {
    return select_in_block(m, k, P) ? zero_job(w.sel.list_cnt, (size_t)P) : zero_job(w.sel.hist, select_clear_words(w.sel));
}

// The pass can also histogram the candidates it keeps; the select's own histogram kernel
// then only serves workers that fall back to their dense row.  That costs LDS atomics and,
// per block and non-empty bin, a global atomic in the pass.  Measured against the
// histogram kernel it saves: at rho = 0.001 (45 candidates per 32768-element block) the
// pass does not change and the select gains 6-8 us; at rho = 0.01 (460 per block) the pass
// loses 55 us and the select gains 13 us; at rho = 0.0725 (3,300 per block) the pass loses
// 120 us and the select gains 85 us; at rho = 0.25 (11,500 per block) the pass loses
// 80 us and the select gains 230 us.  So at both ends, not in between.
// (The blocks of that sweep, and of the rule, are those of 2^15 elements.  Shorter ones, 2^12 .. 2^14, flush more
// often for fewer candidates; there the two are within 4 % of each other, gtopk_local_select in us, histogram
// kernel / pass, by candidates per real block:  m = 1 M  P = 8  6: 54.8 / 54.7  46: 58.1 / 60.5  115: 68.2 / 67.5
// 717: 86.0 / 85.3   m = 3 M  P = 8  115: 96.2 / 97.1  573: 125.1 / 129.6  2867: 179.2 / 170.7   m = 1 M  P = 32
// 229: 131.9 / 127.2  573: 155.2 / 148.9.  Where a row overfills its list the pass's histogram serves the dense row too.)
bool pass_histograms(int64_t m, uint32_t k) {
    const double per_block = 1.4 * (double)k * (double)kChunk / (double)m;
    return per_block <= 128.0 || per_block >= 4096.0;
}

// the candidate lists (or dense rows) of the P workers as the select kernels' source
CandSrc cand_source(const float* rows, int64_t stride, int64_t m, uint32_t k, const StepWs& w,
                    bool producer_hist, bool no_bounds, uint32_t* thr_state = nullptr, bool row_hist = false) {
    return CandSrc{rows, stride, (uint32_t)m, k, w.cap, w.nchunks, w.chunk_log2, w.Lc, w.Ld,
                   w.cand_idx, w.cand_val, w.cand_count, w.tspec, w.run_table, w.run_off,
                   w.ord_idx, w.ord_val, producer_hist, no_bounds, row_hist, reinterpret_cast<uint4*>(thr_state)};
}

// The grids are sized for the candidate lists.  A worker that is selected from its dense
// row has more groups than that; its blocks take several each.  Every emit block finishes
// the select itself: the list of in-bin keys is short.
SelGrid local_grid(const StepWs& w, uint32_t P) {
    const uint32_t gd = w.gdense < 256u ? w.gdense : 256u;
    const uint32_t gx = w.gcand > gd ? w.gcand : gd;
    return SelGrid{P, gx, gx, (uint64_t)w.cap, false};
}

template <bool HIST, bool SUM>
void launch_pass(const float* grad, float* residual, int64_t m, int64_t stride, uint32_t P, const StepWs& w,
                 hipStream_t st) {
    const dim3 grid(w.nchunks, P), block(kSBlock);
#define GTOPK_PASS(ITERS)                                                                                   \
    hipLaunchKernelGGL((k_accum_filter<HIST, ITERS, SUM>), grid, block, 0, st, grad, residual, (uint32_t)m,     \
                       stride, w.tspec, w.cand_idx, w.cand_val, w.cap, w.cand_count, w.run_table, w.nchunks, \
                       w.sel.hist, HIST ? w.sel.hist_dense : w.sel.hist)
    static_assert(kIters == 16, "a chunk of 2^15 elements per block of 16 float4 per lane");
    switch (w.chunk_log2) {
        case 12: GTOPK_PASS(2); break;
        case 13: GTOPK_PASS(4); break;
        case 14: GTOPK_PASS(8); break;
        default: GTOPK_PASS(16); break;
    }
#undef GTOPK_PASS
}

// The speculative thresholds of P rows; before that, clears what `job` says (the candidate counters among it).
// SUM: the rows are residual + grad; else they are `residual` as it stands.  BRACKET: brackets [tspec, thi) instead, and
// samples are kept (see k_sample).
template <bool SUM, bool BRACKET>
void sample_rows(const float* grad, const float* residual, int64_t m, int64_t stride, uint32_t P, uint32_t k,
                 const StepWs& w, const SamplePlan& sp, const ZeroJob& job, uint32_t* tspec, uint32_t* thi,
                 uint32_t* samples, hipStream_t st, uint32_t* thr_state = nullptr) {
    // workers whose threshold is carried over from the previous call skip the sampling (the
    // kernels are launched all the same: who samples is decided on the device)
    const uint4* carry = reinterpret_cast<const uint4*>(thr_state);
    // A row that is summed goes through the pass anyway, and one that overfills its list still gains from the
    // threshold; a row that is not has nothing of a pass whose list will not hold.
    const uint32_t most = SUM ? 0xFFFFFFFFu : (uint32_t)((double)w.cap * (double)sp.sampled / (double)m);
    const uint32_t target_hi = BRACKET ? row_bracket_target_hi(m, k, sp) : 0u;
    if (mid_problem(m, k, P)) {
        const uint32_t zblocks = zero_blocks(job, 4 * kSmallBlock);
        hipLaunchKernelGGL((k_small_sample<kMidSampleTile, true, SUM, BRACKET>), dim3(P + zblocks), dim3(kSmallBlock), 0,
                           st, grad, residual, (uint32_t)m, stride, P, sp.tile_stride, sp.n_tiles, sp.target, most,
                           tspec, w.cand_count, carry, job, target_hi, thi, samples);
    } else {
        zero_async(st, job);
        uint32_t sblocks = ceil_div(sp.n_tiles, (kSampleBlock / kSampleTile) * 8);
        // about 256 blocks in all: every block flushes its own 16384-bin histogram with atomics
        const uint32_t sb_max = P >= 64 ? 4u : (P <= 16 ? 16u : 256u / P);
        if (sblocks > sb_max) sblocks = sb_max;
        if (sblocks < 1) sblocks = 1;
        hipLaunchKernelGGL((k_sample<SUM, BRACKET>), dim3(sblocks, P), dim3(kSampleBlock), 0, st, grad, residual,
                           (uint32_t)m, stride, sp.tile_stride, sp.n_tiles, w.samp_hist, carry, samples);
        hipLaunchKernelGGL(k_sample_pick<BRACKET>, dim3(P), dim3(kSampleBlock), 0, st, w.samp_hist, sp.target, most,
                           tspec, carry, target_hi, thi);
    }
}

// The thresholds and the pass that filters the rows by them (the sums replace the residual; a row that is not
// summed is not written).  Returns whether the pass has histogrammed its candidates.
template <bool SUM>
bool filter_rows(const float* grad, float* residual, int64_t m, int64_t stride, uint32_t P, uint32_t k,
                 const StepWs& w, const ZeroJob& job, hipStream_t st, void* const* events = nullptr,
                 uint32_t* thr_state = nullptr, bool histogram = true) {
    sample_rows<SUM, false>(grad, residual, m, stride, P, k, w, plan_row_sample(m, k, P), job, w.tspec, nullptr, nullptr, st,
                     thr_state);
    mark_stage(1, events, st);

    const bool producer_hist = histogram && pass_histograms(m, k);
    if (producer_hist) launch_pass<true, SUM>(grad, residual, m, stride, P, w, st);
    else launch_pass<false, SUM>(grad, residual, m, stride, P, w, st);
    mark_stage(2, events, st);
    return producer_hist;
}

// `zero_rows`: store +0.0 at the selected entries (the stand-alone call); gtopk_step
// passes false and settles the rows in k_restore_fused.  `job`: what the call needs cleared before
// its select, the candidate counters among it.
int do_local_select(const float* grad, float* residual, int64_t m, int64_t stride, uint32_t P,
                    uint32_t k, uint32_t* out_idx, float* out_val, const StepWs& w, bool zero_rows,
                    const ZeroJob& job, hipStream_t st, void* const* events = nullptr,
                    uint32_t* thr_state = nullptr) {
    const uint32_t entries = select_in_block(m, k, P);
    const bool producer_hist = filter_rows<true>(grad, residual, m, stride, P, k, w, job, st, events, thr_state, entries == 0);
    const CandSrc src = cand_source(residual, stride, m, k, w, producer_hist, false, thr_state);
    if (entries != 0) {
#define GTOPK_SELECT(E) hipLaunchKernelGGL(k_small_select<E>, dim3(P, row_shares(m, k, P)), dim3(kSmallBlock), 0, st, src, k, \
                                           out_idx, out_val, w.sel.T, w.sel.list_cnt)
        if (entries == 4) GTOPK_SELECT(4);
        else if (entries == 8) GTOPK_SELECT(8);
        else GTOPK_SELECT(16);
#undef GTOPK_SELECT
    } else if (run_groups(m, k)) {
        // (the histogram kernel always runs, here and below: where the pass has counted its candidates it serves
        // only the workers that came back with fewer than k of them)
        RunSrc rs;
        static_cast<CandSrc&>(rs) = src;
        // k_bucket: every wave of a block takes a run; k_emit: a block per run; a worker on its
        // dense row uses the blocks there are
        SelGrid gr = local_grid(w, P);
        const uint32_t rb = ceil_div(w.nchunks, kBlock / kWave);
        if (gr.walk_blocks < rb) gr.walk_blocks = rb;
        if (gr.groups < w.nchunks) gr.groups = w.nchunks;
        run_select<RunSrc, false>(rs, w.sel, gr, k, out_idx, out_val, (int64_t)k, 1.0f, nullptr, st);
    } else {
        run_select<CandSrc, false>(src, w.sel, local_grid(w, P), k, out_idx, out_val, (int64_t)k, 1.0f,
                                   nullptr, st);
    }
    // a kernel of its own: while the select runs, a dense row may still be read as a whole
    if (zero_rows)
        hipLaunchKernelGGL(k_zero_selected, dim3(ceil_div(k, kBlock), P), dim3(kBlock), 0, st, out_idx,
                           k, residual, stride);
    return launch_status();
}

// Sample of a union for its speculative threshold: 256 tiles of 64 positions of either
// operand.  Every slot of the union is sampled with probability f = sampled / k, so the
// k-th key of the union has expected sample rank `sampled`; the target adds 5.5 standard
// deviations and 3 % for the tiles' placement error, as for a row (plan_sample).
struct MergeSamplePlan { uint32_t tile_stride, n_tiles, target, blocks; };
inline MergeSamplePlan plan_merge_sample(uint32_t k) {
    MergeSamplePlan p;
    const uint32_t want_tiles = 256;
    p.tile_stride = k / want_tiles;                          // k > 2^19: at least 2048
    if (p.tile_stride < (uint32_t)kSampleTile) p.tile_stride = kSampleTile;
    p.n_tiles = ceil_div(k, p.tile_stride);
    const uint64_t last = (uint64_t)k - (uint64_t)(p.n_tiles - 1) * p.tile_stride;
    const double sampled = (double)(p.n_tiles - 1) * kSampleTile + (double)(last < (uint64_t)kSampleTile ? last : kSampleTile);
    double t = 1.03 * sampled + 5.5 * __builtin_sqrt(sampled) + 2.0;
    if (t > 2.0 * sampled) t = 2.0 * sampled;
    p.target = (uint32_t)t;
    p.blocks = ceil_div(p.n_tiles, kSampleBlock / kSampleTile);
    if (p.blocks > 16) p.blocks = 16;
    if (p.blocks < 1) p.blocks = 1;
    return p;
}

// Lanes per cut point by the number of cut points of the launch (see k_union_cuts).  Measured
// for sets of 1.9 M and 6.4 M entries, in us for (25 k, 12.5 k, 6.2 k, 3.1 k, 1.6 k) and
// (7.3 k, 3.6 k, 1.8 k, 0.9 k, 0.45 k) cut points:
//    2 lanes: 35 31 24 21 14 | 26 22 18 13 16      4 lanes: 41 22 16 13  9 | 17 13 11  8  7
//   16 lanes: 79 40 20 10  7 | 21 10  8  6  5     64 lanes: 131 73 36 18 9 | 41 19 11  6  5
inline void launch_union_cuts(const uint32_t* a_idx, const uint32_t* b_idx, uint32_t k, int64_t in_stride,
                              uint32_t tile, uint32_t ntiles, uint32_t batch, uint32_t* cuts, hipStream_t st) {
    const uint64_t total = (uint64_t)(ntiles + 1) * batch;
    const uint32_t L = total > 20000 ? 2u : (total > 5000 ? 4u : 16u);
    const dim3 grid(ceil_div((ntiles + 1) * L, kBlock), batch);
    if (L == 2)
        hipLaunchKernelGGL(k_union_cuts<2>, grid, dim3(kBlock), 0, st, a_idx, b_idx, k, in_stride, tile, ntiles, cuts);
    else if (L == 4)
        hipLaunchKernelGGL(k_union_cuts<4>, grid, dim3(kBlock), 0, st, a_idx, b_idx, k, in_stride, tile, ntiles, cuts);
    else
        hipLaunchKernelGGL(k_union_cuts<16>, grid, dim3(kBlock), 0, st, a_idx, b_idx, k, in_stride, tile, ntiles, cuts);
}

// Sets that one block merges (k_merge_block).  A call in us, three kernels a round / this, tree of 8 sets and merge of 4 | 16 pairs:
//   k = 300   53.4 / 26.3   20.3 / 9.3 | 20.8 / 9.4     k = 4096  60.8 / 41.0   22.2 / 14.2 | 25.0 / 14.3
//   k = 1000  58.7 / 27.9   21.8 / 9.7 | 21.9 / 9.9     k = 6000  61.2 / 57.3   22.6 / 19.4 | 27.5 / 19.7
//   k = 2000  59.1 / 32.0   22.1 / 11.1 | 22.9 / 11.3   k = 8192  62.2 / 61.0   23.3 / 20.8 | 29.5 / 20.9
// Longer ones, with 32 slots per thread, lose: k = 12,000 63.0 / 102, 24.6 / 34.3 | 33.5 / 34.5.
// More pairs gain more: k = 1000 256 | 4096 pairs  34.7 / 9.9 | 227 / 64.1   k = 8192 64 | 1024 pairs  80.3 / 31.6 | 358 / 99.1.
// Sets of one magnitude, whose keys all fall into one bin, take longer either way: k = 1000, 1 pair  30.6 / 13.9   k = 8192, 1 | 16
// pairs 63.5 / 57.3 | 103 / 57.4.  The one slower kind found: trees of sets that lie behind one another, 8 of 6000 |
// 8192 entries 58 / 60 | 59 / 67.
inline bool merge_in_block(uint32_t k) { return k <= kMergeBlockMaxK; }
template <bool DIVIDE>
void launch_merge_block(const uint32_t* a_idx, const float* a_val, const uint32_t* b_idx, const float* b_val, uint32_t k,
                        uint32_t batch, int64_t in_stride, uint32_t* out_idx, float* out_val, int64_t out_stride,
                        const uint32_t* in_min, bool in_min_inverted, uint32_t* out_min, float divisor, uint32_t* gbits,
                        hipStream_t st) {
#define GTOPK_MERGE_BLOCK(EPT)                                                                                          \
    hipLaunchKernelGGL((k_merge_block<EPT, DIVIDE>), dim3(batch), dim3(kMbBlock), 0, st, a_idx, a_val, b_idx, \
                       b_val, k, in_stride, out_idx, out_val, out_stride, in_min, in_min_inverted, out_min, divisor, gbits)
    if (k <= 1024) GTOPK_MERGE_BLOCK(2);
    else if (k <= 2048) GTOPK_MERGE_BLOCK(4);
    else if (k <= 4096) GTOPK_MERGE_BLOCK(8);
    else GTOPK_MERGE_BLOCK(16);
#undef GTOPK_MERGE_BLOCK
}

// one batch of merges: union + exact select + ordered emit.  `round` picks which of the
// two select states is used (it must be clear on entry); the other one is cleared on the
// side for the next round.
template <bool DIVIDE>
void do_merge_batch(const uint32_t* a_idx, const float* a_val, const uint32_t* b_idx,
                    const float* b_val, uint32_t k, uint32_t batch, int64_t in_stride,
                    uint32_t* out_idx, float* out_val, int64_t out_stride, const MergeWs& w,
                    int round, const uint32_t* in_min, bool in_min_inverted, uint32_t* out_min,
                    float divisor, uint32_t* gbits, hipStream_t st) {
    if (merge_in_block(k)) {
        launch_merge_block<DIVIDE>(a_idx, a_val, b_idx, b_val, k, batch, in_stride, out_idx, out_val, out_stride, in_min,
                                   in_min_inverted, out_min, divisor, gbits, st);
        return;
    }
    const bool odd = (round & 1) != 0;
    uint32_t* zp = odd ? w.sel.hist : w.sel_alt.hist;
    const uint32_t zw = (uint32_t)(odd ? select_clear_words(w.sel) : w.alt_clear_words);
    // w.L is the smallest group the workspace was sized for; a batch of many pairs takes larger ones
    uint32_t L = group_slots_for(2ull * k, groups_for(batch), kMergeMinSlots);
    if (L > 8192u) L = 8192u;
    if (L < w.L) L = w.L;
    const uint32_t groups = ceil_div(2ull * k, L);
    MergedSrc src{w.m_idx, w.m_val, 2 * k, w.m_stride, L, in_min, in_min_inverted};
    SelState ss = odd ? w.sel_alt : w.sel;
    ss.T_out = out_min;
    // The union runs in blocks as large as the histogram kernel's and counts the first digits
    // of the keys it produces, so the select below starts at its second kernel.
    // small sets: one entry of either operand per thread (latency); large sets, or many: cut by
    // output position, eight slots per thread (throughput), see union_by_path; for the
    // largest the blocks' cut points come from a kernel of their own
    if (!union_by_path(k, batch))
        hipLaunchKernelGGL((k_union<1, kUnionHistBlock, true>), dim3(ceil_div(k, kUnionHistBlock), batch),
                           dim3(kUnionHistBlock), 0, st, a_idx, a_val, b_idx, b_val, k, in_stride, w.m_idx,
                           w.m_val, w.m_stride, zp, zw, src, ss);
    else if (k <= kUnionCutsMinK)
        hipLaunchKernelGGL((k_union_path<kUnionPathEpt, false, kUnionHistBlock, true>),
                           dim3(ceil_div(2 * k, kUnionHistBlock * kUnionPathEpt), batch),
                           dim3(kUnionHistBlock), 0, st, a_idx, a_val, b_idx, b_val, k, in_stride, w.m_idx,
                           w.m_val, w.m_stride, (const uint32_t*)nullptr, zp, zw, src, ss);
    else if (!w.f_samp_hist) {
        const uint32_t tile = kUnionHistBlock * kUnionPathEpt, ntiles = ceil_div(2 * k, tile);
        launch_union_cuts(a_idx, b_idx, k, in_stride, tile, ntiles, batch, w.cuts, st);
        hipLaunchKernelGGL((k_union_path<kUnionPathEpt, true, kUnionHistBlock, true>), dim3(ntiles, batch),
                           dim3(kUnionHistBlock), 0, st, a_idx, a_val, b_idx, b_val, k, in_stride, w.m_idx,
                           w.m_val, w.m_stride, (const uint32_t*)w.cuts, zp, zw, src, ss);
    } else {
        // The largest sets.  A sample of the union gives a threshold that a little more than k
        // of its slots are expected to reach; the union keeps only those, tile by tile, and the
        // select works on what is left (FiltSrc).  A pair whose union kept fewer than k slots is
        // then merged and selected once more, from its complete union; for every other pair
        // those launches return at once.
        const uint32_t tile = kUnionHistBlock * kUnionPathEpt, ntiles = ceil_div(2 * k, tile);
        zero_async(st, zero_job(w.f_samp_hist, w.f_clear_words, w.sel_rep.hist, w.rep_clear_words));
        const MergeSamplePlan mp = plan_merge_sample(k);
        hipLaunchKernelGGL(k_merge_sample, dim3(mp.blocks, batch), dim3(kSampleBlock), 0, st, a_idx, a_val,
                           b_idx, b_val, k, in_stride, mp.tile_stride, mp.n_tiles, w.f_samp_hist);
        hipLaunchKernelGGL(k_sample_pick<false>, dim3(batch), dim3(kSampleBlock), 0, st,
                           (const uint32_t*)w.f_samp_hist, mp.target, 0xFFFFFFFFu, w.f_tspec, (const uint4*)nullptr,
                           0u, (uint32_t*)nullptr);
        launch_union_cuts(a_idx, b_idx, k, in_stride, tile, ntiles, batch, w.cuts, st);
        hipLaunchKernelGGL((k_union_path<kUnionPathEpt, true, kUnionHistBlock, true, true>), dim3(ntiles, batch),
                           dim3(kUnionHistBlock), 0, st, a_idx, a_val, b_idx, b_val, k, in_stride, w.m_idx,
                           w.m_val, w.m_stride, (const uint32_t*)w.cuts, zp, zw, src, ss,
                           UnionFilter{w.f_tspec, w.f_tile_cnt, w.f_set_cnt}, (const uint32_t*)nullptr);
        static_assert(kUnionHistBlock * kUnionPathEpt == 8192, "FiltSrc's tiles are the union's: 2^13 slots");
        const FiltSrc fs{w.m_idx, w.m_val, k, w.m_stride, 13u, ntiles, w.f_tile_cnt, w.f_set_cnt, w.f_tspec};
        run_select<FiltSrc, DIVIDE>(fs, ss, SelGrid{batch, ntiles, ntiles, 2ull * k, true}, k, out_idx, out_val,
                                    out_stride, divisor, gbits, st, /*with_hist=*/false);
        // the pairs that came out short
        MergedSrc rsrc = src;
        rsrc.gate_cnt = w.f_set_cnt;
        rsrc.gate_k = k;
        SelState rs = w.sel_rep;
        rs.T_out = out_min;
        hipLaunchKernelGGL((k_union_path<kUnionPathEpt, true, kUnionHistBlock, true>), dim3(ntiles, batch),
                           dim3(kUnionHistBlock), 0, st, a_idx, a_val, b_idx, b_val, k, in_stride, w.m_idx,
                           w.m_val, w.m_stride, (const uint32_t*)w.cuts, (uint32_t*)nullptr, 0u, rsrc, rs,
                           UnionFilter{nullptr, nullptr, nullptr}, (const uint32_t*)w.f_set_cnt);
        run_select<MergedSrc, DIVIDE>(rsrc, rs, SelGrid{batch, groups, groups, 2ull * k, true}, k, out_idx,
                                      out_val, out_stride, divisor, gbits, st, /*with_hist=*/false);
        return;
    }
    run_select<MergedSrc, DIVIDE>(src, ss, SelGrid{batch, groups, groups, 2ull * k, 2ull * k > kInlineFinishMax},
                                  k, out_idx, out_val, out_stride, divisor, gbits, st,
                                  /*with_hist=*/false);
}

// loc_min: the smallest key of each of the P input sets (the local selection's T), or NULL
// when the caller supplied the sets
int do_tree(const uint32_t* loc_idx, const float* loc_val, const uint32_t* loc_min, uint32_t P,
            uint32_t k, uint32_t* g_idx, float* g_val, const StepWs& w, uint32_t* gbits,
            bool pre_cleared, hipStream_t st) {
    const float divisor = (float)P;
    if (P == 1) {
        hipLaunchKernelGGL(k_copy_set, dim3(ceil_div(k, 256)), dim3(256), 0, st, loc_idx, loc_val, k,
                           g_idx, g_val, divisor, gbits);
        return launch_status();
    }
    ZeroJob job = zero_job();
    if (!pre_cleared && !merge_in_block(k))
        job = zero_job(w.mrg.sel.hist, select_clear_words(w.mrg.sel), w.mrg.sel_alt.hist, w.mrg.alt_clear_words);
    bool inverted = false;
    if (loc_min) {
        zero_async(st, job);
    } else if (!merge_in_block(k)) {
        // sets from the caller: find their smallest keys, the first round's lower bounds
        find_min_keys(loc_val, nullptr, (int64_t)k, k, P, w.mrg.inv_min, job, st);
        loc_min = w.mrg.inv_min;
        inverted = true;
    }
    // After every round the surviving sets are stored compactly, so round j always
    // merges set 2p with set 2p+1 of its input: exactly worker p*2^(j+1) with worker
    // p*2^(j+1) + 2^j of the original numbering.
    const uint32_t* in_idx = loc_idx;
    const float* in_val = loc_val;
    uint32_t* ping_i = w.x_idx; float* ping_v = w.x_val;
    uint32_t* pong_i = w.y_idx; float* pong_v = w.y_val;
    const uint32_t* in_min = loc_min;
    int round = 0;
    for (uint32_t pairs = P / 2; pairs >= 1; pairs /= 2, ++round) {
        const bool last = pairs == 1;
        uint32_t* out_min = w.mrg.tmin[round & 1];
        if (last) {
            do_merge_batch<true>(in_idx, in_val, in_idx + k, in_val + k, k, 1, 2 * (int64_t)k, g_idx,
                                 g_val, k, w.mrg, round, in_min, inverted, out_min, divisor, gbits,
                                 st);
        } else {
            do_merge_batch<false>(in_idx, in_val, in_idx + k, in_val + k, k, pairs, 2 * (int64_t)k,
                                  ping_i, ping_v, k, w.mrg, round, in_min, inverted, out_min, 1.0f,
                                  nullptr, st);
            in_min = out_min;
            inverted = false;
            in_idx = ping_i; in_val = ping_v;
            uint32_t* ti = ping_i; ping_i = pong_i; pong_i = ti;
            float* tv = ping_v; ping_v = pong_v; pong_v = tv;
        }
    }
    return launch_status();
}

// gtopk_step at large densities.
int do_grouped_step(const float* grad, float* residual, int64_t m, int64_t stride, uint32_t P, uint32_t k, uint32_t* g_idx,
                    float* g_val, uint32_t* loc_idx, float* loc_val, const StepWs& w, hipStream_t st, void* const* events) {
    const GroupWs gw = carve_grouped(w, m, k, P);
    const GroupSets& gs = gw.gs;
    const uint32_t ng = gs.ngroups;
    const SamplePlan sp = plan_row_sample(m, k, P);
    sample_rows<true, true>(grad, residual, m, stride, P, k, w, sp,
                      zero_job(w.samp_hist, w.samp_words, w.cand_count, (size_t)P, gs.hist, gw.clear_words), gs.lo, gs.hi, gw.samples, st);
    mark_stage(1, events, st);
    hipLaunchKernelGGL(k_group_pass, dim3(ceil_div((uint64_t)m + 3, kGrpPassChunk), P), dim3(kSBlock), 0, st, grad, residual, stride,
                       gs, w.cand_val, w.cap, w.cand_count);
    mark_stage(2, events, st);

    const uint32_t walk_blocks = 1 + ceil_div(ng, kGrpWalkBlock / kWave * kGrpWalkRuns);
    auto finish = [&](const GroupBatch& gb, uint32_t sets, uint32_t samples, double fraction) {
        const double mean = (double)k * fraction;            // expected sample rank of the k-th key of a union
        const GroupSample sm{gb.first + sets, sets / 2, gw.samples, samples,
                             union_bracket_target_lo(mean), union_bracket_target_hi(mean)};
        hipLaunchKernelGGL(k_group_walk, dim3(walk_blocks, sets), dim3(kGrpWalkBlock), 0, st, gs, gb, sm);
        // blocks for the sets that miss their brackets: a wave per group, one block per CU (the others' return)
        uint32_t shares = sets >= 32 ? 8u : (sets <= 4 ? 64u : 256u / sets);
        const uint32_t most = ceil_div(ng, kGrpFinishBlock / kWave);
        if (shares > most) shares = most;
        hipLaunchKernelGGL(k_group_finish, dim3(sets, shares), dim3(kGrpFinishBlock), 0, st, gs, gb);
    };
    GroupBatch gb{0u, k, reinterpret_cast<const uint32_t*>(w.cand_val), w.cap, w.sel.list, w.cap, w.cap, residual, stride,
                  nullptr, nullptr, 0u};
    // (of the rows' sample every fourth element of a tile of 64, every one of a tile of 16)
    finish(gb, P, gw.row_samples, (double)sp.sampled / (double)m / (mid_problem(m, k, P) ? 1.0 : (double)(kSampleTile / kSampleKept)));
    GroupNext nx{P, w.mrg.m_val, w.mrg.m_stride, P > 2 ? gw.samples : nullptr, gw.per_group};
    hipLaunchKernelGGL(k_group_select, dim3(ng, P / 2), dim3(kGrpBlock), 0, st, gs, nx, residual, stride, k, loc_idx, loc_val,
                       gw.bits);
    mark_stage(3, events, st);

    const uint32_t* in_idx = loc_idx;
    const float* in_val = loc_val;
    uint32_t first_in = 0;
    uint32_t* ping_i = w.x_idx; float* ping_v = w.x_val;
    uint32_t* pong_i = w.y_idx; float* pong_v = w.y_val;
    for (uint32_t pairs = P / 2; pairs >= 1; pairs /= 2) {
        const uint32_t first = first_in + 2 * pairs;
        gb = GroupBatch{first, k, reinterpret_cast<const uint32_t*>(w.mrg.m_val), w.mrg.m_stride, w.mrg.sel.list, 2 * k, 0u,
                        nullptr, 0, in_idx, in_val, first_in};
        finish(gb, pairs, ng * gw.per_group, (double)gw.per_group / (double)kGroup);
        if (pairs == 1) {
            hipLaunchKernelGGL(k_group_merge<1>, dim3(ng, 1), dim3(kGrpBlock), 0, st, gs, nx, first, first_in, in_idx, in_val, k,
                               g_idx, g_val, (float)P, gw.gbits);
        } else {
            nx = GroupNext{first + pairs, w.mrg.m_val, w.mrg.m_stride, pairs > 2 ? gw.samples : nullptr, gw.per_group};
            hipLaunchKernelGGL(k_group_merge<2>, dim3(ng, pairs / 2), dim3(kGrpBlock), 0, st, gs, nx, first, first_in, in_idx,
                               in_val, k, ping_i, ping_v, 1.0f, (uint64_t*)nullptr);
        }
        first_in = first;
        in_idx = ping_i; in_val = ping_v;
        uint32_t* ti = ping_i; ping_i = pong_i; pong_i = ti;
        float* tv = ping_v; ping_v = pong_v; pong_v = tv;
    }
    mark_stage(4, events, st);
    hipLaunchKernelGGL(k_group_restore, dim3(ceil_div(ng * kGroupWords, kRestoreWords * (kBlock / kWave)), P), dim3(kBlock), 0, st, residual, stride, gs, gw.bits, gw.gbits);
    const int rc = launch_status();
    mark_stage(5, events, st);
    return rc;
}

}  // namespace

extern "C" {

const char* gtopk_status_string(int status) {
    switch (status) {
        case GTOPK_OK: return "GTOPK_OK";
        case GTOPK_EINVAL: return "GTOPK_EINVAL: invalid argument";
        case GTOPK_EWORKSPACE: return "GTOPK_EWORKSPACE: workspace too small";
        case GTOPK_EALIGN: return "GTOPK_EALIGN: pointer not 16-byte aligned";
        case GTOPK_EHIP: return "GTOPK_EHIP: kernel launch failed";
        default: return "GTOPK: unknown status";
    }
}

size_t gtopk_workspace_bytes(int64_t m, int32_t k, int32_t P) {
    if (!sizes_ok(m, k, P)) return 0;
    return carve_step(nullptr, m, (uint32_t)k, (uint32_t)P).bytes;
}

size_t gtopk_merge_workspace_bytes(int32_t k, int32_t batch) {
    if (k < 1 || k > kMaxMergeK || batch < 1 || batch > 32767) return 0;
    Carver c{nullptr};
    return carve_merge(c, (uint32_t)k, (size_t)batch).bytes;
}

int gtopk_local_select(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P,
                       int32_t k, uint32_t* out_idx, float* out_val, void* ws, size_t ws_bytes,
                       void* stream) {
    if (!grad || !residual || !out_idx || !out_val || !ws) return GTOPK_EINVAL;
    if (!sizes_ok(m, k, P) || stride < m) return GTOPK_EINVAL;
    if (!aligned16(grad) || !aligned16(residual) || !aligned16(out_idx) || !aligned16(out_val) ||
        !aligned16(ws))
        return GTOPK_EALIGN;
    const StepWs w = carve_step(ws, m, (uint32_t)k, (uint32_t)P);
    if (ws_bytes < w.bytes) return GTOPK_EWORKSPACE;
    const ZeroJob sel = local_clear(w, m, (uint32_t)k, (uint32_t)P);
    return do_local_select(grad, residual, m, stride, (uint32_t)P, (uint32_t)k, out_idx, out_val, w, true,
                           zero_job(w.samp_hist, w.samp_words, w.cand_count, (size_t)P, sel.p[0], sel.n[0]), (hipStream_t)stream);
}

int gtopk_merge(const uint32_t* a_idx, const float* a_val, const uint32_t* b_idx, const float* b_val,
                int32_t k, int32_t batch, int64_t in_stride, uint32_t* out_idx, float* out_val,
                int64_t out_stride, void* ws, size_t ws_bytes, void* stream) {
    if (!a_idx || !a_val || !b_idx || !b_val || !out_idx || !out_val || !ws) return GTOPK_EINVAL;
    if (k < 1 || k > kMaxMergeK || batch < 1 || batch > 32767 || in_stride < k || out_stride < k)
        return GTOPK_EINVAL;
    if (!aligned16(a_idx) || !aligned16(a_val) || !aligned16(b_idx) || !aligned16(b_val) ||
        !aligned16(out_idx) || !aligned16(out_val) || !aligned16(ws))
        return GTOPK_EALIGN;
    Carver c{reinterpret_cast<char*>(ws)};
    const MergeWs w = carve_merge(c, (uint32_t)k, (size_t)batch);
    if (ws_bytes < w.bytes) return GTOPK_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t* in_min = merge_in_block((uint32_t)k) ? nullptr : w.inv_min;
    if (in_min)
        find_min_keys(a_val, b_val, in_stride, (uint32_t)k, 2 * (uint32_t)batch, w.inv_min,
                      zero_job(w.sel.hist, select_clear_words(w.sel)), st);
    do_merge_batch<false>(a_idx, a_val, b_idx, b_val, (uint32_t)k, (uint32_t)batch, in_stride,
                          out_idx, out_val, out_stride, w, 0, in_min, true, nullptr, 1.0f, nullptr,
                          st);
    return launch_status();
}

int gtopk_tree(const uint32_t* loc_idx, const float* loc_val, int32_t P, int32_t k, uint32_t* g_idx,
               float* g_val, void* ws, size_t ws_bytes, void* stream) {
    if (!loc_idx || !loc_val || !g_idx || !g_val || !ws) return GTOPK_EINVAL;
    if (k < 1 || k > kMaxMergeK || !is_pow2(P) || P > 65535) return GTOPK_EINVAL;
    if (!aligned16(loc_idx) || !aligned16(loc_val) || !aligned16(g_idx) || !aligned16(g_val) ||
        !aligned16(ws))
        return GTOPK_EALIGN;
    // the tree's scratch sits inside the step workspace; m only sizes the parts it does not use
    const StepWs w = carve_step(ws, (int64_t)k, (uint32_t)k, (uint32_t)P);
    if (ws_bytes < w.bytes) return GTOPK_EWORKSPACE;
    return do_tree(loc_idx, loc_val, nullptr, (uint32_t)P, (uint32_t)k, g_idx, g_val, w, nullptr,
                   false, (hipStream_t)stream);
}

int gtopk_residual_restore(float* residual, int64_t m, int64_t stride, int32_t P, int32_t k,
                           const uint32_t* loc_idx, const float* loc_val, const uint32_t* g_idx,
                           void* stream) {
    if (!residual || !loc_idx || !loc_val || !g_idx) return GTOPK_EINVAL;
    if (!sizes_ok(m, k, P) || stride < m) return GTOPK_EINVAL;
    if (!aligned16(residual) || !aligned16(loc_idx) || !aligned16(loc_val) || !aligned16(g_idx))
        return GTOPK_EALIGN;
    hipLaunchKernelGGL(k_restore, dim3(ceil_div((uint32_t)k, kBlock), (uint32_t)P), dim3(kBlock), 0,
                       (hipStream_t)stream, residual, (uint32_t)m, stride, (uint32_t)k, loc_idx, loc_val,
                       g_idx);
    return launch_status();
}

static int step_impl(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P,
                     int32_t k, uint32_t* g_idx, float* g_val, uint32_t* loc_idx, float* loc_val,
                     void* ws, size_t ws_bytes, void* stream, void* const* events,
                     uint32_t* thr_state = nullptr) {
    if (!grad || !residual || !g_idx || !g_val || !ws) return GTOPK_EINVAL;
    if (!aligned16(thr_state)) return GTOPK_EALIGN;
    if ((loc_idx == nullptr) != (loc_val == nullptr)) return GTOPK_EINVAL;
    if (!sizes_ok(m, k, P) || stride < m) return GTOPK_EINVAL;
    if (!aligned16(grad) || !aligned16(residual) || !aligned16(g_idx) || !aligned16(g_val) ||
        !aligned16(loc_idx) || !aligned16(loc_val) || !aligned16(ws))
        return GTOPK_EALIGN;
    const StepWs w = carve_step(ws, m, (uint32_t)k, (uint32_t)P);
    if (ws_bytes < w.bytes) return GTOPK_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    uint32_t* li = loc_idx ? loc_idx : w.loc_idx;
    float* lv = loc_val ? loc_val : w.loc_val;
    if (!events && !thr_state && small_problem(m, k, P)) {
        // one block per worker samples, picks the threshold and clears the candidate counter
        const SamplePlan sp = plan_sample(m, (uint32_t)k, kSampleTile, kSmallSampleMean, kSmallSampleMin);
        hipLaunchKernelGGL((k_small_sample<kSampleTile, false, true>), dim3(P), dim3(kSmallBlock), 0, st, grad, residual,
                           (uint32_t)m, stride, (uint32_t)P, sp.tile_stride, sp.n_tiles, sp.target, 0xFFFFFFFFu,
                           w.tspec, w.cand_count, (const uint4*)nullptr, ZeroJob{});
        // small blocks: one run per 4096 elements (the run table was carved for that many)
        const uint32_t nruns = ceil_div((uint64_t)m + 3, kSmallChunk);
        hipLaunchKernelGGL((k_accum_filter<false, kSmallIters>), dim3(nruns, P), dim3(kSBlock), 0, st,
                           grad, residual, (uint32_t)m, stride, w.tspec, w.cand_idx, w.cand_val, w.cap,
                           w.cand_count, w.run_table, nruns, w.sel.hist, (uint32_t*)nullptr);
        CandSrc src = cand_source(residual, stride, m, (uint32_t)k, w, false, false);
        src.nchunks = nruns;
        hipLaunchKernelGGL(k_small_select<kSmallEntries>, dim3(P), dim3(kSmallBlock), 0, st, src, (uint32_t)k, li, lv,
                           (uint32_t*)nullptr, (uint32_t*)nullptr);
        // (see tree_round_by_waves; longer sets take the teams of threads)
#define GTOPK_TREE(E) hipLaunchKernelGGL(k_small_tree<E>, dim3(1), dim3(kSmallBlock), 0, st, li, lv, (uint32_t)P, (uint32_t)k, \
                                         g_idx, g_val, (float)P, residual, stride)
        if (k <= 32) GTOPK_TREE(1);
        else if (k <= 64) GTOPK_TREE(2);
        else if (k <= 128) GTOPK_TREE(4);
        else GTOPK_TREE(0);
#undef GTOPK_TREE
        return launch_status();
    }
    mark_stage(0, events, st);
    if (!thr_state && grouped_step(m, (uint32_t)k, (uint32_t)P, w))
        return do_grouped_step(grad, residual, m, stride, (uint32_t)P, (uint32_t)k, g_idx, g_val, li, lv, w, st, events);
    // one clear for everything this step needs zeroed: the sampler's histograms and the
    // candidate counters; both selects' histograms and tickets; the global-set bitmap
    const bool in_block = merge_in_block((uint32_t)k);       // its rounds need no select state
    const ZeroJob sel = local_clear(w, m, (uint32_t)k, (uint32_t)P);
    const ZeroJob job = zero_job(w.samp_hist, w.samp_words, w.cand_count, (size_t)P, sel.p[0], sel.n[0],
                                 w.mrg.sel.hist, in_block ? 0 : select_clear_words(w.mrg.sel),
                                 w.mrg.sel_alt.hist, in_block ? 0 : w.mrg.alt_clear_words, w.gbits, w.gbits_words);
    int rc = do_local_select(grad, residual, m, stride, (uint32_t)P, (uint32_t)k, li, lv, w, false,
                             job, st, events, thr_state);
    if (rc != GTOPK_OK) return rc;
    mark_stage(3, events, st);
    rc = do_tree(li, lv, w.sel.T, (uint32_t)P, (uint32_t)k, g_idx, g_val, w, w.gbits, true, st);
    if (rc != GTOPK_OK) return rc;
    mark_stage(4, events, st);
    hipLaunchKernelGGL(k_restore_fused, dim3(ceil_div((uint32_t)k, kBlock), (uint32_t)P), dim3(kBlock),
                       0, st, residual, stride, (uint32_t)k, li, lv, w.gbits, (const uint32_t*)w.sel.T);
    rc = launch_status();
    mark_stage(5, events, st);
    return rc;
}

int gtopk_step(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P, int32_t k,
               uint32_t* g_idx, float* g_val, uint32_t* loc_idx, float* loc_val, void* ws,
               size_t ws_bytes, void* stream) {
    return step_impl(grad, residual, m, stride, P, k, g_idx, g_val, loc_idx, loc_val, ws, ws_bytes,
                     stream, nullptr);
}

// ---------------------------------------------------------------------------------
// gtopk_step for callers that cannot allocate: the workspace is a file-scope device array
// ---------------------------------------------------------------------------------
}  // extern "C"

// Every GPU the library runs on holds its own copy of this array until the process ends.
// In host code the name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[GTOPK_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};     // device address of `scratch` on each device, once known

// device address of `scratch` on the current device (looked up once per device), or NULL
void* scratch_on_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

extern "C" {

int gtopk_step_static(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P,
                      int32_t k, uint32_t* g_idx, float* g_val, uint32_t* loc_idx, float* loc_val,
                      void* stream) {
    if (!sizes_ok(m, k, P)) return GTOPK_EINVAL;
    const size_t need = carve_step(nullptr, m, (uint32_t)k, (uint32_t)P).bytes;
    if (need > (size_t)GTOPK_STATIC_WORKSPACE_BYTES) return GTOPK_EWORKSPACE;
    void* ws = scratch_on_current_device();
    if (!ws) return GTOPK_EHIP;
    // everything the step needs zeroed is cleared by its first kernel, so what the
    // previous call left in the array does not matter
    return step_impl(grad, residual, m, stride, P, k, g_idx, g_val, loc_idx, loc_val, ws,
                     (size_t)GTOPK_STATIC_WORKSPACE_BYTES, stream, nullptr);
}

int gtopk_step_carry(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P,
                     int32_t k, uint32_t* g_idx, float* g_val, uint32_t* loc_idx, float* loc_val,
                     uint32_t* thr_state, void* ws, size_t ws_bytes, void* stream) {
    if (!thr_state) return GTOPK_EINVAL;
    return step_impl(grad, residual, m, stride, P, k, g_idx, g_val, loc_idx, loc_val, ws, ws_bytes,
                     stream, nullptr, thr_state);
}

int gtopk_step_timed(const float* grad, float* residual, int64_t m, int64_t stride, int32_t P,
                     int32_t k, uint32_t* g_idx, float* g_val, uint32_t* loc_idx, float* loc_val,
                     uint32_t* thr_state, void* ws, size_t ws_bytes, void* stream,
                     void* const* events) {
    if (!events) return GTOPK_EINVAL;
    for (int i = 0; i < GTOPK_STAGE_EVENTS; ++i)
        if (!events[i]) return GTOPK_EINVAL;
    return step_impl(grad, residual, m, stride, P, k, g_idx, g_val, loc_idx, loc_val, ws, ws_bytes,
                     stream, events, thr_state);
}

int gtopk_apply_update(float* weights, int64_t m, int64_t stride, int32_t copies, int32_t k,
                       const uint32_t* g_idx, const float* g_val, float lr, void* stream) {
    if (!weights || !g_idx || !g_val) return GTOPK_EINVAL;
    if (m < 1 || m > ((int64_t)1 << 31) || k < 1 || k > m || stride < m || copies < 1 ||
        copies > 65535)
        return GTOPK_EINVAL;
    if (!aligned16(weights) || !aligned16(g_idx) || !aligned16(g_val)) return GTOPK_EALIGN;
    hipLaunchKernelGGL(k_apply_update, dim3(ceil_div((uint32_t)k, kBlock), (uint32_t)copies),
                       dim3(kBlock), 0, (hipStream_t)stream, weights, (uint32_t)m, stride, (uint32_t)k, g_idx,
                       g_val, lr);
    return launch_status();
}

int gtopk_dense_mask(const uint32_t* g_idx, int32_t k, int64_t m, uint8_t* mask, void* stream) {
    if (!g_idx || !mask) return GTOPK_EINVAL;
    if (m < 1 || m > ((int64_t)1 << 31) || k < 1 || k > m) return GTOPK_EINVAL;
    if (!aligned16(g_idx) || !aligned16(mask)) return GTOPK_EALIGN;
    hipStream_t st = (hipStream_t)stream;
    uint32_t blocks = ceil_div((uint64_t)m, 256 * 16);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_mask_clear, dim3(blocks), dim3(256), 0, st, mask, (uint64_t)m);
    hipLaunchKernelGGL(k_mask_set, dim3(ceil_div((uint32_t)k, kBlock)), dim3(kBlock), 0, st, mask,
                       (uint32_t)m, (uint32_t)k, g_idx);
    return launch_status();
}

size_t gtopk_allreduce_workspace_bytes(int64_t m, int32_t P) {
    if (m < 1 || m > ((int64_t)1 << 31) || P < 1 || P > kAggMaxP) return 0;
    const uint64_t nranges = ceil_div((uint64_t)m, kAggRange);
    return (size_t)(((uint64_t)P * (nranges + 1) * sizeof(uint32_t) + 255) & ~(uint64_t)255);
}

int gtopk_topk_allreduce(const uint32_t* loc_idx, const float* loc_val, int32_t P, int32_t k,
                         int64_t m, float* dense, void* ws, size_t ws_bytes, void* stream) {
    if (!loc_idx || !loc_val || !dense || !ws) return GTOPK_EINVAL;
    if (m < 1 || m > ((int64_t)1 << 31) || k < 1 || k > m || P < 1 || P > kAggMaxP)
        return GTOPK_EINVAL;
    if (!aligned16(loc_idx) || !aligned16(loc_val) || !aligned16(dense) || !aligned16(ws))
        return GTOPK_EALIGN;
    if (ws_bytes < gtopk_allreduce_workspace_bytes(m, P)) return GTOPK_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t nranges = ceil_div((uint64_t)m, kAggRange);
    uint32_t* bounds = reinterpret_cast<uint32_t*>(ws);
    hipLaunchKernelGGL(k_slice_bounds, dim3(ceil_div(nranges + 1, kBlock), (uint32_t)P), dim3(kBlock),
                       0, st, loc_idx, (uint32_t)k, nranges, bounds);
    // up to 32 workers' turns at an element fit a word
    if (P <= kFewP)
        hipLaunchKernelGGL(k_scatter_mean_few, dim3(nranges * (kAggRange / kFewRange)), dim3(kFewBlock), 0, st,
                           loc_idx, loc_val, (uint32_t)P, (uint32_t)k, (uint32_t)m, bounds, nranges, (float)P,
                           dense);
    else
        hipLaunchKernelGGL(k_scatter_mean, dim3(nranges), dim3(kBlock), 0, st, loc_idx, loc_val,
                           (uint32_t)P, (uint32_t)k, (uint32_t)m, bounds, nranges, (float)P, dense);
    return launch_status();
}

// Whether the dense top-k filters its row by a sampled threshold first, as the local selection does,
// and selects from the candidates, instead of reading the whole row in each of its three kernels (54 + 56
// + 58 us at m = 25,557,032; now sample 9 + 5, pass 22, select 27).  A call in us, three reads / filtered,
// on rows of which a tenth (the last line: all) is non-zero:
//   m = 200,001     k = 200     26.4 / 27.7     k = 4000        29.3 / 28.5
//   m = 500,000     k = 500     32.9 / 30.8     k = 30,000      37.7 / 30.8
//   m = 4,000,001   k = 4000    59.1 / 40.6     k = 240,000     68.8 / 45.0
//   m = 25,557,032  k = 25,557  180.7 / 63.6    k = 1,533,421  244.4 / 96.6
//   m = 25,557,032  k = 6.4 M   881.9 / 174.9   k = 23 M       392.4 / 361.3
// A row that its sample shows to be unfit for that (fewer than k non-zeros, masses of few magnitudes) is read three
// times, the first of them by the pass (see k_accum_filter); one whose sample misleads, on top of the pass.
static bool dense_topk_filters(int64_t m) { return m >= ((int64_t)1 << 19); }

int gtopk_dense_topk(const float* dense, int64_t m, int32_t k, uint32_t* g_idx, float* g_val,
                     void* ws, size_t ws_bytes, void* stream) {
    if (!dense || !g_idx || !g_val || !ws) return GTOPK_EINVAL;
    if (!sizes_ok(m, k, 1)) return GTOPK_EINVAL;
    if (!aligned16(dense) || !aligned16(g_idx) || !aligned16(g_val) || !aligned16(ws))
        return GTOPK_EALIGN;
    const StepWs w = carve_step(ws, m, (uint32_t)k, 1);
    if (ws_bytes < w.bytes) return GTOPK_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const ZeroJob job = zero_job(w.samp_hist, w.samp_words, w.cand_count, 1, w.sel.hist, select_clear_words(w.sel));
    const bool filter = dense_topk_filters(m);
    bool producer_hist = false;
    if (filter)
        producer_hist = filter_rows<false>(nullptr, const_cast<float*>(dense), m, m, 1, (uint32_t)k, w, job, st);
    else
        zero_async(st, job);       // a candidate count of zero makes the select read the dense row itself
    const CandSrc src = cand_source(dense, m, m, (uint32_t)k, w, producer_hist, /*no_bounds=*/!filter, nullptr,
                                    /*row_hist=*/filter);
    // one set: the grids follow the dense row's groups (a row whose sample misled is read as one);
    // without a lower bound of the k-th key the list can be long, so large rows are finished once
    const uint32_t gx = filter && w.gcand > w.gdense ? w.gcand : w.gdense;
    const SelGrid gr{1, gx, gx, (uint64_t)m, m > ((int64_t)1 << 20)};
    run_select<CandSrc, false>(src, w.sel, gr, (uint32_t)k, g_idx, g_val, (int64_t)k, 1.0f, nullptr, st);
    return launch_status();
}

int gtopk_debug_candidate_counts(const void* ws, int64_t m, int32_t k, int32_t P,
                                 uint32_t* host_counts, uint32_t* host_capacity) {
    if (!ws || !host_counts || !host_capacity || !sizes_ok(m, k, P)) return GTOPK_EINVAL;
    const StepWs w = carve_step(const_cast<void*>(ws), m, (uint32_t)k, (uint32_t)P);
    *host_capacity = w.cap;
    if (hipMemcpy(host_counts, w.cand_count, sizeof(uint32_t) * (size_t)P, hipMemcpyDeviceToHost) !=
        hipSuccess)
        return GTOPK_EHIP;
    return GTOPK_OK;
}

int gtopk_debug_merge_kept(const void* ws, int32_t k, int32_t batch, uint32_t* host_kept) {
    if (!ws || !host_kept || k < 1 || k > kMaxMergeK || batch < 1 || batch > 32767) return GTOPK_EINVAL;
    Carver c{reinterpret_cast<char*>(const_cast<void*>(ws))};
    const MergeWs w = carve_merge(c, (uint32_t)k, (size_t)batch);
    if (!w.f_set_cnt) return GTOPK_EINVAL;               // merges of this k are not filtered
    if (hipMemcpy(host_kept, w.f_set_cnt, sizeof(uint32_t) * (size_t)batch, hipMemcpyDeviceToHost) !=
        hipSuccess)
        return GTOPK_EHIP;
    return GTOPK_OK;
}

int gtopk_probe_stream(const float* a, float* b, int64_t n, int32_t mode, float* sink,
                       void* stream) {
    if (!a || !b || n < 1 || n % kChunk != 0 || n / kChunk > 0x7fffffff) return GTOPK_EINVAL;
    if (mode < 0 || mode >= GTOPK_PROBE_MODES) return GTOPK_EINVAL;
    if (mode == 1 && !sink) return GTOPK_EINVAL;
    if (!aligned16(a) || !aligned16(b) || !aligned16(sink)) return GTOPK_EALIGN;
    const uint32_t blocks = (uint32_t)(n / kChunk);      // of the pass's shape: 32768 elements each
    hipStream_t st = (hipStream_t)stream;
    switch (mode) {
        case 0: hipLaunchKernelGGL(k_probe_stream<true>, dim3(blocks), dim3(kSBlock), 0, st, a, b, sink); break;
        case 1: hipLaunchKernelGGL(k_probe_stream<false>, dim3(blocks), dim3(kSBlock), 0, st, a, b, sink); break;
        // cache policy
        case 2: hipLaunchKernelGGL((k_probe_stream<true, false, true>), dim3(blocks), dim3(kSBlock), 0, st, a, b, sink); break;
        case 3: hipLaunchKernelGGL((k_probe_stream<true, true, false>), dim3(blocks), dim3(kSBlock), 0, st, a, b, sink); break;
        case 4: hipLaunchKernelGGL((k_probe_stream<true, false, false>), dim3(blocks), dim3(kSBlock), 0, st, a, b, sink); break;
        // block shape (elements per block: 32768, 32768, 8192)
        case 5: hipLaunchKernelGGL((k_probe_stream<true, true, true, 256, 32>), dim3(blocks), dim3(256), 0, st, a, b, sink); break;
        case 6: hipLaunchKernelGGL((k_probe_stream<true, true, true, 1024, 8>), dim3(blocks), dim3(1024), 0, st, a, b, sink); break;
        default: hipLaunchKernelGGL((k_probe_stream<true, true, true, 512, 4>), dim3(blocks * 4), dim3(512), 0, st, a, b, sink); break;
    }
    return launch_status();
}

int gtopk_debug_plan(int64_t m, int32_t k, int32_t P, uint32_t* plan) {
    if (!plan || !sizes_ok(m, k, P)) return GTOPK_EINVAL;
    const SamplePlan sp = plan_row_sample(m, (uint32_t)k, (uint64_t)P);
    plan[0] = sp.tile_stride;
    plan[1] = sp.n_tiles;
    plan[2] = (uint32_t)(mid_problem(m, (uint32_t)k, (uint64_t)P) ? kMidSampleTile : kSampleTile);
    plan[3] = sp.target;
    plan[4] = cand_capacity(m, (uint32_t)k);
    const bool in_block = select_in_block(m, (uint32_t)k, (uint32_t)P) != 0;      // neither of the two next
    plan[5] = !in_block && pass_histograms(m, (uint32_t)k) ? 1u : 0u;
    plan[6] = small_problem(m, k, P) ? 1u : 0u;
    plan[7] = !in_block && run_groups(m, (uint32_t)k) ? 1u : 0u;
    for (int i = 8; i < GTOPK_PLAN_WORDS; ++i) plan[i] = 0u;
    if (P > 1 && merge_filtered((uint32_t)k)) {
        const MergeSamplePlan mp = plan_merge_sample((uint32_t)k);
        plan[11] = 1u;
        plan[12] = mp.tile_stride;
        plan[13] = mp.n_tiles;
        plan[14] = mp.target;
    }
    if (plan[6]) {
        const SamplePlan ss = plan_sample(m, (uint32_t)k, kSampleTile, kSmallSampleMean, kSmallSampleMin);
        plan[8] = ss.tile_stride;
        plan[9] = ss.n_tiles;
        plan[10] = ss.target;
    }
    plan[15] = pass_chunk_log2(m, (uint32_t)k, (uint64_t)P);
    return GTOPK_OK;
}

int gtopk_debug_routes(int64_t m, int32_t k, int32_t P, uint32_t* routes) {
    if (!routes || !sizes_ok(m, k, P)) return GTOPK_EINVAL;
    for (int i = 0; i < GTOPK_ROUTE_WORDS; ++i) routes[i] = 0u;
    routes[0] = small_problem(m, k, P) ? 1u : 0u;
    routes[2] = select_in_block(m, (uint32_t)k, (uint32_t)P);
    routes[3] = merge_in_block((uint32_t)k) ? 1u : 0u;
    const StepWs w = carve_step(nullptr, m, (uint32_t)k, (uint32_t)P);
    if (!routes[0] && grouped_step(m, (uint32_t)k, (uint32_t)P, w)) {
        const GroupWs gw = carve_grouped(w, m, (uint32_t)k, (uint32_t)P);
        const SamplePlan sp = plan_row_sample(m, (uint32_t)k, (uint64_t)P);
        const double mean = (double)k * (double)gw.per_group / (double)kGroup;
        routes[1] = gw.gs.ngroups;
        routes[4] = row_bracket_target_hi(m, (uint32_t)k, sp);
        routes[5] = gw.per_group;
        routes[6] = union_bracket_target_lo(mean);
        routes[7] = union_bracket_target_hi(mean);
    }
    return GTOPK_OK;
}

int gtopk_debug_missed_brackets(const void* ws, int64_t m, int32_t k, int32_t P, uint32_t* host_missed) {
    if (!ws || !host_missed || !sizes_ok(m, k, P)) return GTOPK_EINVAL;
    const StepWs w = carve_step(const_cast<void*>(ws), m, (uint32_t)k, (uint32_t)P);
    if (small_problem(m, k, P) || !grouped_step(m, (uint32_t)k, (uint32_t)P, w)) return GTOPK_EINVAL;
    const size_t sets = 2 * (size_t)P - 1;
    if (hipMemcpy(host_missed, carve_grouped(w, m, (uint32_t)k, (uint32_t)P).gs.d1, sizeof(uint32_t) * sets, hipMemcpyDeviceToHost) !=
        hipSuccess)
        return GTOPK_EHIP;
    for (size_t i = 0; i < sets; ++i) host_missed[i] = host_missed[i] == kMissed ? 1u : 0u;
    return GTOPK_OK;
}

}  // extern "C"
