// Host-side planner: turns one mixed batch (a prefill chunk at its chunk offset plus
// piggybacked decodes, paper Sec. 2.2 / 3.2) into the integer work list the fused
// attention kernel consumes.  Runs once per iteration; every layer reuses the plan.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <new>

#include "tc_internal.h"

namespace tc {

static thread_local std::string g_last_error;

void set_error(const std::string &msg) { g_last_error = msg; }

static tc_status fail(tc_status s, const std::string &msg) {
    set_error(msg);
    return s;
}

tc_status check_pool_matches(const tc_plan *plan, const tc_kv_pool *pool, bool need_ptrs) {
    if (!plan || !pool) return fail(TC_ERR_NULL, "plan or pool is NULL");
    if (pool->num_q_heads != plan->Hq || pool->num_kv_heads != plan->Hkv || pool->head_dim != plan->D ||
        pool->block_size != kBlock || pool->num_blocks != plan->num_blocks || pool->dtype != plan->dtype)
        return fail(TC_ERR_SHAPE, "pool shape differs from the shape the plan was built for");
    if (need_ptrs && (!pool->k_pool || !pool->v_pool)) return fail(TC_ERR_NULL, "k_pool or v_pool is NULL");
    return TC_OK;
}

// Measured rates the planner balances with (one MI355X): a prefill workgroup needs about kTileUs
// microseconds per 64-token KV tile at head_dim 128 (half of that at 64), a piece costs about
// kPieceOverheadTiles tiles on top of its sweep (loading Q, filling the copy pipeline, leaving or combining
// partial results), the decode branch reads about 5 TB/s when it has the chip to itself and about
// kDecodeCuGBs GB/s per compute unit when only a few units run it.
constexpr double kTileUs = 1.8;
constexpr double kPieceOverheadTiles = 3.0;
constexpr double kDecodeCuGBs = 40.0;
constexpr int kMinPieceTiles = 4;   // a levelled piece is never shorter than this
constexpr int kMinBinTiles = 8;     // and a levelled workgroup never holds less than this

// Workgroups of a launch with a prefill chunk that the chip holds at a time.
static int64_t wg_slots(const tc_plan *p) { return p->prefill_waves == kMixedWaves ? kNumCu : (int64_t)kNumCu * small_wg_per_cu(p->D); }

// The KV range of a decode sequence is cut into the fewest splits of at most `split` tokens, equal up
// to a page; the split is the largest of 1024..128 tokens that still yields enough items to fill the chip.
static int choose_split(int64_t decode_token_heads) {
    const int64_t want_items = (int64_t)kNumCu * kDecodeWgPerCu * kDecodeWaves;  // one item per wavefront resident in a decode-only launch (finer splits measured slower)
    for (int split = kMaxSplitPages * kBlock; split > 128; split /= 2)
        if (decode_token_heads / split >= want_items) return split;
    return 128;
}

// First token of split i of a decode sequence of kv tokens cut into ns splits: the sequence's pages are
// dealt out evenly (the first splits get the odd pages), so the splits of a sequence take the same time
// and the waves that run them side by side finish together.  split_begin(kv, ns, ns) >= kv.
static int64_t split_begin(int64_t kv, int ns, int i) {
    const int64_t pages = (kv + kBlock - 1) / kBlock;
    return kBlock * (i * (pages / ns) + std::min<int64_t>(i, pages % ns));
}

// Splits of a decode sequence of kv tokens, to run in workgroups of W waves (W a power of two): pieces of
// at most `split` tokens, their number rounded up to a power of two, so that the runs pack into
// workgroups without gaps; a sequence that W pieces of up to kMaxSplitPages pages can cover is never cut
// into more than W (all of them are then one team, which writes the output rows itself: no partial
// result, no merge item); a longer one gets a multiple of W (whole workgroups).
static int num_splits(int64_t kv, int split, int W) {
    const int64_t ns = (kv + split - 1) / split;
    const int64_t longest = (int64_t)kMaxSplitPages * kBlock;
    if (kv > (int64_t)W * longest) return (int)((ns + W - 1) / W * W);
    int n = 1;
    while (n < ns && n < W) n *= 2;
    return n;
}

// The shortest split, from 128 to 1024 tokens, that cuts the decode sequences into no more than `target` (split, KV head) pairs.
static int shortest_split(const tc_plan *p, int S, int64_t target) {
    int lo = 128 / kBlock, hi = kMaxSplitPages;  // pages
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        int64_t n = 0;
        for (int s = 0; s < S; s++)
            if (p->q_start[s + 1] - p->q_start[s] == 1) n += ((int64_t)p->ctx_len[s] + 1 + mid * kBlock - 1) / (mid * kBlock);
        if (n * p->Hkv <= target) hi = mid; else lo = mid + 1;
    }
    return lo * kBlock;
}

// Workgroups of the decode branch when a split of at most `split` tokens is run by a whole one (W = 1), or two of them by one (W = 2;
// sequences that are a single split then share a workgroup with another, but are counted as if they did not).
static int64_t wide_workgroups(const tc_plan *p, int S, int split, int W, int64_t *single = nullptr) {
    int64_t full = 0, one = 0;
    for (int s = 0; s < S; s++)
        if (p->q_start[s + 1] - p->q_start[s] == 1) {
            const int n = num_splits((int64_t)p->ctx_len[s] + 1, split, W);
            if (n >= W) full += n / W; else one++;
        }
    if (single) *single = one * p->Hkv;
    return (full + one) * p->Hkv;
}

// Splits of up to 1024 tokens run by whole workgroups that fill the last of two to four rounds only in part leave units idle
// in it, and each split costs its start and its combination.  Where two splits to a workgroup (half of its waves each; the halves of up
// to 2048 tokens of a sequence have one result) save the round: the shortest splits that do, else 0.  Not for many sequences
// that are a single split, whose pages then have half as many waves: beside a chunk up to a quarter of the workgroups, without one no
// sequence of up to 2048 tokens.
// Measured (us per step, one split to a workgroup / two; 32/8 heads, head_dim 128, unless stated):
//   beside 128 at 1000   24 of 512-4096 48.4 / 43.6, 40 of lognormal 1500 51.6 / 47.5, 12 of lognormal 6000 58.2 / 52.7, 40/8 heads, head_dim 64
//                        36.6 / 31.9, 28 of lognormal 2500 35.8 / 31.2
//   decodes only         12 of lognormal 6000 52.6 / 48.7, 40/8 heads, head_dim 64 29.9 / 27.5; 10 of 4000-12000 54.2 / 50.2, 6 of 8000-20000
//                        59.2 / 56.9; with shorter sequences, 31 of 489-3912, 52.4 / 52.9, 8/8 heads 50.3 / 52.1, 40 of lognormal 1500 45.9 / 46.7
//   single splits        16/2 heads, 176 short decodes beside 564 first tokens 20.1 / 24.8
// And not where one round of halves takes longer than two of splits: the halves of a sequence of up to 2048 tokens are as long as a split may be
// and have half of the waves, while the second round's splits are the short ones, on the units that had the shortest before.  The line is at 22 pages
// between the longest half and the longest split of the second round.  Measured (us, one to a workgroup / two; that difference in brackets):
//   head_dim 128   64/8 heads, 16 of lognormal 2000 (17) 32.0 / 29.9, 8/8, 22 of 446-1786 (21) 27.1 / 26.0, 40/8, 16 of lognormal 1650 (23) 24.1 / 28.3,
//                  32/8, 23 of 275-2204 (27) 28.8 / 30.1
//   head_dim 64    40/8 heads, 16 of 411-3288 (17) 18.8 / 15.6, 32/32, 4 of 457-3658 (23) 15.3 / 17.7, 40/8, 21 of 268-2146 (28) 15.9 / 17.0, but 8/8,
//                  15 of lognormal 1490 (23) 18.7 / 16.5
// In the geometric mean 241 batches on this side of the line are 8 % faster with two to a workgroup, 37 on the other 2 % slower.
static bool halves_take_longer(const tc_plan *p, int S, int pages, int64_t at_once) {
    int64_t count[kMaxSplitPages + 1] = {};  // splits of so many pages, one to a workgroup
    int half = 0;
    for (int s = 0; s < S; s++)
        if (p->q_start[s + 1] - p->q_start[s] == 1) {
            const int64_t kv = (int64_t)p->ctx_len[s] + 1, pg = (kv + kBlock - 1) / kBlock;
            const int64_t n1 = num_splits(kv, kMaxSplitPages * kBlock, 1), n2 = num_splits(kv, pages * kBlock, 2);
            count[pg / n1] += n1 - pg % n1;
            if (pg % n1) count[pg / n1 + 1] += pg % n1;
            half = std::max(half, (int)((pg + n2 - 1) / n2));
        }
    int second = kMaxSplitPages;  // the longest first: the one after `at_once`
    for (int64_t seen = count[second] * p->Hkv; seen <= at_once && second > 1; seen += count[second] * p->Hkv) second--;
    return half > second + 22;
}
static int two_split_workgroups(const tc_plan *p, int S, int split, int64_t at_once, bool decodes_only) {
    const int64_t rounds = (wide_workgroups(p, S, split, 1) + at_once - 1) / at_once;
    if (split < kMaxSplitPages * kBlock || rounds < 2 || rounds > 4) return 0;
    if (decodes_only && *std::min_element(p->ctx_len.begin(), p->ctx_len.begin() + S) < 2 * kMaxSplitPages * kBlock) return 0;
    const int max_pages = decodes_only ? 40 : kMaxSplitPages;  // two waves for a split: no more than 20 pages each
    // Longer splits are never more workgroups: the shortest are found by halving the range (six counts of the sequences, not 33).
    const int64_t most = (rounds - 1) * at_once;
    int pages = kMaxSplitPages / 2, last = max_pages;
    int64_t single = 0;
    if (wide_workgroups(p, S, last * kBlock, 2) > most) return 0;
    while (pages < last) {
        const int mid = (pages + last) / 2;
        if (wide_workgroups(p, S, mid * kBlock, 2) <= most) last = mid; else pages = mid + 1;
    }
    const int64_t n = wide_workgroups(p, S, pages * kBlock, 2, &single);
    if (single * 4 > n || (rounds == 2 && !decodes_only && halves_take_longer(p, S, pages, at_once))) return 0;
    return pages * kBlock;
}

// A batch of few decodes (no prefill chunk) whose single-wave splits would leave wave slots empty or keep a few waves
// busy long after the others: every split is run by a whole workgroup instead (decode_item_wide), and a sequence of more than
// 1024 tokens is cut into as many splits as it takes to have one workgroup per compute unit (two per unit once
// they would hold more than 900 tokens each).  Returns the split length, or 0 when the single-wave form serves better.
// Measured (32/8 heads, head_dim 128, attention launch with its append, us, single-wave form / this one):
//   8 requests, lognormal lengths of mean 1024  29.6 / 11.5       1 request of 16000 tokens         22.8 / 18
//   24 of lognormal mean 1500                   52.1 / 29.8       32 of 128-384 tokens              10.2 / 9.4
//   96 of lognormal mean 1500 (1.15 M tokens x heads)   106.5 / 101.7     96 of 512-1536 tokens      68.2 / 74.6
// The line: with 3072 splits of 256 tokens or more the single-wave form fills the chip and streams at the HBM rate,
// which this form, whose workgroups all start and combine alike, misses by 5-8 %.  Below that the single-wave form
// serves better where it has no partial results to combine (at most 4096 tokens), this one would have (over 1024), and
// the longest sequence is not far above the mean load of a compute unit (24 requests of 512-1536 tokens: 21.8 / 24.6, 16 of
// them 19.3 / 15.9): the line is at 7/4 of that load, and at 9/4 where this form would give a few units a second workgroup and
// wait for those (head_dim 128, 8/8 heads, 25 requests of 260-1431 tokens, 288 workgroups, factor 2: 20.9 / 24.7).
// Every (sequence, KV head) pair is a workgroup here, however short its sequence, and two of them run on a unit at a time (at
// head_dim 64, with half the registers for a page, they pass twice as fast): with more than three pairs per unit the starts
// and combinations of many short sequences cost more than the shorter wait, unless a pair has 288 tokens on the mean, or single
// waves would be busy for a dozen pages and more.  Measured (32/8 heads unless stated, in pairs):
//   60-70 tokens, 512 pairs 8.3 / 7.5, 1024 11.6 / 14.0, 4096 37.2 / 46.3       1-16 tokens, 4096 pairs 19.0 / 31.7
//   64-256 tokens, 512 pairs 12.3 / 11.5, 2048 38.4 / 41.2                      128-512 tokens, 1024 pairs 34.6 / 33.1, 2048 64.5 / 65.0
//   head_dim 64: 60-70 tokens, 1024 pairs 7.3 / 7.4, 2048 11.7 / 13.5; 16-100, 4096 20.0 / 23.7; 128-512, 2048 33.9 / 33.5
//   32/32 heads, one of 2157 tokens (34 pages a wave) among 29 short ones, 960 pairs 27.5 / 17.0
static int choose_wide_split(const tc_plan *p, int S, int64_t decode_tokens) {
    const int64_t token_heads = decode_tokens * p->Hkv;
    if (token_heads >= (int64_t)kNumCu * kDecodeWgPerCu * kDecodeWaves * 256) return 0;
    const int split = choose_split(token_heads);  // of the single-wave form
    int64_t longest = 0, longest_pages = 0;       // the longest sequence; the pages of the longest single-wave split
    for (int s = 0; s < S; s++) {
        const int64_t kv = (int64_t)p->ctx_len[s] + 1, pages = (kv + kBlock - 1) / kBlock, ns = num_splits(kv, split, kDecodeWaves);
        longest = std::max(longest, kv);
        longest_pages = std::max(longest_pages, (pages + ns - 1) / ns);
    }
    const int64_t pairs = (int64_t)S * p->Hkv;
    const double chip_pairs = pairs * (p->D / 128.0);
    if (chip_pairs > 3 * kNumCu && token_heads < 288 * pairs && longest_pages < 12 + chip_pairs / kNumCu) return 0;
    const int wide = shortest_split(p, S, token_heads > 900 * kNumCu ? 2 * kNumCu : kNumCu);
    const int64_t items = wide_workgroups(p, S, wide, 1);
    const bool few_doubled = p->D == 128 && items > kNumCu && 2 * items < 3 * kNumCu;  // a few units get a second workgroup
    const int64_t max_split = (int64_t)kMaxSplitPages * kBlock;
    if (longest > max_split && longest <= kDecodeWaves * max_split && 4 * longest * kNumCu < (few_doubled ? 9 : 7) * token_heads) return 0;
    return wide;
}

// The same beside a prefill chunk, where a decode workgroup has eight waves and a compute unit to itself.  Eight
// single-wave splits per sequence (up to 8192 tokens; none to combine across workgroups) stream best as long as the longest
// of them is not what the launch waits for: a wave needs about 1.1 us per page then, so a sequence of 4000 tokens takes
// 35 us however little else there is to do.  When that is more than half of what the rest of the batch needs (t_rest_us: the
// longest sweep, or the sweeps spread over the chip and the decode bytes at 5 TB/s), the splits are run by whole
// workgroups, as short as the units that the chunk leaves free can take at once.  Where the pieces of a cut chunk hold most units
// and there is no queue, so that decode workgroups beyond the free units wait for a piece to end, the line is at 0.8.
// Measured (us per step, single-wave splits / whole workgroups; the share is what the longest sequence takes of the rest):
//   three first chunks, 1079 tokens, 16 decodes (lognormal 1024)     64.9 / 40.5    first chunk of 300, 4 decodes          34.8 / 17.6
//   2000 at 0, 32 decodes (lognormal 1500; share 0.7)                89.9 / 75.5    256 at 500, 64 of them (share 0.6)     97.1 / 81.5
//   128 at 1000, 32 decodes of 512-4096, 40/8 heads, 16 layers (0.6)  971 / 922     128 at 2048, 40 of them (share 0.4)    73.6 / 78.2
//   256 at 500, 128 decodes (lognormal 1500; share 0.35)            145.7 / 156.5   128 at 2048, 64 of 512-4096 (0.3)     109.6 / 121.4
//   512 at 2048 in 192 pieces, 16 of 512-4096 (share 0.75)           55.6 / 56.8
// Each (sequence, KV head) pair is a workgroup then, or a unit of the queue, however short its sequence, and each 256 of them beyond
// the first take 2 us (3 where they are drawn) for starting and combining on top: one long sequence must not take hundreds of short
// ones along.  128 at 0, 32/32 heads, four decodes of 8000 and 128 of 40-80 tokens (5120 workgroups) 137.6 / 154.5, one of 6000 and 64
// (2240) 74.1 / 52.1; 701, 333 and 45 at 0, 32/8 heads, head_dim 64, one of 6000 and 400 (3248) 46.5 / 56.5, and 128 39.4 / 27.8.
// At head_dim 64 a split is half the bytes for the same start and combination, and the line is at 0.65: 128 at 1000 with 32
// decodes of 512-4096 tokens (share 0.55) 38.0 / 40.2, 256 at 500 with 64 of lognormal 1500 (0.8) 50.6 / 46.4.
static int choose_wide_split_beside_chunk(const tc_plan *p, int S, double t_rest_us, double t_decode_us, int64_t n_prefill_wg, bool queue) {
    const int W = p->prefill_waves;
    const int64_t slots = wg_slots(p);
    int64_t longest = 0;  // decode sequences that one workgroup covers
    for (int s = 0; s < S; s++)
        if (p->q_start[s + 1] - p->q_start[s] == 1) {
            const int64_t kv = (int64_t)p->ctx_len[s] + 1;
            if (kv <= (int64_t)W * kMaxSplitPages * kBlock) longest = std::max(longest, kv);
        }
    const double t_longest = 1.1 * (p->D / 128.0) * (double)longest / (kBlock * W);
    const double share = !queue && n_prefill_wg > slots / 2 ? 0.8 : p->D == 64 ? 0.65 : 0.5;
    // More sweeps than the chip takes at once: the decode workgroups start when the last of them have, so what their longest wave needs comes
    // on top, unless the decodes themselves keep the chip busy for twice as long.  Alone it counts from 16 us on, 20 at head_dim 64: 1900 and 4700 tokens
    // beside workgroups of eight waves, half as many beside those of four.  (Single-wave splits / whole workgroups): 32/8 heads, 2300 at 0 with 16 of
    // lognormal 1024 88.2 / 65.5, 12 of 512-4096 74.4 / 69.7; 3500 at 0 with 3 of 4000-12000 153.2 / 120.5; 40/8 heads, 1800 at 0 with 32 of lognormal
    // 1024 91.3 / 71.8, with 64 of 500-1500 90.3 / 92.9; head_dim 64, 64/8 heads, 2000 at 2000 with 16 of lognormal 1024 131.0 / 119.8, 1300 at 0 with
    // 32 52.4 / 43.5; 12 of 512-4096 beside 2300 at 1000, 40/8 heads, 70.7 / 75.5, beside 2200 at 0, 32/32 heads, 74.5 / 82.1.
    // Many times as many sweeps: 1240 (128/8 heads, 2480 at 0 with one of 8200) 232.1 / 219.3, 1376 (8700 at 0, 6 of 1700-6900) 738.4 / 694.8, 4176 (128/8,
    // 8344 at 65, 2 of 2400-9500) 2013 / 1969.  Long decode streams: 40/8 heads, 2664 at 0 with 29 of 2600-10400 (160 us of K/V) 216.7 / 226.1, 3136
    // at 0 with 31 of 3800-15400 315.9 / 327.2; 32/8, 10816 at 4394 with 34 of 3600-14400 1590 / 1613.
    const bool late = !queue && n_prefill_wg > slots;
    const double t_rest = std::max(t_rest_us, 8.0);
    const double line = late ? std::max(std::min(share * t_rest, p->D == 64 ? 20.0 : 16.0), 0.5 * t_decode_us) : share * t_rest;
    if (t_longest <= line) return 0;
    const int split = shortest_split(p, S, std::max<int64_t>(slots - n_prefill_wg, slots / 4));
    const int64_t items = wide_workgroups(p, S, split, 1);
    const double t_starts = (queue ? 3.0 : 2.0) * std::max<int64_t>(0, items - slots) / slots;
    return t_longest <= (late ? line + t_starts : share * (t_rest + t_starts)) ? 0 : split;
}

// When a batch has few prefill row blocks (a small chunk, as on a decode-heavy instance), each of
// them sweeps its whole KV range in one workgroup while most of the chip idles, and that sweep is the
// iteration's critical path.  Then the KV range of a row block is cut into k pieces that run as
// separate workgroups; the last of them to finish combines their partial results.  k is the smallest count
// that brings the sweep down to the time the decode branch needs anyway (both estimated from measured
// rates), at most 8, at least 8 tiles per piece, and never more pieces than workgroup slots.
// Tile times the cuts are chosen with: 256 rows, 128 rows.
constexpr double kCutTileUs = 2.0, kCutHalfTileUs = 1.1;
static int prefill_cuts(int n_tiles, int64_t items, int64_t decode_bytes, double tile_us) {
    const int k_cap = (int)std::min<int64_t>(8, kNumCu / items);  // one prefill workgroup per compute unit
    const double t_decode_us = std::max(16.0, (double)decode_bytes / 5.0e6);
    const int want = (int)std::ceil(n_tiles * tile_us / t_decode_us);
    return std::max(1, std::min({want, k_cap, n_tiles / 8}));
}
static void choose_prefill_cuts(std::vector<PlanRowBlock> &blocks, int Hkv, int64_t decode_bytes, double tile_us) {
    const int64_t items = (int64_t)blocks.size() * Hkv;
    for (PlanRowBlock &b : blocks) b.k = prefill_cuts(b.n_tiles, items, decode_bytes, tile_us);
}

// Pieces of a batch whose row blocks would leave a good part of the chip empty or idle (more than a quarter of the compute units and up to
// four times as many, chosen by estimate_chunk).  The row blocks of a KV head, heaviest first, are laid end to end and cut into `bins` runs of equal
// cost; each run is one workgroup, which sweeps its pieces one after the other.  A block that straddles a cut
// becomes pieces of two (rarely more) workgroups.  The same cuts are used for every KV head.
static void level_prefill(std::vector<PlanRowBlock> &blocks, std::vector<PlanPiece> &pieces, int bins) {
    double left = 0;  // tiles not yet given to a workgroup
    for (const PlanRowBlock &b : blocks) left += b.n_tiles;
    const double o = kPieceOverheadTiles;
    int bin = 0;
    double fill = 0, target = 0;
    // cost a workgroup should hold, from what is left when it is opened: the tiles, one overhead per block still
    // to be started or continued, one more per cut still to be made
    auto open_bin = [&](size_t blocks_left) { fill = 0; target = (left + o * (double)(blocks_left + (bins - bin) - 1)) / (bins - bin); };
    open_bin(blocks.size());
    for (size_t i = 0; i < blocks.size(); i++) {
        PlanRowBlock &b = blocks[i];
        b.k = 0;
        int t = 0;
        while (t < b.n_tiles) {
            const int rem = b.n_tiles - t;
            const double room = target - fill - o;
            int take;
            if (bin == bins - 1 || room + 1.0 >= rem) take = rem;  // the rest fits (at most a tile over), or this is the last workgroup
            else if (room < kMinPieceTiles && fill > 0) { bin++; open_bin(blocks.size() - i); continue; }
            else {
                take = std::max((int)room, kMinPieceTiles);
                if (rem - take < kMinPieceTiles) take = rem - kMinPieceTiles;  // do not leave a stub behind
                if (take < kMinPieceTiles) take = rem;
            }
            pieces.push_back({(int)i, t, t + take, b.k++, bin});
            t += take;
            left -= take;
            fill += take + o;
            if (bin < bins - 1 && fill + o + kMinPieceTiles > target) { bin++; open_bin(blocks.size() - i - (t == b.n_tiles ? 1 : 0)); }
        }
    }
}

// tc_mixed_attention_static takes every batch whose partial results fit its array.  Items that run whole leave none, so runs must not be
// what takes a batch out of that array: piece regions that fit it beside the decodes' partial results.  Those are at most one per 1024 tokens
// of a sequence longer than that, in teams or in splits, or as many as there are units to fill with shorter splits.
static int64_t fitting_regions(const tc_plan *p, int S) {
    int64_t partials = 0;
    bool decodes = false;
    for (int s = 0; s < S; s++)
        if (p->q_start[s + 1] - p->q_start[s] == 1) {
            decodes = true;
            if (p->ctx_len[s] >= kMaxSplitPages * kBlock) partials += p->ctx_len[s] / (kMaxSplitPages * kBlock) + 1;
        }
    if (decodes) partials = std::max<int64_t>(partials * p->Hkv, kNumCu);
    const int64_t row_bytes = (int64_t)(p->D + 2) * sizeof(float);
    return std::max<int64_t>(0, (int64_t)kStaticScratchBytes - partials * p->G * row_bytes) / (kPrefillRows * row_bytes);
}

// Rows of a prefill item: 256, or 128 when the chunk is small.  An item of 128 rows keeps one wave per SIMD busy, and such a
// wave sweeps a tile in about 0.6 of the time it takes beside a second one; but there are at least twice as many items,
// by 128 / G against 256 / G positions more than twice where 256 / G is odd, three times for chunks of a few positions more than
// an item of 128 rows holds twice, each starts and ends on its own, and K and V are read that much more often.  So the
// items are counted as they will be made, and halves are taken:
//   sweeps of at most 16 tiles (first chunks; cutting the KV range would cost more than it returns) whose 256-row items take
//   half of the compute units at most: always without decodes (256 rows would be levelled over fewer units); beside decodes
//   where the estimate is lower: the longest sweep, or the unit times of all items and of the decodes spread over the chip.
//   longer sweeps whose 256-row items take an eighth of the units at most (their KV range is cut): where the estimate is lower, for the longest
//   piece and, beside decodes, for all the work spread over the chip.  On a full chip halves make longer pieces (they are cut less,
//   and not at all when they are more than a quarter of the units), but fewer per item, which saves about 7 us of starting and
//   combining at head_dim 128, and 5 more where halves are not cut at all.
// Not beside a decode branch that needs longer than the longest sweep: it needs the units.
// Measured (us per step, 256 rows / 128; 32/8 heads, head_dim 128, unless stated):
//   first chunks   200 tokens 14.9 / 12.3, 500 20.6 / 17.3, 1000 35.4 / 25.9; 40/8 heads: 816 (264 items) 35.7 / 23.9, sixteen of 51
//                  (384 items) 83.3 / 17.2
//   with decodes   1000 with 32 (lognormal 1500) 53.6 / 58.4; 40/8 heads, decodes of 100-900 tokens: 801 with 16 of them 29.5 / 29.2, with
//                  32 30.6 / 33.5; sixteen of 51 with 4 17.7 / 21.6; 400 and 405 with 4 23.2 / 23.1, with 16 24.6 / 28.3; 24/8 heads, the
//                  same with 16 23.3 / 20.6, with 32 24.7 / 27.4
//   cut            64 at 3000 33.2 / 29.1, at 60000 160.2 / 132.3 (cut in eight at most, 256 rows leave units empty); 256 at 3000
//                  36.2 / 32.7, at 8000 54.3 / 52.8, at 20000 94.9 / 100.9, at 60000 227.3 / 269.9; 40/8 heads: 204 at 3000 (72 items,
//                  uncut) 37.6 / 52.5, 102 at 20000 74.3 / 76.3; head_dim 64: 256 at 3000 24.2 / 22.6, at 8000 34.6 / 36.2
//   with decodes   head_dim 64, 8/8 heads, 455 at 9062 with 37 (mean 1400) 39.5 / 50.2; 32/8 heads, 128 at 8000 with 8 (mean 500) 31.6 / 29.4;
//                  head_dim 128, 256 at 2048 with 32 of 512-4096 64.1 / 59.9, 128 53.4 / 52.1 with 24 of them
static int choose_rows_per_item(const tc_plan *p, int S, int64_t decode_bytes) {
    const int whole_pos = kPrefillRows / p->G, half_pos = kPrefillRows / 2 / p->G;
    int64_t whole = 0, half = 0, longest = 0;   // items of 256 and of 128 rows, tokens of the longest sweep
    double whole_tiles = 0, half_tiles = 0;     // tiles of all items' sweeps
    for (int s = 0; s < S; s++) {
        const int q = p->q_start[s + 1] - p->q_start[s];
        if (q <= 1) continue;
        const int64_t nw = (int64_t)((q - 1) / whole_pos + 1) * p->Hkv, nh = (int64_t)((q - 1) / half_pos + 1) * p->Hkv;
        const double mean_tiles = ((double)p->ctx_len[s] + 0.5 * q) / kPrefillTileTokens + 0.5;
        whole += nw;
        half += nh;
        whole_tiles += nw * mean_tiles;
        half_tiles += nh * mean_tiles;
        longest = std::max<int64_t>(longest, (int64_t)p->ctx_len[s] + q);
    }
    if (whole == 0) return kPrefillRows;
    const int tiles = (int)((longest + kPrefillTileTokens - 1) / kPrefillTileTokens);
    if ((double)decode_bytes / 5.0e6 > tiles * kTileUs * (p->D / 128.0)) return kPrefillRows;
    int k_whole = 1, k_half = 1;
    double add_whole = 0;  // what starting and combining the longest pieces takes longer with 256 rows
    const bool d64 = p->D == 64, cut = tiles > 16;
    if (!cut) {
        if (whole * 2 > kNumCu) return kPrefillRows;
        if (decode_bytes == 0) return kPrefillRows / 2;
    } else {
        if (whole * 8 > kNumCu || half > kNumCu) return kPrefillRows;
        k_whole = prefill_cuts(tiles, whole, decode_bytes, kCutTileUs);
        if (half * 4 <= kNumCu) k_half = prefill_cuts(tiles, half, decode_bytes, kCutHalfTileUs);
        add_whole = (p->D / 128.0) * (k_half == 1 ? 12.0 : 7.0);
    }
    // time of a tile in an item of either size, by how full the chip is with them
    const bool half_full = half * k_half > kNumCu / 2, whole_full = whole * k_whole > kNumCu / 2;
    const double half_us = !cut ? (d64 ? 0.62 : 1.1) : (half_full ? 1.08 : 0.95) * (d64 ? 0.61 : 1.0);
    const double whole_us = !cut ? (d64 ? 1.04 : 1.6) : whole_full ? kTileUs * (p->D / 128.0) : (d64 ? 0.75 : 1.25);
    double t_whole = tiles * whole_us / k_whole + add_whole, t_half = tiles * half_us / k_half;
    if (decode_bytes > 0) {  // unit times: a piece takes 3 us beside its tiles, 6 if it leaves a partial result (two thirds at head_dim 64)
        const double s = d64 ? 0.65 : 1.0, decode_us = (double)decode_bytes / ((cut ? 30.0e3 : 20.0e3) * kNumCu);
        t_whole = std::max(t_whole, s * (whole_tiles * (cut ? 1.85 : 1.6) + whole * k_whole * (k_whole > 1 ? 6.0 : 3.0)) / kNumCu + decode_us);
        t_half = std::max(t_half, (half_tiles * half_us + s * half * k_half * (k_half > 1 ? 6.0 : 3.0)) / kNumCu + decode_us);
    }
    return t_half <= t_whole ? kPrefillRows / 2 : kPrefillRows;
}

// Row blocks of `rows` (position, head) rows, heaviest (latest positions, longest KV range) first.
static void make_row_blocks(const tc_plan *p, int S, int rows, std::vector<PlanRowBlock> &blocks) {
    const int pos_per_item = rows / p->G;
    blocks.clear();
    for (int s = 0; s < S; s++) {
        const int q = p->q_start[s + 1] - p->q_start[s];
        if (q <= 1) continue;
        for (int pos0 = 0; pos0 < q; pos0 += pos_per_item) {
            const int npos = std::min(pos_per_item, q - pos0);
            const int64_t cost = (int64_t)p->ctx_len[s] + pos0 + npos;
            blocks.push_back({s, pos0, npos, cost, (int)((cost - 1) / kPrefillTileTokens) + 1, 1, 0});
        }
    }
    std::stable_sort(blocks.begin(), blocks.end(), [](const PlanRowBlock &x, const PlanRowBlock &y) { return x.cost > y.cost; });
}

// What a chunk of more than a quarter of the compute units' worth of items takes in each of its forms, estimated, us:
//   whole     items of 256 rows, one workgroup each.  On a unit of its own the longest sweep is what counts; its tiles take 1.25 us while most
//             of the chip is idle and 1.6-1.7 when all of it sweeps (the clock falls); beyond 256 items, list scheduling.
//   levelled  the sweeps cut into runs of equal length, one per unit: pieces leave partial results and start twice.
//   small     items of 128 rows, workgroups of four waves, two or three to a unit.  A unit's workgroups copy their tiles each for itself and
//             get through 15-20 % less together than one of eight waves does, but a long sweep has a short one beside it and is
//             swept at 1.07-1.2 us a tile while the other is at work or gone.
// Measured (us per step, whole / levelled / small, head_dim 128 unless stated):
//   uneven sweeps, first chunks   32/8 heads, 2048 at 0 52.4 / 51.4 / 46.6, head_dim 64 36.0 / 32.2 / 29.6, 1500 38.9 / 35.4 / 34.5; 16/2 heads, 1207
//                                 33.2 / 31.3 / 26.8; 8/8 heads, 7760 176.6 / 151.8 / 159.3, 6000 122.1 / 96.9 / 107.8; 64/8 heads, 1280 39.8 / 42.1 / 38.4
//   an offset                     32/8 heads, 2048 at 1000 79.1 / 83.8 / 74.1, at 4096 159.3 / 161.4 / 159.1; 1200 at 2000 69.4 / 62.4 / 68.2; 1024 at 4096
//                                 102.5 / 82.1 / 87.9; 1000 at 0 and 900 at 6000 134.3 / 121.7 / 117.5
//   more items than units         32/8 heads, 4096 at 0 131.3 / 151.9 / 143.9; 32/32 heads, 2568 84.0 / 97.2 / 80.8; 64/8 heads, head_dim 64, 1055 at 13870 (264
//                                 items) 407.0 / 249.5 / 322.0
//   decodes                       16/2 heads, 1270 at 18176 with 126 of lognormal 7720 357.8 / 266.7 / 346.5; 32/8 heads, 2048 at 0 with 32 of 500-1500
//                                 60.2 / 62.9 / 58.3, 2200 with 10 of 465 57.8 / 65.8 / 54.2
struct ChunkForms {
    double whole, levelled, small;
    double start;  // start and end of a workgroup
};
static ChunkForms estimate_chunk(const tc_plan *p, const std::vector<PlanRowBlock> &blocks, std::vector<PlanUnits> &units) {
    const bool d64 = p->D == 64;
    const int Hkv = p->Hkv;
    const int64_t items = (int64_t)blocks.size() * Hkv;
    double tiles = 0;
    for (const PlanRowBlock &b : blocks) tiles += b.n_tiles;
    const double load = tiles * Hkv / kNumCu, longest = blocks[0].n_tiles, fill = std::min(1.0, load / longest);
    const double o = d64 ? 3.5 : 5.5;
    ChunkForms t;
    t.start = o;
    if (items <= kNumCu) t.whole = longest * (d64 ? std::max(0.92, 0.85 + 0.2 * fill) : std::max(1.25, 1.05 + 0.65 * fill)) + o;
    else {  // heaviest first, to the unit that is free first; units that are free at the same time are one entry (the KV heads of a block take
        // the same time), so that it costs a heap operation or two per block (1.5 us of the 11 that a plan of 1000 items of 8 KV heads takes; one by one 10)
        const double tile_us = d64 ? 1.03 : 1.6;
        const auto later = [](const PlanUnits &x, const PlanUnits &y) { return x.free_us > y.free_us; };
        units.assign(1, {0.0, kNumCu});
        for (const PlanRowBlock &b : blocks)
            for (int left = Hkv; left > 0;) {
                const PlanUnits first = units.front();
                const int n = std::min(left, first.n);
                left -= n;
                if (n < first.n) units.front().n -= n;  // still the first
                else {
                    std::pop_heap(units.begin(), units.end(), later);
                    units.pop_back();
                }
                units.push_back({first.free_us + (b.n_tiles * tile_us + o), n});
                std::push_heap(units.begin(), units.end(), later);
            }
        t.whole = 0;
        for (const PlanUnits &u : units) t.whole = std::max(t.whole, u.free_us);
    }
    const double full = std::max(0.0, (double)(items - 160) / 96);  // the more items, the more of them are cut
    t.levelled = std::max(load, (double)kMinBinTiles) * (d64 ? 1.03 : 1.7) + (d64 ? 14.0 : 15.0 + 6.0 * full);
    const double small_items = 2.0 * items, slots = (double)kNumCu * small_wg_per_cu(p->D);
    const double alone_us = d64 ? std::min(0.8, std::max(0.66, 0.65 + 0.25 * fill)) : std::min(1.2, std::max(1.07, 1.0 + 0.3 * fill));
    const double shared_us = d64 ? (small_items > slots ? 0.62 : 0.59) : (small_items > slots ? 1.06 : 0.98);
    t.small = std::max(longest * alone_us, 2.0 * load * shared_us) + o;
    return t;
}

// KV tiles that the workgroups which begin on one compute unit sweep together, at most (small workgroups of these row blocks, as they are
// placed, see the records).
static int tiles_of_fullest_unit(const tc_plan *p, const std::vector<PlanRowBlock> &blocks) {
    const int n = (int)blocks.size(), row = std::max(1, kNumCu / p->Hkv), rows = small_wg_per_cu(p->D);
    const bool turn = (int64_t)n * p->Hkv <= (int64_t)rows * kNumCu;
    int most = 0;
    for (int unit = 0; unit < std::min(row, n); unit++) {
        int tiles = 0;
        for (int r = 0, first = 0; r < rows && first + unit < n; r++, first += row)
            tiles += blocks[turn && (r & 1) ? first + std::min(row, n - first) - 1 - unit : first + unit].n_tiles;
        most = std::max(most, tiles);
    }
    return most;
}

// Decode units that workgroups begin with in a launch with a queue: those launched for the decode branch (n_decode_wg), and those of the lightest
// sweeps, which sweep after theirs.  Where the sweeps are uneven a unit of a light one is done in the time that its workgroup would draw it later, but while HBM is idle; drawn
// after the sweeps, the units of all workgroups meet there, and the largest begin when the lightest sweeps end.  A unit streams 43 GB/s on its
// own (head_dim 64: as much), so half of the compute units beginning with one saturate HBM.  The units are in order of their size and the light workgroups take
// them as they come, the lightest the largest, as long as a workgroup ends no later than the longest sweep does, or all the work spread over the chip; units too large
// for any go to an eighth of the workgroups all the same.
// Measured (us per step, all units drawn after the sweeps / this): 32/8 heads, 2048 at 4096 with 64 of lognormal 1024 188.4 / 176.5, head_dim 64 111.6 / 110.2; 40/8,
// 701, 333 and 45 at 0 with 16 of them 37.1 / 35.4; 64/8, head_dim 64, 946 at 24 with 46 of 2490-19924 176 / 171; 808 at 0 with 8 of lognormal 2254 26.7 / 25.9.  A
// quarter more or fewer of the units: 0.3 % slower on the mean of 40 batches, up to 8 %.
template <class Splits>
static int64_t deal_units(const tc_plan *p, int n_wg_head, bool level_runs, int64_t decode_tokens, int64_t n_decode_wg, int64_t n_units, const Splits &splits_of) {
    const PlanScratch &w = p->work;
    const int Hkv = p->Hkv;
    int64_t dealt = n_decode_wg;
    // Level runs are alike, also where each of them is one piece: a unit before some of them comes on top (us, none / units before a few of them: head_dim
    // 64, 128/8 heads, 135 at 2105 with 2 of 3680 25.0 / 31.7, 64/8, 279 at 1392 with 173 of 134 26.7 / 30.5; 8/8, 1649 at 319 with 2 of 2908 36.4 / 41.9).
    if (n_wg_head == 0 || level_runs || dealt + Hkv > std::min<int64_t>(n_units, kNumCu / 2)) return dealt;
    const auto sweep_us = [&](int wg) {  // a piece each, the longest first
        return (w.pieces[wg].t1 - w.pieces[wg].t0) * (p->D == 64 ? 1.03 : 1.65) * (p->rows_per_item == kPrefillRows ? 1.0 : 0.6) + 3.0;
    };
    const double unit_us = 4.0, us_per_token = 4.0 * p->D / 43.0e3;
    double sum = n_units * unit_us + (double)decode_tokens * Hkv * us_per_token;
    for (int i = 0; i < n_wg_head; i++) sum += sweep_us(i) * Hkv;
    int64_t tokens[kNumCu / 2] = {};  // of the units that may be dealt
    for (const PlanTeam &x : w.teams) {
        if (x.wg >= kNumCu / 2) continue;
        const int64_t kv = (int64_t)p->ctx_len[x.seq] + 1;
        tokens[x.wg] += kv * x.n / splits_of(kv);
    }
    const double end = 1.03 * std::max(sweep_us(0), sum / kNumCu), room = end - sweep_us(n_wg_head - 1);
    for (int i = 0; i < n_wg_head && dealt + Hkv <= std::min<int64_t>(n_units, kNumCu / 2); i++) {
        const double unit = unit_us + tokens[dealt] * us_per_token;
        if (sweep_us(n_wg_head - 1 - i) + unit > end && (unit <= room || i * Hkv >= kNumCu / 8)) break;
        dealt += Hkv;
    }
    return dealt;
}

tc_status build_plan(tc_plan *p, const tc_kv_pool *pool, const tc_batch *b) {
    if (!p || !pool || !b) return fail(TC_ERR_NULL, "plan, pool or batch is NULL");
    // an error below leaves the plan describing an empty batch
    p->S = p->T = 0;
    p->n_prefill_seqs = p->n_decode_seqs = 0;
    p->n_prefill = p->n_decode = p->n_merge = p->n_partials = p->n_piece_partials = p->n_merge_prefill = p->n_pieces = p->n_prefill_wg = p->n_counters = p->n_append = p->n_append_prefill = p->n_decode_wg = p->n_dealt = p->n_drawers = 0;
    p->queue_counter = -1;
    p->items_per_wg = kDecodeWaves;
    p->waves_per_item = 1;
    p->rows_per_item = kPrefillRows;
    p->prefill_waves = kMixedWaves;
    p->total_pages = 0;
    p->host_n = 0;
    const int Hq = pool->num_q_heads, Hkv = pool->num_kv_heads, D = pool->head_dim;
    if (pool->dtype != TC_BF16 && pool->dtype != TC_FP16) return fail(TC_ERR_SHAPE, "dtype must be TC_BF16 or TC_FP16");
    if (pool->block_size != kBlock) return fail(TC_ERR_SHAPE, "block_size must be 16");
    if (D != 64 && D != 128) return fail(TC_ERR_SHAPE, "head_dim must be 64 or 128");
    if (Hkv <= 0 || Hq <= 0 || Hq % Hkv) return fail(TC_ERR_SHAPE, "num_q_heads must be a positive multiple of num_kv_heads");
    if (Hkv > 1024) return fail(TC_ERR_SHAPE, "more than 1024 KV heads is not supported");
    const int G = Hq / Hkv;
    if (G > 16) return fail(TC_ERR_SHAPE, "more than 16 query heads per KV head is not supported");
    if (pool->num_blocks <= 0 || pool->num_blocks * kBlock >= (int64_t)1 << 31)
        return fail(TC_ERR_SHAPE, "num_blocks must be in [1, 2^27)");
    p->Hq = Hq; p->Hkv = Hkv; p->D = D; p->G = G; p->dtype = pool->dtype; p->num_blocks = pool->num_blocks;
    if (b->num_seqs < 0) return fail(TC_ERR_SPAN, "negative num_seqs");
    const int S = b->num_seqs;
    if (S > 0 && (!b->q_start || !b->ctx_len || !b->block_table)) return fail(TC_ERR_NULL, "a batch array is NULL");
    if (S > 0 && b->max_blocks <= 0) return fail(TC_ERR_BLOCK, "max_blocks must be positive");
    if (S > 0 && b->q_start[0] != 0) return fail(TC_ERR_SPAN, "q_start[0] must be 0");

    p->q_start.assign(S + 1, 0);
    p->ctx_len.assign(S, 0);
    p->page_off.assign(S + 1, 0);
    int n_prefill_seqs = 0, n_decode_seqs = 0;
    int64_t pages = 0, decode_tokens = 0;
    for (int s = 0; s < S; s++) {
        const int64_t a = b->q_start[s], e = b->q_start[s + 1], ctx = b->ctx_len[s];
        if (e <= a) return fail(TC_ERR_SPAN, "q_start must be strictly increasing (every sequence needs a query token)");
        if (ctx < 0) return fail(TC_ERR_SPAN, "negative ctx_len");
        const int64_t kv = ctx + (e - a);
        if (kv >= ((int64_t)1 << 31) - 64) return fail(TC_ERR_SPAN, "ctx_len + q_len too large");
        const int64_t np = (kv + kBlock - 1) / kBlock;
        if (np > b->max_blocks) return fail(TC_ERR_BLOCK, "max_blocks smaller than the pages a sequence needs");
        p->q_start[s + 1] = (int32_t)e;
        p->ctx_len[s] = (int32_t)ctx;
        pages += np;
        if (pages >= ((int64_t)1 << 31)) return fail(TC_ERR_BLOCK, "too many pages in one batch");
        p->page_off[s + 1] = (int32_t)pages;
        if (e - a == 1) { n_decode_seqs++; decode_tokens += kv; } else n_prefill_seqs++;
    }
    // block ids are checked before anything is written into the plan's image
    for (int s = 0; s < S; s++) {
        const int32_t *row = b->block_table + (int64_t)s * b->max_blocks;
        const int np = p->page_off[s + 1] - p->page_off[s];
        const uint32_t nb = (uint32_t)pool->num_blocks;  // < 2^27: a negative id is a large unsigned one
        uint32_t bad = 0;
        for (int i = 0; i < np; i++) bad |= (uint32_t)((uint32_t)row[i] >= nb);
        if (bad) return fail(TC_ERR_BLOCK, "block table entry outside the pool");
    }
    PlanScratch &w = p->work;

    // ---- prefill row blocks, heaviest (latest positions, longest KV range) first, and their pieces
    const int64_t decode_bytes = decode_tokens * Hkv * D * 4;
    p->rows_per_item = choose_rows_per_item(p, S, decode_bytes);
    make_row_blocks(p, S, p->rows_per_item, w.blocks);
    // The sweeps in runs, at most `bins` per KV head: the number made, or 0 (the blocks as they were) where runs whose regions
    // fit the static scratch would be far fewer.  A cut between two runs makes at most two regions.
    auto level = [&](int bins, bool any_scratch) {
        const int wanted = bins;
        const int64_t fit = any_scratch ? INT64_MAX : fitting_regions(p, S) / Hkv;
        while (bins * 16 >= wanted * 15) {
            w.pieces.clear();
            level_prefill(w.blocks, w.pieces, bins);
            int64_t regions = 0;
            for (const PlanRowBlock &x : w.blocks) regions += x.k > 1 ? x.k : 0;
            if (regions <= fit) return bins;
            bins -= (int)((regions - fit + 1) / 2);
        }
        w.pieces.clear();
        for (PlanRowBlock &x : w.blocks) x.k = 1;
        return 0;
    };
    // Regimes by the number of prefill items (row blocks x KV heads) against the compute units:
    //   at most a quarter:  cut each item's KV range so that more units work on the chunk
    //   up to four times:   whole items, level runs or small workgroups, whichever of those that the batch may have is estimated to take least (estimate_chunk)
    //   more:               whole items; the hardware hands them out heaviest first
    // `queue`: the launch has no more workgroups than the chip has compute units and the decode items are drawn from a
    // queue, a workgroup's worth at a time, by whichever workgroup is free (see the kernel).
    w.pieces.clear();
    int n_wg_per_head = 0;  // > 0: levelled; the prefill workgroups are numbered bin * Hkv + KV head
    bool queue = false;
    if (!w.blocks.empty()) {
        const int64_t items = (int64_t)w.blocks.size() * Hkv;
        if (p->rows_per_item != kPrefillRows) {
            if (items * 4 <= kNumCu) choose_prefill_cuts(w.blocks, Hkv, decode_bytes, kCutHalfTileUs);
            // Four waves to a workgroup where several of them share a unit (us, eight waves / four): 40/8 heads, 1000 at 0 (320 items) 32.0 / 26.9,
            // sixteen of 51 (384) 15.2 / 12.8; head_dim 64, 32/8 heads, 1000 at 0 (256) 18.0 / 17.1, 816 (208) 15.3 / 15.1.  Not where every item has a
            // unit to itself at head_dim 128 (32/8 heads, 1000 at 0 24.3 / 25.0, 816 21.4 / 22.0), nor beside decodes, of which eight
            // waves carry more at a time (972 at 0 with 2 25.2 / 26.4; 19 at 737 with 15 17.9 / 18.6).
            if (decode_tokens == 0 && items > (D == 64 ? kNumCu / 2 : kNumCu)) p->prefill_waves = kSmallWaves;
            // (Items of 128 rows take their unit for half as long: they have a queue from half of the units on.  On fewer units drawing
            // from it costs more than it levels: 270 first tokens with 3 decodes of 100-300, 32/8 heads, in 72 items, without it /
            // with it 15.3 / 16.8 us; at head_dim 64 with 46 of 30-300 12.0 / 13.7; 500 tokens, 128 items, with 16 of 100-900 19.0 / 20.8.)
            queue = decode_tokens > 0 && items <= kNumCu && items * 2 > kNumCu;
        } else if (items * 4 <= kNumCu) {
            choose_prefill_cuts(w.blocks, Hkv, decode_bytes, kCutTileUs);
        } else if (items <= 4 * kNumCu) {
            ChunkForms t = estimate_chunk(p, w.blocks, w.units);
            const double t_decode = (double)decode_bytes / 5.0e6;                                 // alone on the chip
            const double unit_decode = (double)decode_bytes / (kDecodeCuGBs * 1e3) / kNumCu;  // what it takes of every unit beside sweeps
            const double t_whole = std::max(t.whole, t_decode), t_levelled = t.levelled + unit_decode;
            // Levelled: not beside a decode branch that needs about as long (512 at 2048, 16 of 512-4096; 1024 at 2048, 64 decodes, 600 MB of K/V, whole /
            // levelled 143 / 155), and where the items nearly fill the chip beside decodes at all, whose queue levels too, only when the sweeps
            // are very uneven (1700 at 3000 with 32 of lognormal 1024 116.2 / 118.1; 8, 800 at 0 and 746 at 7226 with 21 of 1200 156.0 / 129.2),
            // without decodes not for a few per cent either (1500 at 20000, 40/8 heads, head_dim 64, 326 / 341).
            const double level_below = items * 4 <= 3 * kNumCu ? 0.95 : decode_tokens > 0 ? 0.7 : 0.9;
            // Small workgroups: beside more decodes the queue fills the units whose sweeps end early; long sweeps run at a lower clock in either
            // form than the estimates say (6562 at 16848, 8/8 heads, 526 / 543).
            const double small_below = (w.blocks[0].n_tiles <= 64 ? 0.97 : 0.9) * t_whole;
            bool small = t.small < small_below && t_decode < 0.05 * t.small;
            // That is by a unit's share of all sweeps.  Where some units have two long ones it is theirs that count, a tile of the fullest unit 0.9 us, 0.5 at
            // head_dim 64; for sweeps of up to 24 tiles it makes no difference.  (whole / small:) 16/2 heads, 2652 at 11274 and 2355 at 0 with 5
            // decodes 308 / 359, 64/8, 667 at 1657 and 356 at 0 62.4 / 69.3, head_dim 64, 685 at 12873 and 830 at 0 with 2 decodes 190 / 220.  Of 440 batches
            // that took small workgroups without this, 43 had been faster before (up to 25 %), with it 4 (9 %).
            bool crowded = false;
            if (small) {
                make_row_blocks(p, S, kPrefillRows / 2, w.small_blocks);
                crowded = w.blocks[0].n_tiles > 24 && tiles_of_fullest_unit(p, w.small_blocks) * (D == 64 ? 0.5 : 0.9) + t.start >= small_below;
                small = !crowded;
            }
            double tiles = 0;
            for (const PlanRowBlock &x : w.blocks) tiles += x.n_tiles;
            const double unit_prefill = tiles * Hkv * kTileUs * (D / 128.0) / kNumCu;
            const int cu_decode = decode_tokens ? std::max(1, (int)std::lround(kNumCu * unit_decode / (unit_decode + unit_prefill))) : 0;
            const int64_t by_units = std::max<int64_t>(1, (kNumCu - std::min<int64_t>(cu_decode, kNumCu / 2)) / Hkv);
            const int bins = (int)std::max<int64_t>(1, std::min<int64_t>(by_units, (int64_t)tiles / kMinBinTiles));
            // Where small workgroups are estimated to be faster still, but do not serve beside so many decodes: runs all the same (whole / levelled:
            // 32/8 heads, 1408 at 0 with 3 of 579-4632 41.3 / 39.1; 64/8, 360 at 0 and 335 at 1064 with 2 of 981-7850 39.0 / 34.3; 16/2, head_dim 64,
            // 1424 at 0 with 8 of 462-3698 27.5 / 21.2), if a KV head has eight of them: with fewer, of whole units for every head, too many units have
            // none (32/32 heads, 1136 at 174 with one of 1000 40.9 / 47.2, 776 at 1489 with 2 of 442-3540 58.5 / 63.1).  Instead of crowded small ones up to
            // three quarters of the units (40/8 heads, head_dim 64, 1204 at 4097 whole 82, runs 75); beyond whole items do as well or better (8/8, first
            // chunks of 2837, 3049 and 3264 92 / 108, 16/2, 4014 and 1489 95 / 103).
            const bool instead_of_small = !small && bins >= 8 && (!crowded || items * 4 <= 3 * kNumCu);
            // Every KV head has a unit at least: with more heads than units there is one run a head, which cuts nothing, more of them than run at once, and the queue
            // is for launches that all run from the start (us, runs / as they are: 257/257 heads, 200 at 4000 with 2 decodes 219 / 207; head_dim 64, 300/300, 69
            // at 8000 with 3 193 / 186, 320/320, 106 at 0 and 19 at 13305 with one 301 / 211, 514/257, 138 at 21684 with 2 1095 / 789).
            int runs = 0;
            if (Hkv <= kNumCu && t_levelled < level_below * t_whole && (t_levelled < t.small || instead_of_small) && t_decode < 0.75 * t_levelled) {
                // (Chunks of up to three quarters of the units beside few decodes run like this whatever scratch they need.)
                const bool any_scratch = items * 4 <= 3 * kNumCu && t_decode < 0.25 * w.blocks[0].n_tiles * kTileUs * (D / 128.0);
                runs = level(bins, any_scratch);
            }
            if (runs > 0) {
                n_wg_per_head = runs;
                queue = decode_tokens > 0;
            } else if (small) {
                p->prefill_waves = kSmallWaves;
                p->rows_per_item = kPrefillRows / 2;
                w.blocks.swap(w.small_blocks);
            } else {
                queue = decode_tokens > 0 && items <= kNumCu;
            }
        }
    }
    const auto one_workgroup_per_piece = [&] {  // within a block the pieces share the tiles out evenly
        w.pieces.clear();
        for (size_t i = 0; i < w.blocks.size(); i++) {
            const PlanRowBlock &x = w.blocks[i];
            for (int c = 0; c < x.k; c++)
                w.pieces.push_back({(int)i, (int)((int64_t)x.n_tiles * c / x.k), (int)((int64_t)x.n_tiles * (c + 1) / x.k), c, 0});
        }
        // most tiles first (the hardware starts workgroups in index order)
        std::stable_sort(w.pieces.begin(), w.pieces.end(), [](const PlanPiece &x, const PlanPiece &y) { return x.t1 - x.t0 > y.t1 - y.t0; });
        for (size_t i = 0; i < w.pieces.size(); i++) w.pieces[i].wg = (int)i;
    };
    if (n_wg_per_head <= 0) one_workgroup_per_piece();
    int n_wg_head = w.pieces.empty() ? 0 : w.pieces.back().wg + 1;  // prefill workgroups per KV head (pieces are in workgroup order)

    // ---- decode items.  Consecutive splits of one (sequence, KV head) that share a workgroup form a team:
    // the workgroup combines their results in LDS, and the team writes the output rows itself when it
    // holds all splits of its (sequence, KV head), else one partial result.  A run
    // of W splits (W = waves per workgroup of the launch) is a workgroup of its own; shorter runs
    // (1, 2, 4 .. splits) go as one team into the first open workgroup with room (first fit over a
    // bounded window; the oldest is closed when none has room).  Runs are taken longest split first.
    // Wave slots left free hold padding items (no tokens).
    p->split_tokens = choose_split(decode_tokens * Hkv);
    p->items_per_wg = w.blocks.empty() ? kDecodeWaves : p->prefill_waves;
    if (w.blocks.empty() && n_decode_seqs > 0)
        if (const int split = choose_wide_split(p, S, decode_tokens)) {
            p->split_tokens = split;
            p->items_per_wg = 1;
            p->waves_per_item = kWideWaves;
            if (const int two = two_split_workgroups(p, S, split, 2 * kNumCu, true)) {
                p->split_tokens = two;
                p->items_per_wg = 2;
                p->waves_per_item = kWideWaves / 2;
            }
        }
    const auto decodes_beside_chunk = [&] {
        double longest_piece = 0, tiles = 0;
        for (const PlanPiece &x : w.pieces) {
            longest_piece = std::max<double>(longest_piece, x.t1 - x.t0);
            tiles += (x.t1 - x.t0) * (double)Hkv;
        }
        const double tile_us = kTileUs * (D / 128.0) * (p->rows_per_item == kPrefillRows ? 1.0 : 0.6);  // see choose_rows_per_item
        const double t_decode = (double)decode_bytes / 5.0e6, t_rest = std::max(longest_piece * tile_us, tiles * tile_us / kNumCu + t_decode);
        if (const int split = choose_wide_split_beside_chunk(p, S, t_rest, t_decode, (int64_t)n_wg_head * Hkv, queue)) {
            p->split_tokens = split;
            p->items_per_wg = 1;
            p->waves_per_item = p->prefill_waves;
            const int64_t free_units = kNumCu - (int64_t)n_wg_head * Hkv;
            if (!queue && p->prefill_waves == kMixedWaves && free_units >= kNumCu / 4)
                if (const int two = two_split_workgroups(p, S, split, free_units, false)) {
                    p->split_tokens = two;
                    p->items_per_wg = 2;
                    p->waves_per_item = kMixedWaves / 2;
                }
        }
    };
    if (!w.blocks.empty() && n_decode_seqs > 0) {
        decodes_beside_chunk();
        // Short decodes, which single waves run, beside a few uncut sweeps of at most 12 tiles: workgroups of four waves, two or three to a unit, for
        // both, from 128 (sequence, KV head) pairs on (with fewer the two launches of a step take the host longer than the GPU, in either form).  What such a launch takes is the start and the end of its workgroups, which then lie beside each other.  Measured (us per step, eight waves / four):
        //   32/8 heads, 20 at 0 with 17 of 140-281 15.1 / 13.1, 310 at 0 with 180 of 29-58 20.0 / 18.8, 3 at 2 with 369 of 45-90 35.1 / 32.8; 8/8, 78 at 0 with 63 of 77-623
        //   26.9 / 22.4; 16/2, 4 at 1 with 231 of 24-198 17.3 / 13.0; 32/32, head_dim 64, 288 at 0 with 132 of 7-60 22.2 / 20.0; 40/8, 8 at 0 with 374 of 77-616 111.4 / 108.6
        //   longer decodes: 64/8, head_dim 64, 10 at 67 with 42 of 742-5936 51.9 / 56.2; 8/8, head_dim 64, 163 at 0 with 68 of 384-3078 43.3 / 45.4
        //   long streams: 32/32, 196 at 0 with 396 of 92-738 (2.6 GB) 472.1 / 487.6; sweeps of 15 tiles: 16/2, head_dim 64, 945 at 0 with 81 of 48-390 16.1 / 16.5
        //   run by whole workgroups: 40/8, 157 at 0 with 9 of 745-1491 16.8 / 20.0; cut sweeps: 32/8, 11 at 2659 with 20 of lognormal 140 27.4 / 37.6
        int64_t longest = 0;
        bool cut = n_wg_per_head > 0 || w.blocks[0].n_tiles > 12;
        for (int s = 0; s < S; s++)
            if (p->q_start[s + 1] - p->q_start[s] == 1) longest = std::max(longest, (int64_t)p->ctx_len[s] + 1);
        for (const PlanRowBlock &x : w.blocks) cut |= x.k > 1;
        if (p->waves_per_item == 1 && p->prefill_waves == kMixedWaves && !queue && !cut && longest <= 768 && (int64_t)n_decode_seqs * Hkv * 2 >= kNumCu && decode_bytes < (int64_t)600000000 &&
            (int64_t)w.blocks.size() * Hkv * 4 <= kNumCu) {
            p->prefill_waves = p->items_per_wg = kSmallWaves;
            p->rows_per_item = kPrefillRows / 2;
            make_row_blocks(p, S, p->rows_per_item, w.blocks);
            one_workgroup_per_piece();
            n_wg_head = (int)w.pieces.size();
            decodes_beside_chunk();
        }
    }
    const int64_t n_items = (int64_t)w.blocks.size() * Hkv, slots = wg_slots(p);
    const int W = p->items_per_wg;
    // Beside a chunk a workgroup has a unit to itself and runs eight splits: of up to 1024 tokens they take it 170 us while all units stream, and
    // few such rounds end raggedly.  Where the sequences are long (2000 tokens on the mean) splits are shorter, down to 256 tokens (512 at head_dim 64), until
    // there are eight rounds of them; for sequences that one workgroup covers, so that there are no more partial results.  Measured (us per step, before /
    // with this, both with the queue below): 32/8 heads, 256 at 1234 with 256 of 512-4096 413 / 394; 424 at 2 with 162 of 826-6608 409 / 400; 32/32, 3746 at 0
    // with 25 of 459-3676 287 / 277; 1131 at 2 with 83 of 1525-12200 411 / 399.  Of shorter sequences a wave has few pages for its start: 40/8, 1118 at 24
    // with 389 of lognormal 656 218 / 222, 32/32, 382 at 4379 with 180 of 65-526 187 / 191.  The line is where none loses any more: with 800 tokens in its place 17 batches of
    // 1400-2000 on the mean took 4 % less to 2 % more (geometric mean 1.2 % less; 32/8, 256 at 1234 with 256 of 1999 355.9 / 343.3, 2048 at 4096 with 151 of 1957 302.0 / 306.9),
    // 38 of 640-1400 3 % less to 4 % more (0.3 % more; 40/8, 424 with 286 of 1003 222.6 / 217.7, 32/8, 512 with 467 of 1002 331.4 / 344.0, 32/32, 2048 with 60 of 1176 335.7 / 347.3).
    const int split_long = p->split_tokens;  // of sequences that take several workgroups
    if (!w.blocks.empty() && p->prefill_waves == kMixedWaves && p->waves_per_item == 1 && decode_tokens >= (int64_t)2000 * n_decode_seqs)
        while (p->split_tokens * D > 256 * 128 && (int64_t)p->split_tokens * W * 4 * D * 8 * kNumCu > decode_bytes) p->split_tokens /= 2;
    const auto splits_of = [&](int64_t kv) { return num_splits(kv, kv > (int64_t)W * kMaxSplitPages * kBlock ? split_long : p->split_tokens, W); };
    w.runs.clear();
    for (int s = 0; s < S; s++) {
        if (p->q_start[s + 1] - p->q_start[s] != 1) continue;
        const int64_t kv = (int64_t)p->ctx_len[s] + 1;
        const int ns = splits_of(kv);
        w.runs.push_back({s, 0, ns, (int)std::min<int64_t>(kv, split_begin(kv, ns, 1))});
    }
    // longest split first; sequences with equal splits keep their order, and the KV heads of a sequence follow each other
    std::sort(w.runs.begin(), w.runs.end(), [](const PlanRun &x, const PlanRun &y) { return x.len != y.len ? x.len > y.len : x.seq < y.seq; });
    // (the runs of the KV heads of one sequence are alike: `runs` holds one entry per sequence)
    w.teams.clear();
    w.wg_fill.clear();                          // wave slots taken, per decode workgroup
    w.n_teams.assign((size_t)S * Hkv, 0);       // teams per (sequence, KV head)
    {
        constexpr size_t kOpen = 32;
        w.open.clear();  // workgroups with free wave slots, oldest first
        for (const PlanRun &r : w.runs)
            for (int h = 0; h < Hkv; h++)
                for (int first = 0; first < r.ns; first += W) {
                    const int n = std::min(r.ns - first, W);
                    size_t j = 0;
                    if (n == W) j = w.open.size();  // a full run is a workgroup of its own and never stays open
                    while (j < w.open.size() && w.wg_fill[w.open[j]] + n > W) j++;
                    const bool fresh = j == w.open.size();
                    const int wg = fresh ? (int)w.wg_fill.size() : w.open[j];
                    if (fresh) w.wg_fill.push_back(0);
                    w.teams.push_back({r.seq, h, first, n, w.n_teams[(size_t)r.seq * Hkv + h]++, wg, w.wg_fill[wg]});
                    w.wg_fill[wg] += n;
                    if (fresh && n < W) {
                        if (w.open.size() == kOpen) w.open.erase(w.open.begin());
                        w.open.push_back(wg);
                    } else if (!fresh && w.wg_fill[wg] == W) {
                        w.open.erase(w.open.begin() + j);
                    }
                }
    }
    int64_t n_decode_merge = 0, n_decode_partials = 0;
    for (int32_t nt : w.n_teams)
        if (nt > 1) { n_decode_merge++; n_decode_partials += nt; }

    // ---- section sizes
    int64_t n_prefill = n_items, n_pieces = (int64_t)w.pieces.size() * Hkv, n_decode = (int64_t)w.wg_fill.size() * W,
            n_merge = n_decode_merge, n_partials = n_decode_partials, n_counters = n_decode_merge, n_piece_partials = 0, n_merge_prefill = 0;
    for (const PlanRowBlock &x : w.blocks)
        if (x.k > 1) { n_merge += Hkv; n_merge_prefill += Hkv; n_piece_partials += (int64_t)x.k * Hkv; n_counters += Hkv; }
    if (n_pieces + n_decode >= ((int64_t)1 << 28) || n_partials >= ((int64_t)1 << 28) || n_merge >= ((int64_t)1 << 23) ||
        n_piece_partials >= ((int64_t)1 << 20))
        return fail(TC_ERR_SPAN, "batch too large");
    int64_t n_append = 0;  // append segments: the rows a sequence adds to one page (1..16 consecutive token indices)
    for (int s = 0; s < S; s++) {
        const int64_t first = p->ctx_len[s], last = first + (p->q_start[s + 1] - p->q_start[s]) - 1;
        n_append += last / kBlock - first / kBlock + 1;
    }
    const int64_t n_prefill_wg = (int64_t)n_wg_head * Hkv;
    // With a queue the launch has a decode workgroup for every compute unit the chunk leaves free (none when its row
    // blocks fill the chip): they draw decode items from the start, the prefill workgroups when their pieces are done.
    const int64_t n_decode_units = (int64_t)w.wg_fill.size();  // workgroups' worth of decode items
    // Chunks of few workgroups have a queue where the decode stream is long and many rounds of what the free units take at once, so that the units
    // that stream faster take more of it: from 300 MB and 2.4 rounds on.  Measured (us per step, without / with; 32/8 heads, head_dim 128, unless stated):
    //   3.5 rounds of 890 MB  256 at 1234 with 256 of 512-4096 428 / 413           3.6, 740 MB  40/8, 101 at 0 with 135 of 302-2422 136.7 / 132.7
    //   5.0, 300 MB           312 at 7068 with 13 of lognormal 4371 87.0 / 84.4    2.4, 780 MB  8/8, head_dim 64, 4 at 5 with 79 of 1030-8244 135.4 / 133.9
    //   2.3, 700 MB           32/32, 75 at 29 with 20 of lognormal 2109 124.3 / 125.8    2.1, 590 MB  40 at 24 with 15 of lognormal 9482 106.9 / 110.5
    //   2.8, 240 MB           64/8, head_dim 64, 10 at 356 with 289 of lognormal 431 52.9 / 53.4; smaller ones lose up to 7 % (a draw takes a microsecond)
    // Where sequences take several workgroups and leave partial results, from 3.2 rounds on, or from 800 MB:
    //   2.7, 670 MB           32/32, 77 at 2 with 4 of mean 10210 109.9 / 114.4     3.1, 670 MB   64/8, head_dim 64, 3 with 72 of mean 4553 108.0 / 111.8
    //   2.6, 790 MB           64/8, 10 with 21 of mean 9235 133.7 / 140.4           2.7, 340 MB   64/8, head_dim 64, 5 with 13 of mean 12919 63.2 / 64.6
    //   3.3, 760 MB           40/8, head_dim 64, 23 with 38 of mean 9720 130.0 / 126.2   2.6, 880 MB   40/8, head_dim 64, 161 with 42 of mean 10215 153.0 / 148.2
    // (43 batches between 2.4 and 3.2 rounds and under 800 MB 1.2 % slower on the mean with the queue, 38 without partial results 0.7 % faster).
    // Behind more sweeps than units only the decode workgroups draw (see the kernel), where the sweeps are long enough for what the dies' rates differ by.  Single waves
    // at head_dim 128 from 24 tiles a unit on, 41 us of sweeps: 4711 at 0, 32/32, with 272 of 31-254 334.6 / 323.9; 3797 at 2 with 80 of 77 129.4 / 126.6; 2781 at 0
    // with 12 of 587-4702 93.1 / 92.8; below 2343 at 0 with 5 of 758-6068 67.6 / 68.5.  Whole workgroups, whose units are short, from 40 and from 15 for every 256 units on: 36
    // tiles, 832 units 150.9 / 153.6, 33, 896 132.6 / 137.5, 40, 1376 169.3 / 179.2; 42, 360 124.0 / 123.0, 68, 576 206.6 / 201.0, 60, 865 214.1 / 209.2, 208, 832 419.7 / 408.3.
    // Head_dim 64 from 140 and 60 for every 256 units on: 33 tiles, 680 units 76.3 / 79.8, 56, 660 107.1 / 110.4, 107, 504 153.5 / 156.0, 122, 720 166.3 / 169.4 (55
    // batches below 0.7 % slower on the mean); 144, 476 222.1 / 218.9, 203, 448 245.5 / 240.0, 255, 169 318.3 / 311.3 (13 0.5 % faster, none slower by more than 0.2 %).
    bool late_queue = false;
    if (!queue && n_decode_units > 0 && !w.blocks.empty() && p->prefill_waves == kMixedWaves && (p->waves_per_item == 1 || p->items_per_wg == 1)) {
        if (n_prefill_wg <= kNumCu) queue = decode_bytes >= (int64_t)300000000 && n_decode_units * 5 >= (n_decode_partials > 0 && decode_bytes < (int64_t)800000000 ? 16 : 12) * std::max<int64_t>(kNumCu - n_prefill_wg, 1);
        else {
            int64_t tiles = 0;
            for (const PlanPiece &x : w.pieces) tiles += x.t1 - x.t0;
            const bool waves = p->waves_per_item == 1;
            const int64_t at_least = D == 64 ? 140 : waves ? 24 : 40, per_round = D == 64 ? 60 : waves ? 0 : 15;
            late_queue = tiles * Hkv >= std::max(at_least * kNumCu, per_round * n_decode_units);
        }
    }
    const int64_t n_decode_wg = !queue ? n_decode_units : std::min<int64_t>(n_decode_units, std::max<int64_t>(slots - n_prefill_wg, 0));
    // Who draws is said here and nowhere else: a unit that no launched workgroup has of its own needs somebody to draw it.
    const int64_t n_drawers = queue ? n_prefill_wg + n_decode_wg : late_queue ? n_decode_wg : 0;
    const int64_t n_dealt = queue ? deal_units(p, n_wg_head, n_wg_per_head > 0, decode_tokens, n_decode_wg, n_decode_units, splits_of) : 0;
    const size_t off_records = 0;  // first: a record is a 128-byte line
    const size_t off_append = w.pieces.size() * kRecordInts, off_pages = off_append + (size_t)n_append * kAppendInts;
    const size_t off_valid = off_pages + (size_t)pages;
    const size_t off_prefill = off_valid + (size_t)pages;
    const size_t off_decode = off_prefill + (size_t)n_prefill * kItemInts;
    const size_t off_merge = off_decode + (size_t)n_decode * kItemInts;
    const size_t off_counters = (off_merge + (size_t)n_merge * kItemInts + kCounterLine - 1) / kCounterLine * kCounterLine;
    int counter_stride = kCounterLine;
    while (counter_stride > 1 && n_counters * counter_stride > kCounterInts) counter_stride /= 2;
    const size_t off_queue = ((size_t)n_counters * counter_stride + kCounterLine - 1) / kCounterLine * kCounterLine;  // from off_counters
    const size_t n_counter_ints = queue || late_queue ? off_queue + kCounterLine : (size_t)n_counters * counter_stride;
    const size_t total = std::max<size_t>(off_counters + n_counter_ints, 1);
    if (int err = begin_plan_host(p, total)) return fail(TC_ERR_DEVICE, std::string("host buffer of the plan: ") + hip_error_text(err));
    int32_t *H = p->host;

    // ---- pages and the tokens each holds (16, except the last page of a sequence)
    for (int s = 0; s < S; s++) {
        const int32_t *row = b->block_table + (int64_t)s * b->max_blocks;
        const int np = p->page_off[s + 1] - p->page_off[s];
        std::memcpy(H + off_pages + p->page_off[s], row, (size_t)np * sizeof(int32_t));
        const int kv = p->ctx_len[s] + (p->q_start[s + 1] - p->q_start[s]);
        int32_t *val = H + off_valid + p->page_off[s];
        for (int i = 0; i + 1 < np; i++) val[i] = kBlock;
        val[np - 1] = kv - (np - 1) * kBlock;
    }
    {   // append segments: those of the prefill chunks first (the call that fuses the append into the attention
        // kernel still stores the chunks' rows with the append kernel, and only those)
        int32_t *ap = H + off_append;
        for (int pass = 0; pass < 2; pass++) {
            for (int s = 0; s < S; s++) {
                const int q = p->q_start[s + 1] - p->q_start[s];
                if ((q == 1) != (pass == 1)) continue;
                const int32_t *ids = H + off_pages + p->page_off[s];
                int i = 0;
                while (i < q) {
                    const int64_t pos = (int64_t)p->ctx_len[s] + i;
                    const int tok0 = (int)(pos % kBlock);
                    const int n_tok = std::min(kBlock - tok0, q - i);
                    ap[0] = p->q_start[s] + i; ap[1] = n_tok; ap[2] = tok0; ap[3] = ids[pos / kBlock];
                    ap += kAppendInts;
                    i += n_tok;
                }
            }
            if (pass == 0) p->n_append_prefill = (int)((ap - (H + off_append)) / kAppendInts);
        }
    }

    // ---- prefill items in `blocks` order with the KV head as the fastest index; the merge items and partial
    // slots of cut items; then pieces and workgroups.  Workgroup id mod Hkv names the KV head, so that with
    // eight KV heads each of the eight L2 caches serves one head.
    int32_t next_slot = 0, next_region = 0, next_counter = 0;
    int32_t *mg = H + off_merge;
    {
        int32_t *pf = H + off_prefill;
        int32_t item = 0;
        for (PlanRowBlock &x : w.blocks) {
            x.slot0 = next_region;
            for (int h = 0; h < Hkv; h++, pf += kItemInts, item++) {
                pf[PF_SEQ] = x.seq; pf[PF_KVH] = h; pf[PF_POS0] = x.pos0; pf[PF_NPOS] = x.npos;
                pf[PF_QROW0] = p->q_start[x.seq]; pf[PF_CTX] = p->ctx_len[x.seq];
                pf[PF_PAGEOFF] = p->page_off[x.seq]; pf[PF_NPAGES] = p->page_off[x.seq + 1] - p->page_off[x.seq];
                if (x.k == 1) continue;
                mg[MG_SEQ] = x.seq; mg[MG_KVH] = h; mg[MG_QROW] = p->q_start[x.seq] + x.pos0;
                mg[MG_SLOT0] = next_region; mg[MG_NSPLIT] = x.k; mg[MG_COUNTER] = counter_stride * next_counter++; mg[MG_NPOS] = x.npos; mg[MG_ITEM] = item;
                mg += kItemInts;
                next_region += x.k;
            }
        }
        // the counters of cut blocks were handed out block by block, head by head
        std::vector<int32_t> &first_counter = w.slot0;  // (borrowed) per block
        first_counter.assign(w.blocks.size(), -1);
        {
            int32_t c = 0;
            for (size_t i = 0; i < w.blocks.size(); i++)
                if (w.blocks[i].k > 1) { first_counter[i] = c; c += Hkv; }
        }
        // Records: that of a workgroup's first piece has the workgroup's index, those of its other pieces lie behind all of these.
        // Small workgroups that are all on the chip from the start, the first kNumCu one on each unit and the next ones beside them in
        // the same order: every other row of them is turned round, so that the longest sweep has the shortest beside it.
        {
            const bool turn = p->prefill_waves == kSmallWaves && (int64_t)n_wg_head * Hkv <= slots;
            const int row = std::max(1, kNumCu / Hkv);
            auto place = [&](int wg) {
                const int first = wg / row * row;
                return turn && (wg / row & 1) ? first + std::min(row, n_wg_head - first) - 1 - (wg - first) : wg;
            };
            int32_t next_record = n_wg_head;
            int32_t *before = nullptr;  // the record of the piece before, of the same workgroup
            for (size_t u = 0; u < w.pieces.size(); u++) {
                const PlanPiece &x = w.pieces[u];
                const PlanRowBlock &blk = w.blocks[x.block];
                const bool first = u == 0 || w.pieces[u - 1].wg != x.wg;
                const int32_t index = first ? place(x.wg) : next_record++;
                if (!first) before[RC_NEXT] = index;
                int32_t *r = H + off_records + (size_t)index * kRecordInts;
                r[RC_T0] = x.t0; r[RC_T1] = x.t1; r[RC_K] = blk.k; r[RC_C] = x.c;
                r[RC_REGION] = blk.k > 1 ? blk.slot0 : -1;
                r[RC_COUNTER] = blk.k > 1 ? counter_stride * first_counter[x.block] : 0; r[RC_CSTRIDE] = counter_stride;
                r[RC_NEXT] = -1;
                r[RC_POS0] = blk.pos0; r[RC_NPOS] = blk.npos; r[RC_QROW0] = p->q_start[blk.seq]; r[RC_CTX] = p->ctx_len[blk.seq];
                r[RC_PAGEOFF] = p->page_off[blk.seq];
                const int np = p->page_off[blk.seq + 1] - p->page_off[blk.seq];
                r[RC_NPAGES] = np; r[RC_BLOCK] = x.block; r[RC_BLOCK + 1] = 0;
                const int32_t *ids = H + off_pages + p->page_off[blk.seq];
                constexpr int kTilePages = kPrefillTileTokens / kBlock;
                for (int i = 0; i < kRecordInts - RC_IDS; i++) r[RC_IDS + i] = ids[std::min(x.t0 * kTilePages + i, np - 1)];  // past the end: the last page, never used
                before = r;
            }
        }
    }

    // ---- merge items of the (sequence, KV head) pairs with several teams, then the decode items
    w.slot0.assign((size_t)S * Hkv, -1);     // first partial slot of such a pair
    w.merge_of.assign((size_t)S * Hkv, -1);  // index of its merge item
    for (int s = 0; s < S; s++)
        for (int h = 0; h < Hkv; h++) {
            const int nt = w.n_teams[(size_t)s * Hkv + h];
            if (nt <= 1) continue;
            w.slot0[(size_t)s * Hkv + h] = next_slot;
            w.merge_of[(size_t)s * Hkv + h] = (int32_t)((mg - (H + off_merge)) / kItemInts);
            mg[MG_SEQ] = s; mg[MG_KVH] = h; mg[MG_QROW] = p->q_start[s]; mg[MG_SLOT0] = next_slot; mg[MG_NSPLIT] = nt;
            mg[MG_COUNTER] = counter_stride * next_counter++; mg[MG_NPOS] = 1; mg[MG_ITEM] = -1;
            mg += kItemInts;
            next_slot += nt;
        }
    int32_t *dc0 = H + off_decode;
    for (const PlanTeam &t : w.teams) {
        const int64_t kv = (int64_t)p->ctx_len[t.seq] + 1;
        const int32_t base = w.slot0[(size_t)t.seq * Hkv + t.h], merge = w.merge_of[(size_t)t.seq * Hkv + t.h];
        const int ns = splits_of(kv);
        // split i begins at page i * (pages / ns) + min(i, pages % ns)
        const int64_t pg = (kv + kBlock - 1) / kBlock, each = pg / ns, odd = pg % ns;
        int32_t *dc = dc0 + ((int64_t)t.wg * W + t.at) * kItemInts;
        const int32_t qrow = p->q_start[t.seq], page_off = p->page_off[t.seq], slot = base >= 0 ? base + t.idx : -1;
        int64_t begin = kBlock * ((int64_t)t.first * each + std::min<int64_t>(t.first, odd));
        for (int m = 0; m < t.n; m++, dc += kItemInts) {
            const int i = t.first + m + 1;
            const int64_t end = std::min<int64_t>(kv, kBlock * (i * each + std::min<int64_t>(i, odd)));
            dc[DC_SEQ] = t.seq; dc[DC_KVH] = t.h; dc[DC_BEGIN] = (int32_t)begin; dc[DC_END] = (int32_t)end;
            dc[DC_QROW] = qrow; dc[DC_SLOT] = slot; dc[DC_PAGEOFF] = page_off;
            dc[DC_TEAM] = t.n | (m << 4) | (end == kv ? kTeamTailBit : 0) | ((merge + 1) << 8);
            begin = end;
        }
    }
    for (size_t g = 0; g < w.wg_fill.size(); g++)  // wave slots no team took: padding items (no tokens, a team of their own)
        for (int at = w.wg_fill[g]; at < W; at++) {
            int32_t *dc = dc0 + ((int64_t)g * W + at) * kItemInts;
            dc[DC_SEQ] = -1; dc[DC_KVH] = 0; dc[DC_BEGIN] = dc[DC_END] = 0; dc[DC_QROW] = 0; dc[DC_SLOT] = -1; dc[DC_PAGEOFF] = 0; dc[DC_TEAM] = 1;
        }
    std::memset(H + off_counters, 0, n_counter_ints * sizeof(int32_t));

    p->S = S; p->T = S ? p->q_start[S] : 0;
    p->n_prefill_seqs = n_prefill_seqs; p->n_decode_seqs = n_decode_seqs;
    p->total_pages = pages;
    p->n_prefill = (int)n_prefill; p->n_pieces = (int)n_pieces; p->n_prefill_wg = (int)n_prefill_wg; p->n_decode = (int)n_decode;
    p->n_merge = (int)n_merge; p->n_partials = (int)n_partials; p->n_counters = (int)n_counters; p->n_append = (int)n_append;
    p->n_piece_partials = (int)n_piece_partials; p->n_merge_prefill = (int)n_merge_prefill;
    p->n_decode_wg = (int)n_decode_wg; p->n_dealt = (int)n_dealt; p->n_drawers = (int)n_drawers; p->counter_stride = counter_stride; p->queue_counter = queue || late_queue ? (int)off_queue : -1;
    p->off_records = off_records; p->off_append = off_append; p->off_pages = off_pages; p->off_valid = off_valid; p->off_prefill = off_prefill;
    p->off_decode = off_decode; p->off_merge = off_merge; p->off_counters = off_counters;
    p->host_n = total;
    return TC_OK;
}

}  // namespace tc

extern "C" {

static tc_status create_plan(const tc_kv_pool *pool, const tc_batch *batch, void *stream, bool on_device, tc_plan **out) {
    if (!out) { tc::set_error("out is NULL"); return TC_ERR_NULL; }
    *out = nullptr;
    tc_plan *p = new (std::nothrow) tc_plan();
    if (!p) { tc::set_error("out of host memory"); return TC_ERR_DEVICE; }
    p->on_device = on_device;
    tc_status st = on_device ? tc_plan_update(p, pool, batch, stream) : tc::build_plan(p, pool, batch);
    if (st != TC_OK) { tc_plan_destroy(p); return st; }
    *out = p;
    return TC_OK;
}

tc_status tc_plan_create_host(const tc_kv_pool *pool, const tc_batch *batch, tc_plan **out) {
    return create_plan(pool, batch, nullptr, false, out);
}

tc_status tc_plan_create(const tc_kv_pool *pool, const tc_batch *batch, void *stream, tc_plan **out) {
    return create_plan(pool, batch, stream, true, out);
}

tc_status tc_plan_update(tc_plan *p, const tc_kv_pool *pool, const tc_batch *batch, void *stream) {
    if (!p) { tc::set_error("plan is NULL"); return TC_ERR_NULL; }
    const auto t0 = std::chrono::steady_clock::now();
    tc_status st = tc::build_plan(p, pool, batch);
    const auto t1 = std::chrono::steady_clock::now();
    p->build_ns = std::chrono::duration_cast<std::chrono::nanoseconds>(t1 - t0).count();
    p->upload_ns = 0;
    if (st != TC_OK || !p->on_device) return st;
    int err = tc::upload_plan(p, stream);
    p->upload_ns = std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - t1).count();
    if (err) {
        tc::set_error(std::string("plan upload failed: ") + tc::hip_error_text(err));
        tc_batch none = {};
        (void)tc::build_plan(p, pool, &none);  // an empty plan: every call on it is a no-op
        return TC_ERR_DEVICE;
    }
    return TC_OK;
}

tc_status tc_plan_get_info(const tc_plan *p, tc_plan_info *info) {
    if (!p || !info) { tc::set_error("plan or info is NULL"); return TC_ERR_NULL; }
    std::memset(info, 0, sizeof *info);
    info->num_seqs = p->S; info->total_q = p->T;
    info->num_prefill_seqs = p->n_prefill_seqs; info->num_decode_seqs = p->n_decode_seqs;
    info->num_prefill_items = p->n_prefill; info->num_decode_items = p->n_decode;
    info->num_merge_items = p->n_merge; info->num_partials = p->n_partials; info->num_piece_partials = p->n_piece_partials;
    info->split_tokens = p->split_tokens; info->rows_per_prefill_item = p->rows_per_item;
    info->grid_blocks = p->grid_blocks(); info->block_threads = p->launch_threads();
    info->waves_per_item = p->waves_per_item;
    info->total_pages = p->total_pages;
    info->num_prefill_pieces = p->n_pieces;
    info->num_prefill_workgroups = p->n_prefill_wg;
    info->num_counters = p->n_counters;
    info->decode_queue = p->n_drawers > p->n_decode_wg;  // the prefill workgroups draw too
    info->build_ns = p->build_ns;
    info->upload_ns = p->upload_ns;
    return TC_OK;
}

// The pieces and workgroups of the launch, from the records that it reads: workgroup w * Hkv + h runs record w and those behind it for KV head h.
static void copy_pieces(const tc_plan *p, int32_t *pieces, size_t cap_pieces, int32_t *first, size_t cap_first) {
    size_t n = 0;
    for (int wg = 0; wg < p->n_prefill_wg; wg++) {
        const int h = wg % p->Hkv;
        if ((size_t)wg < cap_first) first[wg] = (int32_t)n;
        for (int i = wg / p->Hkv; i >= 0; n++) {
            const int32_t *r = p->host + p->off_records + (size_t)i * tc::kRecordInts;
            i = r[tc::RC_NEXT];
            if (n >= cap_pieces) continue;
            const bool cut = r[tc::RC_REGION] >= 0;
            int32_t *q = pieces + n * tc::kItemInts;
            q[tc::PP_ITEM] = r[tc::RC_BLOCK] * p->Hkv + h; q[tc::PP_T0] = r[tc::RC_T0]; q[tc::PP_T1] = r[tc::RC_T1];
            q[tc::PP_SLOT] = cut ? r[tc::RC_REGION] + h * r[tc::RC_K] : -1;
            q[tc::PP_K] = r[tc::RC_K]; q[tc::PP_C] = r[tc::RC_C];
            q[tc::PP_COUNTER] = cut ? (r[tc::RC_COUNTER] + h * r[tc::RC_CSTRIDE]) / p->counter_stride : -1;
            q[tc::PP_LAST] = i < 0;
        }
    }
}

tc_status tc_plan_copy_items(const tc_plan *p, int32_t kind, int32_t *dst, size_t cap_items) {
    if (!p || !dst) { tc::set_error("plan or dst is NULL"); return TC_ERR_NULL; }
    size_t off, n;
    if (kind == 0) { off = p->off_prefill; n = p->n_prefill; }
    else if (kind == 1) { off = p->off_decode; n = p->n_decode; }
    else if (kind == 2) { off = p->off_merge; n = p->n_merge; }
    else if (kind == 3) { copy_pieces(p, dst, cap_items, nullptr, 0); return TC_OK; }
    else if (kind == 4) { copy_pieces(p, nullptr, 0, dst, cap_items); return TC_OK; }  // plain int32, not 8-int items
    else { tc::set_error("kind must be 0, 1, 2, 3 or 4"); return TC_ERR_ARG; }
    n = std::min(n, cap_items);
    if (n) std::memcpy(dst, p->host + off, n * tc::kItemInts * sizeof(int32_t));
    if (kind == 2)  // the image says where a counter lies, the item which one it is
        for (size_t i = 0; i < n; i++) dst[i * tc::kItemInts + tc::MG_COUNTER] /= p->counter_stride;
    return TC_OK;
}

size_t tc_plan_workspace_bytes(const tc_plan *p) { return p ? p->workspace_bytes() : 0; }

void tc_plan_destroy(tc_plan *p) {
    if (!p) return;
    tc::free_plan_buffers(p);
    delete p;
}

const char *tc_status_str(tc_status s) {
    switch (s) {
        case TC_OK: return "TC_OK";
        case TC_ERR_NULL: return "TC_ERR_NULL";
        case TC_ERR_SHAPE: return "TC_ERR_SHAPE";
        case TC_ERR_SPAN: return "TC_ERR_SPAN";
        case TC_ERR_BLOCK: return "TC_ERR_BLOCK";
        case TC_ERR_WORKSPACE: return "TC_ERR_WORKSPACE";
        case TC_ERR_DEVICE: return "TC_ERR_DEVICE";
        case TC_ERR_ARG: return "TC_ERR_ARG";
    }
    return "TC_ERR_UNKNOWN";
}

const char *tc_last_error(void) { return tc::g_last_error.c_str(); }

int32_t tc_version(void) { return 2; }

}  // extern "C"
