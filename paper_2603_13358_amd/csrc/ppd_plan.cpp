// Host planner of the one-launch mixed step: classifies sequences, splits key ranges, orders tiles.
//
// Per sequence (L cached, n new; paper section 4.1 with L = the paper's n and n = its m): n*G <= 16 query
// columns -> narrow tiles (decode is n = 1), else row blocks of 256/G rows on the MFMA path.  A tile is
// (sequence, KV head, row block, key range); key ranges are split only as far as filling and balancing the
// workgroups needs, and tiles run longest-first from nine queues (one of narrow tiles, eight of row-block tiles,
// one per XCD) so that HBM-bound narrow tiles and MFMA-bound row-block tiles run side by side on the chip.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <unordered_map>

#include "ppd_internal.h"

namespace ppd {

ppd_status validate_shape(const ppd_shape* s, const char** err) {
    static const char* kNull = "shape is NULL";
    static const char* kDim = "head_dim must be 64 or 128";
    static const char* kPageSz = "page_size must be 16";
    static const char* kHeads = "num_q_heads must be G * num_kv_heads with 1 <= G <= 8, num_kv_heads >= 1";
    static const char* kPages = "num_pages must be >= 1 and the pool below 2^40 elements";
    const char* dummy;
    if (!err) err = &dummy;
    if (!s) { *err = kNull; return PPD_ERR_NULL; }
    if (s->head_dim != 64 && s->head_dim != 128) { *err = kDim; return PPD_ERR_SHAPE; }
    if (s->page_size != kPage) { *err = kPageSz; return PPD_ERR_SHAPE; }
    if (s->num_kv_heads < 1 || s->num_q_heads < 1 || s->num_q_heads % s->num_kv_heads != 0) {
        *err = kHeads; return PPD_ERR_SHAPE;
    }
    int G = s->num_q_heads / s->num_kv_heads;
    if (G < 1 || G > 8) { *err = kHeads; return PPD_ERR_SHAPE; }
    if (s->num_kv_heads > 1024) { *err = kHeads; return PPD_ERR_SHAPE; }
    if (s->num_pages < 1 || s->num_pages > (int64_t(1) << 40) / (2LL * s->num_kv_heads * kPage * s->head_dim)) {
        *err = kPages; return PPD_ERR_SHAPE;
    }
    return PPD_OK;
}

static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Splits [0, len) into pieces of at most ~chunk tokens with boundaries on multiples of kTileTokens.
static void split_range(int64_t len, int64_t chunk, std::vector<int32_t>* bounds) {
    bounds->clear();
    int64_t nsplit = std::max<int64_t>(1, (len + chunk - 1) / chunk);
    int64_t per = round_up((len + nsplit - 1) / nsplit, kTileTokens);
    for (int64_t b = 0; b < len; b += per) bounds->push_back((int32_t)b);
    bounds->push_back((int32_t)len);
}

// Split size of the MFMA row-block tiles.  Every split costs a partial (fp32 o, m, l per column) that the tile
// writes and a separate merge launch reads back; not splitting leaves few, long tiles that may not fill or balance
// the workgroups.  The choice is made by estimate: for each candidate size the row blocks are cut (all KV heads
// alike), their tiles list-scheduled longest-first, at kTileStartUs + kTileIterUs per 64 keys, onto the
// workgroups that will take MFMA tiles first in the launch; the launch then takes the longer of that schedule and
// of all work spread evenly over all workgroups (narrow tiles included: a compute unit streams ~45 GB/s, HBM
// delivers ~6.5 TB/s to all of them together), plus the cost of the partials.  Candidates run from whole key ranges
// downwards and stop once there are far more tiles than workgroups.  Constants fitted to measured launches
// (append-prefill batches of 2..16 sequences, 256 workgroups): the estimate is within ~8 % of the kernel time and
// ranks the candidates of one batch correctly.
struct RowBlock { int64_t vis_end; int32_t nrows; };

// Compute units (of the 32 of an XCD) whose workgroups take narrow tiles first.  A workgroup of the mixed kernel
// fills a compute unit (8 waves of up to 256 registers), so the two kinds are split by physical unit: narrow tiles are
// bound by the bytes a unit keeps in flight (about 45 GB/s each), MFMA tiles by compute, and the split is sized so that
// both kinds finish together; whoever finishes first steals from the other anyway.
// A unit streams FP8 pages at about 38 GB/s: its loads are 8 bytes per lane instead of 16 and 8, and a unit's memory
// pipeline moves fewer bytes per second with narrower loads (about 58 GB/s at best, with contiguous 16-byte loads).
static double unit_bytes_per_us(int elem_bytes) { return elem_bytes == 1 ? 38e3 : 45e3; }

// What 64 keys of a row block are priced at.  The loop itself takes 1.9 us on either format while every unit runs it (the
// chip is then at its power limit) and less beside streaming units; the three prices below are fits of three
// different estimates, not measurements of it.
//  - the split of the units: swept over seven mixed steps on bf16 pages the best split lay within two units of what 1.5 gives, and
//    2.3 cost 1-4 % (60 decodes beside 4 turns, 64 query heads, 16 -> 18 units: 358 -> 346 us; 128 long decodes beside 4 long
//    turns, 14 -> 18: 3249 -> 3133 us a layer pair); on FP8 pages 2.3 is within 1 % of the best.
//  - the units left to row blocks while their split size is chosen: with 1.5 it splits more row blocks, and one batch in
//    forty then needs more room for its partials than the fixed scratch array has.
//  - the tiles of that choice: kTileIterUs there, with the cost of a tile's start beside it.
static double split_of_units_iter_us(int elem_bytes) { return elem_bytes == 1 ? 2.3 : 1.5; }
constexpr double kChunkChoiceIterUs = 2.3;
static int narrow_units(double narrow_bytes, double mfma_iters, int elem_bytes, double iter_us) {
    if (narrow_bytes == 0) return 0;
    if (mfma_iters == 0) return 32;
    const double narrow_cu_us = narrow_bytes / unit_bytes_per_us(elem_bytes);  // CU-microseconds
    const double mfma_us = mfma_iters * iter_us / kWgPerCu;
    const int cus = (int)std::lround(32.0 * narrow_cu_us / (narrow_cu_us + mfma_us));
    return std::min(std::max(cus, 2), 20);            // HBM saturates well before all units stream
}

static int64_t choose_mfma_chunk(const std::vector<RowBlock>& blocks, int G, int Hkv, int D, int slots,
                                 double narrow_bytes, int elem_bytes) {
    constexpr double kTileStartUs = 16.0;
    // 1.7 us per 64 keys at D = 128; at D = 64 the two products halve and the softmax stays (measured ~0.65x)
    const double kTileIterUs = 1.7 * (0.3 + 0.7 * D / 128.0);
    constexpr double kMergeLaunchUs = 12.0, kPartialBytesPerUs = 2.5e6;
    constexpr double kHbmBytesPerUs = 6.5e6;
    const double kUnitBytesPerUs = unit_bytes_per_us(elem_bytes);
    static const int64_t kCandidates[] = {32768, 24576, 16384, 12288, 8192, 6144, 4096, 3072, 2048, 1024, 512};
    const double narrow_work = narrow_bytes / kUnitBytesPerUs;  // unit-microseconds
    const double narrow_floor = narrow_bytes / kHbmBytesPerUs;  // however many units stream
    int64_t best_chunk = kCandidates[0];
    double best = -1.0, even_first = -1.0;
    std::vector<double> tiles, load;
    std::vector<int32_t> bounds;
    for (int64_t c : kCandidates) {
        tiles.clear();
        double partial_bytes = 0, mfma_work = 0, iters = 0;
        for (const RowBlock& rb : blocks) {
            split_range(rb.vis_end, c, &bounds);
            const int nsplit = (int)bounds.size() - 1;
            for (int k = 0; k < nsplit; ++k) {
                const double it = (double)((bounds[k + 1] - bounds[k] + kTileTokens - 1) / kTileTokens);
                tiles.push_back(kTileStartUs + kTileIterUs * it);
                mfma_work += tiles.back() * Hkv;
                iters += it * Hkv;
            }
            if (nsplit > 1) partial_bytes += (double)rb.nrows * G * (D + 2) * 4.0 * nsplit * Hkv;
        }
        // the workgroups that take MFMA tiles first, as the launch will split them
        const int S = std::max(1, slots - narrow_units(narrow_bytes, iters, elem_bytes, kChunkChoiceIterUs) * slots / 32);
        std::sort(tiles.begin(), tiles.end(), std::greater<double>());
        load.assign((size_t)S, 0.0);  // min-heap of workgroup finish times; the earliest workgroup takes the next tile
        for (double t : tiles)
            for (int h = 0; h < Hkv; ++h) {
                load[0] += t;
                for (size_t at = 0;;) {  // sift the grown root down
                    size_t kid = 2 * at + 1;
                    if (kid >= (size_t)S) break;
                    if (kid + 1 < (size_t)S && load[kid + 1] < load[kid]) ++kid;
                    if (load[at] <= load[kid]) break;
                    std::swap(load[at], load[kid]);
                    at = kid;
                }
            }
        const double makespan = *std::max_element(load.begin(), load.end());
        const double even = std::max((mfma_work + narrow_work) / slots, narrow_floor);
        const double est = std::max(makespan, even) +
                           (partial_bytes > 0 ? kMergeLaunchUs + partial_bytes / kPartialBytesPerUs : 0.0);
        if (best < 0 || est < 0.99 * best) {  // a smaller chunk has to win clearly
            best = est;
            best_chunk = c;
        }
        if ((int64_t)tiles.size() * Hkv > 16LL * S) break;  // plenty of tiles already: smaller pieces only add partials
        // Smaller pieces only add tiles, so `even` never falls below what the first candidate gives, and no later
        // estimate can be below it: once the best estimate is within 1 % of that bound nothing can still win.
        if (even_first < 0) even_first = even;
        if (0.99 * best <= even_first) break;
    }
    return best_chunk;
}

// Split size of the narrow tiles of a launch that has nothing else and fewer (sequence, KV head) pairs than twice the
// workgroups: the few-sequences, long-context corner, where the fixed rule below leaves compute units idle or
// the last round of tiles nearly empty.  Estimate per candidate: tiles longest-first in rounds of `slots`; a round
// takes kStartUs plus its longest tile at what a unit streams (kUnitBytesPerUs, or its share of kHbmBytesPerUs
// when more units stream than HBM can feed); a split range costs a merge launch plus kMergeSplitUs per split
// (the merge walks the splits of a column one after the other).  Constants fitted to 114 measured launches
// (1..16 sequences x 4K..256K context x six split sizes; log-error 11 % rms, the pick within 3 % of the best
// measured size in all 19 batches).
static int64_t choose_narrow_chunk(const std::vector<int64_t>& lengths, int Hkv, int D, int slots, int elem_bytes) {
    constexpr double kStartUs = 7.0, kHbmBytesPerUs = 7.0e6;
    const double kUnitBytesPerUs = elem_bytes == 1 ? 44e3 : 55e3;
    constexpr double kMergeUs = 4.0, kMergeSplitUs = 0.3;
    static const int64_t kCandidates[] = {8192, 6144, 4096, 3072, 2048, 1536, 1024, 768, 512};
    const double bytes_per_key = 2.0 * D * elem_bytes;
    int64_t best_chunk = kCandidates[0];
    double best = -1.0;
    std::vector<int32_t> tiles, bounds;
    for (int64_t c : kCandidates) {
        tiles.clear();
        int max_split = 1;
        for (int64_t len : lengths) {
            split_range(len, c, &bounds);
            const int nsplit = (int)bounds.size() - 1;
            max_split = std::max(max_split, nsplit);
            for (int k = 0; k < nsplit; ++k)
                for (int h = 0; h < Hkv; ++h) tiles.push_back(bounds[k + 1] - bounds[k]);
        }
        if ((int64_t)tiles.size() > 8LL * slots && best >= 0) break;  // more than enough tiles: stop refining
        std::sort(tiles.begin(), tiles.end(), std::greater<int32_t>());
        double est = max_split > 1 ? kMergeUs + kMergeSplitUs * max_split : 0.0;
        for (size_t j = 0; j < tiles.size(); j += (size_t)slots) {
            const double streaming = (double)std::min<size_t>((size_t)slots, tiles.size() - j);
            const double rate = std::min(kUnitBytesPerUs, kHbmBytesPerUs / streaming);
            est += kStartUs + tiles[j] * bytes_per_key / rate;
        }
        if (best < 0 || est < 0.99 * best) {  // a smaller chunk has to win clearly
            best = est;
            best_chunk = c;
        }
    }
    return best_chunk;
}

// Whether the tiles of a decode-only launch run on four waves (kStreamingWaves; D = 128, bf16 pages, a multiple of 8 KV heads)
// instead of eight.  Where every unit streams long tiles one after the other, HBM is the bound, and it delivers more to half the waves, each with one more
// page in flight: us of 128 sequences of 7000-8000 keys by 8 heads 597 -> 574 (6.6 -> 6.9 TB/s), 64 of 3200-6400 192.8 -> 187.0, 128
// of 1000-8000 345 -> 339, 256 of them 697 -> 687.  A unit alone streams less that way (42 against 52 GB/s): launches of less than
// two rounds stay on eight waves (16 sequences of 3200-6400 keys 70 -> 83), and so do tiles below 3072 keys, where the gain ends
// (256 of 1600-2000 297 -> 298, 32 of 3200-6400, 512 tiles of 2400, 103.9 -> 107.2).  For the same reason the last round counts:
// while fewer than 70 % of the units have a tile they lose what the full ones won, unless what is left by then is short.  Equal
// tiles, four waves against eight: 2.2 rounds 225 against 206 us, 3.2 277 and 261, 5.1 439 and 423, 2.97 330 and 338.  And the KV
// heads: where they are not a multiple of the 8 XCDs the full rounds win nothing (220 drawn launches under the rule: 8 heads 1.8 % on
// average, -1.5 at worst, 16 heads 1.7 %, 12 heads 0.1, 4 heads -0.3, 1, 2 and 6 heads -0.1 to -0.5).
// By the device's workgroups, not by a grid override: the two forms round differently, and that option stays scheduling only.
static bool long_tiles_on_four_waves(const Plan& plan, int64_t wgs, int head_dim, int num_kv_heads, int elem_bytes) {
    const int n = plan.queue_begin[kQueues];
    if (head_dim != 128 || elem_bytes != 2 || num_kv_heads % kXcds != 0 || n < 2 * wgs || plan.queue_begin[kWaveQueue] != n) return false;
    auto keys = [&](int64_t i) { return (int64_t)(plan.items[i].kv_end - plan.items[i].kv_begin); };
    int64_t sum = 0;
    for (int i = 0; i < n; ++i) sum += keys(i);
    if (sum / n < 3072) return false;
    const int64_t last = n % wgs;  // tiles of the last round, the shortest ones
    return last == 0 || 10 * last >= 7 * wgs || 7 * keys(n - last) <= sum / wgs;
}

// Whether a decode-only launch of more slots than workgroups hands its second round out by index (ppd_narrow_kernel) instead of
// by claims.  Asked where no other form takes the launch: on bf16 pages the shortest tiles of about one length run pipelined, so the figures
// below 640 keys (1280 at D = 64) there are what led to the rule and now apply to one-wave slots and lengths further apart.  Workgroup b gets slot b and slot 2 * wgs - 1 - b.  By index where that costs no more than any order must:
//  * at most two rounds, of tiles below 1536 keys of bf16 pages or 3072 of FP8 pages (figures at the kernel);
//  * the heaviest workgroup's two slots are at most 96 KiB of K/V above what no order can undercut -- the longest slot, the mean
//    of the workgroups, or the two shortest slots of which two must share a workgroup -- where a slot's fixed cost counts as
//    128 KiB.  Equal and evenly spread lengths pair off to almost nothing above it; a long tile among short ones gets another
//    behind it, where claims would leave it alone (us of 64 sequences of 800 keys, one of them 2.4 and 4 times as long, claimed
//    43.8 and 49.0, by index 46.0 and 58.3; of log-normal lengths around 800 keys 40.6 and 42.5, at D = 64 25.6 and 28.6; 202 of
//    205 keys on single waves and 10 of 530 39.1 and 46.1);
//  * in a second round of less than a quarter, slots there below 256 KiB: a few workgroups decide such a step, and claims give
//    them to those that are done first (264, 288, 304 and 320 tiles by 256 workgroups, by index against claimed: 1500
//    keys of bf16 pages -4.1, -2.6, -1.0, +0.7 %, 1000 keys -3.1, -1.2, +0.4, +1.9, 600 keys -1.3, -0.4, +1.2, +2.5, 300 keys +6
//    at 288; 3000 keys of FP8 pages -2.2, -1.3, -1.3, -0.4, 1200 keys -0.1, +1.2, +1.6, +2.3; D = 64, 1200 keys of bf16 pages
//    -1.8, +1.2, +1.1, +1.4, 1000 keys +0.8, +1.3, +2.7, +3.3); of three eighths where they are of one-wave tiles (264, 320 and
//    400 slots of 300 keys, bf16 pages -3.9, -0.8 and +1.1 %, D = 64 -4.1, -2.8 and -0.5).
// Over 558 launches of 33-64 sequences (equal, spread and log-normal around 250-3000 keys, both formats and head sizes) 5.4 % less
// time than claims on average, over 800 of 264-500 sequences on single waves 2.4 %, -3.1 % at worst; every second round by index 5.1
// and 1.9 % on average and up to 17 % more time at worst.
static bool second_round_by_index(const Plan& plan, int64_t wgs, int head_dim, int elem_bytes) {
    const int n_wg = plan.queue_begin[kWaveQueue], n_items = plan.queue_begin[kQueues];
    const int64_t slots = n_wg + ((int64_t)n_items - n_wg + kNarrowKernelWaves - 1) / kNarrowKernelWaves;
    if (slots <= wgs || slots > 2 * wgs) return false;
    constexpr int64_t kFixed = 128 * 1024, kAbove = 96 * 1024, kShort = 256 * 1024;
    const int64_t key_bytes = 2LL * head_dim * elem_bytes;
    std::vector<int64_t> cost((size_t)slots, 0);
    int64_t keys = 0;
    for (int i = 0; i < n_items; ++i) {
        const int64_t k = plan.items[i].kv_end - plan.items[i].kv_begin;
        cost[i < n_wg ? i : n_wg + (i - n_wg) / kNarrowKernelWaves] += k * key_bytes;
        keys += k;
    }
    if (keys / n_items * elem_bytes >= 3072) return false;
    if (8 * slots < (wgs < n_wg ? 10 : 11) * wgs && cost[wgs] >= kShort) return false;
    int64_t sum = 0, longest = 0, heaviest = 0;
    for (int64_t b = 0; b < slots; ++b) {
        if (b >= n_wg) cost[b] = cost[b] * 3 / 2 + kFixed;  // single waves start and stream slower: 370 keys of FP8 pages, D = 64, 16 us
        cost[b] += kFixed;
        sum += cost[b];
    }
    for (int64_t b = 0; b < slots; ++b) {
        longest = std::max(longest, cost[b]);
        if (b < wgs) heaviest = std::max(heaviest, cost[b] + (2 * wgs - 1 - b < slots ? cost[2 * wgs - 1 - b] : 0));
    }
    // (tiles are in order of their length, but a slot of eight one-wave tiles may take longer than the whole-workgroup tiles before it)
    if (!std::is_sorted(cost.begin(), cost.end(), std::greater<int64_t>())) std::sort(cost.begin(), cost.end(), std::greater<int64_t>());
    return heaviest <= std::max({longest, sum / wgs, cost[wgs - 1] + cost[wgs]}) + kAbove;
}

// Whether the whole-workgroup tiles of a decode-only launch on bf16 pages run in ppd_pipelined_kernel where a workgroup gets more than one.
// What it saves is the gap between two tiles, which counts while tiles are short; and it holds three tiles ahead, so that a workgroup
// with one far longer than the others keeps what an idle one could have run.  Not, against tiles one after the other:
//  * above 320 KiB on average, 625 keys at D = 128 and 1250 at D = 64 (181 drawn launches of 257-2500 tiles: up to 300 keys 8-13 % less time,
//    300-900 2-3, 900-2500 1 % more; at D = 64 300-900 9, 900-1300 7);
//  * the longest above 3 times the average, from 150 KiB on 1.7 and from 200 on 1.5 (beyond 3 11 % more; 1000 tiles of 519 keys, the longest 1.66
//    times that, 47.9 -> 50.5 us, 846 around 420 keys 38.7 -> 42.8);
//  * a workgroup's first three tiles, which go by index (up, down and up the list, the longest ones with two more behind them), 96 KiB above what no
//    order can undercut, a tile's fixed cost counted as 64 KiB (544 tiles of 263 keys, an eighth of them 2.3 times that, 20.7 -> 22.4 us, 576 20.5 -> 22.1; of 294
//    drawn launches of two to three rounds 7 of 68 above it were slower by more than 1 %, by up to 8.3, and 3 of 226 below, by up to 2.8);
//  * more than eight columns (of several rows) in a second round, or with split ranges: 3 and 1 % less time on average there, up to 3 and
//    6.7 % more.
// Of 1800 drawn launches that it takes (bf16 pages, both head sizes, 1-16 KV heads, up to four rows, 400 with split ranges) 7 are slower by
// more than 1 %, by 2.8 at most; they take 0.91 of the time (0.95 with split ranges).
static bool tiles_pipelined(const Plan& plan, int64_t wgs, int head_dim, int G, int elem_bytes) {
    const int64_t n = plan.queue_begin[kQueues];
    if (elem_bytes != 2 || n <= wgs || plan.queue_begin[kWaveQueue] != n) return false;
    constexpr int64_t kFixed = 64 << 10, kAbove = 96 << 10, kLongest = 320 << 10, kEven = 200 << 10, kShort = 150 << 10;
    const int64_t key_bytes = 2LL * head_dim * elem_bytes;
    auto bytes = [&](int64_t i) { return (plan.items[i].kv_end - plan.items[i].kv_begin) * key_bytes; };
    int64_t sum = 0;
    int32_t columns = 0;
    for (int64_t i = 0; i < n; ++i) {
        sum += bytes(i);
        columns = std::max(columns, plan.items[i].nrows * G);
    }
    static_assert(kMaxPipelinedKeys >= 3 * kLongest / (2 * 64 * 2), "a wave's share of the longest tile fits its page ids");
    const int64_t mean = sum / n, tenths = mean <= kShort ? 30 : mean <= kEven ? 17 : 15;
    if (mean > kLongest || bytes(0) * n * 10 > sum * tenths) return false;
    if (columns > 8 && (n <= 2 * wgs || !plan.groups.empty())) return false;
    auto cost = [&](int64_t i) { return i < n ? bytes(i) + kFixed : 0; };
    const int64_t least = std::max({cost(0), sum / wgs + n * kFixed / wgs, cost(wgs - 1) + cost(wgs), cost(2 * wgs - 2) + cost(2 * wgs - 1) + cost(2 * wgs)});
    for (int64_t b = 0; b < wgs; ++b)
        if (cost(b) + cost(2 * wgs - 1 - b) + cost(2 * wgs + b) > least + kAbove) return false;
    return true;
}

// Whether every tile of a decode-only launch runs on one wave (ppd_wave_kernel), and in units of how many neighbours (0: no).  By
// estimate, against the tiles on whole workgroups:
//  * on whole workgroups a launch takes 6 us, 2.15 per round of tiles (3.3 on FP8 pages; tiles that the list already has on single waves
//    count an eighth), and its bytes at 7.2 TB/s;
//  * on waves it takes the longer of two flows of the bytes out of HBM at 6.7 TB/s: to the compute units, of which none takes more
//    than 40 GB/s (FP8 pages at D = 64: 24), and to the waves' chains of tiles, of which none takes more than 12 GB/s (6 at D = 64; FP8
//    pages 8 and 5).  All take the same until the one with the least to read is done, and the others share what it took; then 4 us (6),
//    and 4 more in the second round of bf16 pages.
// What has to come out (8 %, 6 in the second round, on FP8 pages 4, at D = 64 6, in units of one 10) is where no drawn launch that was taken is
// slower by more than two runs differ: of 2200 launches (bf16 and FP8 pages, both head sizes, 1-16 KV heads, up to four rows, equal, spread and
// log-normal lengths around 60-4000 keys, a few longer ones among equal ones) 2 are, by 1.2 and 2.3 %.  bf16 pages take 0.81 of the time (800
// launches), FP8 pages 0.79 (900 of 640 tiles and more) and 0.64 (500 of fewer).  With one rate for both head sizes of FP8 pages and 4 %
// everywhere 73 of 2300 were slower: 1296 tiles of 3239 keys of FP8 pages at D = 64 107 -> 128 us, 5296 tiles of 669 keys of bf16 pages 283 -> 299.
// Not by the estimate:
//  * Split ranges stay on whole workgroups, which merge them.
//  * More tiles than one round of the chip's waves and fewer than two stay there.  That is not where waves stop winning: 257 sequences of
//    64-700 keys by 8 heads 65 us against 76, 511 125 against 139, FP8 pages 39 against 60 and 67 against 90, and of 120 drawn launches that
//    the estimate would take on average 0.97 of the time on bf16 pages (0.86-1.06) and 0.80 on FP8 pages (0.52-1.06).  The line stands
//    because whole workgroups give the mixed kernel's results bit for bit, which batches of that size are tested for.
//  * Two rounds of waves and more on bf16 pages at D = 128: 2.5 % less time on average where HBM bounds both, and 34 of 197 launches slower, by up to 5.6 %.
//    And two rounds of which the list has seven eighths on single waves already (5539 tiles of 80 keys of FP8 pages at D = 64 21.6 -> 24.7 us), and
//    lists that are all on them (at most 384 keys each, and 1536 of them: 80 launches that the estimate would take -15 to +23 %, 2.6 % more on average).
//  * Below two and a half tiles for each compute unit on bf16 pages, where ppd_pipelined_kernel runs them.
//  * Up to two tiles for each workgroup on FP8 pages, a longest one of more than 176 keys: the second round by index (second_round_by_index) takes 9 us
//    there at D = 64 and 11 at D = 128, a wave 4.5 and 20 ns a key (443 tiles of 197 keys 8.7 -> 9.7 us, 436 of 204 at D = 128 11.3 -> 11.8; 424 of 164 9.1 -> 8.7).
// Units of two where there are fewer than six tiles for each compute unit: more units have work then (640-1100 tiles 1.3 % less time).
// By the device's workgroups, not by a grid override: the forms round differently, and that option stays scheduling only.
static int32_t tiles_on_waves(const Plan& plan, int64_t wgs, int head_dim, int elem_bytes) {
    const int64_t n = plan.queue_begin[kQueues], n_wg = plan.queue_begin[kWaveQueue];
    const bool fp8 = elem_bytes == 1;
    if (fp8 ? n <= wgs : 2 * n < 5 * wgs) return 0;
    const bool rounds_of_waves = n > kWaves * wgs;
    if ((rounds_of_waves && n < 2 * kWaves * wgs) || n_wg == 0 || !plan.groups.empty()) return 0;
    if (rounds_of_waves && (8 * n_wg < n || (!fp8 && head_dim == 128))) return 0;
    if (fp8 && n <= 2 * wgs && plan.items[0].kv_end - plan.items[0].kv_begin > 176) return 0;
    const double key_bytes = 2.0 * head_dim * elem_bytes;
    constexpr double kHbm = 6.7e6;  // bytes per us
    const double unit_rate = fp8 && head_dim == 64 ? 24e3 : 40e3;
    const double wave_rate = fp8 ? (head_dim == 64 ? 5e3 : 8e3) : (head_dim == 64 ? 6e3 : 12e3);
    const int64_t unit = n >= 6 * wgs ? 4 : 2 * n >= 5 * wgs ? 2 : 1, groups = kWaves / unit;
    auto bytes_of = [&](int64_t i) { return (plan.items[i].kv_end - plan.items[i].kv_begin) * key_bytes; };
    double bytes = 0;
    for (int64_t i = 0; i < n; ++i) bytes += bytes_of(i);
    const double rounds = ((double)n_wg + (double)(n - n_wg) / kWaves) / (double)wgs;
    const double on_workgroups = 6.0 + (fp8 ? 3.3 : 2.15) * rounds + bytes / 7.2e6;
    const double wins = unit == 1 ? 0.90 : fp8 ? (head_dim == 64 ? 0.94 : 0.96) : rounds_of_waves ? 0.94 : 0.92;
    const double fixed = (fp8 ? 6.0 : 4.0) + (rounds_of_waves && !fp8 ? 4.0 : 0.0);
    const double at_most = wins * on_workgroups - fixed;  // us, of the flows
    // Neither flow is over before HBM has delivered all bytes and a wave the longest tile.  That answers most launches, and the flows take
    // the host as long as the rest of a small plan (64 sequences of FP8 pages by 8 heads 65.6 -> 32.1 us, 31.7 without the estimate).
    if (std::max(bytes / kHbm, bytes_of(0) / wave_rate) >= at_most) return 0;
    // As ppd_wave_kernel deals the units, in ascending order where no chain has two of them.
    std::vector<double> units((size_t)wgs, 0.0), chains((size_t)(wgs * groups), 0.0);
    for (int64_t u = 0; u * unit < n; ++u) {
        const int64_t round = u / wgs, at = u % wgs, wg = round & 1 ? wgs - 1 - at : at;
        for (int64_t i = u * unit; i < std::min(n, (u + 1) * unit); ++i) units[wgs - 1 - wg] += bytes_of(i);
        chains[wgs * groups - 1 - (round % groups * wgs + at)] += bytes_of(u * unit);  // (groups is even: a chain is one place of every round)
    }
    auto flow = [&](std::vector<double>& loads, double each, int64_t readers) {  // us; a load is that of `readers` waves
        if (!std::is_sorted(loads.begin(), loads.end())) std::sort(loads.begin(), loads.end());
        double t = 0, level = 0;
        for (size_t i = 0; i < loads.size(); ++i) {
            t += (loads[i] - level) * std::max(1 / each, (double)((loads.size() - i) * readers) * (1 / kHbm));
            level = loads[i];
        }
        return t;
    };
    return std::max(flow(units, unit_rate, 1), flow(chains, wave_rate, unit)) < at_most ? (int32_t)unit : 0;
}

ppd_status build_plan(const ppd_shape& s, const int32_t* L, const int32_t* n, int32_t B, const PlanOptions& o,
                      Plan* plan, const char** err) {
    static const char* kNull = "L / n is NULL";
    static const char* kNeg = "n_i must be >= 1 and L_i >= 0";
    static const char* kBig = "L_i + n_i and the total row count must stay below 2^30";
    static const char* kTiles = "the batch needs more than 2^22 tiles: too large for one launch";
    static const char* kChunk = "chunk options must be 0 or a positive multiple of 64 (mfma_chunk <= 32768); grid >= 0";
    const char* dummy;
    if (!err) err = &dummy;
    plan->items.clear();
    plan->groups.clear();
    plan->units.clear();
    std::memset(&plan->stats, 0, sizeof plan->stats);
    std::memset(plan->queue_begin, 0, sizeof plan->queue_begin);
    if (B < 0) { *err = kNeg; return PPD_ERR_RANGE; }
    if (B > 0 && (!L || !n)) { *err = kNull; return PPD_ERR_NULL; }
    if (o.narrow_chunk < 0 || o.narrow_chunk % kTileTokens || o.mfma_chunk < 0 || o.mfma_chunk % kTileTokens ||
        o.mfma_chunk > kMaxMfmaChunk || o.grid < 0 || o.num_cus < 1) {
        *err = kChunk; return PPD_ERR_RANGE;
    }
    const int D = s.head_dim, Hq = s.num_q_heads, Hkv = s.num_kv_heads, G = Hq / Hkv;
    const int64_t kv_tok_bytes_head = 2LL * D * (o.kv_elem_bytes == 1 ? 1 : 2);  // K and V of one token of one KV head
    int64_t rows = 0;
    double flops = 0;
    int64_t kv_tokens = 0;
    for (int i = 0; i < B; ++i) {
        if (n[i] < 1 || L[i] < 0) { *err = kNeg; return PPD_ERR_RANGE; }
        if ((int64_t)L[i] + n[i] >= (1 << 30)) { *err = kBig; return PPD_ERR_RANGE; }
        rows += n[i];
        kv_tokens += (int64_t)L[i] + n[i];
        flops += 4.0 * Hq * D * ((double)n[i] * L[i] + (double)n[i] * ((double)n[i] + 1) / 2);
    }
    if (rows >= (1 << 30)) { *err = kBig; return PPD_ERR_RANGE; }

    auto is_narrow = [&](int i) { return o.force_kind != 1 && (int64_t)n[i] * G <= kNarrowCols; };
    const int rows_per_block = kMfmaCols / G;

    double narrow_tokens = 0;          // keys of the narrow tiles, counted once per KV head
    std::vector<int64_t> narrow_lengths;
    std::vector<RowBlock> row_blocks;  // of one KV head
    for (int i = 0; i < B; ++i) {
        if (is_narrow(i)) {
            narrow_tokens += (double)Hkv * (L[i] + n[i]);
            narrow_lengths.push_back((int64_t)L[i] + n[i]);
        } else {
            const int64_t blocks = ((int64_t)n[i] + rows_per_block - 1) / rows_per_block;
            if (((int64_t)row_blocks.size() + blocks) * Hkv > kMaxTiles) { *err = kTiles; return PPD_ERR_RANGE; }
            for (int r0 = 0; r0 < n[i]; r0 += rows_per_block) {
                const int nrows = std::min(rows_per_block, n[i] - r0);
                const int64_t vis_end = (int64_t)L[i] + r0 + nrows;
                row_blocks.push_back(RowBlock{vis_end, nrows});
            }
        }
    }
    if ((int64_t)(row_blocks.size() + narrow_lengths.size()) * Hkv > kMaxTiles) { *err = kTiles; return PPD_ERR_RANGE; }
    const int slots = o.grid > 0 ? o.grid : kWgPerCu * o.num_cus;  // resident workgroups
    // Narrow tiles: every split costs a partial and, above all, a gap in the workgroup's stream of loads (claim,
    // page ids, first loads: ~8 us), so key ranges stay whole unless the batch is too small to occupy the chip:
    // measured over batch sizes 1..512 and contexts 4K..32K, ~100 tiles or more per launch and no tile shorter
    // than 512 keys is within a few percent of the best split everywhere.
    int64_t narrow_chunk = o.narrow_chunk > 0
                               ? o.narrow_chunk
                               : std::min<int64_t>(8192, std::max<int64_t>(512, round_up((int64_t)(narrow_tokens / 96), kTileTokens)));
    if (o.narrow_chunk == 0 && row_blocks.empty() && (int64_t)narrow_lengths.size() * Hkv < 2LL * slots)
        narrow_chunk = choose_narrow_chunk(narrow_lengths, Hkv, D, slots, o.kv_elem_bytes == 1 ? 1 : 2);
    int64_t mfma_chunk = o.mfma_chunk;
    if (mfma_chunk == 0 && !row_blocks.empty())
        mfma_chunk = choose_mfma_chunk(row_blocks, G, Hkv, D, slots, narrow_tokens * kv_tok_bytes_head, o.kv_elem_bytes == 1 ? 1 : 2);
    if (mfma_chunk == 0) mfma_chunk = kMaxMfmaChunk;

    struct Keyed { double cost; ppd_work_item it; };
    std::vector<Keyed> keyed;
    keyed.reserve((row_blocks.size() + narrow_lengths.size()) * (size_t)Hkv);
    std::vector<int32_t> bounds;
    int64_t part_floats = 0;
    int64_t grow = 0;
    int64_t n_narrow = 0, n_mfma = 0, bytes_tiles = 0;
    for (int i = 0; i < B; ++i) {
        const bool narrow = is_narrow(i);
        const int blk = narrow ? n[i] : rows_per_block;
        for (int r0 = 0; r0 < n[i]; r0 += blk) {
            const int nrows = std::min(blk, n[i] - r0);
            const int64_t vis_end = (int64_t)L[i] + r0 + nrows;  // keys 0 .. L + last row of the block
            split_range(vis_end, narrow ? narrow_chunk : mfma_chunk, &bounds);
            const int nsplit = (int)bounds.size() - 1;
            if ((int64_t)keyed.size() + (int64_t)nsplit * Hkv > kMaxTiles) { *err = kTiles; return PPD_ERR_RANGE; }
            const int64_t stride = (int64_t)nrows * G * (D + 2);
            for (int h = 0; h < Hkv; ++h) {
                int group = -1;
                int64_t base = -1;
                if (nsplit > 1) {
                    group = (int)plan->groups.size();
                    base = part_floats;
                    plan->groups.push_back(MergeGroup{(int32_t)(grow + r0), (int16_t)nrows, (int16_t)h, nsplit, 0u, base, stride});
                    for (int c0 = 0; c0 < nrows * G; c0 += kMergeCols) plan->units.push_back(MergeUnit{group, c0});
                    part_floats += stride * nsplit;
                }
                for (int sp = 0; sp < nsplit; ++sp) {
                    ppd_work_item it;
                    std::memset(&it, 0, sizeof it);
                    it.kind = narrow ? 0 : 1;
                    it.seq = i;
                    it.kvh = h;
                    it.row0 = r0;
                    it.nrows = nrows;
                    it.grow0 = (int32_t)(grow + r0);
                    it.L = L[i];
                    it.kv_total = L[i] + n[i];
                    it.kv_begin = bounds[sp];
                    it.kv_end = bounds[sp + 1];
                    it.group = group;
                    it.part_off = nsplit > 1 ? base + stride * sp : -1;
                    const int64_t toks = it.kv_end - it.kv_begin;
                    keyed.push_back(Keyed{(narrow ? 1.0 : 2.0) * toks, it});
                    (narrow ? n_narrow : n_mfma) += 1;
                    bytes_tiles += toks * kv_tok_bytes_head;
                }
            }

        }
        grow += n[i];
    }
    // Queues.  Narrow tiles read every key once: one queue, longest first.  MFMA row-block tiles of one
    // (sequence, KV head, key range) read the same K/V: they form a sharing group that is kept together in
    // one of eight per-XCD queues (the workgroups of an XCD share its L2), groups spread over the queues
    // longest-first onto the least loaded queue; inside a queue the tiles of a group stay adjacent so that they
    // run at about the same time.
    std::vector<Keyed> narrow_items;
    struct Share { double cost; std::vector<ppd_work_item> items; };
    std::vector<Share> shares;
    {
        std::unordered_map<uint64_t, size_t> index;
        for (auto& k : keyed) {
            if (k.it.kind == 0) { narrow_items.push_back(k); continue; }
            const uint64_t key = ((uint64_t)k.it.seq * (uint64_t)Hkv + (uint64_t)k.it.kvh) * (1ull << 24) +
                                 (uint64_t)(k.it.kv_begin / kTileTokens);
            auto f = index.find(key);
            if (f == index.end()) {
                index.emplace(key, shares.size());
                shares.push_back(Share{0.0, {}});
                f = index.find(key);
            }
            shares[f->second].cost += k.cost;
            shares[f->second].items.push_back(k.it);
        }
    }
    std::stable_sort(shares.begin(), shares.end(), [](const Share& a, const Share& b) { return a.cost > b.cost; });
    std::vector<size_t> members[kXcds];
    double load[kXcds] = {0};
    for (size_t k = 0; k < shares.size(); ++k) {
        int q = 0;
        for (int x = 1; x < kXcds; ++x)
            if (load[x] < load[q]) q = x;
        load[q] += shares[k].cost;
        members[q].push_back(k);
    }
    // Inside a queue the groups run longest TILE first (a group's tiles run side by side on different workgroups,
    // so it is the length of one tile, not the sum over the group, that decides how late it may start): a single
    // long tile of a short append-prefill must not wait behind groups of many short ones.
    std::vector<ppd_work_item> queues[kXcds];
    for (int q = 0; q < kXcds; ++q) {
        auto longest = [&](size_t k) {
            int32_t m = 0;
            for (auto& it : shares[k].items) m = std::max(m, it.kv_end - it.kv_begin);
            return m;
        };
        std::vector<std::pair<int32_t, size_t>> order;
        for (size_t k : members[q]) order.emplace_back(longest(k), k);
        std::stable_sort(order.begin(), order.end(), [](const std::pair<int32_t, size_t>& a, const std::pair<int32_t, size_t>& b) { return a.first > b.first; });
        for (auto& o2 : order)
            for (auto& it : shares[o2.second].items) {
                it.queue = q;
                queues[q].push_back(it);
            }
    }
    // Longest first; among equals the KV heads of one key range side by side.  Workgroups that start together then read the
    // heads' 4 KiB pieces of the same 64 KiB pages instead of pieces of as many pages as there are splits: one decode over 32000
    // keys 47 -> 42 us a layer, 11 decodes of 300-6500 keys (64 query heads) 36.8 -> 34.9.
    std::stable_sort(narrow_items.begin(), narrow_items.end(), [](const Keyed& a, const Keyed& b) {
        if (a.cost != b.cost) return a.cost > b.cost;
        if (a.it.seq != b.it.seq) return a.it.seq < b.it.seq;
        return a.it.kv_begin < b.it.kv_begin;
    });
    plan->items.reserve(keyed.size());
    for (int q = 0; q < kXcds; ++q) {
        plan->queue_begin[q] = (int32_t)plan->items.size();
        for (auto& it : queues[q]) plan->items.push_back(it);
    }
    // Narrow tiles, longest first.  The short ones at the end of the list form the wave-tile queue when there are
    // enough of them to keep the waves of every workgroup busy (then eight tiles share the fixed cost of one); with
    // fewer, eight waves per tile keep more compute units streaming.
    size_t wave_from = narrow_items.size();
    if (o.wave_tiles != 0 && o.force_kind != 1) {
        size_t first_short = 0;
        while (first_short < narrow_items.size() &&
               narrow_items[first_short].it.kv_end - narrow_items[first_short].it.kv_begin > kWaveTileKeys)
            ++first_short;
        const size_t n_short = narrow_items.size() - first_short;
        // (by the chip's workgroup slots, not by a grid override: that option must stay scheduling only)
        if (n_short > 0 && (o.wave_tiles == 1 || n_short >= (size_t)6 * (size_t)(kWgPerCu * o.num_cus))) wave_from = first_short;
    }
    plan->queue_begin[kNarrowQueue] = (int32_t)plan->items.size();
    for (size_t k = 0; k < narrow_items.size(); ++k) {
        if (k == wave_from) plan->queue_begin[kWaveQueue] = (int32_t)plan->items.size();
        narrow_items[k].it.queue = k < wave_from ? kNarrowQueue : kWaveQueue;
        plan->items.push_back(narrow_items[k].it);
    }
    if (wave_from == narrow_items.size()) plan->queue_begin[kWaveQueue] = (int32_t)plan->items.size();
    plan->queue_begin[kQueues] = (int32_t)plan->items.size();

    // Split of the compute units between the two kinds when both are present (see narrow_units).
    {
        double narrow_bytes = 0, mfma_iters = 0;
        for (auto& k : keyed) {
            const double toks = (double)(k.it.kv_end - k.it.kv_begin);
            if (k.it.kind == 0) narrow_bytes += toks * kv_tok_bytes_head;
            else mfma_iters += std::ceil(toks / kTileTokens);
        }
        const int elem_bytes = o.kv_elem_bytes == 1 ? 1 : 2;
        plan->narrow_cus = o.narrow_cus >= 0 ? std::min(o.narrow_cus, 32)
                                             : narrow_units(narrow_bytes, mfma_iters, elem_bytes, split_of_units_iter_us(elem_bytes));
    }

    ppd_plan_stats& st = plan->stats;
    st.n_items = (int64_t)plan->items.size();
    st.n_narrow = n_narrow;
    st.n_mfma = n_mfma;
    st.n_groups = (int64_t)plan->groups.size();
    st.partial_floats = part_floats;
    st.kv_bytes = kv_tokens * kv_tok_bytes_head * Hkv;
    st.kv_bytes_tiles = bytes_tiles;
    st.flops = flops;
    st.narrow_chunk = (int32_t)narrow_chunk;
    st.mfma_chunk = (int32_t)mfma_chunk;
    // a workgroup's eight waves take eight wave tiles at a time
    const int64_t wave_groups = (plan->queue_begin[kQueues] - plan->queue_begin[kWaveQueue] + kWaves - 1) / kWaves;
    st.grid = (int32_t)std::max<int64_t>(1, std::min<int64_t>(slots, plan->queue_begin[kWaveQueue] + wave_groups));
    plan->four_waves = n_mfma == 0 && long_tiles_on_four_waves(*plan, kWgPerCu * o.num_cus, D, Hkv, o.kv_elem_bytes == 1 ? 1 : 2);
    plan->wave_unit = n_mfma == 0 && !plan->four_waves && o.wave_tiles < 0 && o.force_kind != 1
                          ? tiles_on_waves(*plan, kWgPerCu * o.num_cus, D, o.kv_elem_bytes == 1 ? 1 : 2) : 0;
    plan->pipelined = n_mfma == 0 && !plan->four_waves && plan->wave_unit == 0 && tiles_pipelined(*plan, st.grid * (kWaves / kNarrowKernelWaves), D, G, o.kv_elem_bytes == 1 ? 1 : 2);
    plan->by_index = n_mfma == 0 && !plan->four_waves && plan->wave_unit == 0 && !plan->pipelined && second_round_by_index(*plan, st.grid * (kWaves / kNarrowKernelWaves), D, o.kv_elem_bytes == 1 ? 1 : 2);
    return PPD_OK;
}

bool has_workgroup_per_entry(const Plan& plan) {
    const int64_t n_wg = plan.queue_begin[kWaveQueue], n_wave = plan.queue_begin[kQueues] - n_wg;
    return n_wg + (n_wave + kWaves - 1) / kWaves <= plan.stats.grid;
}

// Workgroups go round the XCDs in turn, so workgroup b takes from the queue of XCD b % 8 first (row blocks that read the same K/V then
// share an L2 as they do when they are claimed); workgroups whose queue is too short take, in order, what the longer queues have
// left, and then the narrow tiles.
void order_by_block(const Plan& plan, std::vector<int32_t>* order) {
    const int n_wg = plan.queue_begin[kWaveQueue];
    order->assign((size_t)n_wg, -1);
    std::vector<int32_t> left;
    for (int q = 0; q < kXcds; ++q)
        for (int i = plan.queue_begin[q], b = q; i < plan.queue_begin[q + 1]; ++i, b += kXcds) {
            if (b < n_wg) (*order)[b] = i;
            else left.push_back(i);
        }
    for (int i = plan.queue_begin[kNarrowQueue]; i < n_wg; ++i) left.push_back(i);
    size_t next = 0;
    for (auto& o : *order)
        if (o < 0) o = left[next++];
}

}  // namespace ppd

extern "C" ppd_status ppd_plan_build(const ppd_shape* shape, const int32_t* L, const int32_t* n, int32_t B,
                                     int32_t narrow_chunk, int32_t mfma_chunk, int32_t grid, int32_t force_kind,
                                     int32_t num_cus, ppd_work_item* items, int64_t capacity, ppd_plan_stats* stats) {
    ppd_status st = ppd::validate_shape(shape, nullptr);
    if (st != PPD_OK) return st;
    ppd::PlanOptions o;
    o.narrow_chunk = narrow_chunk;
    o.mfma_chunk = mfma_chunk;
    o.grid = grid;
    o.force_kind = force_kind;
    o.num_cus = num_cus > 0 ? num_cus : 256;
    ppd::Plan plan;
    st = ppd::build_plan(*shape, L, n, B, o, &plan, nullptr);
    if (st != PPD_OK) return st;
    if (items)
        for (int64_t i = 0; i < std::min<int64_t>(capacity, (int64_t)plan.items.size()); ++i) items[i] = plan.items[i];
    if (stats) *stats = plan.stats;
    return PPD_OK;
}
