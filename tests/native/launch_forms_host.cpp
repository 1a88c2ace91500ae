// Host-only checks of how a step is launched (built and run by tests/test_launch_forms.py): ppd_api.hip as it
// is, compiled against the stand-in runtime of host_runtime/, whose launches are recorded instead of run.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <vector>

#include "../../paper_2603_13358_amd/csrc/ppd_api.hip"

static size_t g_allocations = 0;
void* operator new(size_t bytes) {
    ++g_allocations;
    if (void* p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(size_t bytes, const std::nothrow_t&) noexcept {
    ++g_allocations;
    return std::malloc(bytes ? bytes : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

static ppd::KParams g_params;
static int g_grid = 0, g_merges = 0;

std::function<void()> sim_bind(const void* f, void** args) {
    if (f != reinterpret_cast<const void*>(&ppd_upload_kernel)) std::abort();
    auto host = *static_cast<const uint4**>(args[0]);
    auto dev = *static_cast<uint4**>(args[1]);
    auto granules = *static_cast<int64_t*>(args[2]);
    auto counters = *static_cast<uint32_t**>(args[3]);
    auto read = *static_cast<uint32_t**>(args[4]);
    auto serial = *static_cast<uint32_t*>(args[5]);
    return [=] { ppd_upload_kernel(host, dev, granules, counters, read, serial); };
}

namespace ppd {
int prepare_mixed_kernels() { return 0; }
int launch_mixed(const KParams& p, int, int grid, void*, bool) {
    g_params = p;
    g_grid = grid;
    return 0;
}
int launch_narrow(const KParams& p, int, int grid, void*, bool) {
    g_params = p;
    g_grid = grid;
    return 0;
}
int launch_mfma_only(const KParams& p, int, int, void*) {
    g_params = p;
    return 0;
}
int launch_stream_only(const KParams& p, int, int, void*) {
    g_params = p;
    return 0;
}
int launch_merge(const MergeParams&, void*) {
    ++g_merges;
    return 0;
}
int launch_kv_append(const uint16_t*, const uint16_t*, void*, const int64_t*, int64_t, int, int, int64_t, int, int64_t, uint32_t*,
                     void*, bool, float, float) { return 0; }
}  // namespace ppd

#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("%s:%d: not so: %s\n", __FILE__, __LINE__, #x); \
            std::fflush(stdout);                                      \
            std::_Exit(1);                                            \
        }                                                             \
    } while (0)

struct Step {
    bool by_index, four_waves, merges_itself, merge_launched;
    int64_t items, groups;
};

// One decode step of sequences that see `keys` keys each.
static Step step(std::vector<int32_t> keys, int head_dim, bool fp8, int64_t chunk, int64_t grid, bool use_static = false, int hkv = 8) {
    alignas(16) static char device[16];
    const ppd_shape s = {4 * hkv, hkv, head_dim, 16, 1 << 20};
    ppd_ctx* ctx = nullptr;
    CHECK(ppd_create(&s, 0, &ctx) == PPD_OK);
    if (fp8) CHECK(ppd_set_kv_format(ctx, PPD_KV_FP8_E4M3, 1.f, 1.f) == PPD_OK);
    CHECK(ppd_set_option(ctx, "narrow_chunk", chunk) == PPD_OK && ppd_set_option(ctx, "grid", grid) == PPD_OK);
    for (auto& k : keys) k -= 1;
    const std::vector<int32_t> n(keys.size(), 1);
    g_merges = 0;
    auto fn = use_static ? ppd_mixed_attention_static : ppd_mixed_attention;
    CHECK(fn(ctx, device, device, reinterpret_cast<const int32_t*>(device), 1 << 16, keys.data(), n.data(), (int32_t)keys.size(), 1.f, device, nullptr) == PPD_OK);
    sim.null_stream.run();
    ppd_plan_stats st;
    CHECK(ppd_get_plan_stats(ctx, &st) == PPD_OK && st.n_mfma == 0);
    ppd_destroy(ctx);
    // one form at most, and only where it has what it hands out
    CHECK((g_params.by_index != 0) + (g_params.four_waves != 0) + (g_params.wave_unit != 0) + (g_params.pipelined != 0) <= 1);
    CHECK(!g_params.merge_groups || (g_params.by_index | g_params.four_waves | g_params.wave_unit | g_params.pipelined) == 0);
    CHECK(!(g_params.by_index || g_params.pipelined) || st.n_items > g_grid);
    return Step{g_params.by_index != 0, g_params.four_waves != 0, g_params.merge_groups != nullptr, g_merges == 1, st.n_items, st.n_groups};
}

static std::vector<int32_t> lengths(int count, int32_t keys, int n_long = 0, int32_t longer = 0) {
    std::vector<int32_t> v((size_t)count, keys);
    for (int i = 0; i < n_long; ++i) v[i] = longer;
    return v;
}

// Whatever the lengths and the grid, split ranges are merged exactly once: by a form that can, or by the merge launch.  Which
// form runs does not depend on the grid.
static void merged_once() {
    std::mt19937 rng(1);
    int four = 0, itself = 0, launched = 0;
    for (int trial = 0; trial < 150; ++trial) {
        const int D = rng() % 4 ? 128 : 64;
        const bool fp8 = rng() % 4 == 0, use_static = rng() % 4 == 0;
        const int64_t chunks[] = {0, 64, 1024, 4096, 8192};
        const int64_t chunk = chunks[rng() % 5];
        const int32_t longest = 200 << (rng() % 8);
        std::vector<int32_t> keys((size_t)(1 + rng() % 120));
        const int32_t low = rng() % 2 ? longest / 2 : 0;
        for (auto& k : keys) k = 1 + low + (int32_t)(rng() % (longest - low));
        if (use_static && (chunk == 64 || chunk == 0)) continue;  // (plans that do not fit the static array)
        const Step a = step(keys, D, fp8, chunk, 0, use_static);
        for (int64_t grid : {256, 512, 600, 4096, 65536}) {
            const Step b = step(keys, D, fp8, chunk, grid, use_static);
            if (chunk > 0) CHECK(b.four_waves == a.four_waves);  // (an automatic split size goes by the grid)
            CHECK(!(b.four_waves && b.merges_itself));
            CHECK((b.groups > 0) == (b.merges_itself || b.merge_launched) && !(b.merges_itself && b.merge_launched));
            if (b.items <= 256) CHECK(!b.four_waves);
            four += b.four_waves;
            itself += b.merges_itself;
            launched += b.merge_launched;
        }
    }
    std::printf("four waves %d, merged in the launch %d, by the merge launch %d\n", four, itself, launched);
    CHECK(four > 20 && itself > 20 && launched > 20);
}

// Long tiles run on four waves (256 workgroups) where their last round is nearly full or short.
static void four_waves() {
    auto four = [&](const std::vector<int32_t>& keys, int D = 128, bool fp8 = false) { return step(keys, D, fp8, 16384, 0).four_waves; };
    CHECK(four(lengths(64, 3072)) && !four(lengths(64, 3071)) && !four(lengths(63, 5000)));  // two full rounds, less
    for (int hkv : {4, 8, 12, 16}) CHECK(step(lengths(1536 / hkv, 5000), 128, false, 16384, 0, false, hkv).four_waves == (hkv % 8 == 0));
    CHECK(!four(lengths(64, 5000), 64) && !four(lengths(64, 8000), 128, true));
    CHECK(!four(lengths(65, 5000)) && !four(lengths(86, 5000)) && four(lengths(87, 5000)) && four(lengths(96, 5000)));
    CHECK(!four(lengths(97, 5000)) && !four(lengths(200, 5000)) && four(lengths(230, 4000)));  // the eighth round: a seventh of the mean load
    std::vector<int32_t> keys = lengths(72, 5000);                                            // the last round is short
    for (int i = 64; i < 72; ++i) keys[i] = 1400;
    CHECK(four(keys));
    keys[70] = 1500;
    CHECK(!four(keys));
}

// The second round of a decode-only launch (256 workgroups) is handed out by index where its pairs are balanced, and the tiles do not run
// pipelined (bf16 pages, up to 640 keys of about one length here, 1280 at D = 64).
static void second_round() {
    const int64_t whole = 16384;  // no range is split
    auto by_index = [&](const std::vector<int32_t>& keys, int D = 128, bool fp8 = false) { return step(keys, D, fp8, whole, 0).by_index; };
    CHECK(!by_index(lengths(32, 800)) && !by_index(lengths(65, 800)));                     // one round, more than two
    CHECK(by_index(lengths(64, 800)) && by_index(lengths(64, 1535)) && !by_index(lengths(64, 1536)));
    CHECK(by_index(lengths(64, 3071), 128, true) && !by_index(lengths(64, 3072), 128, true));
    CHECK(by_index(lengths(64, 1535), 64) && !by_index(lengths(64, 1536), 64));
    CHECK(by_index(lengths(40, 1500)) && !by_index(lengths(39, 1500)));
    CHECK(by_index(lengths(39, 1023), 128, true) && !by_index(lengths(39, 1024), 128, true));
    CHECK(by_index(lengths(33, 2047), 64, true) && !by_index(lengths(33, 2048), 64, true));
    CHECK(by_index(lengths(33, 1023), 128, true) && !by_index(lengths(33, 1024), 128, true));
    for (int32_t keys : {500, 800, 1300})                                                  // another tile behind a long one
        for (int n_long : {1, 8})
            for (bool fp8 : {false, true})
                for (int D : {64, 128}) {
                    CHECK(!by_index(lengths(64, keys, n_long, 4 * keys), D, fp8));
                    CHECK(by_index(lengths(64, keys, n_long, keys + 32), D, fp8) != (!fp8 && keys * D <= 640 * 128));  // (those run pipelined)
                }
    CHECK(!by_index(lengths(52, 800, 14, 1600)));                                          // 16 long tiles of 112 would get one
    CHECK(by_index(lengths(52, 800, 12, 1600)));                                           // none of 96 would
    CHECK(by_index(lengths(300, 60)) && !by_index(lengths(351, 205)) && by_index(lengths(352, 205)));  // slots of eight one-wave tiles
    CHECK(!by_index(lengths(212, 205, 10, 530)));
    std::vector<int32_t> even(64);
    for (int i = 0; i < 64; ++i) even[i] = 64 + i * 24;                                     // evenly spread: the pairs balance
    CHECK(by_index(even));
}

// Tiles run on single waves (256 compute units) where that is estimated to be faster: not below 640 tiles, not where a wave's chain
// or a unit's bytes would outlast the rest, not where the list has all of them on single waves.
static void on_waves() {
    auto unit = [&](const std::vector<int32_t>& keys, int D = 128, bool fp8 = false, int64_t chunk = 0, int64_t grid = 0) {
        const Step s = step(keys, D, fp8, chunk, grid);
        CHECK((s.groups > 0) == (s.merges_itself || s.merge_launched) && !(s.merges_itself && s.merge_launched));
        CHECK(!g_params.wave_unit || (g_grid <= 256 || grid > 256) && !s.merges_itself);
        return g_params.wave_unit;
    };
    for (bool fp8 : {false, true}) {
        for (int D : {64, 128}) {
            CHECK(unit(lengths(79, 100), D, fp8) == (fp8 ? 1 : 0) && unit(lengths(80, 100), D, fp8) == 2);
            CHECK(unit(lengths(32, 100), D, fp8) == 0 && unit(lengths(33, 70), D, fp8) == (fp8 ? 1 : 0) && unit(lengths(33, 700), D, fp8) == 0);
            CHECK(unit(lengths(191, 100), D, fp8) == 2 && unit(lengths(192, 100), D, fp8) == 0);         // all in the list of one-wave tiles
            CHECK(unit(lengths(192, 100, 16, 400), D, fp8) == 4);                                          // not all
            CHECK(unit(lengths(192, 100, 16, 400), D, fp8, 0, 7) == 4 && unit(lengths(192, 100, 16, 400), D, fp8, 0, 4096) == 4);
            CHECK(unit(lengths(100, 100, 1, 4000), D, fp8) == 0 && unit(lengths(192, 300, 64, 8000), D, fp8) == 0);
        }
        CHECK(unit(lengths(80, 200), 128, fp8, 320) == 2 && unit(lengths(80, 200, 1, 330), 128, fp8, 320) == 0);  // a split range
    }
    std::vector<int32_t> even(256);
    for (int i = 0; i < 256; ++i) even[i] = 64 + i * 636 / 255;
    for (bool fp8 : {false, true})
        for (int D : {64, 128}) {  // rounds of the waves
            CHECK(unit(lengths(256, 440), D, fp8) == 4 && unit(lengths(257, 440), D, fp8) == 0 && unit(lengths(511, 440), D, fp8) == 0);
            CHECK(unit(lengths(512, 440), D, fp8) == (D == 128 && !fp8 ? 0 : 4));
        }
    for (int D : {64, 128}) {
        CHECK(unit(lengths(520, 100, 64, 400), D, true) == 0 && unit(lengths(520, 100, 65, 400), D, true) == 4);  // an eighth not on single waves as it is
        CHECK(unit(lengths(64, 176), D, true) == 1 && unit(lengths(64, 177), D, true) == 0 && unit(lengths(65, 177), D, true) == 1);  // a second round by index
    }
    // where whole workgroups were measured to be faster
    CHECK(unit(lengths(162, 3239), 64, true) == 0 && unit(lengths(145, 1726), 64, true) == 0 && unit(lengths(128, 1124), 64) == 0);
    CHECK(unit(lengths(662, 669)) == 0 && unit(lengths(576, 590)) == 0);
    CHECK(unit(even) == 4 && unit(even, 128, true) == 4 && unit(even, 64) == 4);
    CHECK(unit(lengths(256, 3500)) == 0 && unit(lengths(64, 2000)) == 0);
    auto longer = [&](int count, int32_t low, int32_t high, int D, bool fp8) {  // test_long_decode_tiles_on_single_waves
        std::vector<int32_t> keys;
        for (int32_t end : {2049, 2048, 2047, 2046, 1025, 1024, 1023, 1022, 15, 1})
            if (end <= high) keys.push_back(end);
        while ((int)keys.size() < count) keys.push_back(low + (int32_t)keys.size() * 37 % (high - low + 1));
        return unit(keys, D, fp8);
    };
    CHECK(longer(256, 900, 1100, 64, false) == 4 && longer(200, 900, 1100, 64, false) == 4);
    CHECK(longer(128, 1900, 2100, 128, true) == 2 && longer(256, 1900, 2100, 64, true) == 4);
}

// Where no order could make single waves win, the planner finds that out without laying the tiles out on the waves: the plan takes the memory
// of one that must not ask ("wave_tiles" 0; no tile here is in the list of one-wave tiles).
static void estimate() {
    auto allocations = [&](const std::vector<int32_t>& L, int D, int elem_bytes, int32_t wave_tiles, int32_t* unit) {
        const ppd_shape s = {64, 8, D, 16, 1 << 20};
        const std::vector<int32_t> n(L.size(), 1);
        ppd::PlanOptions o;
        o.kv_elem_bytes = elem_bytes;
        o.wave_tiles = wave_tiles;
        ppd::Plan plan;
        for (int call = 0; call < 2; ++call) {  // the second one finds the plan's own tables allocated
            g_allocations = 0;
            CHECK(ppd::build_plan(s, L.data(), n.data(), (int32_t)L.size(), o, &plan, nullptr) == PPD_OK);
        }
        *unit = plan.wave_unit;
        return g_allocations;
    };
    auto asks = [&](const std::vector<int32_t>& L, int D, int elem_bytes) {
        int32_t unit, never;
        const size_t with = allocations(L, D, elem_bytes, -1, &unit), without = allocations(L, D, elem_bytes, 0, &never);
        CHECK(never == 0 && with >= without && (unit == 0 || with > without));
        return with > without;
    };
    std::mt19937 rng(3);
    std::vector<int32_t> spread(64);
    for (auto& l : spread) l = 64 + (int32_t)(rng() % 637);
    for (int D : {64, 128}) CHECK(!asks(spread, D, 1) && !asks(lengths(64, 5000), D, 1) && !asks(lengths(79, 3000, 1, 20000), D, 1));
    CHECK(!asks(lengths(36, 300), 128, 1) && !asks(lengths(100, 400, 1, 6000), 128, 2) && !asks(lengths(200, 4000), 128, 2));
    CHECK(asks(lengths(33, 70), 128, 1) && asks(lengths(80, 100), 128, 2));
}

// More tiles than workgroups run pipelined where they are short and of a length, on bf16 pages and whole workgroups.
static void pipelined() {
    auto runs = [&](const std::vector<int32_t>& keys, int D = 128, bool fp8 = false, int64_t grid = 0, int hkv = 8) {
        step(keys, D, fp8, 8192, grid, false, hkv);
        CHECK(!g_params.pipelined || (!g_params.wave_unit && !g_params.four_waves && !g_params.merge_groups && g_params.n_wg == g_params.n_items && g_grid < g_params.n_items));
        return g_params.pipelined != 0;
    };
    CHECK(!runs(lengths(32, 200)) && runs(lengths(33, 200)) && runs(lengths(79, 200)) && runs(lengths(20, 200), 128, false, 100));
    CHECK(!runs(lengths(33, 200), 128, true) && runs(lengths(33, 640)) && !runs(lengths(33, 641)) && runs(lengths(33, 1280), 64) && !runs(lengths(33, 1281), 64));
    CHECK(runs(lengths(40, 400, 4, 630)) && !runs(lengths(40, 400, 4, 640)) && runs(lengths(40, 300, 4, 540)) && !runs(lengths(40, 300, 4, 600)));
    CHECK(runs(lengths(40, 200, 4, 600)) && !runs(lengths(40, 200, 4, 800)));
    CHECK(runs(lengths(65, 200, 1, 390)) && !runs(lengths(65, 200, 1, 400)) && runs(lengths(72, 200, 9, 390)) && !runs(lengths(72, 200, 9, 400)));  // a long tile and two more behind it
    CHECK(!runs(lengths(72, 220, 9, 520)) && !runs(lengths(125, 480, 12, 862)) && !runs(lengths(106, 417, 11, 700)));  // measured to be slower
    CHECK(!runs(lengths(64, 5000)) && !runs(lengths(256, 100)) && !runs(lengths(256, 440)));
    auto split = [&](int count, int D, int64_t chunk, int64_t grid) {  // test_pipelined_tiles_of_split_ranges
        std::vector<int32_t> keys;
        for (int i = 0; i < count; ++i) keys.push_back(300 + i * 389 % 700);
        const Step s = step(keys, D, false, chunk, grid);
        CHECK(g_params.pipelined && !s.merges_itself && s.merge_launched);
        return s.groups;
    };
    CHECK(split(34, 128, 0, 0) == 176 && split(40, 64, 256, 48) == 320 && split(37, 128, 256, 100) == 296);
}

// The list of a launch of the mixed kernel with a workgroup for every entry is in the order of its workgroups: every tile once, workgroup b
// with tile b / 8 of the queue of XCD b % 8 while that has one, the one-wave tiles behind the others.
static void by_block() {
    alignas(16) static char device[16];
    std::mt19937 rng(2);
    int in_order = 0, claimed = 0;
    for (int trial = 0; trial < 300; ++trial) {
        const int hkv = 1 << (rng() % 4), mode = rng() % 3 ? 0 : 1;
        const ppd_shape s = {4 * hkv, hkv, 128, 16, 1 << 20};
        ppd_ctx* ctx = nullptr;
        CHECK(ppd_create(&s, 0, &ctx) == PPD_OK);
        CHECK(ppd_set_option(ctx, "launch_mode", mode) == PPD_OK && ppd_set_option(ctx, "narrow_kernel", 0) == PPD_OK);
        const int kinds = mode == 0 ? rng() % 3 : rng() % 2;  // decodes, turns, both (which launch_mode 1 runs as two kernels)
        std::vector<int32_t> L, n;
        for (int i = 1 + rng() % (1 << (rng() % 7)); i > 0; --i) {
            const bool turn = kinds == 1 || (kinds == 2 && rng() % 2);
            L.push_back((int32_t)(rng() % 3000));
            n.push_back(turn ? 64 + (int32_t)(rng() % 300) : 1);
        }
        CHECK(ppd_mixed_attention(ctx, device, device, reinterpret_cast<const int32_t*>(device), 1 << 16, L.data(), n.data(), (int32_t)L.size(), 1.f, device, nullptr) == PPD_OK);
        sim.null_stream.run();
        const ppd::Plan& plan = ctx->plan;
        const ppd_work_item* const list = g_params.items;
        const int n_wg = plan.queue_begin[ppd::kWaveQueue], n_items = plan.queue_begin[ppd::kQueues];
        const bool enough = n_wg + (n_items - n_wg + ppd::kWaves - 1) / ppd::kWaves <= g_grid;
        CHECK((g_params.by_block != 0) == enough && g_params.n_wg == n_wg && g_params.n_items == n_items);
        std::vector<int> times((size_t)n_items, 0);
        for (int b = 0; b < n_items; ++b) {
            int i = 0;
            while (i < n_items && (times[i] || std::memcmp(&plan.items[i], &list[b], sizeof(ppd_work_item)) != 0)) ++i;
            CHECK(i < n_items);
            times[i] = 1;
            const int q = b % ppd::kXcds, at = plan.queue_begin[q] + b / ppd::kXcds;
            if (!enough || b >= n_wg) CHECK(i == b);
            else if (at < plan.queue_begin[q + 1]) CHECK(i == at);
        }
        in_order += enough && plan.stats.n_mfma > 0;
        claimed += !enough;
        ppd_destroy(ctx);
    }
    std::printf("in the workgroups' order %d, claimed %d\n", in_order, claimed);
    CHECK(in_order > 30 && claimed > 30);
}

// A plan serves every launch mode that plans alike (here "wave_tiles" 0, which the modes of two kernels imply): a step run eagerly in one
// mode can be captured in another, and what is launched then finds the list in its own order, the queues' or the workgroups'.
static void modes_share_a_plan() {
    alignas(16) static char device[16];
    std::mt19937 rng(4);
    int in_order = 0;
    for (int trial = 0; trial < 200; ++trial) {
        const ppd_shape s = {32, 8, 128, 16, 1 << 20};
        ppd_ctx* ctx = nullptr;
        CHECK(ppd_create(&s, 0, &ctx) == PPD_OK && ppd_set_option(ctx, "wave_tiles", 0) == PPD_OK && ppd_set_option(ctx, "grid", rng() % 4 ? 0 : 65536) == PPD_OK);
        const int kinds = rng() % 3;  // decodes, turns, both
        std::vector<int32_t> L, n;
        for (int i = 1 + rng() % (1 << (rng() % 7)); i > 0; --i) {
            const bool turn = kinds == 1 || (kinds == 2 && rng() % 2);
            L.push_back((int32_t)(rng() % 3000));
            n.push_back(turn ? 64 + (int32_t)(rng() % 300) : 1);
        }
        for (int call = 0; call < 6; ++call) {
            const bool use_static = trial % 2 != 0;
            const int mode = (int)(rng() % 3);
            sim.capturing = call > 0;
            CHECK(ppd_set_option(ctx, "launch_mode", mode) == PPD_OK);
            auto fn = use_static ? ppd_mixed_attention_static : ppd_mixed_attention;
            const ppd_status st = fn(ctx, device, device, reinterpret_cast<const int32_t*>(device), 1 << 16, L.data(), n.data(), (int32_t)L.size(), 1.f, device, nullptr);
            if (call == 0 && use_static && st == PPD_ERR_WORKSPACE) break;  // (the split partials of a large grid)
            CHECK(st == PPD_OK);
            sim.null_stream.run();
            const ppd::Plan& plan = ctx->plan;
            const bool mixed = mode == 0 ? plan.stats.n_mfma > 0 : mode == 1 && (plan.stats.n_narrow == 0 || plan.stats.n_mfma == 0);
            CHECK((g_params.by_block != 0) == (mixed && plan.stats.n_items <= plan.stats.grid));
            std::vector<int32_t> order;
            if (g_params.by_block) ppd::order_by_block(plan, &order);
            for (int b = 0; b < plan.stats.n_items; ++b)
                CHECK(std::memcmp(&g_params.items[b], &plan.items[g_params.by_block ? order[b] : b], sizeof(ppd_work_item)) == 0);
            CHECK(std::memcmp(g_params.queue_begin, plan.queue_begin, sizeof plan.queue_begin) == 0);
            in_order += g_params.by_block && kinds > 0;
        }
        sim.capturing = false;
        ppd_destroy(ctx);
    }
    CHECK(in_order > 100);
    // a list that the fixed scratch array holds in one order only is claimed there
    for (int decodes : {2200, 2400}) {
        const ppd_shape s = {32, 8, 128, 16, 1 << 20};
        std::vector<int32_t> L((size_t)decodes + 1, 99), n((size_t)decodes + 1, 1);
        n[0] = 64;
        for (bool use_static : {false, true}) {
            ppd_ctx* ctx = nullptr;
            CHECK(ppd_create(&s, 0, &ctx) == PPD_OK);
            for (auto& o : std::vector<std::pair<const char*, int64_t>>{{"wave_tiles", 0}, {"grid", 65536}, {"mfma_chunk", 32768}, {"narrow_chunk", 8192}})
                CHECK(ppd_set_option(ctx, o.first, o.second) == PPD_OK);
            auto fn = use_static ? ppd_mixed_attention_static : ppd_mixed_attention;
            CHECK(fn(ctx, device, device, reinterpret_cast<const int32_t*>(device), 1 << 16, L.data(), n.data(), (int32_t)L.size(), 1.f, device, nullptr) == PPD_OK);
            sim.null_stream.run();
            CHECK(ctx->plan.stats.n_items == 8 * (decodes + 1) && (g_params.by_block != 0) == (!use_static || decodes == 2200));
            ppd_destroy(ctx);
        }
    }
}

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "merged_once") merged_once();
    else if (what == "four_waves") four_waves();
    else if (what == "second_round") second_round();
    else if (what == "on_waves") on_waves();
    else if (what == "estimate") estimate();
    else if (what == "pipelined") pipelined();
    else if (what == "by_block") by_block();
    else if (what == "modes_share_a_plan") modes_share_a_plan();
    else return 2;
    std::printf("ok\n");
    return 0;
}
