// Host-only checks of how a plan gets to the device (built and run by tests/test_plan_upload.py): ppd_api.hip as it is,
// compiled against the stand-in runtime of host_runtime/, whose streams run only when the test lets them.  The attention
// launches are replaced by checks that the work list on the device is the one of their own call.
#include <hip/hip_runtime.h>

#include <chrono>
#include <random>
#include <thread>
#include <vector>

#include "../../paper_2603_13358_amd/csrc/ppd_api.hip"

static std::vector<int32_t> g_L;  // cached lengths of the call being made
static int g_ran = 0, g_wrong = 0;

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
static int check_plan(const KParams& p, void* stream) {
    const std::vector<int32_t> L = g_L;
    sim.of(static_cast<hipStream_t>(stream))->push([p, L] {
        ++g_ran;
        bool good = p.n_items == (int)L.size() && p.queue_begin[kQueues] == p.n_items;
        for (int i = 0; good && i < p.n_items; ++i)
            good = p.items[i].seq >= 0 && p.items[i].seq < (int)L.size() && p.items[i].L == L[p.items[i].seq];
        if (!good) ++g_wrong;
    });
    return (int)hipGetLastError();
}
int launch_mixed(const KParams& p, int, int, void* stream, bool) { return check_plan(p, stream); }
int launch_narrow(const KParams& p, int, int, void* stream, bool) { return check_plan(p, stream); }
int launch_mfma_only(const KParams&, int, int, void*) { return 0; }
int launch_stream_only(const KParams&, int, int, void*) { return 0; }
int launch_merge(const MergeParams&, void*) { return 0; }
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

static ppd_ctx* make_ctx() {
    const ppd_shape s = {8, 1, 64, 16, 1 << 20};
    ppd_ctx* ctx = nullptr;
    CHECK(ppd_create(&s, 0, &ctx) == PPD_OK);
    return ctx;
}

// One decode step of `tiles` sequences of `L` cached tokens (one tile each).
static ppd_status step(ppd_ctx* ctx, int tiles, int32_t L, bool use_static = false, hipStream_t s = nullptr) {
    alignas(16) static char device[16];
    g_L.assign((size_t)tiles, L);
    const std::vector<int32_t> n((size_t)tiles, 1);
    auto fn = use_static ? ppd_mixed_attention_static : ppd_mixed_attention;
    return fn(ctx, device, device, reinterpret_cast<const int32_t*>(device), 64, g_L.data(), n.data(), tiles, 1.f, device, s);
}

static void finish(ppd_ctx* ctx) {
    sim.null_stream.run();
    CHECK(g_wrong == 0);
    ppd_destroy(ctx);
}

// Runs what the null stream holds a while after now, i.e. while the caller waits inside a call.
static std::thread device_after(int ms, size_t count = SIZE_MAX) {
    return std::thread([=] {
        std::this_thread::sleep_for(std::chrono::milliseconds(ms));
        sim.null_stream.run(count);
    });
}

// An error that an earlier HIP call of the thread left pending meets the upload of every staging buffer: whatever those
// calls return, the plans after them run their own work lists.
static void pending_error(bool use_static) {
    ppd_ctx* ctx = make_ctx();
    const int slots = use_static ? 1 : kStagingSlots;
    for (int k = 0; k < slots; ++k) {
        sim.pending = hipErrorInvalidValue;
        (void)step(ctx, 6, 100 + k, use_static);
        sim.pending = hipSuccess;
        sim.null_stream.run();
    }
    CHECK(step(ctx, 6, 100 + slots - 1, use_static) == PPD_OK);  // the last one again
    for (int k = 1; k < slots; ++k) CHECK(step(ctx, 6, 120 + k, use_static) == PPD_OK);
    std::thread device = device_after(100);
    for (int k = 0; k < 2 * slots; ++k) CHECK(step(ctx, 7, 200 + k, use_static) == PPD_OK);
    device.join();
    finish(ctx);
}

// The same on a context that shares the static array: the other context's plan is gone, it must not be taken for resident.
static void pending_error_and_two_contexts() {
    ppd_ctx *a = make_ctx(), *b = make_ctx();
    CHECK(step(a, 5, 40, true) == PPD_OK);
    sim.null_stream.run();
    sim.pending = hipErrorInvalidValue;
    (void)step(b, 9, 60, true);
    sim.pending = hipSuccess;
    sim.null_stream.run();
    CHECK(step(a, 5, 40, true) == PPD_OK);
    finish(a);
    ppd_destroy(b);
}

// An upload that could not be launched leaves its buffer free, and the call can be made again.
static void failed_launch(bool use_static) {
    ppd_ctx* ctx = make_ctx();
    for (int k = 0; k < 6; ++k) {
        sim.launch_status = hipErrorLaunchFailure;
        CHECK(step(ctx, 5, 40 + k, use_static) == PPD_ERR_HIP);
        sim.launch_status = sim.pending = hipSuccess;
        CHECK(step(ctx, 5, 40 + k, use_static) == PPD_OK);
        sim.null_stream.run();
    }
    finish(ctx);
}

// Plans that just fit the buffers of an earlier one: the upload moves 16 bytes per lane and a plan is any multiple of 4.
static void sizes_that_just_fit() {
    for (int first : {3, 50, 292}) {
        const int bytes = first * (int)sizeof(ppd_work_item) + (int)sizeof(ppd::Plan::queue_begin);
        const int fits = (bytes + bytes / 4 + 4096 - (int)sizeof(ppd::Plan::queue_begin)) / (int)sizeof(ppd_work_item);
        // on the device: the second plan fills what the first one allocated
        ppd_ctx* ctx = make_ctx();
        CHECK(step(ctx, first, 40) == PPD_OK);
        for (int tiles = fits - 1; tiles <= fits + 1; ++tiles) {
            CHECK(step(ctx, tiles, 41) == PPD_OK);
            sim.null_stream.run();
        }
        finish(ctx);
        // in the staging buffer: the device buffer has grown in between, then the first staging buffer is used again
        for (int tiles = fits - 1; tiles <= fits + 1; ++tiles) {
            ctx = make_ctx();
            CHECK(step(ctx, first, 40) == PPD_OK);
            for (int k = 1; k < kStagingSlots; ++k) CHECK(step(ctx, 4 * fits, 50 + k) == PPD_OK);
            sim.null_stream.run();
            CHECK(step(ctx, tiles, 60) == PPD_OK);
            finish(ctx);
        }
    }
    std::mt19937 rng(5);
    ppd_ctx* ctx = make_ctx();
    for (int k = 0; k < 400; ++k) {
        CHECK(step(ctx, 1 + (int)(rng() % (1 + 2 * k)), k) == PPD_OK);
        sim.null_stream.run();
    }
    finish(ctx);
}

// A host that runs ahead of the device waits for the one upload whose buffer it needs: not for the layers enqueued after
// it, nor for work on streams of others.
static void run_ahead(bool use_static) {
    ppd_ctx* ctx = make_ctx();
    const int slots = use_static ? 1 : kStagingSlots;
    sim.device_syncs = 0;
    for (int k = 0; k < slots; ++k)
        for (int layer = 0; layer < 3; ++layer) CHECK(step(ctx, 6, 100 + k, use_static) == PPD_OK);
    const size_t before = sim.null_stream.waiting();
    std::thread device = device_after(100, 1);  // the oldest upload, and nothing after it
    CHECK(step(ctx, 6, 200, use_static) == PPD_OK);
    device.join();
    CHECK(sim.device_syncs == 0);
    ppd_plan_stats stats;
    CHECK(ppd_get_plan_stats(ctx, &stats) == PPD_OK && stats.plan_host_us < 50000);  // the plan's own time, not the wait
    CHECK(sim.null_stream.waiting() > before - 1);  // what was enqueued is still there, and the new plan's work behind it
    finish(ctx);
}

int main(int argc, char** argv) {
    (void)argc;
    const std::string what = argv[1];
    if (what == "pending_error") {
        pending_error(false);
        pending_error(true);
    }
    if (what == "two_contexts") pending_error_and_two_contexts();
    if (what == "run_ahead") {
        run_ahead(false);
        run_ahead(true);
    }
    if (what == "sizes") sizes_that_just_fit();
    if (what == "failed_launch") {
        failed_launch(false);
        failed_launch(true);
    }
    std::printf("ok, %d launches\n", g_ran);
    return 0;
}
