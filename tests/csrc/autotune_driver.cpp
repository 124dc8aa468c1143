// What ca_autotune's choices do to batches of several shapes, without a GPU: the
// host core against the stand-in runtime, with times that the test sets.
// Test infrastructure only.
#include "ca_host.h"

#define launch_strips stub_launch_strips
#define hipEventElapsedTime stub_event_elapsed
#define main harness_main
namespace ca {
hipError_t stub_launch_strips(const StripArgs &, size_t, hipStream_t, hipEvent_t, hipEvent_t);
}
#include "host_harness.cpp"
#undef launch_strips
#undef hipEventElapsedTime
#undef main

namespace {

int g_strip_launches = 0;        // since the last call or timing
std::vector<int> g_tiles;        // their items a workgroup
float (*g_time)() = nullptr;     // of what was launched since the last timing

}  // namespace

namespace ca {
hipError_t launch_strips(const StripArgs &a, size_t lds, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    ++g_strip_launches;
    g_tiles.push_back(a.items_per_group);
    return stub_launch_strips(a, lds, s, e0, e1);
}
}  // namespace ca

hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = g_time ? g_time() : 0.01f;
    g_strip_launches = 0;
    g_tiles.clear();
    return hipSuccess;
}

namespace {

typedef std::vector<std::pair<int32_t, int32_t>> Sizes;

// Strip launches of a call on these frames (tune: of ca_autotune, then a call).
int launches(ca_ctx *ctx, const Sizes &sizes, bool tune)
{
    std::vector<ca_frame_desc> dims;
    size_t total = 0;
    for (const auto &wh : sizes) {
        ca_frame_desc d;
        std::memset(&d, 0, sizeof(d));
        d.width = wh.first;
        d.height = wh.second;
        d.row_stride = 3 * d.width;
        d.pixel_stride = 3;
        d.byte_offset = (int64_t)total;
        d.frame_uid = dims.size();
        total += (size_t)3 * d.width * d.height;
        dims.push_back(d);
    }
    ca_params p;
    ca_default_params(&p);
    const int32_t n = (int32_t)dims.size();
    void *frames = nullptr, *out = nullptr;
    CHECK(hipMalloc(&frames, total) == hipSuccess);
    CHECK(hipMalloc(&out, sizeof(ca_result) * dims.size()) == hipSuccess);
    int32_t schedule = -1;
    if (tune)
        CHECK(ca_autotune(ctx, static_cast<uint8_t *>(frames), dims.data(), n, &p, 2, nullptr,
                          &schedule)
              == CA_OK);
    g_strip_launches = 0;
    g_tiles.clear();
    CHECK(ca_estimate_area(ctx, static_cast<uint8_t *>(frames), dims.data(), n, &p,
                           static_cast<ca_result *>(out), nullptr)
          == CA_OK);
    CHECK(hipFree(frames) == hipSuccess && hipFree(out) == hipSuccess);
    return g_strip_launches;
}

// A tile of four strips wins while a shape is timed alone; of whole calls, one
// launch does, or (the other) a launch for each shape.
bool all_tiles_four()
{
    for (const int t : g_tiles)
        if (t != 4)
            return false;
    return true;
}
float one_launch_wins()
{
    if (g_tiles.empty())   // the persistent kernel
        return 5.0f;
    bool tiled = false;
    for (const int t : g_tiles)
        tiled = tiled || t != 1;
    const bool alone = g_tiles.size() == 3;   // a warm-up and two timed launches
    return alone ? (all_tiles_four() ? 1.0f : 2.0f) : tiled ? 3.0f : 2.0f;
}
float tiles_win()
{
    if (g_tiles.empty())
        return 5.0f;
    const bool alone = g_tiles.size() == 3;
    return alone ? (all_tiles_four() ? 1.0f : 2.0f) : all_tiles_four() ? 1.0f : 3.0f;
}

}  // namespace

int main()
{
    const Sizes one(1, {1280, 720});
    const Sizes two = {{1280, 720}, {640, 480}, {1280, 720}, {640, 480}};
    {
        ca_ctx *ctx = nullptr;
        CHECK(ca_create(&ctx, 0, 0) == CA_OK);
        CHECK(launches(ctx, two, false) == 1);
        // another batch's tuning leaves this one's launch alone
        g_time = one_launch_wins;
        CHECK(launches(ctx, one, true) == 1);
        int32_t tile = 0;
        CHECK(ca_get_tuning(ctx, 1280, 720, 16, 16, &tile) == CA_OK && tile == 4);
        if (launches(ctx, two, false) != 1)
            fail("%s", "a shape's tile splits an untuned batch of several shapes");
        // and so does its own, where one launch is the faster
        if (launches(ctx, two, true) != 1)
            fail("%s", "the faster single launch is not kept");
        ca_destroy(ctx);
    }
    {
        ca_ctx *ctx = nullptr;
        CHECK(ca_create(&ctx, 0, 0) == CA_OK);
        g_time = tiles_win;
        if (launches(ctx, two, true) != 2 || !all_tiles_four())
            fail("%s", "the faster launches with tiles are not kept");
        // asked for by the option, either way
        CHECK(ca_set_option(ctx, CA_OPT_STRIPS_PER_GROUP, 1) == CA_OK);
        CHECK(launches(ctx, two, false) == 1);
        CHECK(ca_set_option(ctx, CA_OPT_STRIPS_PER_GROUP, 2) == CA_OK);
        CHECK(launches(ctx, two, false) == 2);
        ca_destroy(ctx);
    }
    std::printf("ok autotune of shapes\n");
    return 0;
}
