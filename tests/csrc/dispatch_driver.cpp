// How batches of several frame shapes are dispatched, without a GPU: the host
// core and the entry point without allocation against the stand-in runtime of
// host_harness.cpp, whose strip launches are recorded on their way.
// Test infrastructure only.
#include "ca_host.h"

#define launch_strips stub_launch_strips
#define launch_cnn_strips stub_launch_cnn_strips
#define launch_cnn2d_strips stub_launch_cnn2d_strips
#define scratch_setup stub_scratch_setup
#define main harness_main
namespace ca {
hipError_t stub_launch_strips(const StripArgs &, size_t, hipStream_t, hipEvent_t, hipEvent_t);
hipError_t stub_launch_cnn_strips(const CnnStripArgs &, int, hipStream_t, hipEvent_t, hipEvent_t);
hipError_t stub_launch_cnn2d_strips(const Cnn2dStripArgs &, hipStream_t, hipEvent_t, hipEvent_t);
}  // namespace ca
namespace cahost {
int stub_scratch_setup(int);
}
#include "host_harness.cpp"
#undef launch_strips
#undef launch_cnn_strips
#undef launch_cnn2d_strips
#undef scratch_setup
#undef main

// the entry point without allocation; its scratch counts as device memory
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) x
inline hipError_t hipGetSymbolAddress(void **p, uint8_t *symbol)
{
    *p = symbol;
    g_allocs[reinterpret_cast<uintptr_t>(symbol)] = {CA_NOALLOC_SCRATCH_BYTES, true, false};
    return hipSuccess;
}
#include "ca_noalloc.hip"

namespace {

struct Launch {
    int scorer;
    int mixed;                   // taken for a batch of several shapes
    int spread;                  // of the handcrafted strips
    std::vector<int32_t> order;  // the frames, where a list gives them
};
std::vector<Launch> g_launches;

template <class Args>
void record(int scorer, const Args &a, int mixed, int spread, const int32_t *list)
{
    Launch l = {scorer, mixed, spread, {}};
    if (list)
        l.order.assign(list, list + a.n_items / (a.n_h + a.n_v));
    g_launches.push_back(l);
}

}  // namespace

namespace ca {

hipError_t launch_strips(const StripArgs &a, size_t lds, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    record(0, a, a.spread != kSpreadSlices, a.spread, a.frame_list);
    return stub_launch_strips(a, lds, s, e0, e1);
}
hipError_t launch_cnn_strips(const CnnStripArgs &a, int groups, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1)
{
    record(1, a, a.mixed, 0, nullptr);
    return stub_launch_cnn_strips(a, groups, s, e0, e1);
}
hipError_t launch_cnn2d_strips(const Cnn2dStripArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    record(2, a, a.mixed, 0, nullptr);
    return stub_launch_cnn2d_strips(a, s, e0, e1);
}

}  // namespace ca

namespace {

typedef std::vector<std::pair<int32_t, int32_t>> Sizes;

struct Bench {
    ca_ctx *ctx = nullptr;
    Bench()
    {
        CHECK(ca_create(&ctx, 0, 0) == CA_OK);
        set_model(ctx);
        std::vector<float> prm(CA_CNN2D_PARAMS, 0.01f);
        CHECK(ca_set_model_2d(ctx, prm.data(), CA_CNN2D_PARAMS) == CA_OK);
    }
    ~Bench() { ca_destroy(ctx); }
};

ca_params params_of(int scorer)
{
    ca_params p;
    ca_default_params(&p);
    p.n_hstrips = 32;
    p.n_vstrips = 31;
    p.scorer = scorer;
    return p;
}

// The strip launches of one call on frames of these sizes.
std::vector<Launch> call(ca_ctx *ctx, const Sizes &sizes, int scorer, bool noalloc)
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
    const int32_t n = (int32_t)dims.size();
    void *frames = nullptr, *out = nullptr;
    CHECK(hipMalloc(&frames, total) == hipSuccess);
    CHECK(hipMalloc(&out, sizeof(ca_result) * dims.size()) == hipSuccess);
    const ca_params p = params_of(scorer);
    g_launches.clear();
    CHECK((noalloc ? ca_estimate_area_noalloc : ca_estimate_area)(
              ctx, static_cast<const uint8_t *>(frames), dims.data(), n, &p,
              static_cast<ca_result *>(out), nullptr)
          == CA_OK);
    CHECK(hipFree(frames) == hipSuccess && hipFree(out) == hipSuccess);
    return g_launches;
}

// One frame of each of these streams through a server's batch.
std::vector<Launch> served(ca_ctx *ctx, const Sizes &sizes, int scorer)
{
    ca_server_config cfg = config(64, 2, (size_t)1 << 30, scorer);
    cfg.params = params_of(scorer);
    ca_server *srv = nullptr;
    CHECK(ca_server_create(ctx, &cfg, &srv) == CA_OK);
    std::vector<void *> frames;
    for (size_t i = 0; i < sizes.size(); ++i) {
        int32_t admitted = 0;
        CHECK(ca_server_open(srv, (int32_t)i, sizes[i].first, sizes[i].second, &admitted) == CA_OK
              && admitted);
        void *f = nullptr;
        CHECK(hipMalloc(&f, (size_t)3 * sizes[i].first * sizes[i].second) == hipSuccess);
        frames.push_back(f);
        CHECK(ca_server_submit(srv, (int32_t)i, 0, static_cast<uint8_t *>(f),
                               3 * (int64_t)sizes[i].first, 1)
              == CA_OK);
    }
    g_launches.clear();
    std::vector<ca_served> got;
    for (int i = 0; i < 100 && got.size() < sizes.size(); ++i)
        step(srv, got);
    CHECK(got.size() == sizes.size());
    ca_server_destroy(srv);
    for (void *f : frames)
        CHECK(hipFree(f) == hipSuccess);
    return g_launches;
}

void expect_mixed(const std::vector<Launch> &l, const Sizes &sizes, bool mixed, const char *what)
{
    if (l.size() != 1 || l[0].mixed != (mixed ? 1 : 0))
        fail("not dispatched as it should be: %s", what);
    if (!mixed || l[0].scorer != 0)
        return;
    // every frame once, the largest first
    if (l[0].order.size() != sizes.size())
        fail("without its list of frames: %s", what);
    int64_t last = INT64_MAX;
    std::set<int32_t> seen;
    for (const int32_t f : l[0].order) {
        CHECK(f >= 0 && f < (int32_t)sizes.size() && seen.insert(f).second);
        const int64_t area = (int64_t)sizes[f].first * sizes[f].second;
        if (area > last)
            fail("not the largest frames first: %s", what);
        last = area;
    }
}

}  // namespace

int main()
{
    const Sizes one(6, {1920, 1080});
    const Sizes four = {{720, 576}, {1280, 720}, {1920, 1080}, {720, 576}, {3840, 2160}, {1280, 720}};
    Sizes turned, many;   // equal areas, other shapes; enough for whole frames to the XCDs
    for (int i = 0; i < 8; ++i)
        turned.push_back(i % 3 ? std::make_pair(1920, 1080) : std::make_pair(1080, 1920));
    for (int i = 0; i < 64; ++i)
        many.push_back(four[i % 6]);
    cahost::scratch_setup(0);
    Bench b;
    const struct {
        const Sizes &sizes;
        bool mixed;
        const char *name;
    } batches[] = {{one, false, "one shape"}, {four, true, "four shapes"},
                   {turned, true, "one area, two shapes"}, {many, true, "many frames"}};
    for (const auto &t : batches)
        for (int scorer = 0; scorer < 3; ++scorer) {
            std::vector<int> spreads;
            for (int route = 0; route < 3; ++route) {
                const std::string what = std::string(t.name) + (route == 0   ? ", cached plan"
                                                                : route == 1 ? ", no allocation"
                                                                             : ", served");
                const auto l = route == 2 ? served(b.ctx, t.sizes, scorer)
                                          : call(b.ctx, t.sizes, scorer, route == 1);
                expect_mixed(l, t.sizes, t.mixed, what.c_str());
                spreads.push_back(l[0].spread);
            }
            if (spreads[0] != spreads[1] || spreads[0] != spreads[2])
                fail("dealt differently by route: %s", t.name);
        }
    std::printf("ok dispatch of shapes\n");
    return 0;
}
