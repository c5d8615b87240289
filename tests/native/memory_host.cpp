// The library's host side (osc_host.hip) on a pretended device of 1000 MB,
// without a GPU: the workspace kept between template builds gives way to every
// other allocation, on any context of the device, but not while a build uses it.
#include <cstdio>
#include <cstdlib>
#include <map>

// the host compiler's place for the library's one device array
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (x)

#include "../../paper_1311_7579_amd/csrc/osc_host.hip"

namespace {

constexpr size_t kMB = 1000 * 1000, kDevice = 1000 * kMB;
int g_current = 0;
hipError_t g_last = hipSuccess;
std::map<void*, std::pair<int, size_t>> g_blocks;   // device, bytes

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n)
{
    size_t used = 0;
    for (const auto& b : g_blocks)
        if (b.second.first == g_current) used += b.second.second;
    if (used + n > kDevice) return g_last = hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_blocks[*p] = {g_current, n};
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (!g_blocks.erase(p)) std::abort();
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int* d) { *d = g_current; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_current = d; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    *p = {};
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* s)
{
    *p = const_cast<void*>(s);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = reinterpret_cast<hipStream_t>(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = reinterpret_cast<hipEvent_t>(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t)
{
    return hipSuccess;
}
}

namespace osc {
hipError_t launch_tiles(int, bool, bool, const SetConsts&, const PathConsts&, const BinConsts&,
                        int64_t, const double*, const uint8_t*, const double*, const double*,
                        const uint16_t*, const double*, double*, double*, hipStream_t, hipEvent_t,
                        hipEvent_t)
{
    return hipGetLastError();   // as after a launch
}
hipError_t launch_bin_slots(int64_t, const double*, const BinConsts&, uint16_t*, hipStream_t)
{
    return hipGetLastError();
}
hipError_t launch_layered_tiles(int, bool, const SetConsts&, const LayerPath&, const BinConsts&,
                                int64_t, const double*, const uint8_t*, const double*,
                                const double*, double*, double*, hipStream_t, hipEvent_t,
                                hipEvent_t)
{
    return hipSuccess;
}
// 1 MB of scratch for each 1024 events
MergePlan plan_merge(const int64_t* tiles, int, int nbt, int64_t)
{
    MergePlan p;
    p.nbt = nbt;
    p.tile_set_stride = tiles[0] * int64_t(kMB / sizeof(double));
    return p;
}
size_t merge_scratch_bytes(const MergePlan& p, int64_t n_sets)
{
    return size_t(n_sets) * size_t(p.tile_set_stride) * sizeof(double);
}
hipError_t launch_merge(const MergePlan&, int64_t, double*, double*, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_merge_serve(const MergePlan&, double*, const ServeFinish&, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_serve_finish(const ServeFinish&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_poisson_nll(const double*, int64_t, double, const double*, int64_t, int, double*,
                              hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_validate_sample(int64_t, const double*, const uint8_t*, unsigned long long*,
                                  hipStream_t)
{
    return hipSuccess;
}
hipError_t occupancy(int, int, int* n) { *n = 1; return hipSuccess; }
hipError_t set_kernel_attributes(size_t) { return hipSuccess; }
}  // namespace osc

int main()
{
    osc_ctx *a = nullptr, *b = nullptr, *other = nullptr;
    osc_create(&a, 0);
    osc_create(&b, 0);
    osc_create(&other, 1);
    const osc_params p{0.307, 0.5, 0.02, 2.5e-3, 7.5e-5, 0.0};
    osc_set_params(a, &p, 1);
    double d = 0.0;
    uint8_t f = 0;
    const osc_binning bins{10, 0.0, 1.0, 0.0};
    const auto sample = [&](int64_t n) { return osc_sample{n, &d, &f, &d, &d, 295.0, 2.6, 0.5}; };
    const auto build = [&](osc_ctx* ctx, size_t mb) {
        (void)hipSetDevice(ctx->device);
        osc::host::BuildSpace s;
        return int(s.acquire(ctx, mb * kMB));
    };
    const auto kept = [&] {
        std::printf("kept %zu %zu %zu\n", a->build_cap / kMB, b->build_cap / kMB,
                    other->build_cap / kMB);
    };
    std::printf("builds %d %d %d\n", build(a, 500), build(b, 300), build(other, 400));
    kept();
    // 300 million events: 600 MB of slots; nothing of the other device's
    const osc_sample big = sample(300 * 1000 * 1000);
    osc_binned* binned = nullptr;
    std::printf("binned %d\n", int(osc_binned_create(a, &big, &bins, &binned)));
    kept();
    osc_binned_destroy(binned);
    // 700 MB of scratch
    std::printf("build %d\n", build(b, 400));
    const osc_sample s700 = sample(700 * 1024);
    std::printf("fill %d\n", int(osc_fill_pdf(a, &s700, 0, &bins, OSC_FP64, &d, nullptr, nullptr)));
    kept();
    // a workspace in use stays, and the failure leaves no error behind
    std::printf("build %d\n", build(b, 200));
    {
        osc::host::BuildSpace s;
        std::printf("held %d\n", int(s.acquire(b, 250 * kMB)));
        void* const held = s.ptr();
        std::printf("binned %d\n", int(osc_binned_create(a, &big, &bins, &binned)));
        std::printf("same %d\n", int(s.ptr() == held && g_blocks.count(held) == 1));
    }
    const osc_sample small = sample(2048);
    std::printf("fill %d\n", int(osc_fill_pdf(a, &small, 0, &bins, OSC_FP64, &d, nullptr, nullptr)));
    osc_destroy(b);
    osc_destroy(a);
    osc_destroy(other);
    std::printf("left %zu\n", g_blocks.size());
    return 0;
}
