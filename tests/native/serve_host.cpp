// The serving form's host side (osc_serve.hip holds no device code) against a
// pretended device, without a GPU: requests are finished by the block counter
// and the flag as the merge kernel does it, from a thread of this program.
//   serve_host lost  a request whose blocks stop half way, then one on its slot
//   serve_host idle  CPU time while one long request is in flight
#include <sys/resource.h>

#include <cstdio>
#include <cstring>

#include "../../paper_1311_7579_amd/csrc/osc_serve.hip"

namespace {

constexpr int kBins = 6;

struct Plan {
    int blocks = kBins + 2;   // blocks that run
    double delay_s = 0.0;     // before the first of them
};
Plan g_plan;
std::atomic<int> g_running{0};
std::vector<std::thread> g_threads;

// merge_serve_kernel: each block stores its total and takes a ticket; the one
// that finds itself last ends the request.
void device(osc::ServeFinish f, Plan plan, double value)
{
    std::this_thread::sleep_for(std::chrono::duration<double>(plan.delay_s));
    for (int b = 0; b < plan.blocks; ++b) {
        f.hist[b] = value + b;
        const unsigned before = (*f.ticket)++;
        if (before + 1u != unsigned(kBins + 2)) continue;
        *f.ticket = 0;
        std::memcpy(f.host, f.hist, (kBins + 2) * sizeof(double));
        __atomic_store_n(f.flag, f.seq, __ATOMIC_RELEASE);
    }
    --g_running;
}

double cpu_s()
{
    rusage u{};
    getrusage(RUSAGE_SELF, &u);
    return double(u.ru_utime.tv_sec + u.ru_stime.tv_sec) +
           1e-6 * double(u.ru_utime.tv_usec + u.ru_stime.tv_usec);
}

}  // namespace

extern "C" {
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n)
{
    return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return g_running ? hipErrorNotReady : hipSuccess; }
osc_status osc_validate_params(const osc_params*, int32_t) { return OSC_OK; }
}

namespace osc {
namespace host {
hipError_t device_malloc(void** p, size_t n, const osc_ctx*) { return hipMalloc(p, n); }
SetConsts set_consts(const osc_params& p)
{
    SetConsts s{};
    s.T0 = p.delta_cp;
    return s;
}
bool sample_ok(const osc_sample*, bool) { return true; }
bool binning_ok(const osc_ctx*, const osc_binning*) { return true; }
int ctx_device(const osc_ctx*) { return 0; }
size_t fill_scratch_bytes(int64_t, int) { return 1024; }
hipError_t enqueue_bin_slots(const osc_sample*, const osc_binning*, uint16_t*, hipStream_t)
{
    return hipSuccess;
}
hipError_t enqueue_served(const SetConsts& sc, const osc_sample*, const uint16_t*,
                          const osc_binning*, bool, double*, const ServeFinish& f, hipStream_t)
{
    ++g_running;
    g_threads.emplace_back(device, f, g_plan, sc.T0);
    return hipSuccess;
}
}  // namespace host
}  // namespace osc

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    int ctx = 0;
    osc_sample sample{};
    const osc_binning bins{kBins, 0.0, 1.0, 0.0};
    const osc_server_config cfg{1, 16, 1 << 20};
    osc_server* sv = nullptr;
    if (osc_server_create(reinterpret_cast<osc_ctx*>(&ctx), &sample, 1, &bins, &cfg, &sv) != OSC_OK)
        return 2;
    osc_params p{};
    double h[kBins + 2];
    const auto run = [&](Plan plan, double value) {
        g_plan = plan;
        p.delta_cp = value;
        uint64_t t = 0;
        osc_server_submit(sv, &p, 0, OSC_FP64, &t);
        return int(osc_server_wait(sv, t, h, nullptr, nullptr, nullptr));
    };
    if (what == "lost") {
        std::printf("%d\n", run({}, 100.0));
        std::printf("%d\n", run({5, 0.0}, 200.0));
        for (double value : {300.0, 400.0}) {
            std::printf("%d", run({}, value));
            for (double v : h) std::printf(" %g", v - value);
            std::printf("\n");
        }
    } else {
        const double t0 = now_s(), c0 = cpu_s();
        const int st = run({kBins + 2, 0.5}, 1.0);
        std::printf("%d %.4f\n", st, (cpu_s() - c0) / (now_s() - t0));
    }
    osc_server_destroy(sv);
    for (std::thread& t : g_threads) t.join();
    return 0;
}
