// HIP kernels of libosc for gfx950 (CDNA4, wave64).
//
// One wave64 owns one tile of kTileEvents consecutive events (four or eight
// share it where tiles are few).  Lane l of
// tile t handles events t*T + m*64 + l, m = 0..K-1 (coalesced SoA loads,
// software-pipelined one group of kGroup events ahead), computes the oscillation
// probability of each event in FP64 (flavour basis, one amplitude element
// per event), optionally writes it, and adds w * P into a per-wave
// histogram held in LDS (kHistLanes accumulators per bin, each shared by
// kLaneShare lanes that add in ascending lane order: masked LDS atomic adds,
// one lane group after the other).  The accumulators of the tile meet in a
// fixed binary tree; a merge kernel adds the tile results per bin in a
// fixed binary tree.  Every addition has a fixed place in that order, so
// the bits of the histogram do not depend on the launch shape or timing.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "osc_device.h"
#include "osc_host_common.h"
#include "osc_internal.h"
#include "osc_launch.h"

namespace osc {

namespace {

using namespace dev;

// Register budget for kTileWavesPerSimd resident waves per SIMD.
template <int MODE, bool WRITE_P, bool MIXED = false, int SPLIT = 1>
__global__ __launch_bounds__(kTileLanes * SPLIT)
__attribute__((amdgpu_waves_per_eu(kTileWavesPerSimd)))
void tile_kernel(
    SetConsts sc, PathConsts pc, BinConsts bc, int64_t n,
    const double* __restrict__ e_true, const uint8_t* __restrict__ flags,
    const double* __restrict__ weight, const double* __restrict__ e_reco,
    const uint16_t* __restrict__ bins, const double* __restrict__ value,
    double* __restrict__ p_out, double* __restrict__ partial)
{
    extern __shared__ double hist[];
    __shared__ Tables<MIXED> tabs;

    const int thread = threadIdx.x;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int nbt = bc.nb + 2;
    const TileArrays t = tile_arrays(tile, n, e_true, flags, weight, e_reco, bins, value, p_out);
    const int wave = __builtin_amdgcn_readfirstlane(thread / kTileLanes);
    const int lane = thread % kTileLanes;
    const TileBufs bufs = tile_bufs<MODE>(t.n, t.e_true, t.flags, t.weight, t.e_reco, t.bins,
                                          t.value, t.p_out);

    if (MODE != kHist) {
        load_tab(sc, tabs, thread);
        if constexpr (!MIXED) load_sincos(tabs, thread);
    }
    if (MODE != kReweight) hist_zero<kTileLanes * SPLIT>(hist, thread, nbt);
    __syncthreads();

    const ConstDensityProb<MIXED> prob{&sc, &tabs, pc.kA, pc.kL,
                                       MIXED ? PolyRegs{} : PolyRegs::in_vgprs()};
    if constexpr (SPLIT > 1)
        split_tile_events<MODE, WRITE_P, SPLIT>(prob, bc, hist, bufs, wave, lane, t.n);
    else if (t.n == kTileEvents)
        tile_events<MODE, WRITE_P, true, WRITE_P>(prob, bc, hist, thread, t.n, t.e_true, t.flags,
                                                  t.weight, t.e_reco, t.bins, t.value, t.p_out);
    else
        tile_events<MODE, WRITE_P, false, WRITE_P>(prob, bc, hist, thread, t.n, t.e_true, t.flags,
                                                   t.weight, t.e_reco, t.bins, t.value, t.p_out);

    if (MODE != kReweight) {
        if (SPLIT == 1) __syncthreads();   // split tiles end with a barrier
        tile_write<kTileLanes * SPLIT>(hist, thread, nbt, tile, partial, gridDim.x == 1);
    }
}

// The same tile body with P through a layered path (FP64 only).  The event
// loop stays rolled: 16 unrolled copies of the layer loop would not fit the
// instruction cache.
template <int MODE, bool WRITE_P, int SPLIT = 1>
__global__ __launch_bounds__(kTileLanes * SPLIT)
__attribute__((amdgpu_waves_per_eu(kLayeredWavesPerSimd)))
void layered_tile_kernel(SetConsts sc, LayerPath lp, BinConsts bc, int64_t n,
                         const double* __restrict__ e_true, const uint8_t* __restrict__ flags,
                         const double* __restrict__ weight, const double* __restrict__ e_reco,
                         double* __restrict__ p_out, double* __restrict__ partial)
{
    extern __shared__ double hist[];
    __shared__ LayeredTables tabs;

    const int thread = threadIdx.x;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int nbt = bc.nb + 2;
    const TileArrays t =
        tile_arrays(tile, n, e_true, flags, weight, e_reco, nullptr, nullptr, p_out);
    const int wave = __builtin_amdgcn_readfirstlane(thread / kTileLanes);
    const int lane = thread % kTileLanes;
    const TileBufs bufs = tile_bufs<MODE>(t.n, t.e_true, t.flags, t.weight, t.e_reco, nullptr,
                                          nullptr, t.p_out);

    load_tab(lp, tabs, thread);
    load_sincos(tabs, thread);
    if (MODE != kReweight) hist_zero<kTileLanes * SPLIT>(hist, thread, nbt);
    __syncthreads();

    const LayeredProb prob{&sc, &tabs, &lp};
    if constexpr (SPLIT > 1)
        split_tile_events<MODE, WRITE_P, SPLIT>(prob, bc, hist, bufs, wave, lane, t.n);
    else if (t.n == kTileEvents)
        tile_events<MODE, WRITE_P, true, true>(prob, bc, hist, thread, t.n, t.e_true, t.flags,
                                               t.weight, t.e_reco, nullptr, nullptr, t.p_out);
    else
        tile_events<MODE, WRITE_P, false, true>(prob, bc, hist, thread, t.n, t.e_true, t.flags,
                                                t.weight, t.e_reco, nullptr, nullptr, t.p_out);

    if (MODE != kReweight) {
        if (SPLIT == 1) __syncthreads();   // split tiles end with a barrier
        tile_write<kTileLanes * SPLIT>(hist, thread, nbt, tile, partial, gridDim.x == 1);
    }
}

template <bool FINAL, int WAVES, int ROWS>
__global__ __launch_bounds__(WAVES * 64) void merge_level_kernel(MergeLevel L,
                                                                 const double* __restrict__ in,
                                                                 double* __restrict__ out)
{
    merge_level_block<WAVES, ROWS>(
        L, in, [&](int64_t set, int s, int64_t c, int bin, double total) {
            if (FINAL)
                out[(set * L.n_samples + s) * L.nbt + bin] = total;
            else
                out[set * L.set_stride_out + partial_index(L.out_row0[s] + c, bin, L.nbt)] = total;
        });
}

// Ends a served request, by one wave (see ServeFinish).  The burst of 64
// requests on samples of 1e4 to 2e7 events takes 1.7 ms (26 us a request) and
// a lone request on 1e5 events 35 us; with a likelihood kernel, a copy and a
// callback after the merge, and the dispatcher asleep between looks, they took
// 3.2 ms (51 us) and 132 us, bound by the runtime calls.  The histogram is read
// with device-scope loads: its entries may come from other blocks of this
// launch.
__device__ __forceinline__ void serve_finish(const ServeFinish& f, int nbt, int lane)
{
    const auto hist = [&](int b) {
        return __hip_atomic_load(&f.hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int b = lane; b < nbt; b += 64) f.host[b] = hist(b);
    if (f.data) {
        const double nll = poisson_nll(hist, f.data, f.mu_scale, nbt - 2, lane);
        if (lane == 0) f.host[nbt] = nll;
    }
    __threadfence_system();   // every lane's results reach the host before the flag
    if (lane == 0)
        __hip_atomic_store(f.flag, f.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The final merge level of a served request (one set, one sample).  The block
// that finishes last (each block stores its total before it takes a ticket)
// ends the request, so that a request of up to 4096 tiles takes two launches and
// neither a copy nor a callback.
template <int WAVES, int ROWS>
__global__ __launch_bounds__(WAVES * 64) void merge_serve_kernel(MergeLevel L,
                                                                 const double* __restrict__ in,
                                                                 ServeFinish f)
{
    __shared__ bool last;
    merge_level_block<WAVES, ROWS>(L, in, [&](int64_t, int, int64_t, int bin, double total) {
        __hip_atomic_store(&f.hist[bin], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned before =
            __hip_atomic_fetch_add(f.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        last = before + 1u == gridDim.x * gridDim.y;
        // nobody else takes a ticket any more: clear it for the next request
        if (last) __hip_atomic_store(f.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
    __syncthreads();
    if (last && threadIdx.x < 64) serve_finish(f, L.nbt, threadIdx.x);
}

// Ends a served request whose single tile wrote the histogram itself.
__global__ __launch_bounds__(64) void serve_finish_kernel(ServeFinish f, int nbt)
{
    serve_finish(f, nbt, threadIdx.x);
}

// Eq. (2) as a product of Poisson probabilities over the regular bins; one
// wave per histogram.
__global__ __launch_bounds__(64) void poisson_nll_kernel(const double* __restrict__ hist,
                                                         double scale, int64_t n_data,
                                                         const double* __restrict__ data,
                                                         int nbins, double* __restrict__ out)
{
    const int64_t k = blockIdx.x;
    const int lane = threadIdx.x;
    const double* h = hist + k * (nbins + 2);
    const double nll =
        poisson_nll([&](int b) { return h[b]; }, data + (k % n_data) * nbins, scale, nbins, lane);
    if (lane == 0) out[k] = nll;
}

// The cached histogram slot of every event of a sample: the LDS slot
// (hslot) its contribution goes to in the per-event kernels, from the bin
// of e_reco by the exact rule (a correctly rounded division) and the
// accumulator of its lane, event index mod kHistLanes (tiles start at
// multiples of kTileEvents, so an event's lane is its index mod 64).
__global__ __launch_bounds__(256) void bin_slot_kernel(int64_t n, const double* __restrict__ e_reco,
                                                       BinConsts bc, uint16_t* __restrict__ out)
{
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        out[i] = uint16_t(hslot(lds_bin(bin_floor_exact(e_reco[i], bc), bc),
                                int(i & (kHistLanes - 1))));
}

// One-time domain check of a sample: counts of events whose true energy
// is not finite and positive, and of events with an invalid flag byte.
// Grid-stride loop; per-wave sums, one integer atomic per wave and counter
// (integer sums: the totals do not depend on the order).
__global__ __launch_bounds__(256) void validate_sample_kernel(int64_t n,
                                                              const double* __restrict__ e_true,
                                                              const uint8_t* __restrict__ flags,
                                                              unsigned long long* __restrict__ bad)
{
    unsigned long long be = 0, bf = 0;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x) {
        const double e = e_true[i];
        const uint32_t f = flags[i];
        be += (e > 0.0 && e <= __DBL_MAX__) ? 0ull : 1ull;   // NaN fails both tests
        bf += ((f < 32u) && ((kValidFlags >> (f & 31u)) & 1u)) ? 0ull : 1ull;
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        be += __shfl_xor(be, s, 64);
        bf += __shfl_xor(bf, s, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (be) atomicAdd(&bad[0], be);
        if (bf) atomicAdd(&bad[1], bf);
    }
}

}  // namespace

hipError_t launch_validate_sample(int64_t n, const double* e_true, const uint8_t* flags,
                                  unsigned long long* bad, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(validate_sample_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, n,
                       e_true, flags, bad);
    return hipGetLastError();
}

hipError_t launch_bin_slots(int64_t n, const double* e_reco, const BinConsts& bc, uint16_t* out,
                            hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(bin_slot_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, n, e_reco,
                       bc, out);
    return hipGetLastError();
}

hipError_t launch_poisson_nll(const double* hist, int64_t n_hist, double scale,
                              const double* data, int64_t n_data, int nbins, double* out,
                              hipStream_t stream)
{
    if (n_hist == 0) return hipSuccess;
    hipLaunchKernelGGL(poisson_nll_kernel, dim3(unsigned(n_hist)), dim3(64), 0, stream, hist,
                       scale, n_data, data, nbins, out);
    return hipGetLastError();
}

namespace {

// Waves that share a tile.  Few tiles leave the chip's 1024 SIMDs with a wave
// or less each, and a wave's 16 events then run one after the other at the
// latency of their dependent arithmetic and loads; more waves per tile cost
// barriers between their additions and tables filled per tile.  Per-event
// kernel with one wave | four | eight a tile (us, FP64, 50 bins, no P unless
// said): 1e4 events 10.6 | 6.6 | 6.1, 7.7e5 12.1 | 9.0 | 8.9, 1e6 11.6 | 10.3
// | 11.1, 6e6 36.2 | 35.0 | 46.8, 1e7 57.4 | 57.3 | 81.6; with P written 2e6
// 17.5 | 17.3 | 19.2, 3e6 22.4 | 22.8 | 26.3; P alone 1e3 8.2 | 4.0 | 4.0,
// 6e6 31.1 | 30.0 | 32.2; five layers 1e4 33.5 | 13.1 | 10.8, 4e6 99 | 98 | 97.
// The FP32-mixed tier, computed bins and 20 to 600 bins take the same lines: at
// worst 5 % over one wave (6.2e6 events, mixed, computed bins, 20 bins: 34.3 |
// 36.0), and far under it with many bins (6.2e6, 600 bins: 115 | 58).
//
// Given values (kHist) have no arithmetic to share, and four waves only pay
// where one-wave blocks, each with a histogram of its own, would wait for LDS
// (kHistLdsSplit: five eighths of the chip's 256 x 160 KB).  One wave | four |
// eight: 1e6 events of 50 bins 7.3 | 7.5 | 7.2, 2e6 11.8 | 12.5 | 13.9, 3e6 of 20
// bins 15.1 | 16.2 | 16.8, of 200 bins 20.6 | 17.3 | 18.7, 6.2e6 of 100 bins 27.0
// | 25.6 | 27.5, 4e6 of 600 bins 40.5 | 26.7 | 25.9.
constexpr int64_t kHistLdsSplit = 26 << 20;
int tile_split(int64_t ntiles, int mode, bool write_p, size_t hist_bytes)
{
    if (mode == kReweight) return ntiles <= 6144 ? 4 : 1;
    if (mode == kHist) {
        if (ntiles <= 1024) return 8;
        return ntiles <= 6144 && ntiles * int64_t(hist_bytes) > kHistLdsSplit ? 4 : 1;
    }
    if (ntiles <= 768) return 8;
    return ntiles <= (write_p ? 2048 : 6144) ? 4 : 1;
}

// The same for a layered path: with one layer to solve, the barriers between
// the waves' additions weigh more against the arithmetic.  One layer, histogram,
// one wave | eight: 1e6 events 19.9 | 15.7, 1.6e6 25.7 | 24.6, 2e6 26.1 | 28.1,
// 4.1e6 40.2 | 50.1; two layers that differ 2.5e6 48.3 | 41.8, 4.1e6 62.0 | 63.4;
// one layer, P alone 2.5e6 23.8 | 20.3, 4.1e6 31.4 | 33.3.
int layered_split(int64_t ntiles, int mode, const LayerPath& lp)
{
    return ntiles <= (lp.n == 1 && mode != kReweight ? 1600 : 4096) ? 8 : 1;
}

template <int N>
using Int = std::integral_constant<int, N>;

}  // namespace

hipError_t launch_tiles(int mode, bool write_p, bool mixed, const SetConsts& sc,
                        const PathConsts& pc, const BinConsts& bc, int64_t n,
                        const double* e_true, const uint8_t* flags, const double* weight,
                        const double* e_reco, const uint16_t* bins, const double* value,
                        double* p_out, double* partial, hipStream_t stream, hipEvent_t ev_begin,
                        hipEvent_t ev_end)
{
    const int64_t ntiles = (n + kTileEvents - 1) / kTileEvents;
    if (ntiles == 0) return hipSuccess;
    const size_t lds = mode == kReweight ? 0 : size_t(bc.nb + 2) * kHistLanes * sizeof(double);
    const auto launch = [&](auto m, auto w, auto x) {
        const auto with = [&](auto split) {
            constexpr int kSplit = decltype(split)::value;
            hipExtLaunchKernelGGL(
                (tile_kernel<decltype(m)::value, decltype(w)::value, decltype(x)::value, kSplit>),
                dim3{unsigned(ntiles)}, dim3{unsigned(kTileLanes * kSplit)}, lds, stream, ev_begin,
                ev_end, 0, sc, pc, bc, n, e_true, flags, weight, e_reco, bins, value, p_out,
                partial);
        };
        constexpr int kMode = decltype(m)::value;
        const int split = tile_split(ntiles, kMode, decltype(w)::value, lds);
        if (split == 4) return with(Int<4>{});
        if constexpr (kMode != kReweight)
            if (split == 8) return with(Int<8>{});
        with(Int<1>{});
    };
    using std::false_type;
    using std::true_type;
    const auto by_output = [&](auto m) {
        if (write_p && mixed) launch(m, true_type{}, true_type{});
        else if (write_p) launch(m, true_type{}, false_type{});
        else if (mixed) launch(m, false_type{}, true_type{});
        else launch(m, false_type{}, false_type{});
    };
    if (mode == kReweight) launch(Int<kReweight>{}, true_type{}, false_type{});
    else if (mode == kPdf) by_output(Int<kPdf>{});
    else if (mode == kPdfBinned) by_output(Int<kPdfBinned>{});
    else launch(Int<kHist>{}, false_type{}, false_type{});
    return hipGetLastError();
}

hipError_t launch_layered_tiles(int mode, bool write_p, const SetConsts& sc,
                                const LayerPath& lp, const BinConsts& bc, int64_t n,
                                const double* e_true, const uint8_t* flags, const double* weight,
                                const double* e_reco, double* p_out, double* partial,
                                hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end)
{
    const int64_t ntiles = (n + kTileEvents - 1) / kTileEvents;
    if (ntiles == 0) return hipSuccess;
    const size_t lds = mode == kReweight ? 0 : size_t(bc.nb + 2) * kHistLanes * sizeof(double);
    const auto launch = [&](auto m, auto w) {
        const auto with = [&](auto split) {
            constexpr int kSplit = decltype(split)::value;
            hipExtLaunchKernelGGL(
                (layered_tile_kernel<decltype(m)::value, decltype(w)::value, kSplit>),
                dim3{unsigned(ntiles)}, dim3{unsigned(kTileLanes * kSplit)}, lds, stream, ev_begin,
                ev_end, 0, sc, lp, bc, n, e_true, flags, weight, e_reco, p_out, partial);
        };
        if (layered_split(ntiles, decltype(m)::value, lp) == 8) return with(Int<8>{});
        with(Int<1>{});
    };
    if (mode == kReweight) launch(Int<kReweight>{}, std::true_type{});
    else if (write_p) launch(Int<kPdf>{}, std::true_type{});
    else launch(Int<kPdf>{}, std::false_type{});
    return hipGetLastError();
}

// A level that is not the last divides every sample's row count by kScratchChunk
// (rounding up), so two levels reduce the largest accepted sample to one row.
constexpr int64_t kScratchChunk = 16384;
static_assert(kMaxEvents / kTileEvents <= kScratchChunk * kScratchChunk && kMaxMergeLevels >= 2,
              "the merge plan's level capacity covers every accepted sample");

namespace {

// Threads and rows per thread of a merge block, for samples of up to `rows`
// rows: few waves for few rows (most of a large block's threads would only
// wait for the others), and one launch instead of two up to 32768 rows: at
// 19532 rows x 52 bins 10.2 us from the per-event kernel's end against 12.9
// with two levels.  Above that one level's 64 rows a thread do not fit the
// registers of 1024 threads, and two levels are faster: 5e7 given values of 50
// bins (48829 rows) 252 us with two levels of 16 rows a thread, 256 of 32, 263
// with one level; 7e7 339, 340 and 353.  With blocks enough to fill the chip several times
// (`many`) 4097 to 8192 rows take 256 threads of 32 rows too: the 256-set x
// 4-sample batch (rows 98 to 4883) merges in 297 instead of 388 us with 1024
// threads of 16.
struct MergeShape {
    int waves, rows;
};
MergeShape merge_shape(int64_t rows, bool many)
{
    if (rows <= 1024) return {1, 16};
    if (rows <= 4096) return {4, 16};
    if (many && rows <= 8192) return {4, 32};
    if (rows > 16384 && rows <= 32768) return {16, 32};
    return {16, 16};
}

}  // namespace

MergePlan plan_merge(const int64_t* tiles, int n_samples, int nbt, int64_t n_sets)
{
    const bool many = n_sets * n_samples * nbt >= 4096;
    auto align = [](int64_t r) { return (r + kLayoutChunk - 1) / kLayoutChunk * kLayoutChunk; };
    MergePlan p;
    p.nbt = nbt;
    p.n_samples = n_samples;
    int64_t rows[kMaxBatchSamples], row0[kMaxBatchSamples];
    int64_t in_rows = 0;
    for (int s = 0; s < n_samples; ++s) {
        rows[s] = tiles[s];
        row0[s] = in_rows;
        in_rows += align(rows[s]);
    }
    // The level buffers are sized for chunks of kScratchChunk rows, the figure
    // that include/osc.h states and budgets are counted in; the chunks of the
    // levels are at least as large wherever a second level is needed.
    int64_t level_rows = 0;
    bool level_buffers = false;
    for (int s = 0; s < n_samples; ++s) {
        level_rows += align((rows[s] + kScratchChunk - 1) / kScratchChunk + (rows[s] == 0));
        level_buffers |= rows[s] > kScratchChunk;
    }
    p.level_set_stride = level_buffers ? level_rows * nbt : 0;
    for (bool first = true;; first = false) {
        MergeLevel& L = p.levels[p.n_levels];
        L = MergeLevel{};
        L.n_samples = n_samples;
        L.nbt = nbt;
        int64_t most = 0;
        for (int s = 0; s < n_samples; ++s) most = std::max(most, rows[s]);
        const MergeShape shape = merge_shape(most, many);
        const int64_t chunk = int64_t(shape.waves) * 64 * shape.rows;
        p.waves[p.n_levels] = shape.waves;
        p.thread_rows[p.n_levels] = shape.rows;
        int64_t chunks = 0, out_rows = 0;
        bool final_level = true;
        for (int s = 0; s < n_samples; ++s) {
            const int64_t r = rows[s];
            const int64_t ch = r > chunk ? (r + chunk - 1) / chunk : 1;
            L.rows[s] = r;
            L.in_row0[s] = row0[s];
            L.chunk0[s] = chunks;
            L.out_row0[s] = out_rows;
            chunks += ch;
            out_rows += align(ch);
            if (ch > 1) final_level = false;
            rows[s] = ch;
            row0[s] = L.out_row0[s];
        }
        L.total_chunks = chunks;
        L.set_stride_in = in_rows * nbt;
        L.set_stride_out = final_level ? 0 : out_rows * nbt;
        if (first) p.tile_set_stride = L.set_stride_in;
        ++p.n_levels;
        in_rows = out_rows;
        if (final_level) break;
    }
    return p;
}

size_t merge_scratch_bytes(const MergePlan& p, int64_t n_sets)
{
    return size_t(n_sets) * size_t(p.tile_set_stride + 2 * p.level_set_stride) * sizeof(double);
}

hipError_t launch_serve_finish(const ServeFinish& finish, int nbt, hipStream_t stream)
{
    hipLaunchKernelGGL(serve_finish_kernel, dim3(1), dim3(64), 0, stream, finish, nbt);
    return hipGetLastError();
}

namespace {

// Runs the merge levels with the final one writing hist_out, or, with
// `finish`, ending a served request.  Blocks of 16 waves leave that end to a
// kernel of its own: the likelihood in it takes 208 registers, which capped at
// the 128 of a 1024-thread block spilled 48, and a block needed a CU to itself
// among the other requests' waves.
hipError_t run_merge(const MergePlan& p, int64_t n_sets, double* scratch, double* hist_out,
                     const ServeFinish* finish, hipStream_t stream)
{
    double* bufs[2] = {scratch + n_sets * p.tile_set_stride,
                       scratch + n_sets * (p.tile_set_stride + p.level_set_stride)};
    if (finish) hist_out = finish->hist;
    const double* in = scratch;
    for (int l = 0; l < p.n_levels; ++l) {
        const MergeLevel& L = p.levels[l];
        const dim3 grid{unsigned(L.total_chunks), unsigned(p.nbt), unsigned(n_sets)};
        const bool final_level = l + 1 == p.n_levels;
        double* out = final_level ? hist_out : bufs[l % 2];
        const auto launch = [&](auto waves, auto rows) {
            constexpr int W = decltype(waves)::value, R = decltype(rows)::value;
            if constexpr (W < 16 && R == 16)
                if (final_level && finish) {
                    hipLaunchKernelGGL((merge_serve_kernel<W, R>), grid, dim3(W * 64), 0, stream,
                                       L, in, *finish);
                    finish = nullptr;
                    return;
                }
            if (final_level)
                hipLaunchKernelGGL((merge_level_kernel<true, W, R>), grid, dim3(W * 64), 0, stream,
                                   L, in, out);
            else
                hipLaunchKernelGGL((merge_level_kernel<false, W, R>), grid, dim3(W * 64), 0, stream,
                                   L, in, out);
        };
        if (p.waves[l] == 1) launch(Int<1>{}, Int<16>{});
        else if (p.waves[l] == 4 && p.thread_rows[l] == 16) launch(Int<4>{}, Int<16>{});
        else if (p.waves[l] == 4) launch(Int<4>{}, Int<32>{});
        else if (p.thread_rows[l] == 16) launch(Int<16>{}, Int<16>{});
        else launch(Int<16>{}, Int<32>{});
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        in = out;
    }
    return finish ? launch_serve_finish(*finish, p.nbt, stream) : hipSuccess;
}

}  // namespace

hipError_t launch_merge(const MergePlan& p, int64_t n_sets, double* scratch, double* hist_out,
                        hipStream_t stream)
{
    return run_merge(p, n_sets, scratch, hist_out, nullptr, stream);
}

hipError_t launch_merge_serve(const MergePlan& p, double* scratch, const ServeFinish& finish,
                              hipStream_t stream)
{
    return run_merge(p, 1, scratch, nullptr, &finish, stream);
}

hipError_t occupancy(int mode, int nbins, int* blocks_per_cu)
{
    const size_t lds = mode == kReweight ? 0 : size_t(nbins + 2) * kHistLanes * sizeof(double);
    const void* f = mode == kReweight ? reinterpret_cast<const void*>(&tile_kernel<kReweight, true>)
                  : mode == kPdf      ? reinterpret_cast<const void*>(&tile_kernel<kPdf, true>)
                                      : reinterpret_cast<const void*>(&tile_kernel<kHist, false>);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, kTileLanes, lds);
}

namespace {

// Raises the limit of kernels that keep histograms in dynamic LDS.
template <class... F>
hipError_t raise_lds_limit(int bytes, F... kernels)
{
    for (const void* f : {reinterpret_cast<const void*>(kernels)...}) {
        const hipError_t e =
            hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Those with SPLIT waves a tile.
template <int SPLIT>
hipError_t raise_tile_limits(int bytes)
{
    return raise_lds_limit(
        bytes, &tile_kernel<kPdf, true, false, SPLIT>, &tile_kernel<kPdf, false, false, SPLIT>,
        &tile_kernel<kPdf, true, true, SPLIT>, &tile_kernel<kPdf, false, true, SPLIT>,
        &tile_kernel<kHist, false, false, SPLIT>, &tile_kernel<kPdfBinned, true, false, SPLIT>,
        &tile_kernel<kPdfBinned, false, false, SPLIT>,
        &tile_kernel<kPdfBinned, true, true, SPLIT>, &tile_kernel<kPdfBinned, false, true, SPLIT>);
}

template <int SPLIT>
hipError_t raise_layered_limits(int bytes)
{
    return raise_lds_limit(bytes, &layered_tile_kernel<kPdf, true, SPLIT>,
                           &layered_tile_kernel<kPdf, false, SPLIT>);
}

}  // namespace

hipError_t set_kernel_attributes(size_t max_dyn_lds)
{
    const int bytes = int(max_dyn_lds);
    hipError_t e = raise_tile_limits<1>(bytes);
    if (e == hipSuccess) e = raise_tile_limits<4>(bytes);
    if (e == hipSuccess) e = raise_tile_limits<8>(bytes);
    if (e == hipSuccess) e = raise_layered_limits<1>(bytes);
    if (e == hipSuccess) e = raise_layered_limits<8>(bytes);
    return e;
}

}  // namespace osc
