// Bin-centre reweighting (Sec. 1.1.1): the approximation that event-by-event
// reweighting replaces.  A sample is reduced once to a migration template
// T[r][c][t] -- the Monte Carlo weight of channel c (alpha + 3 beta + 9 anti)
// in true-energy bin t and reconstructed-energy bin r -- and a parameter set
// is applied by evaluating P once per channel at every true-bin centre:
//   hist[r] = sum over k = c nt + t of fl(T[r][k] * P[k]).
//
// Template build (once, deterministic): every event gets a cell key, a
// stable radix sort of (key, weight) puts the weights of a cell in a row in
// ascending event order, and a wave adds each cell's row with the bits of
// one addition after the other.
// Per call: one kernel for the 18 nt probabilities (the same per-event
// arithmetic as the fused kernel), one wave per reconstructed bin for the
// contraction (lane-strided sums, then the wave's binary tree).
#include <hipcub/hipcub.hpp>
#include <rocprim/rocprim.hpp>

#include <cstdint>
#include <new>

#include "../../include/osc.h"
#include "osc_device.h"
#include "osc_host_common.h"
#include "osc_internal.h"

namespace osc {
namespace {

using namespace dev;

constexpr int kTemplateChannels = 18;

struct TrueBins {
    double lo, wb;
    int32_t nt;
};

// Cell key of every event: (r * 18 + c) * nt + t, or n_cells when the flag
// byte is invalid or the true energy is outside the true binning.
__global__ __launch_bounds__(256) void template_keys_kernel(
    int64_t n, const double* __restrict__ e_true, const uint8_t* __restrict__ flags,
    const double* __restrict__ e_reco, TrueBins tb, BinConsts rb, uint32_t n_cells,
    uint32_t* __restrict__ keys)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t f = flags[i];
    const bool valid = (f < 32u) && ((kValidFlags >> (f & 31u)) & 1u);
    double kt, kr;
    {
#pragma clang fp contract(off)
        kt = __builtin_floor((e_true[i] - tb.lo) / tb.wb);
        kr = __builtin_floor((e_reco[i] * rb.scale - rb.lo) / rb.wb);
    }
    const bool inside = kt >= 0.0 && kt < double(tb.nt);
    const int r = (kr < 0.0) ? rb.nb : ((kr < double(rb.nb)) ? int(kr) : rb.nb + 1);
    const uint32_t c = (f & 3u) + 3u * ((f >> 2) & 3u) + 9u * ((f >> 4) & 1u);
    keys[i] = (valid && inside)
                  ? (uint32_t(r) * kTemplateChannels + c) * uint32_t(tb.nt) + uint32_t(kt)
                  : n_cells;
}

// First and one-past-last position of every cell in the sorted keys, and in
// *used the number of keys below n_cells (they sort first; *used is 0
// beforehand).
__global__ __launch_bounds__(256) void template_bounds_kernel(int64_t n,
                                                              const uint32_t* __restrict__ keys,
                                                              uint32_t n_cells,
                                                              uint2* __restrict__ rows,
                                                              uint32_t* __restrict__ used)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t k = keys[i];
    if (k >= n_cells) return;
    const uint32_t next = i + 1 < n ? keys[i + 1] : n_cells;
    if (i == 0 || keys[i - 1] != k) rows[k].x = uint32_t(i);
    if (next != k) rows[k].y = uint32_t(i + 1);
    if (next >= n_cells) *used = uint32_t(i + 1);
}

// The weight sum of a cell is defined as one FP64 addition after the other,
// from +0.0 in event order: 1e5 dependent additions for the fullest cells.
// Most of them need not wait for each other.  While the sum s stays in one
// binade [2^k, 2^(k+1)), s is a multiple of g = 2^(k-52) and adding w >= 0
// adds r(w), w rounded to a multiple of g, which does not depend on s unless
// w lies exactly half way between two multiples (the tie then goes by the
// parity of s / g).  r(w) = fl(s + w) - s for any such s, both operations
// exact enough to recover the rounding w - r(w).  So the r of a block of
// values are formed independently from the s before the block and added in
// any order (sums of multiples of g below 2^(k+1) are exact), and the result
// stands if no w was negative, NaN or a tie and the new sum is still below
// 2^(k+1).  Otherwise the block is added row by row of 64, and a row that
// fails the same test one value after the other.  About one value in s / w
// is a tie, so that is the rule for the first thousand values of a cell and
// rare afterwards.

// Sum over the lanes of a wave in any order (for exact sums): DPP within
// rows of 16, then the four rows through SGPRs.
__device__ __forceinline__ double lanes_sum(double v)
{
    const auto step = [&](auto ctrl) {
        constexpr int c = decltype(ctrl)::value;
        v = v + __hiloint2double(
                    __builtin_amdgcn_mov_dpp(__double2hiint(v), c, 0xf, 0xf, true),
                    __builtin_amdgcn_mov_dpp(__double2loint(v), c, 0xf, 0xf, true));
    };
    step(std::integral_constant<int, 0xB1>{});    // quad_perm [1, 0, 3, 2]
    step(std::integral_constant<int, 0x4E>{});    // quad_perm [2, 3, 0, 1]
    step(std::integral_constant<int, 0x141>{});   // row_half_mirror
    step(std::integral_constant<int, 0x140>{});   // row_mirror
    const auto lane = [&](int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                                __builtin_amdgcn_readlane(__double2loint(v), l));
    };
    return (lane(0) + lane(16)) + (lane(32) + lane(48));
}

struct RowSum {
    double s;       // the sum before the block
    double acc;     // this lane's part of the block's r(w)
    bool bad;       // this lane has a value that does not fit the scheme
    double half_g;
    __device__ __forceinline__ explicit RowSum(double s0) : s(s0), acc(0.0)
    {
        const int e = (__double2hiint(s0) >> 20) & 0x7ff;
        bad = e < 64 || e > 2040 || __double2hiint(s0) < 0;
        half_g = __hiloint2double((e > 53 ? e - 53 : 0) << 20, 0);
    }
    __device__ __forceinline__ void add(double w)
    {
        const double t = s + w;
        const double r = t - s;
        bad = bad || !(w >= 0.0) || __builtin_fabs(w - r) == half_g;
        acc = acc + r;
    }
    // The end of the binade of the sum before the block.
    __device__ __forceinline__ double top() const
    {
        return __hiloint2double((__double2hiint(s) & 0x7ff00000) + 0x00100000, 0);
    }
    // The sum after the block (the same in every lane); false if it has to
    // be formed in smaller steps.
    __device__ __forceinline__ bool finish(double& out) const
    {
        if (__any(bad)) return false;
        out = s + lanes_sum(acc);
        return out < top();
    }
};

// One value after the other: the 64 lanes of v.
__device__ __forceinline__ double sum_in_order(double s, double v)
{
    const int hi = __double2hiint(v), lo = __double2loint(v);
#pragma unroll
    for (int j = 0; j < 64; ++j)
        s = s + __hiloint2double(__builtin_amdgcn_readlane(hi, j),
                                 __builtin_amdgcn_readlane(lo, j));
    return s;
}

// s plus the 64 lanes of v, in order.
__device__ __forceinline__ double add_row(double s, double v)
{
    RowSum row(s);
    row.add(v);
    double total;
    return row.finish(total) ? total : sum_in_order(s, v);
}

// s plus the block v (kSumRows rows of 64 values, the first at `first` of
// len; +0.0 past the end, which adds nothing).
constexpr int kSumRows = 16;
constexpr uint32_t kSumBlock = kSumRows * 64;

__device__ __forceinline__ void load_block(const double* __restrict__ ws, uint32_t first,
                                           uint32_t len, int lane, double (&v)[kSumRows])
{
#pragma unroll
    for (int j = 0; j < kSumRows; ++j) {
        const uint32_t i = first + j * 64 + lane;
        v[j] = i < len ? ws[i] : 0.0;
    }
}

// s plus the values of block v that are among the len of its row.  If the
// block does not stand as a whole, its rows of 64 follow one by one, read back
// from `rows` (LDS of the wave's own).
__device__ __forceinline__ double add_block(double s, const double (&v)[kSumRows],
                                            double* __restrict__ rows, uint32_t first,
                                            uint32_t len, int lane)
{
    RowSum block(s);
#pragma unroll
    for (int j = 0; j < kSumRows; ++j) block.add(v[j]);
    double total;
    if (block.finish(total)) return total;
    if (first >= len) return s;
#pragma unroll
    for (int j = 0; j < kSumRows; ++j) rows[j * 64 + lane] = v[j];
    const uint32_t n = min(kSumBlock, len - first);
    double next = rows[lane];
#pragma unroll 1
    for (uint32_t at = 0; at < n; at += 64) {
        const double row = next;
        if (at + 64 < n) next = rows[at + 64 + lane];
        s = add_row(s, row);
    }
    return s;
}

// Weight sum of every cell.  A first kernel has a lane add each short row and
// lists the longer ones; a second one has a wave add a middling row block by
// block, and a workgroup's eight waves a long one, each wave forming a block's
// part of 8192 values at a time from the sum before them (if that does not
// stand, the waves go on one after the other).  The next values are loaded
// before these are added.  Bound by the chain of the fullest cells, above all
// by their first few thousand values, where ties are frequent.  1e7 events in
// 187200 cells: one thread a cell with 16 loads ahead 5900 us; one kernel whose
// waves each took the middling rows of their own 64 cells in turn, rows of a
// block read again from memory, 240; listed and spread over all waves 167;
// the block's rows kept in LDS 148.  Long rows from 4096, 8192, 16384 or 32768
// values (the whole build): 673, 644, 654, 671 us.
constexpr uint32_t kShortRow = 32;
constexpr uint32_t kLongRow = 8192;
constexpr int kSumWaves = 8;
constexpr unsigned kSumBlocks = 512;

// The cells that the first kernel leaves: counts[0] middling ones, counts[1]
// long ones (both 0 beforehand).
struct RowLists {
    uint32_t *counts, *middling, *longs;
};

__global__ __launch_bounds__(256) void template_short_kernel(uint32_t n_cells,
                                                             const uint2* __restrict__ rows,
                                                             const double* __restrict__ ws,
                                                             double* __restrict__ T,
                                                             RowLists lists)
{
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const uint2 row = cell < n_cells ? rows[cell] : uint2{0u, 0u};
    const uint32_t len = row.y - row.x;
    const auto list = [&](bool mine, uint32_t* count, uint32_t* to) {
        const uint64_t mask = __ballot(mine);
        if (!mask) return;
        const int leader = __builtin_ctzll(mask);
        uint32_t at = 0;
        if (lane == leader) at = atomicAdd(count, uint32_t(__builtin_popcountll(mask)));
        at = __builtin_amdgcn_readlane(at, leader);
        if (mine) to[at + __builtin_popcountll(mask & ((uint64_t(1) << lane) - 1))] = cell;
    };
    list(len > kShortRow && len <= kLongRow, lists.counts, lists.middling);
    list(len > kLongRow, lists.counts + 1, lists.longs);
    if (cell >= n_cells || len > kShortRow) return;
    double s = 0.0;
    uint32_t i = row.x;
    for (; row.y - i >= 8u; i += 8u) {
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ws[i + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) s = s + v[j];
    }
    for (; i < row.y; ++i) s = s + ws[i];
    T[cell] = s;
}

__global__ __launch_bounds__(kSumWaves * 64) void template_sum_kernel(
    const uint2* __restrict__ rows, const double* __restrict__ ws, double* __restrict__ T,
    RowLists lists)
{
    __shared__ double part[kSumWaves], rows_lds[kSumWaves][kSumBlock];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const uint32_t n_long = lists.counts[1], n_middling = lists.counts[0];
    for (uint32_t k = blockIdx.x; k < n_long; k += gridDim.x) {
        const uint32_t cell = lists.longs[k];
        const uint2 row = rows[cell];
        const double* w = ws + row.x;
        const uint32_t n = row.y - row.x;
        double next[kSumRows], v[kSumRows], c = 0.0;
        load_block(w, wave * kSumBlock, n, lane, next);
        for (uint32_t first = 0; first < n; first += kSumWaves * kSumBlock) {
            const uint32_t mine = first + wave * kSumBlock;
#pragma unroll
            for (int j = 0; j < kSumRows; ++j) v[j] = next[j];
            if (first + kSumWaves * kSumBlock < n)
                load_block(w, mine + kSumWaves * kSumBlock, n, lane, next);
            RowSum block(c);
#pragma unroll
            for (int j = 0; j < kSumRows; ++j) block.add(v[j]);
            // a NaN part marks a block that does not stand
            const bool bad = __any(block.bad);
            const double sum = lanes_sum(block.acc);
            if (lane == 0) part[wave] = bad ? __builtin_nan("") : sum;
            __syncthreads();
            double total = 0.0;
#pragma unroll
            for (int j = 0; j < kSumWaves; ++j) total = total + part[j];
            total = c + total;
            __syncthreads();
            if (total < block.top()) {
                c = total;
            } else {
                for (int j = 0; j < kSumWaves; ++j) {
                    if (wave == j) {
                        c = add_block(c, v, rows_lds[wave], mine, n, lane);
                        if (lane == 0) part[0] = c;
                    }
                    __syncthreads();
                    c = part[0];
                    __syncthreads();
                }
            }
        }
        if (threadIdx.x == 0) T[cell] = c;
    }
    for (uint32_t k = blockIdx.x * kSumWaves + wave; k < n_middling; k += gridDim.x * kSumWaves) {
        const uint32_t cell = lists.middling[k];
        const uint2 row = rows[cell];
        const double* w = ws + row.x;
        const uint32_t n = row.y - row.x;
        double next[kSumRows], v[kSumRows], c = 0.0;
        load_block(w, 0, n, lane, next);
        for (uint32_t first = 0; first < n; first += kSumBlock) {
#pragma unroll
            for (int j = 0; j < kSumRows; ++j) v[j] = next[j];
            if (first + kSumBlock < n) load_block(w, first + kSumBlock, n, lane, next);
            c = add_block(c, v, rows_lds[wave], first, n, lane);
        }
        if (lane == 0) T[cell] = c;
    }
}

// P of the 18 channels at the centre of every true bin, layout P[c][t].
__global__ __launch_bounds__(64) void centre_probs_kernel(SetConsts sc, PathConsts pc, TrueBins tb,
                                                          double* __restrict__ P)
{
    __shared__ TileTables tabs;
    load_tab(sc, tabs, threadIdx.x);
    load_sincos(tabs, threadIdx.x);
    __syncthreads();
    const int64_t k = int64_t(blockIdx.x) * 64 + threadIdx.x;
    if (k >= int64_t(kTemplateChannels) * tb.nt) return;
    const uint32_t c = uint32_t(k / tb.nt), t = uint32_t(k - int64_t(c) * tb.nt);
    double E;
    {
#pragma clang fp contract(off)
        const double off = (double(t) + 0.5) * tb.wb;
        E = tb.lo + off;
    }
    const uint32_t f = (c % 3u) | (((c / 3u) % 3u) << 2) | ((c / 9u) << 4);
    P[k] = event_prob(sc, tabs, pc.kA, pc.kL, E, f);
}

// hist[r] for one reconstructed bin per block: lane l of the first wave adds
// the terms k = l, l + 64, ... in ascending k, then the wave's binary tree.
// All waves form the terms, kContractRows rows of 64 at a time in LDS, while
// the first one adds the rows of the round before: a round costs one load's
// latency and 64 dependent additions, not a load's latency for every 8 terms
// of a lane (the form with one wave a bin).  That took 4.8 us on 200 true x 52
// reconstructed bins and 53 us on 4000 x 22; this takes 3.8 and 26, of which
// the additions in order are 0.2 and 4.  Rounds of 8192 terms take 23 on
// the large one, but longer where a round is not full (500 true bins).
// Terms beyond K are +0.0, which leaves a sum that began at +0.0 as it is.
constexpr int kContractWaves = 8;
constexpr int kContractPer = 8;   // terms of one thread in a round
constexpr int kContractRows = kContractWaves * kContractPer;
constexpr int kContractGroup = 8;

__global__ __launch_bounds__(kContractWaves * 64) void bincentre_contract_kernel(
    const double* __restrict__ T, const double* __restrict__ P, int64_t K,
    double* __restrict__ hist)
{
    __shared__ double terms[2][kContractRows * 64];
    const int r = blockIdx.x, thread = threadIdx.x;
    const double* row = T + int64_t(r) * K;
    double t[kContractPer], p[kContractPer];
    const auto load = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < kContractPer; ++j) {
            const int64_t k = k0 + j * (kContractWaves * 64) + thread;
            t[j] = k < K ? row[k] : 0.0;
            p[j] = k < K ? P[k] : 0.0;
        }
    };
    const auto store = [&](double* to) {
#pragma unroll
        for (int j = 0; j < kContractPer; ++j)
            to[j * (kContractWaves * 64) + thread] = t[j] * p[j];
    };
    constexpr int64_t kRound = kContractRows * 64;
    double acc = 0.0;
    load(0);
    store(terms[0]);
    __syncthreads();
    for (int64_t k0 = 0, i = 0; k0 < K; k0 += kRound, ++i) {
        const bool more = k0 + kRound < K;
        if (more) load(k0 + kRound);
        if (thread < 64) {
            const int rows = int(min(int64_t(kContractRows), (K - k0 + 63) / 64));
            const double* from = terms[i & 1] + thread;
            for (int g = 0; g < rows; g += kContractGroup)
#pragma unroll
                for (int j = 0; j < kContractGroup; ++j) {
#pragma clang fp contract(off)
                    acc = acc + from[(g + j) * 64];
                }
        }
        if (more) store(terms[(i + 1) & 1]);
        __syncthreads();
    }
    if (thread >= 64) return;
    acc = wave_tree(acc);
    if (thread == 0) hist[r] = acc;
}

}  // namespace
}  // namespace osc

struct osc_template {
    osc_ctx* ctx = nullptr;
    int device = 0;
    osc::TrueBins tb{};
    int32_t nr = 0;
    osc::PathConsts pc{};
    double* d_T = nullptr;   // [nr + 2][18][nt]
    double* d_P = nullptr;   // [18][nt], used when the caller passes no table
};

namespace {

using osc::host::device_malloc;

bool true_binning_ok(const osc_binning* b)
{
    if (!b || b->nbins < 1 || b->nbins > 65536) return false;
    if (!(b->lo >= 0.0) || !(b->hi > b->lo) || !(b->hi < 1e300)) return false;
    if (b->e_scale != 0.0) return false;
    const double wb = (b->hi - b->lo) / double(b->nbins);
    return wb > 0.0 && wb < 1e300;
}

// The stable sort of (cell key, weight) by the lowest end_bit bits of the key;
// with tmp null only *bytes, the workspace, is set.  hipCUB takes 8 bits of the
// key in a pass and merge sort up to about 2^20 values; rocPRIM's radix sort
// underneath it also takes 9 bits, which saves a pass for keys of 9, 17 and 18
// (or 25 to 27) bits.  Template builds with hipCUB's choice | 9 bits (us): 18 bits,
// 1e7 events 623 | 534, 5e6 477 | 423, 2e6 292 | 273; 20 bits, 5e6 501 | 508, 2e6
// 352 | 378; any width, 1e6 336-393 | 225-306, 4e5 267-292 | 193-232, 2e5 184-219
// | 171-225, 4e4 141-187 | 148-214.
using NineBits = rocprim::radix_sort_config<
    rocprim::default_config, rocprim::default_config,
    rocprim::radix_sort_onesweep_config<rocprim::kernel_config<512, 8>,
                                        rocprim::kernel_config<512, 12>, 9,
                                        rocprim::block_radix_rank_algorithm::match>,
    0>;

hipError_t sort_cells(void* tmp, size_t* bytes, const uint32_t* keys, uint32_t* keys_out,
                      const double* weights, double* weights_out, int64_t n, int end_bit,
                      hipStream_t stream)
{
    const bool fewer_passes = (end_bit + 8) / 9 < (end_bit + 7) / 8;
    if (n > (1 << 18) && (n <= (1 << 20) || fewer_passes))
        return rocprim::radix_sort_pairs<NineBits>(tmp, *bytes, keys, keys_out, weights,
                                                   weights_out, size_t(n), 0u, unsigned(end_bit),
                                                   stream);
    return hipcub::DeviceRadixSort::SortPairs(tmp, *bytes, keys, keys_out, weights, weights_out,
                                              int(n), 0, end_bit, stream);
}

unsigned blocks_for(int64_t n, int threads) { return unsigned((n + threads - 1) / threads); }

}  // namespace

extern "C" {

osc_status osc_template_create(osc_ctx* ctx, const osc_sample* sample,
                               const osc_binning* true_binning,
                               const osc_binning* reco_binning, osc_template** out,
                               int64_t* n_used)
{
    if (!out) return OSC_ERR_INVALID_ARG;
    *out = nullptr;
    if (!ctx || !osc::host::sample_ok(sample, true) || !true_binning_ok(true_binning) ||
        !osc::host::binning_ok(ctx, reco_binning))
        return OSC_ERR_INVALID_ARG;
    if (sample->n > int64_t(INT32_MAX)) return OSC_ERR_INVALID_ARG;
    const int64_t nt = true_binning->nbins, nrt = int64_t(reco_binning->nbins) + 2;
    const int64_t cells = nrt * osc::kTemplateChannels * nt;
    if (cells >= int64_t(UINT32_MAX)) return OSC_ERR_INVALID_ARG;
    const uint32_t n_cells = uint32_t(cells);
    const int device = osc::host::ctx_device(ctx);
    if (hipSetDevice(device) != hipSuccess) return OSC_ERR_DEVICE;

    osc_template* tp = new (std::nothrow) osc_template();
    if (!tp) return OSC_ERR_OUT_OF_MEMORY;
    tp->ctx = ctx;
    tp->device = device;
    tp->tb = osc::TrueBins{true_binning->lo,
                           (true_binning->hi - true_binning->lo) / double(true_binning->nbins),
                           true_binning->nbins};
    tp->nr = reco_binning->nbins;
    tp->pc = osc::host::path_consts(sample);
    if (device_malloc(&tp->d_T, size_t(cells) * sizeof(double)) != hipSuccess ||
        device_malloc(&tp->d_P, size_t(osc::kTemplateChannels * nt) * sizeof(double)) != hipSuccess) {
        osc_template_destroy(tp);
        return OSC_ERR_OUT_OF_MEMORY;
    }

    const int64_t n = sample->n;
    int end_bit = 1;
    while (end_bit < 32 && (uint64_t(1) << end_bit) <= uint64_t(n_cells)) ++end_bit;
    // the sample may have been written by work still in flight on any stream
    osc_status st = hipDeviceSynchronize() == hipSuccess ? OSC_OK : OSC_ERR_DEVICE;
    uint32_t used = 0;
    if (st == OSC_OK) {
        size_t sort_bytes = 0;
        if (n > 0 && sort_cells(nullptr, &sort_bytes, nullptr, nullptr, nullptr, nullptr, n, end_bit,
                                nullptr) != hipSuccess)
            st = OSC_ERR_DEVICE;
        // one workspace: the cells' rows, the count of used events and those
        // of the listed rows, the
        // keys before and after the sort, the sorted weights, the sort's own
        const auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
        const size_t rows_b = up(size_t(n_cells) * sizeof(uint2) + 3 * sizeof(uint32_t));
        const size_t keys_b = up(size_t(n) * sizeof(uint32_t));
        const size_t ws_b = up(size_t(n) * sizeof(double));
        osc::host::BuildSpace space;
        if (st == OSC_OK) st = space.acquire(ctx, rows_b + 2 * keys_b + ws_b + up(sort_bytes));
        if (st == OSC_OK) {
            char* at = static_cast<char*>(space.ptr());
            const hipStream_t s = space.stream();
            uint2* rows = reinterpret_cast<uint2*>(at);
            uint32_t* d_used = reinterpret_cast<uint32_t*>(rows + n_cells);
            uint32_t* keys = reinterpret_cast<uint32_t*>(at + rows_b);
            uint32_t* skeys = reinterpret_cast<uint32_t*>(at + rows_b + keys_b);
            double* ws = reinterpret_cast<double*>(at + rows_b + 2 * keys_b);
            void* tmp = at + rows_b + 2 * keys_b + ws_b;
            hipError_t e = hipMemsetAsync(rows, 0, rows_b, s);
            if (e == hipSuccess && n > 0) {
                hipLaunchKernelGGL(osc::template_keys_kernel, dim3(blocks_for(n, 256)), dim3(256),
                                   0, s, n, sample->e_true, sample->flags, sample->e_reco, tp->tb,
                                   osc::host::bin_consts(reco_binning), n_cells, keys);
                e = hipGetLastError();
                if (e == hipSuccess)
                    e = sort_cells(tmp, &sort_bytes, keys, skeys, sample->weight, ws, n, end_bit, s);
                if (e == hipSuccess) {
                    hipLaunchKernelGGL(osc::template_bounds_kernel, dim3(blocks_for(n, 256)),
                                       dim3(256), 0, s, n, skeys, n_cells, rows, d_used);
                    e = hipGetLastError();
                }
            }
            if (e == hipSuccess) {
                // the unsorted keys' place holds the lists: every listed row
                // has more than kShortRow events, a long one more than kLongRow
                const osc::RowLists lists{d_used + 1, keys, keys + n / osc::kShortRow};
                hipLaunchKernelGGL(osc::template_short_kernel, dim3(blocks_for(n_cells, 256)),
                                   dim3(256), 0, s, n_cells, rows, ws, tp->d_T, lists);
                e = hipGetLastError();
                if (e == hipSuccess && n > int64_t(osc::kShortRow)) {
                    hipLaunchKernelGGL(osc::template_sum_kernel, dim3(osc::kSumBlocks),
                                       dim3(osc::kSumWaves * 64), 0, s, rows, ws, tp->d_T, lists);
                    e = hipGetLastError();
                }
            }
            if (e == hipSuccess)
                e = hipMemcpyAsync(&used, d_used, sizeof used, hipMemcpyDeviceToHost, s);
            // also after an error: the workspace is the next build's from here on
            const hipError_t done = hipStreamSynchronize(s);
            if (e == hipSuccess) e = done;
            if (e != hipSuccess) st = OSC_ERR_DEVICE;
        }
    }
    if (st == OSC_OK && n_used) *n_used = used;
    if (st != OSC_OK) {
        osc_template_destroy(tp);
        return st;
    }
    *out = tp;
    return OSC_OK;
}

osc_status osc_template_destroy(osc_template* t)
{
    if (!t) return OSC_OK;
    osc_status st = OSC_OK;
    if (hipSetDevice(t->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess)
        st = OSC_ERR_DEVICE;
    if (t->d_T) (void)hipFree(t->d_T);
    if (t->d_P) (void)hipFree(t->d_P);
    delete t;
    return st;
}

osc_status osc_template_copy(const osc_template* t, double* dst, void* stream)
{
    if (!t || !dst) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(t->device) != hipSuccess) return OSC_ERR_DEVICE;
    const size_t cells = size_t(t->nr + 2) * osc::kTemplateChannels * size_t(t->tb.nt);
    return hipMemcpyAsync(dst, t->d_T, cells * sizeof(double), hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(stream)) == hipSuccess
               ? OSC_OK
               : OSC_ERR_DEVICE;
}

osc_status osc_fill_pdf_bincentre(osc_ctx* ctx, const osc_template* t, int32_t set,
                                  double* hist_out, double* p_centre_out, void* stream)
{
    if (!ctx || !t || !hist_out || t->ctx != ctx) return OSC_ERR_INVALID_ARG;
    osc::SetConsts sc;
    if (!osc::host::ctx_set(ctx, set, &sc)) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(t->device) != hipSuccess) return OSC_ERR_DEVICE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* P = p_centre_out ? p_centre_out : t->d_P;
    const int64_t K = int64_t(osc::kTemplateChannels) * t->tb.nt;
    hipLaunchKernelGGL(osc::centre_probs_kernel, dim3(blocks_for(K, 64)), dim3(64), 0, s, sc,
                       t->pc, t->tb, P);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(osc::bincentre_contract_kernel, dim3(unsigned(t->nr + 2)),
                           dim3(osc::kContractWaves * 64), 0, s, t->d_T, P, K, hist_out);
        e = hipGetLastError();
    }
    return e == hipSuccess ? OSC_OK : OSC_ERR_DEVICE;
}

}  // extern "C"
