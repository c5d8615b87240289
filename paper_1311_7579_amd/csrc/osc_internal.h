// Internal layout shared by the host side and the kernels of libosc.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace osc {

// Reduction contract of the binned PDF: a tile is kTileLanes lanes x
// kLaneEvents events per lane (one wave64 per tile, or several that share it).
constexpr int kTileLanes = 64;
#ifndef OSC_LANE_EVENTS
#define OSC_LANE_EVENTS 16
#endif
constexpr int kLaneEvents = OSC_LANE_EVENTS;
constexpr int kTileEvents = kTileLanes * kLaneEvents;
// Histogram accumulators per bin of a tile: lane l adds into accumulator
// l mod kHistLanes, so kLaneShare lanes share one accumulator and add into
// it in ascending lane order.  Small accumulator rows keep the LDS per wave
// low (occupancy is bounded by registers, not by the histograms).  The
// value is part of the reduction contract (the bits of every histogram
// depend on it); the macro exists for build-time tuning sweeps.
#ifndef OSC_HIST_LANES
#define OSC_HIST_LANES 8
#endif
constexpr int kHistLanes = OSC_HIST_LANES;
constexpr int kLaneShare = kTileLanes / kHistLanes;
// Waves per SIMD the per-event kernels are compiled for (register caps
// that the compiler meets without spilling).
#ifndef OSC_TILE_WAVES
#define OSC_TILE_WAVES 6
#endif
constexpr int kTileWavesPerSimd = OSC_TILE_WAVES;
constexpr int kBatchWavesPerSimd = 4;
// 128 registers: with a few more the blocks of eight waves fit one to a CU
// instead of two (3e6 events through 12 layers 168 instead of 132 us).
constexpr int kLayeredWavesPerSimd = 4;

// Largest event count accepted.
constexpr int64_t kMaxEvents = int64_t(1) << 32;
// Histogram merge: one block per (chunk of rows, bin, parameter set) forms
// one aligned subtree of the tile tree: thread t adds kRows contiguous rows as
// a binary tree in registers, and the block's threads meet in a binary tree
// (the 64 lanes of a wave, then the waves).  The shape of a block changes no
// bits, so it follows the largest sample's row count (merge_shape).  A chunk
// is at most 1024 threads x 32 rows; one level serves samples up to 32768
// tiles (3.4e7 events), a second one the rest.  Rows are stored bin-major
// within chunks of kLayoutChunk rows (partial_index), so a thread's rows of
// one bin are contiguous.
constexpr int kLayoutChunk = 128;
constexpr int kMaxBatchSamples = 16;
// Largest number of parameter sets of one batch (the merge grid's z extent).
constexpr int kMaxBatchSets = 65535;

// One level of the merge for n_samples samples (x any number of parameter
// sets, one set per grid layer z): sample s has rows[s] input rows stored
// from row in_row0[s] (a multiple of kLayoutChunk) of the set's input
// region, takes blocks chunk0[s] .. and produces ceil(rows[s] / chunk rows)
// (at least one) output rows, stored from row out_row0[s]
// (a multiple of kLayoutChunk) of the set's output region.  The final level
// writes hist[set][sample][bin] instead.
struct MergeLevel {
    int32_t n_samples;
    int32_t nbt;
    int64_t total_chunks;                 // blocks per (bin, set)
    int64_t set_stride_in, set_stride_out;
    int64_t rows[kMaxBatchSamples];
    int64_t in_row0[kMaxBatchSamples];
    int64_t chunk0[kMaxBatchSamples];
    int64_t out_row0[kMaxBatchSamples];
};

// How a served request ends on the device: its finished histogram and, with a
// data row, -2 ln L are copied to host memory, and then `seq` is stored to
// *flag, on which the host waits.
struct ServeFinish {
    unsigned* ticket;      // device counter of finished blocks, 0 between requests
    double* hist;          // device, nbt entries
    double* host;          // pinned host memory: nbt entries, then -2 ln L
    unsigned* flag;        // pinned host memory
    unsigned seq;
    const double* data;    // nbt - 2 counts, or null
    double mu_scale;
};

// Position of the result of (tile, bin) among the tile results.
__host__ __device__ inline int64_t partial_index(int64_t tile, int bin, int nbt)
{
    return (tile / kLayoutChunk) * int64_t(nbt) * kLayoutChunk + int64_t(bin) * kLayoutChunk +
           (tile % kLayoutChunk);
}

// One flavour channel (beta <- alpha) of the vacuum mass matrix H0 =
// U diag(0, dm21, dm31) U^+ in the flavour basis, for neutrinos.
// With M = H0 + A e_e e_e^T:
//   M_ba      = m + A [a = b = e]
//   (M^2)_ba  = m2 + A g + A^2 [a = b = e],  g = [b = e] H0_ea + H0_be [a = e]
// Antineutrinos use the complex conjugates and the opposite sign of A.
// dee = [a = b = e] is stored as 0.0 / 1.0 so that the kernel applies it
// with FMAs.  The kernels expand these 9 entries into the flag-indexed LDS
// tables of TileTables (conjugated copies for antineutrinos, [a = b]).
struct Chan {
    double m_re, m_im;
    double m2_re, m2_im;
    double g_re, g_im;
    double dee;
};

constexpr int kChannels = 9;   // index 3 beta + alpha

// H0 in the real basis of the layered path.  With U = W O, W = R23
// diag(1, 1, e^{i delta}) and O real (up to column phases, which drop out),
// W^+ H0 W is real symmetric, and a rotation of its last two axes, on which
// A e_e e_e^T does not act, clears its (0, 2) entry:
//   M = [[a0 + A, b0, 0], [b0, a1, b1], [0, b1, a2]].
// w[f] is row f of the basis, <f| in it: (1, 0, 0) for nu_e, (0, w1, w2)
// (complex) for nu_mu and nu_tau.
struct Tridiagonal {
    double a0, a1, a2, b0, b1;
    double b00, b01, b11;   // b0 b0, b0 b1, b1 b1
    double w[3][5];   // [flavour]: w0, Re w1, Im w1, Re w2, Im w2
};

// Parameter-only quantities of one oscillation parameter set.
// Characteristic polynomial of M: x^3 - tr x^2 + c1 x - det with
//   tr = T0 + A,  c1 = C0 + A CA,  det = A DA;
// a quarter of its discriminant is the quartic (((D4 A + D3) A + D2) A +
// D1) A + D0.  The FP32-mixed tier's seeds take q/2, q = 2 tr^3 - 9 tr c1 +
// 27 det, as ((A + QH2) A + QH1) A + QH0; the FP64 tier's seed of the
// isolated root works in FP32 in a = A + A0:
//   p = tr^2 - 3 c1 = a^2 + pm,  q/2 = a^3 + k1 a + k0,  tr/3 = a/3 + t3
// (A0 is minus the A of the smallest p, pm that p; the a^2 term of q/2
// vanishes there).
struct SetConsts {
    double T0, C0, CA, DA;
    double QH0, QH1, QH2;
    double D0, D1, D2, D3, D4;
    double A0;
    float pm, k1, k0, t3;
    Chan ch[kChannels];
};

// sin and cos of k pi / 32, k = 0..63: the anchors of the FP64 phase
// sine/cosine, correctly rounded (sin of 0 .. pi/2 below, the rest by
// symmetry).  The table lives in device memory with the code: as a kernel
// argument its 1 KB was copied by the host and fetched from there by every
// launch.
struct SinCos {
    double s, c;
};
struct SinCosTable {
    SinCos e[64];
};
constexpr double kSinQuarter[17] = {
    0.0, 0.0980171403295606, 0.19509032201612828,
    0.2902846772544624, 0.3826834323650898, 0.47139673682599764,
    0.5555702330196022, 0.6343932841636455, 0.7071067811865476,
    0.773010453362737, 0.8314696123025452, 0.881921264348355,
    0.9238795325112867, 0.9569403357322088, 0.9807852804032304,
    0.9951847266721969, 1.0};
constexpr double anchor_sin(int k)
{
    const int q = k & 63, r = q & 31, m = r > 16 ? 32 - r : r;
    return q < 32 ? kSinQuarter[m] : -kSinQuarter[m];
}
constexpr SinCosTable make_anchors()
{
    SinCosTable t{};
    for (int k = 0; k < 64; ++k) t.e[k] = SinCos{anchor_sin(k), anchor_sin(k + 16)};
    return t;
}

// Path constants of one sample.
struct PathConsts {
    double kA;   // matter term per GeV: A = +-kA * E (eV^2)
    double kL;   // phase per eV^2 per 1/GeV in units of pi/32:
                 // phase = (pi/32) * kL * lambda / E
};

// A path of piecewise-constant density: layers in the order the neutrino
// crosses them, each with its own PathConsts.  A path that reads the same
// from both ends (as paths through the Earth do) is given as its first half:
// the first `pairs` layers are crossed again, in reverse, after the last.
constexpr int kMaxLayers = 32;
struct LayerPath {
    int32_t n, pairs;
    Tridiagonal tri;
    PathConsts layer[kMaxLayers];
};

// The fast bin index is exact for quotients below this magnitude, so no
// binning may have more regular bins (under/overflow included).
constexpr double kFastBinLimit = 4096.0;
constexpr int32_t kMaxBins = 4094;

struct BinConsts {
    double lo;
    double wb;      // (hi - lo) / nbins, computed on the host in FP64
    double inv_wb;  // 1 / wb rounded to FP64 (fast path of the bin index)
    double scale;   // 1 + e_scale rounded to FP64; the bin is taken for x * scale
    int32_t nb;     // regular bins; entries nb and nb + 1 are under/overflow
};

// Flag bytes f < 32 with alpha = f & 3 < 3 and beta = (f >> 2) & 3 < 3, as
// a bit mask over f.
constexpr uint32_t kValidFlags = 0x07770777u;

// Tables a per-event kernel keeps in LDS, built by each block from a
// SetConsts and the anchors:
//  * the channel entry of each flag byte below 28 (complex conjugates for
//    antineutrinos: the imaginary parts negated), with dba = [alpha = beta];
//    invalid flag bytes have a zero entry with dba = NaN, so P comes out
//    NaN, and bytes >= 28 use entry 27, which is invalid.  An entry is cut
//    into 16-byte parts, one array each; entry f sits at f + (f >> 4), so
//    that the same channel of neutrinos and antineutrinos lies in different
//    LDS banks (with entries 16 apart the benchmark step took 65.3 instead
//    of 61.8 us);
//  * sct: the phase sine/cosine anchors.
// The decode of a flag byte is then one min, the entry's offset and, for
// the sign of A, bit 4 moved to the sign bit.
constexpr int kFlagEntries = 28;
constexpr int kEntrySlots = kFlagEntries + 1;
struct alignas(16) Pair {
    double a, b;
};
struct TileTables {
    Pair m[kEntrySlots];    // M_ba of H0, real and imaginary part
    Pair m2[kEntrySlots];   // (H0^2)_ba
    Pair g[kEntrySlots];    // d(M^2)_ba / dA
    Pair d[kEntrySlots];    // [a = b = e], [a = b]
    SinCos sct[64];
};

// Tables of the layered kernel: the basis rows of the flavours (see
// Tridiagonal; row 3, for invalid flavours, is NaN) and the anchors.
struct LayeredTables {
    double w[4][5];
    SinCos sct[64];
};

// The FP32-mixed tier assembles the amplitude in FP32 from the same channel
// entries rounded to FP32 (M_ba and (M^2)_ba are then formed from them in
// FP32), and its phases use the hardware sine and cosine, so its tables
// hold FP32 channel entries and no sin/cos anchors:
//  * ch: entries 3 beta + alpha for neutrinos, 9 + 3 beta + alpha for
//    antineutrinos; entry 18 (invalid flag bytes) is zero with dba = NaN;
//  * flag: for each flag byte f < 32 the byte offset of its ch entry and
//    the sign bit of A (set for antineutrinos); bytes >= 32 use entry 31,
//    which is invalid.
// (The FP64 tier's indexing by flag byte ran the mixed kernel 2 % slower:
// its two 16-byte reads per event leave less to save.)
struct ChanF {
    float m_re, m_im;
    float m2_re, m2_im;
    float g_re, g_im;
    float dee, dba;
};
constexpr int kMixedChannels = 2 * kChannels + 1;
constexpr int kInvalidChannel = 2 * kChannels;
constexpr int kMixedFlags = 32;
struct FlagInfo {
    uint32_t ch_off;   // byte offset into the table's ch array
    uint32_t sign;     // 0 or 0x80000000: the sign bit of A
};
struct TileTablesMixed {
    ChanF ch[kMixedChannels];
    FlagInfo flag[kMixedFlags];
};
template <bool MIXED>
struct TablesOf {
    using type = TileTables;
};
template <>
struct TablesOf<true> {
    using type = TileTablesMixed;
};
template <bool MIXED>
using Tables = typename TablesOf<MIXED>::type;

}  // namespace osc
