// Host side of libosc: the C ABI of include/osc.h, argument validation,
// the parameter-only precompute (Sec. 2.1 of arXiv:1311.7579 computes these
// on the CPU and ships them to the GPU), device scratch, kernel launches.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/osc.h"
#include "osc_host_common.h"
#include "osc_internal.h"
#include "osc_launch.h"

namespace {

// hbar*c = 197.3269804 MeV fm; N_A = 6.02214076e23 / mol (CODATA 2018);
// G_F / (hbar c)^3 = 1.1663787e-5 GeV^-2.
constexpr double kHbarcEvM = 197.3269804e-9;
constexpr double kAvogadro = 6.02214076e23;
constexpr double kFermiGeV = 1.1663787e-5;

// The phase m^2 L / 2E in natural units per (eV^2 / GeV) over L_km
// kilometres, in units of pi/32 (the form the kernels take), rounded once
// from extended precision.
double phase_steps(double L_km)
{
    const long double pi = 3.141592653589793238462643383279502884L;
    const long double k = 1.0e3L / static_cast<long double>(kHbarcEvM) / 2.0e9L;
    return static_cast<double>(k * static_cast<long double>(L_km) * (32.0L / pi));
}

// 2 sqrt(2) G_F N_e E per (g/cm^3 * GeV * Ye), in eV^2
double matter_constant()
{
    const double hbarc_ev_cm = kHbarcEvM * 1.0e2;
    const double ne_ev3 = kAvogadro * hbarc_ev_cm * hbarc_ev_cm * hbarc_ev_cm;  // per g/cm^3
    return 2.0 * std::sqrt(2.0) * (kFermiGeV * 1.0e-18) * ne_ev3 * 1.0e9;
}

bool is_finite(double x) { return std::isfinite(x); }

bool params_ok(const osc_params& p)
{
    const double s[3] = {p.sin2_th12, p.sin2_th23, p.sin2_th13};
    for (double v : s)
        if (!is_finite(v) || v < 0.0 || v > 1.0) return false;
    if (!is_finite(p.dm2_21) || !(p.dm2_21 > 0.0)) return false;
    if (!is_finite(p.dm2_32) || p.dm2_32 == 0.0) return false;
    const double dm31 = p.dm2_32 + p.dm2_21;
    if (!is_finite(dm31) || dm31 == 0.0) return false;
    if (!is_finite(p.delta_cp)) return false;
    return true;
}

// The parameter-only quantities are formed in extended precision and rounded
// once: their errors are the same for every event of a set and for every layer
// of a path, so they add up where the events' own do not, and event_prob's Y
// cancels the matrix elements down to the half distance of two levels.  rms
// error of P at 295, 810 and 1300 km, E log-uniform on 0.1-10 GeV, in 1e-16:
// 3.2, 7.9 and 12.4 with these in double, 2.9, 7.6 and 12.2 with only the cubic's
// so, 2.7, 6.9 and 11.3 with all; 0.14 -> 0.17 us a set (0.32 with the smaller
// term of the matrix elements in extended precision too, for the same errors).
using Ext = long double;

// Square root: a Newton correction of the one in double (18 -> 5 ns).
Ext root(Ext y)
{
    const double s = std::sqrt(double(y));
    return s > 0.0 ? s + (y - Ext(s) * s) * (0.5 / s) : 0.0L;
}

struct Mixing {
    Ext S12, C12, S23, C23, S13, C13;   // squared sines and cosines
    Ext s23, c23, s13, c13;
    double cd, sd;                      // cos and sin of delta
    Ext dm21, dm31;
    explicit Mixing(const osc_params& p)
        : S12(p.sin2_th12), C12(1.0L - S12), S23(p.sin2_th23), C23(1.0L - S23), S13(p.sin2_th13),
          C13(1.0L - S13), s23(root(S23)), c23(root(C23)), s13(root(S13)), c13(root(C13)),
          cd(std::cos(p.delta_cp)),
          sd(std::sin(p.delta_cp)), dm21(p.dm2_21), dm31(Ext(p.dm2_32) + p.dm2_21)
    {
    }
};

// The eigenvalue solver's constants (see SetConsts) from T0, C0, CA and DA,
// in extended precision: their sums cancel.
void seed_consts(osc::SetConsts& sc)
{
    typedef long double R;
    const R T = sc.T0, C = sc.C0, a = sc.CA, d = sc.DA;
    // p = tr^2 - 3 c1 = A^2 + p1 A + p0 about its minimum at A = -A0
    const R p1 = 2.0L * T - 3.0L * a, p0 = T * T - 3.0L * C;
    sc.A0 = static_cast<double>(0.5L * p1);
    const R A0 = sc.A0;
    sc.pm = static_cast<float>(p0 + A0 * (A0 - p1));
    // q/2 = tr^3 - 4.5 tr c1 + 13.5 det = A^3 + q2 A^2 + q1 A + q0
    const R q2 = 3.0L * T - 4.5L * a;
    const R q1 = 3.0L * T * T - 4.5L * (C + T * a) + 13.5L * d;
    const R q0 = T * (T * T - 4.5L * C);
    sc.k1 = static_cast<float>(q1 + A0 * (3.0L * A0 - 2.0L * q2));
    sc.k0 = static_cast<float>(q0 + A0 * (-q1 + A0 * (q2 - A0)));
    sc.t3 = static_cast<float>((T - A0) / 3.0L);
    // the discriminant tr^2 c1^2 - 4 c1^3 - 4 tr^3 det + 18 tr c1 det -
    // 27 det^2 by powers of A, over 4
    sc.D0 = static_cast<double>(0.25L * C * C * (T * T - 4.0L * C));
    sc.D1 = static_cast<double>(0.25L * (2.0L * T * C * (C + T * a) - 12.0L * C * C * a -
                                         4.0L * T * T * T * d + 18.0L * T * C * d));
    sc.D2 = static_cast<double>(0.25L * (C * C + 4.0L * T * C * a + T * T * a * a -
                                         12.0L * C * a * a - 12.0L * T * T * d +
                                         18.0L * d * (C + T * a) - 27.0L * d * d));
    sc.D3 = static_cast<double>(0.25L * (2.0L * C * a + 2.0L * T * a * a - 4.0L * a * a * a -
                                         12.0L * T * d + 18.0L * a * d));
    sc.D4 = static_cast<double>(0.25L * (a * a - 4.0L * d));
}

// H0 in the layered path's real tridiagonal basis (see Tridiagonal).
void tridiagonal_consts(const osc_params& p, osc::Tridiagonal& t)
{
    const Mixing m(p);
    const Ext sc12 = root(m.S12 * m.C12);
    // K = O diag(0, dm21, dm31) O^T, O = R13 R12
    const Ext k00 = m.dm21 * m.S12 * m.C13 + m.dm31 * m.S13, k01 = m.dm21 * sc12 * m.c13,
              k02 = m.s13 * m.c13 * (m.dm31 - m.dm21 * m.S12), k11 = m.dm21 * m.C12,
              k12 = -m.dm21 * sc12 * m.s13,
              k22 = m.dm21 * m.S12 * m.S13 + m.dm31 * m.C13;
    // rotate axes 1 and 2 so that K(0, 2) vanishes
    const Ext h = std::hypot(k01, k02);
    const Ext c = h > 0.0L ? k01 / h : 1.0L, s = h > 0.0L ? k02 / h : 0.0L;
    t.a0 = double(k00);
    t.b0 = double(h);
    t.a1 = double(c * c * k11 + 2.0L * c * s * k12 + s * s * k22);
    t.a2 = double(s * s * k11 - 2.0L * c * s * k12 + c * c * k22);
    t.b1 = double((c * c - s * s) * k12 + c * s * (k22 - k11));
    t.b00 = t.b0 * t.b0;
    t.b01 = t.b0 * t.b1;
    t.b11 = t.b1 * t.b1;
    // rows of R23 diag(1, 1, e^{i delta}) times that rotation: x on axis 1, y
    // e^{i delta} on axis 2
    const Ext x[3] = {0.0L, m.c23, -m.s23}, y[3] = {0.0L, m.s23, m.c23};
    for (int f = 0; f < 3; ++f) {
        const Ext re = y[f] * m.cd, im = y[f] * m.sd;
        const double w[5] = {f == 0 ? 1.0 : 0.0, double(c * x[f] + s * re), double(s * im),
                             double(c * re - s * x[f]), double(c * im)};
        std::copy(w, w + 5, t.w[f]);
    }
}

}  // namespace

// Parameter-only quantities of one set for the kernels.
osc::SetConsts osc::host::set_consts(const osc_params& p)
{
    const Mixing m(p);
    osc::SetConsts sc{};
    sc.T0 = double(m.dm21 + m.dm31);   // trace of H
    sc.C0 = double(m.dm21 * m.dm31);   // sum of principal 2x2 minors of H
    // d c1 / dA = H_mm + H_tt and d det / dA = cofactor_ee(H)
    sc.CA = double(m.dm21 * (1.0L - m.S12 * m.C13) + m.dm31 * m.C13);
    sc.DA = double(m.dm21 * m.dm31 * m.C12 * m.C13);

    // Elements ee, me, mm, te, tm, tt of dm31 U_b2 U_a2^* (PDG form; without
    // e^{i delta}, which me and te carry) and of dm21 U_b1 U_a1^*, the smaller
    // term of the two, in double.
    const Ext ls = m.dm31 * m.s13 * m.c13, lc = m.dm31 * m.C13;
    const Ext l2[6] = {m.dm31 * m.S13, m.s23 * ls, m.S23 * lc, m.c23 * ls, m.s23 * m.c23 * lc,
                       m.C23 * lc};
    const double d = p.dm2_21, S12 = p.sin2_th12, S23 = p.sin2_th23, S13 = p.sin2_th13,
                 C12 = double(m.C12), C23 = double(m.C23), C13 = double(m.C13),
                 s23 = double(m.s23), c23 = double(m.c23), c13 = double(m.c13),
                 sc12 = std::sqrt(S12 * C12), sc23 = s23 * c23, w = sc12 * double(m.s13),
                 u = S12 * double(m.s13) * c13, t = 2.0 * sc23 * w * m.cd;
    const double re1[6] = {d * (S12 * C13),
                           d * (sc12 * c13 * c23 - u * s23 * m.cd),
                           d * (C12 * C23 + S12 * S23 * S13 - t),
                           -d * (sc12 * c13 * s23 + u * c23 * m.cd),
                           d * (sc23 * (S12 * S13 - C12) + w * m.cd * (S23 - C23)),
                           d * (C12 * S23 + S12 * C23 * S13 + t)};
    const double im1[6] = {0.0, -d * u * s23 * m.sd, 0.0, -d * u * c23 * m.sd, -d * w * m.sd, 0.0};
    for (int b = 0, k = 0; b < 3; ++b)
        for (int a = 0; a <= b; ++a, ++k) {
            const bool phase = a == 0 && b > 0;
            const Ext r2 = phase ? l2[k] * m.cd : l2[k], i2 = phase ? l2[k] * m.sd : 0.0L;
            osc::Chan c{};
            c.m_re = double(r2 + re1[k]);
            c.m_im = double(i2 + im1[k]);
            c.m2_re = double(m.dm31 * r2 + d * re1[k]);
            c.m2_im = double(m.dm31 * i2 + d * im1[k]);
            if (a == 0) c.g_re = (b == 0 ? 2.0 : 1.0) * c.m_re, c.g_im = c.m_im;
            c.dee = b == 0 ? 1.0 : 0.0;
            sc.ch[3 * b + a] = c;
            c.m_im = -c.m_im, c.m2_im = -c.m2_im, c.g_im = -c.g_im;
            if (a < b) sc.ch[3 * a + b] = c;
        }
    // q/2 = tr^3 - 4.5 tr c1 + 13.5 det as a cubic in A
    sc.QH2 = 3.0 * sc.T0 - 4.5 * sc.CA;
    sc.QH1 = 3.0 * sc.T0 * sc.T0 - 4.5 * (sc.C0 + sc.T0 * sc.CA) + 13.5 * sc.DA;
    sc.QH0 = sc.T0 * (sc.T0 * sc.T0 - 4.5 * sc.C0);
    seed_consts(sc);
    return sc;
}

namespace {

struct Scratch {
    void* ptr = nullptr;
    size_t cap = 0;
    hipEvent_t done = nullptr;      // recorded after the slot's last use
    bool recorded = false;
    hipStream_t last = nullptr;     // stream of the slot's last use
};

constexpr int kScratchSlots = 4;

// hipEvents around the kernels of one call (profiling only)
struct ProfRec {
    hipEvent_t start = nullptr, mid = nullptr, end = nullptr;
};

}  // namespace

struct osc_ctx {
    int device = 0;
    size_t max_dyn_lds = 0;
    int32_t max_nbins = 0;
    std::vector<osc_params> params;
    std::vector<osc::SetConsts> consts;
    Scratch slots[kScratchSlots];
    int next_slot = 0;
    // While every call has used one stream (`sole`), the stream order alone
    // protects the scratch slots and no event is recorded per call.
    bool one_stream = true;
    bool used = false;
    hipStream_t sole = nullptr;
    double* noalloc = nullptr;      // this device's address of the static scratch array
    bool profiling = false;
    std::vector<ProfRec> prof;
    std::mutex mu;
    // one-time builds (osc::host::BuildSpace)
    std::mutex build_mu;
    void* build_ptr = nullptr;
    size_t build_cap = 0;
    hipStream_t build_stream = nullptr;
    osc_ctx* next = nullptr;        // list of the live contexts
};

namespace {

using osc::host::device_malloc;

osc_status device_status(hipError_t e) { return e == hipSuccess ? OSC_OK : OSC_ERR_DEVICE; }

void drop_profile(osc_ctx* ctx)
{
    for (ProfRec& r : ctx->prof) {
        for (hipEvent_t e : {r.start, r.mid, r.end})
            if (e) (void)hipEventDestroy(e);
    }
    ctx->prof.clear();
}

// Starts a profiling record when profiling is on.  `start` and `mid` are
// handed to the launch of the per-event kernel, which records its own
// begin and end time in them (the dispatch's timestamps, so the interval
// is the kernel's execution alone); `end` is recorded on the stream after
// the merge.
ProfRec* prof_begin(osc_ctx* ctx, hipStream_t)
{
    if (!ctx->profiling) return nullptr;
    ProfRec r;
    if (hipEventCreate(&r.start) != hipSuccess || hipEventCreate(&r.mid) != hipSuccess ||
        hipEventCreate(&r.end) != hipSuccess) {
        for (hipEvent_t e : {r.start, r.mid, r.end})
            if (e) (void)hipEventDestroy(e);
        return nullptr;
    }
    ctx->prof.push_back(r);
    return &ctx->prof.back();
}

// A call without a merge: the record ends with the per-event kernel.
void prof_no_merge(ProfRec* r)
{
    if (!r) return;
    (void)hipEventDestroy(r->end);
    r->end = nullptr;
}

void prof_mark(hipEvent_t ev, hipStream_t stream)
{
    if (ev) (void)hipEventRecord(ev, stream);
}

// Scratch for one call on `stream`: slots are used round-robin.  While the
// context has seen a single stream, that stream's order already puts every
// use of a slot after the previous one.  The first call on a second stream
// waits once for the device to go idle (the first stream may have been
// destroyed since, so no event can be recorded on it now); from then on
// every call records the slot's event after its use, and a slot last used
// on another stream orders the new stream after that use.
osc_status acquire_scratch(osc_ctx* ctx, size_t bytes, hipStream_t stream, Scratch** out)
{
    if (ctx->one_stream) {
        if (!ctx->used) {
            ctx->used = true;
            ctx->sole = stream;
        } else if (stream != ctx->sole) {
            if (hipDeviceSynchronize() != hipSuccess) return OSC_ERR_DEVICE;
            ctx->one_stream = false;
        }
    }
    Scratch& s = ctx->slots[ctx->next_slot];
    ctx->next_slot = (ctx->next_slot + 1) % kScratchSlots;
    if (s.done == nullptr && hipEventCreateWithFlags(&s.done, hipEventDisableTiming) != hipSuccess)
        return OSC_ERR_DEVICE;
    if (s.cap < bytes) {
        if (s.ptr) {
            // the slot's last use is on `stream` (one stream) or behind its event
            const hipError_t e = ctx->one_stream ? hipStreamSynchronize(stream)
                                 : s.recorded    ? hipEventSynchronize(s.done)
                                                 : hipSuccess;
            if (e != hipSuccess) return OSC_ERR_DEVICE;
            if (hipFree(s.ptr) != hipSuccess) return OSC_ERR_DEVICE;
            s.ptr = nullptr;
            s.cap = 0;
        }
        const size_t want = (bytes + (size_t(1) << 20) - 1) & ~((size_t(1) << 20) - 1);
        if (device_malloc(&s.ptr, want) != hipSuccess) return OSC_ERR_OUT_OF_MEMORY;
        s.cap = want;
        s.recorded = false;
    } else if (s.recorded && s.last != stream) {
        if (hipStreamWaitEvent(stream, s.done, 0) != hipSuccess) return OSC_ERR_DEVICE;
    }
    *out = &s;
    return OSC_OK;
}

osc_status release_scratch(osc_ctx* ctx, Scratch* s, hipStream_t stream)
{
    if (ctx->one_stream) return OSC_OK;
    if (hipEventRecord(s->done, stream) != hipSuccess) return OSC_ERR_DEVICE;
    s->recorded = true;
    s->last = stream;
    return OSC_OK;
}

}  // namespace

namespace {

constexpr size_t kBuildKeepBytes = size_t(512) << 20;

// The live contexts, for device_malloc.  Taken before a context's build_mu is
// tried, never the other way round with a wait.
std::mutex g_contexts_mu;
osc_ctx* g_contexts = nullptr;

void free_build_space(osc_ctx* ctx)
{
    if (ctx->build_ptr) (void)hipFree(ctx->build_ptr);
    ctx->build_ptr = nullptr;
    ctx->build_cap = 0;
}

}  // namespace

hipError_t osc::host::device_malloc(void** p, size_t bytes, const osc_ctx* building)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();   // or the next launch's check would find it
    int device = -1;
    if (hipGetDevice(&device) == hipSuccess) {
        bool freed = false;
        std::lock_guard<std::mutex> lock(g_contexts_mu);
        for (osc_ctx* c = g_contexts; c; c = c->next) {
            if (c == building || c->device != device || !c->build_mu.try_lock()) continue;
            freed = freed || c->build_ptr;
            free_build_space(c);
            c->build_mu.unlock();
        }
        if (freed) e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

osc_status osc::host::BuildSpace::acquire(osc_ctx* ctx, size_t bytes)
{
    ctx->build_mu.lock();
    ctx_ = ctx;
    if (!ctx->build_stream &&
        hipStreamCreateWithFlags(&ctx->build_stream, hipStreamNonBlocking) != hipSuccess)
        return OSC_ERR_DEVICE;
    if (ctx->build_cap >= bytes) return OSC_OK;
    free_build_space(ctx);
    if (device_malloc(&ctx->build_ptr, bytes, ctx) != hipSuccess) return OSC_ERR_OUT_OF_MEMORY;
    ctx->build_cap = bytes;
    return OSC_OK;
}

osc::host::BuildSpace::~BuildSpace()
{
    if (!ctx_) return;
    if (ctx_->build_cap > kBuildKeepBytes) free_build_space(ctx_);
    ctx_->build_mu.unlock();
}

void* osc::host::BuildSpace::ptr() const { return ctx_->build_ptr; }
hipStream_t osc::host::BuildSpace::stream() const { return ctx_->build_stream; }

bool osc::host::sample_ok(const osc_sample* s, bool needs_hist_inputs)
{
    if (!s || s->n < 0 || s->n > osc::kMaxEvents) return false;
    if (!is_finite(s->L_km) || s->L_km < 0.0) return false;
    if (!is_finite(s->rho_gcc) || s->rho_gcc < 0.0) return false;
    if (!is_finite(s->Ye) || s->Ye < 0.0 || s->Ye > 1.0) return false;
    if (s->n > 0) {
        if (!s->e_true || !s->flags) return false;
        if (needs_hist_inputs && (!s->weight || !s->e_reco)) return false;
    }
    return true;
}

bool osc::host::binning_ok(const osc_ctx* ctx, const osc_binning* b)
{
    if (!b || b->nbins < 1 || b->nbins > ctx->max_nbins) return false;
    if (!is_finite(b->lo) || !is_finite(b->hi) || !(b->lo < b->hi)) return false;
    const double wb = (b->hi - b->lo) / double(b->nbins);
    if (!is_finite(b->e_scale) || !(b->e_scale > -1.0)) return false;
    return is_finite(wb) && wb > 0.0;
}

osc::PathConsts osc::host::path_consts(const osc_sample* s)
{
    return osc::PathConsts{matter_constant() * s->Ye * s->rho_gcc, phase_steps(s->L_km)};
}

osc::BinConsts osc::host::bin_consts(const osc_binning* b)
{
    const double wb = (b->hi - b->lo) / double(b->nbins);
    return osc::BinConsts{b->lo, wb, 1.0 / wb, 1.0 + b->e_scale, b->nbins};
}

int osc::host::ctx_device(const osc_ctx* ctx) { return ctx->device; }

bool osc::host::ctx_set(osc_ctx* ctx, int32_t set, osc::SetConsts* out)
{
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return false;
    *out = ctx->consts[size_t(set)];
    return true;
}

size_t osc::host::fill_scratch_bytes(int64_t n, int nbins)
{
    const int64_t tiles = (n + osc::kTileEvents - 1) / osc::kTileEvents;
    return osc::merge_scratch_bytes(osc::plan_merge(&tiles, 1, nbins + 2), 1);
}

hipError_t osc::host::enqueue_served(const osc::SetConsts& sc, const osc_sample* sample,
                                     const uint16_t* bins, const osc_binning* binning, bool mixed,
                                     double* scratch, const osc::ServeFinish& finish,
                                     hipStream_t stream)
{
    const osc::BinConsts bc = bin_consts(binning);
    const int64_t tiles = (sample->n + osc::kTileEvents - 1) / osc::kTileEvents;
    hipError_t e = osc::launch_tiles(3, false, mixed, sc, path_consts(sample), bc, sample->n,
                                     sample->e_true, sample->flags, sample->weight, nullptr, bins,
                                     nullptr, nullptr, tiles == 1 ? finish.hist : scratch, stream);
    if (e != hipSuccess) return e;
    if (tiles == 1) return osc::launch_serve_finish(finish, bc.nb + 2, stream);
    return osc::launch_merge_serve(osc::plan_merge(&tiles, 1, bc.nb + 2), scratch, finish, stream);
}

hipError_t osc::host::enqueue_bin_slots(const osc_sample* sample, const osc_binning* binning,
                                        uint16_t* bins, hipStream_t stream)
{
    return osc::launch_bin_slots(sample->n, sample->e_reco, bin_consts(binning), bins, stream);
}

namespace {

using osc::host::bin_consts;
using osc::host::binning_ok;
using osc::host::path_consts;
using osc::host::sample_ok;
using osc::host::set_consts;

// The per-event kernel and the merge of one histogram on `stream`, with
// the tile results and level buffers in `partials` (merge_scratch_bytes of
// `plan`; a sample of one tile needs neither: its result is the histogram).
// t0 / t1 (nullable) receive the per-event kernel's own begin and
// end times.
hipError_t enqueue_hist(int mode, bool write_p, bool mixed, const osc::SetConsts& sc,
                        const osc::PathConsts& pc, const osc::BinConsts& bc, int64_t n,
                        const double* e_true, const uint8_t* flags, const double* weight,
                        const double* e_reco, const uint16_t* bins, const double* value,
                        double* p_out, double* hist_out, const osc::MergePlan* plan,
                        double* partials, hipStream_t stream, const osc::LayerPath* lp,
                        hipEvent_t t0, hipEvent_t t1)
{
    if (!plan) partials = hist_out;
    hipError_t e = lp ? osc::launch_layered_tiles(mode, write_p, sc, *lp, bc, n, e_true, flags,
                                                  weight, e_reco, p_out, partials, stream, t0,
                                                  t1)
                      : osc::launch_tiles(mode, write_p, mixed, sc, pc, bc, n, e_true, flags,
                                          weight, e_reco, bins, value, p_out, partials, stream,
                                          t0, t1);
    if (e == hipSuccess && plan) e = osc::launch_merge(*plan, 1, partials, hist_out, stream);
    return e;
}

// Tile partials + merge for one histogram on `stream`, in a scratch slot of
// the context.
osc_status run_hist(osc_ctx* ctx, int mode, bool write_p, bool mixed, const osc::SetConsts& sc,
                    const osc::PathConsts& pc, const osc::BinConsts& bc, int64_t n,
                    const double* e_true, const uint8_t* flags, const double* weight,
                    const double* e_reco, const uint16_t* bins, const double* value,
                    double* p_out, double* hist_out, hipStream_t stream,
                    const osc::LayerPath* lp = nullptr)
{
    const int64_t tiles = (n + osc::kTileEvents - 1) / osc::kTileEvents;
    if (tiles == 1) {   // one launch, no scratch, nothing to merge
        ProfRec* pr = prof_begin(ctx, stream);
        const hipError_t e = enqueue_hist(mode, write_p, mixed, sc, pc, bc, n, e_true, flags,
                                          weight, e_reco, bins, value, p_out, hist_out, nullptr,
                                          nullptr, stream, lp, pr ? pr->start : nullptr,
                                          pr ? pr->mid : nullptr);
        prof_no_merge(pr);
        return device_status(e);
    }
    const osc::MergePlan plan = osc::plan_merge(&tiles, 1, bc.nb + 2);
    Scratch* s = nullptr;
    osc_status st = acquire_scratch(ctx, osc::merge_scratch_bytes(plan, 1), stream, &s);
    if (st != OSC_OK) return st;
    ProfRec* pr = prof_begin(ctx, stream);
    const hipError_t e = enqueue_hist(mode, write_p, mixed, sc, pc, bc, n, e_true, flags, weight,
                                      e_reco, bins, value, p_out, hist_out, &plan,
                                      static_cast<double*>(s->ptr), stream, lp,
                                      pr ? pr->start : nullptr, pr ? pr->mid : nullptr);
    if (pr) prof_mark(pr->end, stream);
    st = release_scratch(ctx, s, stream);
    if (e != hipSuccess) return OSC_ERR_DEVICE;
    return st;
}

// ---- The entry point that allocates nothing --------------------------------
// osc_fill_pdf_noalloc keeps its tile results and merge level buffers in
// this file-scope array instead of a scratch slot of the context.  Each GPU
// the library runs on holds its own copy for the life of the process.  In
// host code the name stands for a host-side shadow, not a device address:
// kernels are only ever given the address that hipGetSymbolAddress returns
// for the current device (noalloc_address).
static __device__ __align__(256) double scratch[OSC_NOALLOC_SCRATCH_BYTES / sizeof(double)];

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
double* g_noalloc_ptr[kMaxDevices] = {};

// The device address of `scratch` on `device`, which must be current;
// resolved once per device.  nullptr when the runtime cannot resolve it.
double* noalloc_address(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[device]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_noalloc_ptr[device] = static_cast<double*>(ptr);
    }
    return g_noalloc_ptr[device];
}

}  // namespace

extern "C" {

osc_status osc_create(osc_ctx** out, int device)
{
    if (!out) return OSC_ERR_INVALID_ARG;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) return OSC_ERR_DEVICE;
    if (device < 0 || device >= count) return OSC_ERR_DEVICE;
    if (hipSetDevice(device) != hipSuccess) return OSC_ERR_DEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return OSC_ERR_DEVICE;
    osc_ctx* ctx = new (std::nothrow) osc_ctx();
    if (!ctx) return OSC_ERR_OUT_OF_MEMORY;
    ctx->device = device;
    ctx->noalloc = noalloc_address(device);
    // per-wave histograms: (nbins + 2) x kHistLanes accumulators x 8 B of
    // dynamic LDS, next to the static tables (channels, sin/cos); what they
    // leave of the reserve stays unused, so that the bin counts accepted do not
    // follow the tables' layout
    constexpr size_t static_lds = 3008;
    static_assert(sizeof(osc::TileTables) <= static_lds &&
                  sizeof(osc::TileTablesMixed) <= static_lds &&
                  sizeof(osc::LayeredTables) <= static_lds, "the tables fit the reserve");
    size_t lds = prop.sharedMemPerBlock > static_lds ? prop.sharedMemPerBlock - static_lds : 0;
    if (osc::set_kernel_attributes(lds) != hipSuccess) {
        // keep to the default 64 KiB per workgroup when the larger limit is refused
        (void)hipGetLastError();
        lds = std::min<size_t>(lds, 65536 - static_lds);
    }
    const size_t row = size_t(osc::kHistLanes) * sizeof(double);
    ctx->max_nbins = std::min<int32_t>(int32_t(lds / row) - 2, osc::kMaxBins);
    ctx->max_dyn_lds = lds;
    if (ctx->max_nbins < 1) {
        delete ctx;
        return OSC_ERR_DEVICE;
    }
    {
        std::lock_guard<std::mutex> lock(g_contexts_mu);
        ctx->next = g_contexts;
        g_contexts = ctx;
    }
    *out = ctx;
    return OSC_OK;
}

osc_status osc_destroy(osc_ctx* ctx)
{
    if (!ctx) return OSC_OK;
    osc_status st = OSC_OK;
    {
        std::lock_guard<std::mutex> lock(g_contexts_mu);
        osc_ctx** at = &g_contexts;
        while (*at && *at != ctx) at = &(*at)->next;
        if (*at) *at = ctx->next;
    }
    (void)hipSetDevice(ctx->device);
    drop_profile(ctx);
    // one stream: it may have been destroyed since its last call, so wait
    // for the device
    if (ctx->one_stream && ctx->used && hipDeviceSynchronize() != hipSuccess) st = OSC_ERR_DEVICE;
    for (Scratch& s : ctx->slots) {
        if (s.recorded && hipEventSynchronize(s.done) != hipSuccess) st = OSC_ERR_DEVICE;
        if (s.ptr && hipFree(s.ptr) != hipSuccess) st = OSC_ERR_DEVICE;
        if (s.done && hipEventDestroy(s.done) != hipSuccess) st = OSC_ERR_DEVICE;
    }
    if (ctx->build_ptr && hipFree(ctx->build_ptr) != hipSuccess) st = OSC_ERR_DEVICE;
    if (ctx->build_stream && hipStreamDestroy(ctx->build_stream) != hipSuccess) st = OSC_ERR_DEVICE;
    delete ctx;
    return st;
}

osc_status osc_validate_params(const osc_params* sets, int32_t n_sets)
{
    if (!sets || n_sets < 1) return OSC_ERR_INVALID_ARG;
    for (int32_t k = 0; k < n_sets; ++k)
        if (!params_ok(sets[k])) return OSC_ERR_INVALID_ARG;
    return OSC_OK;
}

osc_status osc_set_params(osc_ctx* ctx, const osc_params* sets, int32_t n_sets)
{
    if (!ctx) return OSC_ERR_INVALID_ARG;
    osc_status st = osc_validate_params(sets, n_sets);
    if (st != OSC_OK) return st;
    std::lock_guard<std::mutex> lock(ctx->mu);
    try {
        ctx->params.assign(sets, sets + n_sets);
        ctx->consts.resize(size_t(n_sets));
    } catch (...) {
        return OSC_ERR_OUT_OF_MEMORY;
    }
    for (int32_t k = 0; k < n_sets; ++k) ctx->consts[size_t(k)] = set_consts(sets[k]);
    return OSC_OK;
}

osc_status osc_reweight(osc_ctx* ctx, const osc_sample* sample, int32_t set, double* p_out,
                        void* stream)
{
    if (!ctx || !sample_ok(sample, false)) return OSC_ERR_INVALID_ARG;
    if (sample->n > 0 && !p_out) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const osc::BinConsts bc{0.0, 1.0, 1.0, 1.0, 1};
    const hipStream_t hs = static_cast<hipStream_t>(stream);
    ProfRec* pr = prof_begin(ctx, hs);
    const hipError_t e = osc::launch_tiles(0, true, false, ctx->consts[size_t(set)],
                                           path_consts(sample), bc,
                                           sample->n, sample->e_true, sample->flags, nullptr,
                                           nullptr, nullptr, nullptr, p_out, nullptr, hs,
                                           pr ? pr->start : nullptr, pr ? pr->mid : nullptr);
    prof_no_merge(pr);
    return device_status(e);
}

osc_status osc_fill_pdf(osc_ctx* ctx, const osc_sample* sample, int32_t set,
                        const osc_binning* binning, osc_precision precision, double* hist_out,
                        double* p_out, void* stream)
{
    if (!ctx || !sample_ok(sample, true) || !hist_out) return OSC_ERR_INVALID_ARG;
    if (!binning_ok(ctx, binning)) return OSC_ERR_INVALID_ARG;
    if (precision != OSC_FP64 && precision != OSC_FP32_MIXED) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    return run_hist(ctx, 1, p_out != nullptr, precision == OSC_FP32_MIXED, ctx->consts[size_t(set)],
                    path_consts(sample),
                    bin_consts(binning), sample->n, sample->e_true, sample->flags, sample->weight,
                    sample->e_reco, nullptr, nullptr, p_out, hist_out,
                    static_cast<hipStream_t>(stream));
}

osc_status osc_fill_pdf_noalloc(osc_ctx* ctx, const osc_sample* sample, int32_t set,
                                const osc_binning* binning, osc_precision precision,
                                double* hist_out, double* p_out, void* stream)
{
    if (!ctx || !sample_ok(sample, true) || !hist_out) return OSC_ERR_INVALID_ARG;
    if (!binning_ok(ctx, binning)) return OSC_ERR_INVALID_ARG;
    if (precision != OSC_FP64 && precision != OSC_FP32_MIXED) return OSC_ERR_INVALID_ARG;
    const osc::BinConsts bc = bin_consts(binning);
    const int64_t tiles = (sample->n + osc::kTileEvents - 1) / osc::kTileEvents;
    const osc::MergePlan plan = osc::plan_merge(&tiles, 1, bc.nb + 2);
    if (osc::merge_scratch_bytes(plan, 1) > OSC_NOALLOC_SCRATCH_BYTES) return OSC_ERR_BUDGET;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (!ctx->noalloc) return OSC_ERR_DEVICE;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const hipError_t e = enqueue_hist(
        1, p_out != nullptr, precision == OSC_FP32_MIXED, ctx->consts[size_t(set)],
        path_consts(sample), bc, sample->n, sample->e_true, sample->flags, sample->weight,
        sample->e_reco, nullptr, nullptr, p_out, hist_out, tiles == 1 ? nullptr : &plan,
        ctx->noalloc,
        static_cast<hipStream_t>(stream), nullptr, nullptr, nullptr);
    return device_status(e);
}

struct osc_binned {
    osc_ctx* ctx = nullptr;
    osc_sample sample{};        // e_reco is not read after creation
    osc_binning binning{};
    uint16_t* slots = nullptr;  // n cached histogram slots (device)
};

osc_status osc_binned_create(osc_ctx* ctx, const osc_sample* sample, const osc_binning* binning,
                             osc_binned** out)
{
    if (!out) return OSC_ERR_INVALID_ARG;
    *out = nullptr;
    if (!ctx || !sample_ok(sample, true) || !binning_ok(ctx, binning)) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    osc_binned* b = new (std::nothrow) osc_binned();
    if (!b) return OSC_ERR_OUT_OF_MEMORY;
    b->ctx = ctx;
    b->sample = *sample;
    b->binning = *binning;
    if (sample->n > 0 &&
        device_malloc(&b->slots, size_t(sample->n) * sizeof(uint16_t)) != hipSuccess) {
        delete b;
        return OSC_ERR_OUT_OF_MEMORY;
    }
    // synchronous: after earlier work on the device (the caller's uploads),
    // and the slots are ready on return
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess)
        e = osc::host::enqueue_bin_slots(sample, binning, b->slots, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        if (b->slots) (void)hipFree(b->slots);
        delete b;
        return OSC_ERR_DEVICE;
    }
    *out = b;
    return OSC_OK;
}

osc_status osc_binned_destroy(osc_binned* b)
{
    if (!b) return OSC_OK;
    osc_status st = OSC_OK;
    if (b->slots) {
        if (hipSetDevice(b->ctx->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
            hipFree(b->slots) != hipSuccess)
            st = OSC_ERR_DEVICE;
    }
    delete b;
    return st;
}

osc_status osc_fill_pdf_binned(osc_ctx* ctx, const osc_binned* b, int32_t set,
                               osc_precision precision, double* hist_out, double* p_out,
                               void* stream)
{
    if (!ctx || !b || b->ctx != ctx || !hist_out) return OSC_ERR_INVALID_ARG;
    if (precision != OSC_FP64 && precision != OSC_FP32_MIXED) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const osc_sample& s = b->sample;
    return run_hist(ctx, 3, p_out != nullptr, precision == OSC_FP32_MIXED,
                    ctx->consts[size_t(set)], path_consts(&s), bin_consts(&b->binning), s.n,
                    s.e_true, s.flags, s.weight, nullptr, b->slots, nullptr, p_out, hist_out,
                    static_cast<hipStream_t>(stream));
}

namespace {

// Layers of a piecewise-constant path: 1..kMaxLayers layers, each with
// L >= 0, rho >= 0 (finite) and 0 <= Ye <= 1.
bool layers_ok(const osc_layer* layers, int32_t n_layers)
{
    if (!layers || n_layers < 1 || n_layers > osc::kMaxLayers) return false;
    for (int32_t j = 0; j < n_layers; ++j) {
        const osc_layer& l = layers[j];
        if (!is_finite(l.L_km) || l.L_km < 0.0 || !is_finite(l.rho_gcc) || l.rho_gcc < 0.0 ||
            !is_finite(l.Ye) || l.Ye < 0.0 || l.Ye > 1.0)
            return false;
    }
    return true;
}

osc::LayerPath layer_path(const osc_params& p, const osc_layer* layers, int32_t n_layers)
{
    osc::LayerPath lp{};
    lp.n = n_layers;
    tridiagonal_consts(p, lp.tri);
    for (int32_t j = 0; j < n_layers; ++j)
        lp.layer[j] = osc::PathConsts{matter_constant() * layers[j].Ye * layers[j].rho_gcc,
                                      phase_steps(layers[j].L_km)};
    // a path that reads the same from both ends: its first half, crossed twice
    bool mirrored = true;
    for (int32_t j = 0; j < n_layers / 2; ++j) {
        const osc::PathConsts &a = lp.layer[j], &b = lp.layer[n_layers - 1 - j];
        mirrored = mirrored && a.kA == b.kA && a.kL == b.kL;
    }
    if (mirrored) {
        lp.pairs = n_layers / 2;
        lp.n = n_layers - lp.pairs;
    }
    return lp;
}

}  // namespace

osc_status osc_reweight_layered(osc_ctx* ctx, const osc_sample* sample, const osc_layer* layers,
                                int32_t n_layers, int32_t set, double* p_out, void* stream)
{
    if (!ctx || !sample_ok(sample, false) || !layers_ok(layers, n_layers))
        return OSC_ERR_INVALID_ARG;
    if (sample->n > 0 && !p_out) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const osc::BinConsts bc{0.0, 1.0, 1.0, 1.0, 1};
    const hipStream_t hs = static_cast<hipStream_t>(stream);
    ProfRec* pr = prof_begin(ctx, hs);
    const hipError_t e = osc::launch_layered_tiles(
        0, true, ctx->consts[size_t(set)], layer_path(ctx->params[size_t(set)], layers, n_layers), bc, sample->n,
        sample->e_true, sample->flags, nullptr, nullptr, p_out, nullptr, hs,
        pr ? pr->start : nullptr, pr ? pr->mid : nullptr);
    prof_no_merge(pr);
    return device_status(e);
}

osc_status osc_fill_pdf_layered(osc_ctx* ctx, const osc_sample* sample, const osc_layer* layers,
                                int32_t n_layers, int32_t set, const osc_binning* binning,
                                double* hist_out, double* p_out, void* stream)
{
    if (!ctx || !sample_ok(sample, true) || !hist_out || !layers_ok(layers, n_layers))
        return OSC_ERR_INVALID_ARG;
    if (!binning_ok(ctx, binning)) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (set < 0 || size_t(set) >= ctx->consts.size()) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const osc::LayerPath lp = layer_path(ctx->params[size_t(set)], layers, n_layers);
    return run_hist(ctx, 1, p_out != nullptr, false, ctx->consts[size_t(set)], osc::PathConsts{},
                    bin_consts(binning), sample->n, sample->e_true, sample->flags,
                    sample->weight, sample->e_reco, nullptr, nullptr, p_out, hist_out,
                    static_cast<hipStream_t>(stream), &lp);
}

osc_status osc_fill_hist(osc_ctx* ctx, int64_t n, const double* value, const double* weight,
                         const double* e_reco, const osc_binning* binning, double* hist_out,
                         void* stream)
{
    if (!ctx || n < 0 || n > osc::kMaxEvents || !hist_out) return OSC_ERR_INVALID_ARG;
    if (n > 0 && (!value || !weight || !e_reco)) return OSC_ERR_INVALID_ARG;
    if (!binning_ok(ctx, binning)) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const osc::SetConsts sc{};
    const osc::PathConsts pc{0.0, 0.0};
    return run_hist(ctx, 2, false, false, sc, pc, bin_consts(binning), n, nullptr, nullptr, weight,
                    e_reco, nullptr, value, nullptr, hist_out, static_cast<hipStream_t>(stream));
}

osc_status osc_profile_enable(osc_ctx* ctx, int on)
{
    if (!ctx) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    drop_profile(ctx);
    ctx->profiling = on != 0;
    return OSC_OK;
}

osc_status osc_profile_read(osc_ctx* ctx, double* event_kernel_ms, int64_t* event_kernel_launches,
                            double* merge_kernel_ms, int64_t* merge_kernel_launches)
{
    if (!ctx) return OSC_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(ctx->mu);
    double tile_ms = 0.0, merge_ms = 0.0;
    int64_t tiles = 0, merges = 0;
    osc_status st = OSC_OK;
    for (const ProfRec& r : ctx->prof) {
        float ms = 0.0f;
        if (hipEventSynchronize(r.mid) != hipSuccess ||
            hipEventElapsedTime(&ms, r.start, r.mid) != hipSuccess) {
            st = OSC_ERR_DEVICE;
            break;
        }
        tile_ms += ms;
        ++tiles;
        if (r.end) {
            if (hipEventSynchronize(r.end) != hipSuccess ||
                hipEventElapsedTime(&ms, r.mid, r.end) != hipSuccess) {
                st = OSC_ERR_DEVICE;
                break;
            }
            merge_ms += ms;
            ++merges;
        }
    }
    drop_profile(ctx);
    if (event_kernel_ms) *event_kernel_ms = tile_ms;
    if (event_kernel_launches) *event_kernel_launches = tiles;
    if (merge_kernel_ms) *merge_kernel_ms = merge_ms;
    if (merge_kernel_launches) *merge_kernel_launches = merges;
    return st;
}

osc_status osc_poisson_nll(osc_ctx* ctx, const double* hist, int64_t n_hist, double mu_scale,
                           const double* data, int64_t n_data, int32_t nbins, double* nll_out,
                           void* stream)
{
    if (!ctx || n_hist < 0 || n_data < 1 || nbins < 1 || nbins > ctx->max_nbins)
        return OSC_ERR_INVALID_ARG;
    if (!is_finite(mu_scale) || !(mu_scale > 0.0)) return OSC_ERR_INVALID_ARG;
    if (n_hist > 0 && (!hist || !data || !nll_out)) return OSC_ERR_INVALID_ARG;
    if (n_hist > int64_t(1) << 31) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    return device_status(osc::launch_poisson_nll(hist, n_hist, mu_scale, data, n_data, nbins,
                                                 nll_out, static_cast<hipStream_t>(stream)));
}

osc_status osc_validate_sample(osc_ctx* ctx, const osc_sample* sample, int64_t* bad_energy,
                               int64_t* bad_flags, void* stream)
{
    if (!ctx || !sample_ok(sample, false)) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    const hipStream_t hs = static_cast<hipStream_t>(stream);
    unsigned long long* d = nullptr;
    unsigned long long h[2] = {0, 0};
    if (device_malloc(&d, sizeof h) != hipSuccess) return OSC_ERR_OUT_OF_MEMORY;
    hipError_t e = hipMemsetAsync(d, 0, sizeof h, hs);
    if (e == hipSuccess)
        e = osc::launch_validate_sample(sample->n, sample->e_true, sample->flags, d, hs);
    if (e == hipSuccess) e = hipMemcpyAsync(h, d, sizeof h, hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    (void)hipFree(d);
    if (e != hipSuccess) return OSC_ERR_DEVICE;
    if (bad_energy) *bad_energy = int64_t(h[0]);
    if (bad_flags) *bad_flags = int64_t(h[1]);
    return OSC_OK;
}

void osc_reduction_layout(int32_t* tile_lanes, int32_t* lane_events, int32_t* accumulators)
{
    if (tile_lanes) *tile_lanes = osc::kTileLanes;
    if (lane_events) *lane_events = osc::kLaneEvents;
    if (accumulators) *accumulators = osc::kHistLanes;
}

int32_t osc_max_nbins(const osc_ctx* ctx) { return ctx ? ctx->max_nbins : 0; }

osc_status osc_occupancy(const osc_ctx* ctx, int32_t nbins, int with_hist, int32_t* waves_per_cu)
{
    if (!ctx || !waves_per_cu) return OSC_ERR_INVALID_ARG;
    if (with_hist && (nbins < 1 || nbins > ctx->max_nbins)) return OSC_ERR_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return OSC_ERR_DEVICE;
    int blocks = 0;
    if (osc::occupancy(with_hist ? 1 : 0, nbins, &blocks) != hipSuccess) return OSC_ERR_DEVICE;
    *waves_per_cu = blocks;
    return OSC_OK;
}

const char* osc_status_string(osc_status status)
{
    switch (status) {
        case OSC_OK: return "ok";
        case OSC_ERR_INVALID_ARG: return "invalid argument";
        case OSC_ERR_OUT_OF_MEMORY: return "out of device memory";
        case OSC_ERR_DEVICE: return "no usable device or HIP runtime error";
        case OSC_ERR_BUDGET: return "over memory budget";
        case OSC_ERR_NOT_READY: return "not ready";
    }
    return "unknown status";
}

}  // extern "C"
