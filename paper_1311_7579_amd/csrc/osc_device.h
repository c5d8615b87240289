// Device-side building blocks of libosc shared by the plain and the batched
// kernels: the per-event probability (FP64 and FP32-mixed tiers), the bin
// index, the per-wave LDS histograms and the tile body.  Both kernels
// run the same code, so a batched (set, sample) histogram equals the plain
// one bit for bit.
#pragma once

#include <type_traits>

#include "osc_internal.h"

namespace osc {
namespace dev {


// Events of one lane computed together in one straight-line block (and
// loaded one block ahead).  One event per block keeps the register count
// low enough for six waves per SIMD, which hides latency better than
// interleaving events within a wave.
constexpr int kGroup = 1;
static_assert(kLaneEvents % kGroup == 0, "the group size divides the events per lane");

// ---------------------------------------------------------------------------
// FP64 sine and cosine of a phase given in units of pi/32 as the product
// a b (|a b| < 2^50).  The nearest integer n to the exact product
// comes out of one FMA against 1.5 * 2^52 (n lands in the low mantissa
// bits), u = a b - n (|u| <= 1/2) out of a second one, so the reduction is
// exact up to the final rounding of u.  With r = u pi/32 (|r| <= pi/64):
//   sin r      = u (pi/32 + u^2 (P3 + P5 u^2 + P7 u^4))   (Taylor, scaled
//                to u; truncation below 7e-18),
//   cos r - 1  = u^2 (Q2 + Q4 u^2 + Q6 u^4)        (least-maximum absolute
//                error fit on |u| <= 1/2, error below 8e-18),
// and the angle-addition formulas with the anchor k = n mod 64 from LDS:
//   sin = s_k + s_k (cos r - 1) + c_k sin r,
//   cos = c_k + c_k (cos r - 1) - s_k sin r.
// ---------------------------------------------------------------------------
constexpr double kRoundMagic = 6755399441055744.0;        // 1.5 * 2^52
constexpr double kStep = 0.09817477042468103;             // fl(pi / 32)
constexpr double kP3 = -0.0001577060784927359;            // -(pi/32)^3 / 3!
constexpr double kP5 = 7.600081085793214e-08;             //  (pi/32)^5 / 5!
constexpr double kP7 = -1.7440893260086657e-11;           // -(pi/32)^7 / 7!
constexpr double kQ2 = -0.0048191427739688;
constexpr double kQ4 = 3.870689497756199e-06;
constexpr double kQ6 = -1.2434575820615234e-09;

__device__ __forceinline__ double flip_sign(double v, uint32_t sign_bit)
{
    return __hiloint2double(__double2hiint(v) ^ int(sign_bit), __double2loint(v));
}

struct Phase {
    double u;     // the phase less n
    int anchor;   // n mod 64
};

__device__ __forceinline__ Phase reduce_phase(double a, double b)
{
    const double t = __builtin_fma(a, b, kRoundMagic);
    const double n = t - kRoundMagic;
    return {__builtin_fma(a, b, -n), __double2loint(t) & 63};
}

// p7 and q6 are kP7 and kQ6; a caller that evaluates many phases passes
// them from VGPRs (see PolyRegs), so that each polynomial step reads at most
// one constant from an SGPR pair (the VALU reads one per instruction).
__device__ __forceinline__ void phase_sincos(const Phase& ph, const SinCos* __restrict__ table,
                                             double& sn, double& cs, double p7 = kP7,
                                             double q6 = kQ6)
{
    const double u = ph.u;
    const SinCos k = table[ph.anchor];
    const double z = u * u;
    const double s = u * __builtin_fma(z, __builtin_fma(z, __builtin_fma(z, p7, kP5), kP3), kStep);
    const double cm = z * __builtin_fma(z, __builtin_fma(z, q6, kQ4), kQ2);
    sn = __builtin_fma(k.s, cm, __builtin_fma(k.c, s, k.s));
    cs = __builtin_fma(k.c, cm, __builtin_fma(-k.s, s, k.c));
}

__device__ constexpr SinCosTable kAnchors = make_anchors();

// Copy the sin/cos anchors into LDS (the 64 lanes of a wave, one each).
template <class Tab>
__device__ __forceinline__ void load_sincos(Tab& T, int lane)
{
    if (lane < 64) T.sct[lane] = kAnchors.e[lane];
}

// Mixed tier: the phase (a b in units of pi/32, so a b / 64 in revolutions)
// is reduced to |rev| <= 1/2 in FP64 as above, rounded to FP32, and the FP32
// hardware sine and cosine (argument in revolutions) finish the job.
__device__ __forceinline__ void phase_sincos_mixed(double a, double b_rev, float& sn, float& cs)
{
    const double t = __builtin_fma(a, b_rev, kRoundMagic);
    const double n = t - kRoundMagic;
    const float rev = float(__builtin_fma(a, b_rev, -n));
    sn = __builtin_amdgcn_sinf(rev);
    cs = __builtin_amdgcn_cosf(rev);
}

// 1/y to within a few ulp: hardware reciprocal estimate r (relative error
// e ~ 3e-7) and one third-order correction r (1 + e + e^2), e = 1 - y r,
// which leaves ~e^3 (y normal, not huge).
__device__ __forceinline__ double recip(double y)
{
    const double r = __builtin_amdgcn_rcp(y);
    const double e = fma(-y, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// y^-1/2 of a positive y: the hardware estimate r (relative error e/2 ~
// 3e-7) corrected with the third-order series r (1 + e/2 + 3/8 e^2), e = 1 -
// y r^2.
__device__ __forceinline__ double rsqrt_refined(double y)
{
    const double r = __builtin_amdgcn_rsq(y);
    const double e = fma(-(y * r), r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
}

// 1/y with one Newton-Raphson correction (relative error ~1e-13): enough
// where the quotient is a small correction to a root.
__device__ __forceinline__ double recip_coarse(double y)
{
    const double r = __builtin_amdgcn_rcp(y);
    return fma(r, fma(-y, r, 1.0), r);
}

// arccos(x) / (6 pi) on [-1, 1] in FP32 (the seed angle theta/3 in
// revolutions for the hardware cosine): Abramowitz & Stegun 4.4.45 on |x|
// (error <= 6.7e-5 rad; the FP64 refinement below absorbs seed errors far
// larger than that) with its coefficients scaled by 1 / (6 pi), and
// acos(-x) = pi - acos(x).
__device__ __forceinline__ float acos_seed_rev(float x)
{
    constexpr float c = 0.053051647697298445f;   // 1 / (6 pi)
    const float ax = __builtin_fabsf(x);
    float p = -0.0187293f * c;
    p = __builtin_fmaf(p, ax, 0.0742610f * c);
    p = __builtin_fmaf(p, ax, -0.2121144f * c);
    p = __builtin_fmaf(p, ax, 1.5707288f * c);
    const float r = __builtin_amdgcn_sqrtf(1.0f - ax) * p;
    return x < 0.0f ? (1.0f / 6.0f) - r : r;
}

// A value the compiler cannot see through, kept in an SGPR pair.  3.0 is
// not an inline constant of the FP64 VALU; as a literal it only fits the
// two-address v_fmac form, which costs a register copy whenever the
// addend stays live.  From an SGPR the three-address v_fma takes it.
__device__ __forceinline__ double sgpr_value(double v)
{
    asm("" : "+s"(v));
    return v;
}

// The same, kept in a VGPR: loop-invariant
// operands that would otherwise be the second SGPR operand of an instruction
// (and be copied into a VGPR on every use).
__device__ __forceinline__ double vgpr_value(double v)
{
    asm("" : "+v"(v));
    return v;
}

// The innermost sine and cosine coefficients of phase_sincos, which a
// kernel that evaluates many phases loads into VGPRs once.
struct PolyRegs {
    double p7 = kP7, q6 = kQ6;
    static __device__ __forceinline__ PolyRegs in_vgprs()
    {
        return PolyRegs{vgpr_value(kP7), vgpr_value(kQ6)};
    }
};

// The eigenvalues of M in the FP64 tier come from one root of the characteristic cubic f(x) =
// x^3 - tr x^2 + c1 x - det and the cubic's discriminant.  Of three real
// roots one, x, is isolated: at least half the spread away from both
// others (the top one where q > 0, the bottom one where q < 0).  It is
// x = tr/3 + sign(q) sqrt(p) (2/3) cos(acos(|r|) / 3), r = q / (2 p^1.5),
// and (2/3) cos(acos(|r|) / 3) is smooth on [0, 1] (no arccos near its end
// points, no cosine): a polynomial of degree 6 gives it to 5e-8.  With a =
// A + A0 (A0 the minimum of p over A) p = a^2 + pm and q/2 = a^3 + k1 a + k0
// have no cancellation, so all of the seed runs in FP32 from fl32(a); it
// errs by at most ~3e-6 of the spread, typically 1e-7.  Each chord step
// x -= f(x) / f'(seed), with FP64 f and an FP32 1/f', squares that error and
// then multiplies it by it again: two steps reach FP64 rounding.
// The other two roots are not solved for: their sum is tr - x = -e, their
// product g = c1 - x (tr - x), f'(x) = (x - l1)(x - l2), and half their
// distance is del = sqrt(disc) / f'(x) with disc a quarter of the
// discriminant, a quartic in A with host coefficients.  Near a level crossing
// of a small mixing angle the quartic cancels, so that del errs by about
// 2^-53 (spread / gap)^2 of itself (in 2^-53: 6 at the atmospheric resonance of
// Table 1, 150 with sin2_th13 = 1e-3, 2e4 with 1e-5); psi, del times L/2E, is
// then as far off as an ulp of the largest phase times spread / gap, as with
// both roots solved for: P was compared with 64-bit-mantissa references at gaps
// from 8e-4 of the spread and 300 to 12000 km, and its error is the same or
// smaller than theirs.
struct Levels {
    double x;     // the isolated eigenvalue
    double e;     // x - tr: minus the sum of the other two
    double g;     // their product
    double fp;    // f'(x) > 0
    double disc;  // discriminant / 4 = (fp del)^2
};

// Two eigenvalues closer than about 7e-4 of the spread (1 - |r| below this,
// near an exact level crossing, which needs a zero mixing angle) are not
// resolved by the characteristic cubic; such an event's P comes out NaN.
constexpr float kUnresolved = 0x1p-19f;

// q / (2 p^1.5) = cos 3 theta of the cubic, in FP32 (also gives the seed's
// a, p^-1/2 and p).
struct SeedAngle {
    float a, p, rs, r;
};

__device__ __forceinline__ SeedAngle seed_angle(const SetConsts& sc, double A)
{
    SeedAngle s;
    s.a = float(A + sc.A0);
    const float a2 = s.a * s.a;
    s.p = a2 + sc.pm;
    const float qh = __builtin_fmaf(s.a, a2 + sc.k1, sc.k0);     // q / 2
    s.rs = __builtin_amdgcn_rsqf(s.p);
    s.r = qh * s.rs * (s.rs * s.rs);
    return s;
}

__device__ __forceinline__ Levels matter_levels(const SetConsts& sc, double A)
{
    Levels v;
    const double tr = sc.T0 + A, c1 = fma(A, sc.CA, sc.C0), det = A * sc.DA;
    v.disc = fma(A, fma(A, fma(A, fma(A, sc.D4, sc.D3), sc.D2), sc.D1), sc.D0);
    // the seed, in FP32
    const SeedAngle sa = seed_angle(sc, A);
    const float ar = __builtin_fabsf(sa.r);
    float G = -0.0006958966f;
    G = __builtin_fmaf(G, ar, 0.003408973f);
    G = __builtin_fmaf(G, ar, -0.008384795f);
    G = __builtin_fmaf(G, ar, 0.015869704f);
    G = __builtin_fmaf(G, ar, -0.031987853f);
    G = __builtin_fmaf(G, ar, 0.11110617f);
    G = __builtin_fmaf(G, ar, 0.57735032f);
    const float kf = __builtin_copysignf(sa.p * sa.rs, sa.r);
    float xf = __builtin_fmaf(kf, G, __builtin_fmaf(sa.a, 1.0f / 3.0f, sc.t3));
    if (ar > 1.0f - kUnresolved) xf = __builtin_nanf("");
    // f'(seed) = p (3 G^2 - 1/3)
    const double inv = double(__builtin_amdgcn_rcpf(sa.p * __builtin_fmaf(3.0f * G, G, -1.0f / 3.0f)));
    double x = double(xf);
#pragma unroll
    for (int k = 0; k < 2; ++k) x = fma(-fma(fma(x - tr, x, c1), x, -det), inv, x);
    v.x = x;
    v.e = x - tr;
    v.g = fma(v.e, x, c1);
    v.fp = fma(x, x + v.e, v.g);
    return v;
}

// The entry of flag byte f in one of the LDS channel arrays.
template <class Part>
__device__ __forceinline__ Part channel_part(const Part* table, uint32_t f)
{
    static_assert(sizeof(Part) == 16, "entries are 16-byte parts");
    const uint32_t ci = min(f, uint32_t(kFlagEntries - 1));
    return *reinterpret_cast<const Part*>(reinterpret_cast<const unsigned char*>(table) +
                                          ((ci << 4) + (ci & 16u)));
}

// +kA E for neutrinos, -kA E for antineutrinos (bit 4 of the flag byte,
// moved to the sign bit; one shift and one bit-field insert).
__device__ __forceinline__ double matter_term(double kA, double E, uint32_t f)
{
    return __builtin_copysign(kA * E, __hiloint2double(int(f << 27), 0));
}

// P(alpha -> beta) of one event.  With the isolated eigenvalue x, the mean mu
// and half-distance del of the other two, b = x - mu, and the phases theta =
// b L/2E and psi = del L/2E, the evolution operator is, up to the common
// phase exp(-i mu L/2E),
//   (1 - X) cos psi - i (sin psi / del) Y + exp(-i theta) X,
//   X = (M^2 + e M + g) / f'(x)     (the spectral projector of x),
//   Y = (M - mu)(1 - X) = M - mu - b X.
// sin psi / del has no singularity as the two eigenvalues close in.  Only
// the element (beta, alpha) is formed.
// What P's error is made of, at large phases: the roundings of x, tr and b, of
// 1/E and of X's factor 1/f'.  So 1/E and 1/f' share one reciprocal estimate, of
// E f', but each is corrected with its own residual, and b's rounding (b_lo)
// enters theta after its reduction.  del needs fewer bits.  Mean ratio of the
// rms error to that of two solved roots, over 400 sets at 295 to 2500 km: 0.89
// for E log-uniform on 0.1-10 GeV (1.27 with both inverses from one inverse
// square root; 1.00 without b_lo), 0.62 for uniform E.
// Bound by VALU issue: about 131 FP64 issue slots per event and wave (the
// benchmark step's loop, an FP32 instruction counted as half), against 158
// with two roots from trigonometric seeds, a Halley step each and the
// projectors of two roots: 1e7 events, P alone 61.7 -> 54.7 us a call, the
// step on binned events with P written 76.7 -> 68.9 us (52.4 and 67.3 with both
// inverses from one inverse square root and without b_lo).  1/f' of the chord
// steps and the seed are FP32, which steer an FP64 iteration.
__device__ __forceinline__ double event_prob(const SetConsts& sc, const TileTables& T, double kA,
                                             double kL, double E, uint32_t f,
                                             const PolyRegs& pr = PolyRegs{})
{
    // flag byte (alpha bits 0-1, beta bits 2-3, antineutrino bit 4) -> the
    // channel entry (conjugated for antineutrinos) and the sign of A
    const Pair m = channel_part(T.m, f), m2 = channel_part(T.m2, f), g = channel_part(T.g, f),
               d = channel_part(T.d, f);
    const double A = matter_term(kA, E, f);
    const double dba = d.b;   // [alpha = beta]; NaN for an invalid flag byte

    // amplitude inputs: M_ba and (M^2)_ba
    const double mre = fma(A, d.a, m.a), mim = m.b;
    const double m2re = fma(A, fma(A, d.a, g.a), m2.a);
    const double m2im = fma(A, g.b, m2.b);

    const Levels v = matter_levels(sc, A);
    // 1/E and 1/f' from one reciprocal, each with its own last bits
    const double r = __builtin_amdgcn_rcp(E * v.fp);
    const double rE = v.fp * r, rf = E * r;
    const double eE = fma(-E, rE, 1.0), ef = fma(-v.fp, rf, 1.0);
    const double invE = fma(rE, fma(eE, eE, eE), rE);
    const double inv_fp = fma(rf, fma(ef, ef, ef), rf);
    const double y = rsqrt_refined(v.disc);             // 1 / sqrt(disc)
    const double del = (v.disc * y) * inv_fp, inv_del = v.fp * y;
    const double b = fma(0.5, v.e, v.x), b_lo = fma(0.5, v.e, v.x - b);
    const double ph = kL * invE;                        // phase per eV^2 in units of pi/32

    const double Xr = fma(v.g, dba, fma(v.e, mre, m2re)) * inv_fp;
    const double Xi = fma(v.e, mim, m2im) * inv_fp;
    const double Yr = fma(-b, Xr, fma(v.e, 0.5 * dba, mre));
    const double Yi = fma(-b, Xi, mim);
    double s1, c1, s2, c2;
    Phase theta = reduce_phase(b, ph);
    theta.u = fma(b_lo, ph, theta.u);
    phase_sincos(theta, T.sct, s1, c1, pr.p7, pr.q6);
    phase_sincos(reduce_phase(del, ph), T.sct, s2, c2, pr.p7, pr.q6);   // psi
    const double sg = s2 * inv_del, w = c1 - c2;
    const double zr = fma(sg, Yi, fma(s1, Xi, fma(w, Xr, dba * c2)));
    const double zi = fma(-sg, Yr, fma(-s1, Xr, w * Xi));
    return fma(zi, zi, zr * zr);
}

// The eigenvalues in the FP32-mixed tier: roots of f(x) = x^3 - tr x^2 +
// c1 x - det.  Two roots are seeded in FP32 from the trigonometric
// solution x = tr/3 + (2/3) sqrt(p) cos(theta - 2 pi k / 3),
// theta = acos(q / (2 p^1.5)) / 3 (p = tr^2 - 3 c1, q = 2 tr^3 - 9 tr c1 +
// 27 det, qh = q / 2), each refined in FP64 by one
// Halley step on f; the third root follows from the trace.  The two roots'
// divisions of each step share one reciprocal: 1/a = b / (a b), 1/b = a /
// (a b).  A wave skips the Newton step when every lane's Halley corrections
// were at most 2^-12 of its smallest root distance.  Halley converges
// cubically, so the roots are then within about (2^-12)^3 ~ 1.5e-11 of that
// distance, far below what the FP32 amplitude assembly resolves, and the
// phases stay within ~1e-8 rad up to 1e3 rad.  (The FP64 tier's isolated
// root and amplitude together moved P of this tier by up to 2e-7; its root alone
// in front of this amplitude has not been measured.)
constexpr double kHalleyOnly = 0x1p-12;
// Waves with a matter term above this (eV^2, about 4 times the largest
// vacuum splitting) assemble the amplitude in FP64.
constexpr double kMixedWideA = 0.01;

struct MixedRoots {
    double tr, c1, det, x0, x1;
    double x2, d01, d12;   // the third root, x0 - x1 and x1 - x2

    __device__ __forceinline__ void finish()
    {
        x2 = (tr - x0) - x1;
        d01 = x0 - x1;
        d12 = x1 - x2;
    }
};

// Constants of a set that the batched kernel keeps in VGPRs over its events
// where it runs two sets side by side (second constant operands of an FMA,
// which it otherwise copied there for every event): the 256-set x 4-sample
// batch 8.83 -> 8.69 ms.
struct MixedRegs {
    double C0, QH1, QH0;
    static __device__ __forceinline__ MixedRegs of(const SetConsts& sc)
    {
        return MixedRegs{sc.C0, sc.QH1, sc.QH0};
    }
    static __device__ __forceinline__ MixedRegs in_vgprs(const SetConsts& sc)
    {
        return MixedRegs{vgpr_value(sc.C0), vgpr_value(sc.QH1), vgpr_value(sc.QH0)};
    }
};

__device__ __forceinline__ MixedRoots halley_roots(const SetConsts& sc, const MixedRegs& regs,
                                                   double A, uint64_t& open)
{
    MixedRoots v;
    const double tr = sc.T0 + A, c1 = fma(A, sc.CA, regs.C0), det = A * sc.DA;
    const double qh = fma(fma(A + sc.QH2, A, regs.QH1), A, regs.QH0);
    const double p = fma(tr, tr, -3.0 * c1);
    const float pf = float(p), qf = float(qh);
    const float rs = __builtin_amdgcn_rsqf(pf);                 // p^-1/2
    float rf = qf * (rs * rs * rs);                             // q / (2 p^3/2)
    rf = __builtin_fminf(1.0f, __builtin_fmaxf(-1.0f, rf));
    // theta in revolutions for the hardware cosine: acos(r) / (3 * 2 pi)
    const float th = acos_seed_rev(rf);
    // the seeds in FP32 (their FP32 rounding, ~6e-8 of |x|, is far below
    // their error of ~1e-4 of the roots' spread)
    const float kf = (2.0f / 3.0f) * (pf * rs);
    const float t3f = float(tr) * (1.0f / 3.0f);
    double x0 = double(__builtin_fmaf(kf, __builtin_amdgcn_cosf(th), t3f));
    double x1 = double(__builtin_fmaf(kf, __builtin_amdgcn_cosf(th - 0.33333333f), t3f));
    const double three = sgpr_value(3.0);
    // Halley: x -= 2 f f' / (2 f'^2 - f f'')
    const double f0 = fma(fma(x0 - tr, x0, c1), x0, -det);
    const double f1 = fma(fma(x1 - tr, x1, c1), x1, -det);
    // m = tr - 3x = -f''/2, and f' = x (3x - 2 tr) + c1 = c1 - x (m + tr)
    const double m0 = fma(-three, x0, tr), m1 = fma(-three, x1, tr);
    const double g0 = fma(-x0, m0 + tr, c1);
    const double g1 = fma(-x1, m1 + tr, c1);
    const double d0 = fma(g0, g0, f0 * m0);
    const double d1 = fma(g1, g1, f1 * m1);
    const double r = recip_coarse(d0 * d1);
    const double h0 = (f0 * g0) * (d1 * r), h1 = (f1 * g1) * (d0 * r);
    x0 -= h0;
    x1 -= h1;
    v.tr = tr;
    v.c1 = c1;
    v.det = det;
    v.x0 = x0;
    v.x1 = x1;
    v.finish();
    // x0 > x1 > x2: the smallest root distance is one of these
    const double dmin = __builtin_fmin(__builtin_fabs(v.d01), __builtin_fabs(v.d12));
    open = __builtin_amdgcn_ballot_w64(
        !(__builtin_fmax(__builtin_fabs(h0), __builtin_fabs(h1)) <= kHalleyOnly * dmin));
    return v;
}

// One Newton step x -= f / f' on both roots.
__device__ __forceinline__ void newton_roots(const SetConsts& sc, double A, MixedRoots& v)
{
    const double three = sgpr_value(3.0);
    const double tr2 = 2.0 * v.tr;
    const double f0 = fma(fma(v.x0 - v.tr, v.x0, v.c1), v.x0, -v.det);
    const double f1 = fma(fma(v.x1 - v.tr, v.x1, v.c1), v.x1, -v.det);
    const double g0 = fma(v.x0, fma(three, v.x0, -tr2), v.c1);
    const double g1 = fma(v.x1, fma(three, v.x1, -tr2), v.c1);
    const double r = recip_coarse(g0 * g1);
    v.x0 -= f0 * (g1 * r);
    v.x1 -= f1 * (g0 * r);
    // the FP64 tier's rule, so that both give NaN on the same events
    // (every such lane's Halley step is large, so its wave comes here)
    if (__builtin_fabsf(seed_angle(sc, A).r) > 1.0f - kUnresolved) v.x0 = __builtin_nan("");
    v.finish();
}

// P of one event in the FP32-mixed tier.  The evolution operator is sum_k
// exp(-i phi_k) X_k with the spectral projectors X_k = (M - l_j)(M - l_l) /
// ((l_k - l_j)(l_k - l_l)); the common phase exp(-i phi_0) drops out, and
// the projectors sum to the identity, so S' = [a = b] + (exp(-i dphi1) - 1)
// X1 + (exp(-i dphi2) - 1) X2.  Eigenvalues and phase differences are FP64,
// the rest FP32.  `wide` (the same for the whole wave): the amplitude in FP64.
template <bool WIDE>
__device__ __forceinline__ double mixed_amplitude(const MixedRoots& v, const ChanF& c, double A,
                                                  double kL, double E)
{
    const double l0 = v.x0, l1 = v.x1, l2 = v.x2;
    const double d01 = v.d01, d02 = l0 - l2, d12 = v.d12;
    const double Q = d01 * d02 * d12;
    const double R = recip(E * Q);
    const double invE = Q * R, invQ = E * R;
    const double ph = kL * (1.0 / 64.0) * invE;   // phase per eV^2 in units of 2 pi
    // numerator coefficients: N_k = (M^2)_ba - (l_j + l_l) M_ba + l_j l_l [a = b]
    const double u1 = l0 + l2, v1 = l0 * l2;
    const double u2 = l0 + l1, v2 = l0 * l1;
    const double iD1 = -d02 * invQ, iD2 = d01 * invQ;

    float s1, c1, s2, c2;
    phase_sincos_mixed(-d01, ph, s1, c1);
    phase_sincos_mixed(-d02, ph, s2, c2);
    if constexpr (WIDE) {
        // Matter terms well above the vacuum splittings: the projector
        // numerators cancel over about |A| / dm^2_31, beyond what FP32
        // resolves, so such waves form them and the sum in FP64 (from
        // the same FP32 channel entries and FP32 phases).
        const double d_dee = c.dee, d_dba = c.dba;
        const double d_mre = fma(A, d_dee, double(c.m_re));
        const double d_mim = c.m_im;
        const double d_m2re = fma(A, fma(A, d_dee, double(c.g_re)), double(c.m2_re));
        const double d_m2im = fma(A, double(c.g_im), double(c.m2_im));
        const double x1r = fma(v1, d_dba, fma(-u1, d_mre, d_m2re)) * iD1;
        const double x1i = fma(-u1, d_mim, d_m2im) * iD1;
        const double x2r = fma(v2, d_dba, fma(-u2, d_mre, d_m2re)) * iD2;
        const double x2i = fma(-u2, d_mim, d_m2im) * iD2;
        const double e1 = double(c1) - 1.0, e2 = double(c2) - 1.0;
        const double ds1 = s1, ds2 = s2;
        const double sr = d_dba + e1 * x1r + ds1 * x1i + e2 * x2r + ds2 * x2i;
        const double si = e1 * x1i - ds1 * x1r + e2 * x2i - ds2 * x2r;
        return sr * sr + si * si;
    } else {
        // amplitude inputs M_ba and (M^2)_ba and the assembly in FP32 from
        // FP32-rounded inputs
        const float Ar = float(A);
        const float mre = __builtin_fmaf(Ar, c.dee, c.m_re), mim = c.m_im;
        const float m2re = __builtin_fmaf(Ar, __builtin_fmaf(Ar, c.dee, c.g_re), c.m2_re);
        const float m2im = __builtin_fmaf(Ar, c.g_im, c.m2_im);
        const float fdba = c.dba;
        const float fu1 = float(u1), fu2 = float(u2);
        const float fv1 = float(v1), fv2 = float(v2);
        const float fi1 = float(iD1), fi2 = float(iD2);
        const float x1r = __builtin_fmaf(fv1, fdba, __builtin_fmaf(-fu1, mre, m2re)) * fi1;
        const float x1i = __builtin_fmaf(-fu1, mim, m2im) * fi1;
        const float x2r = __builtin_fmaf(fv2, fdba, __builtin_fmaf(-fu2, mre, m2re)) * fi2;
        const float x2i = __builtin_fmaf(-fu2, mim, m2im) * fi2;
        const float e1 = c1 - 1.0f, e2 = c2 - 1.0f;
        const float sr = fdba + e1 * x1r + s1 * x1i + e2 * x2r + s2 * x2i;
        const float si = e1 * x1i - s1 * x1r + e2 * x2i - s2 * x2r;
        return double(sr * sr + si * si);
    }
}

// P of one event under NS parameter sets.  The sets share the event's flag
// decode and matter term, and the arithmetic of two sets runs side by side:
// only the rare steps (Newton, wide matter terms) are branches, taken by the
// wave for each set as it would alone.
template <int NS>
__device__ __forceinline__ void event_probs_mixed(const SetConsts* const (&sc)[NS],
                                                  const TileTablesMixed* const (&T)[NS],
                                                  const MixedRegs (&regs)[NS], double kA,
                                                  double kL, double E, uint32_t f, double (&P)[NS])
{
    const FlagInfo fl = T[0]->flag[min(f, uint32_t(kMixedFlags - 1))];
    const double A = flip_sign(kA * E, fl.sign);
    ChanF c[NS];
    MixedRoots v[NS];
    uint64_t open[NS], any_open = 0;   // lanes whose roots need the Newton step
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        c[k] = *reinterpret_cast<const ChanF*>(
            reinterpret_cast<const unsigned char*>(T[k]->ch) + fl.ch_off);
        v[k] = halley_roots(*sc[k], regs[k], A, open[k]);
        any_open |= open[k];
    }
    if (__builtin_expect(any_open != 0, 0)) {
#pragma unroll
        for (int k = 0; k < NS; ++k)
            if (open[k]) newton_roots(*sc[k], A, v[k]);
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(__builtin_fabs(A) > kMixedWideA) != 0, 0)) {
#pragma unroll
        for (int k = 0; k < NS; ++k) P[k] = mixed_amplitude<true>(v[k], c[k], A, kL, E);
        return;
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) P[k] = mixed_amplitude<false>(v[k], c[k], A, kL, E);
}

__device__ __forceinline__ double event_prob_mixed(const SetConsts& sc, const TileTablesMixed& T,
                                                   double kA, double kL, double E, uint32_t f)
{
    const SetConsts* const s[1] = {&sc};
    const TileTablesMixed* const t[1] = {&T};
    double P[1];
    const MixedRegs r[1] = {MixedRegs::of(sc)};
    event_probs_mixed<1>(s, t, r, kA, kL, E, f, P);
    return P[0];
}

// P of one event through one constant-density layer: the policy the tile
// body calls (MIXED selects the FP32-mixed amplitude assembly).
template <bool MIXED>
struct ConstDensityProb {
    static constexpr bool kDecidesByWave = MIXED;   // ballots over the wave's events
    const SetConsts* sc;
    const Tables<MIXED>* tabs;
    double kA, kL;
    PolyRegs pr;
    __device__ __forceinline__ double operator()(double E, uint32_t f) const
    {
        if constexpr (MIXED)
            return event_prob_mixed(*sc, *tabs, kA, kL, E, f);
        else
            return event_prob(*sc, *tabs, kA, kL, E, f, pr);
    }
};

// P(alpha -> beta) of one event through layers of constant density.  The
// evolution operator of the path is the product of the layers' operators,
// so only column alpha of it is needed: v = <basis|alpha> is propagated layer
// by layer, in the basis where M is real and tridiagonal (Tridiagonal).
// Antineutrinos: the operators are the complex conjugates of those of H0 -
// |A| e_e e_e^T with the phases reversed, and |S|^2 is that of the conjugate.
//
// With N = M - mu, the operator of one layer is, up to a phase (notation of
// event_prob; its eigenvalues on N are b and +-del),
//   cos psi - i (sin psi / del) N + kappa (N^2 - del^2)
//     = c0 + N (kappa N - i s),   s = sin psi / del,
//   kappa = (exp(-i theta) - cos psi + i s b) / f'(x),  c0 = cos psi - kappa del^2,
// two products with a real tridiagonal matrix per vector (propagate).
//
// M is symmetric, so every layer's operator is, and a path that reads the
// same from both ends gives S = T^T T or T^T S_mid T with T the first
// half's operator: S_beta,alpha = (T beta) . (S_mid T alpha).  Both vectors go
// through each layer of the first half with one set of coefficients.
//
// Bound by VALU issue: about 97 FP64 issue slots for a layer's coefficients
// and 58 for a vector through it, or 96 for two (by the operator's elements:
// 24 to form them, 36 a vector; two times 58 took 3 % longer over five layers
// and 8 % over 12 and 31).  With complex 3x3 products in the flavour basis and
// every layer solved, 1e7 events took 424 us through the five-layer Earth path
// (now 231) and 3e6 events 300 us through 12 layers (now 133).
struct Vec3 {
    double r[3], i[3];
};

struct LayerOp {
    double p0, p1, p2, b0, b1;   // N
    double c0r, c0i, s, kr, ki;
};

// N u + start, component by component (real part or imaginary part).
__device__ __forceinline__ void add_times(const LayerOp& o, const double (&u)[3], double (&d)[3])
{
    d[0] = fma(o.p0, u[0], fma(o.b0, u[1], d[0]));
    d[1] = fma(o.p1, u[1], fma(o.b0, u[0], fma(o.b1, u[2], d[1])));
    d[2] = fma(o.p2, u[2], fma(o.b1, u[1], d[2]));
}

__device__ __forceinline__ void propagate(const LayerOp& o, Vec3& v)
{
    Vec3 y, t;
    y.r[0] = fma(o.p0, v.r[0], o.b0 * v.r[1]);
    y.i[0] = fma(o.p0, v.i[0], o.b0 * v.i[1]);
    y.r[1] = fma(o.p1, v.r[1], fma(o.b0, v.r[0], o.b1 * v.r[2]));
    y.i[1] = fma(o.p1, v.i[1], fma(o.b0, v.i[0], o.b1 * v.i[2]));
    y.r[2] = fma(o.p2, v.r[2], o.b1 * v.r[1]);
    y.i[2] = fma(o.p2, v.i[2], o.b1 * v.i[1]);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        t.r[j] = fma(o.s, v.i[j], fma(o.kr, y.r[j], -(o.ki * y.i[j])));
        t.i[j] = fma(-o.s, v.r[j], fma(o.kr, y.i[j], o.ki * y.r[j]));
        const double r = fma(o.c0r, v.r[j], -(o.c0i * v.i[j]));
        v.i[j] = fma(o.c0r, v.i[j], o.c0i * v.r[j]);
        v.r[j] = r;
    }
    add_times(o, t.r, v.r);
    add_times(o, t.i, v.i);
}

// Both vectors through one layer, by the operator's six elements (it is
// symmetric): S = c0 + kappa N^2 - i s N.
__device__ __forceinline__ void propagate_both(const LayerOp& o, const Tridiagonal& tri, Vec3& v,
                                               Vec3& u)
{
    // N^2
    const double n00 = fma(o.p0, o.p0, tri.b00), n11 = fma(o.p1, o.p1, tri.b00 + tri.b11),
                 n22 = fma(o.p2, o.p2, tri.b11), n01 = o.b0 * (o.p0 + o.p1),
                 n12 = o.b1 * (o.p1 + o.p2), n02 = tri.b01;
    const double r00 = fma(o.kr, n00, o.c0r), r11 = fma(o.kr, n11, o.c0r),
                 r22 = fma(o.kr, n22, o.c0r), r01 = o.kr * n01, r12 = o.kr * n12,
                 r02 = o.kr * n02;
    const double i00 = fma(o.ki, n00, fma(-o.s, o.p0, o.c0i)),
                 i11 = fma(o.ki, n11, fma(-o.s, o.p1, o.c0i)),
                 i22 = fma(o.ki, n22, fma(-o.s, o.p2, o.c0i)),
                 i01 = fma(o.ki, n01, -(o.s * o.b0)), i12 = fma(o.ki, n12, -(o.s * o.b1)),
                 i02 = o.ki * n02;
    const auto row = [](double ar, double ai, double br, double bi, double cr, double ci,
                        const Vec3& x, double& re, double& im) {
        re = fma(ar, x.r[0], fma(-ai, x.i[0], fma(br, x.r[1], fma(-bi, x.i[1],
             fma(cr, x.r[2], -(ci * x.i[2]))))));
        im = fma(ar, x.i[0], fma(ai, x.r[0], fma(br, x.i[1], fma(bi, x.r[1],
             fma(cr, x.i[2], ci * x.r[2])))));
    };
    const auto apply = [&](Vec3& x) {
        Vec3 y;
        row(r00, i00, r01, i01, r02, i02, x, y.r[0], y.i[0]);
        row(r01, i01, r11, i11, r12, i12, x, y.r[1], y.i[1]);
        row(r02, i02, r12, i12, r22, i22, x, y.r[2], y.i[2]);
        x = y;
    };
    apply(v);
    apply(u);
}

__device__ __forceinline__ double event_prob_layered(const SetConsts& sc, const LayeredTables& T,
                                                     const LayerPath& lp, double E, uint32_t f)
{
    const uint32_t fv = f < 32u ? f : 3u;   // invalid bytes take the NaN row
    const double(&wa)[5] = T.w[fv & 3u];
    const double(&wb)[5] = T.w[(fv >> 2) & 3u];
    Vec3 v{{wa[0], wa[1], wa[3]}, {0.0, -wa[2], -wa[4]}};
    Vec3 u{{wb[0], wb[1], wb[3]}, {0.0, wb[2], wb[4]}};
    const double invE = matter_term(1.0, recip(E), f);   // negative for antineutrinos
    for (int k = 0; k < lp.n; ++k) {
        const PathConsts pc = lp.layer[k];
        const double A = matter_term(pc.kA, E, f);
        const Levels lv = matter_levels(sc, A);
        const double y = rsqrt_refined(lv.disc);   // 1 / sqrt(disc)
        const double inv_fp = recip(lv.fp);
        const double del = (lv.disc * y) * inv_fp;
        const double b = fma(0.5, lv.e, lv.x);
        const double ph = pc.kL * invE;
        double s1, c1, s2, c2;
        phase_sincos(reduce_phase(b, ph), T.sct, s1, c1);     // theta
        phase_sincos(reduce_phase(del, ph), T.sct, s2, c2);   // psi
        LayerOp o;
        o.s = s2 * (lv.fp * y);
        o.kr = (c1 - c2) * inv_fp;
        o.ki = fma(o.s, b, -s1) * inv_fp;
        const double del2 = del * del;
        o.c0r = fma(-o.kr, del2, c2);
        o.c0i = -(o.ki * del2);
        o.p0 = fma(0.5, lv.e, lp.tri.a0 + A);
        o.p1 = fma(0.5, lv.e, lp.tri.a1);
        o.p2 = fma(0.5, lv.e, lp.tri.a2);
        o.b0 = lp.tri.b0;
        o.b1 = lp.tri.b1;
        if (k < lp.pairs)
            propagate_both(o, lp.tri, v, u);
        else
            propagate(o, v);
    }
    double zr = 0.0, zi = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        zr = fma(u.r[j], v.r[j], fma(-u.i[j], v.i[j], zr));
        zi = fma(u.r[j], v.i[j], fma(u.i[j], v.r[j], zi));
    }
    return fma(zi, zi, zr * zr);
}

// P of one event through a layered path (FP64).
struct LayeredProb {
    static constexpr bool kDecidesByWave = false;
    const SetConsts* sc;
    const LayeredTables* tabs;
    const LayerPath* lp;
    __device__ __forceinline__ double operator()(double E, uint32_t f) const
    {
        return event_prob_layered(*sc, *tabs, *lp, E, f);
    }
};

// Bin of x: floor(fl(fl(x * scale - lo) / wb)) with under/overflow.  The
// quotient is first formed as fl(x * scale - lo) * fl(1 / wb); that is
// within 3 u |q| (u = 2^-53) of the correctly rounded quotient q, so the
// floors agree unless an integer lies within that distance.  Below
// kFastBinLimit = 2^12 in magnitude the distance is under 1.5 * 2^-40;
// lanes within 2^-38 of an integer are flagged and redone with the
// correctly rounded division.  Beyond 2^12 the bin is overflow (or
// underflow) either way, since no binning has that many bins.
__device__ __forceinline__ double bin_floor_fast(double x, const BinConsts& bc, bool& edge)
{
#pragma clang fp contract(off)
    const double d = x * bc.scale - bc.lo;   // scaled energy, then the offset: two roundings
    const double q = d * bc.inv_wb;
    const double k = __builtin_floor(q);
    edge = (__builtin_fabs((q - k) - 0.5) > 0.5 - 0x1p-38) && (__builtin_fabs(q) < kFastBinLimit);
    return k;
}

__device__ __forceinline__ double bin_floor_exact(double x, const BinConsts& bc)
{
#pragma clang fp contract(off)
    return __builtin_floor((x * bc.scale - bc.lo) / bc.wb);
}

// Row of floor value k in the LDS histograms: 0 underflow, 1 + k regular,
// nb + 1 overflow (NaN included: fmin returns the non-NaN operand).
__device__ __forceinline__ int lds_bin(double k, const BinConsts& bc)
{
    return int(__builtin_fmax(__builtin_fmin(k, double(bc.nb)), -1.0)) + 1;
}

// LDS row of output bin r (output order: nb regular bins, underflow, overflow).
__device__ __forceinline__ int lds_row_of_output(int r, int nb)
{
    return r < nb ? r + 1 : (r == nb ? 0 : nb + 1);
}

// Histogram accumulator slot: bin-major rows of kHistLanes accumulators,
// the accumulator index XOR-swizzled by the row so that both the per-lane
// accumulation and the per-bin transposed reads spread over the LDS banks.
// The swizzle uses row - 1 (the floor value k of the row), so that the
// row's +1 becomes a constant offset of the LDS instruction.
__device__ __forceinline__ int hslot(int row, int acc)
{
    return row * kHistLanes + (acc ^ ((row - 1) & (kHistLanes - 1)));
}

// complete binary tree over the kHistLanes accumulators of one bin
template <int N, int J0>
__device__ __forceinline__ double lane_tree(const double* h, int bin)
{
    if constexpr (N == 1) {
        return h[hslot(bin, J0)];
    } else {
        const double left = lane_tree<N / 2, J0>(h, bin);
        const double right = lane_tree<N / 2, J0 + N / 2>(h, bin);
        return left + right;
    }
}

// kPdfBinned: kPdf with the events' histogram slots read from a cached
// per-sample array (one 16-bit LDS slot index per event, see bin_slot)
// instead of computed from the reco energy.
enum Mode { kReweight = 0, kPdf = 1, kHist = 2, kPdfBinned = 3 };

constexpr bool reads_bins(int mode) { return mode == kPdfBinned; }
constexpr bool has_hist(int mode) { return mode != kReweight; }

struct EventIn {
    double e;       // true energy (or the given value in kHist mode)
    double w;
    double x;       // reco energy (kPdf, kHist)
    uint32_t f;
    uint32_t slot;  // cached histogram slot (kPdfBinned)
};

// The arrays of one tile as raw buffer resources (base in SGPRs, size in
// bytes as the bound): an event's loads and its P store then take the form
// buffer_load v, lane_offset, rsrc, group_offset -- the lane offset is
// loop-invariant, the group offset lives in an SGPR, and no per-event
// address arithmetic runs on the VALU.  Accesses past the bound read 0 and
// write nothing (the tail guards below still decide what is used).
constexpr int kBufDword3 = 0x00020000;   // gfx9 family: raw buffer, 32-bit data format
constexpr int kBufNonTemporal = 2;        // cache-policy operand: the nt bit
typedef unsigned int BufU2 __attribute__((ext_vector_type(2)));

struct TileBufs {
    __amdgpu_buffer_rsrc_t e, f, w, x, p;
};

template <int MODE>
__device__ __forceinline__ TileBufs tile_bufs(uint32_t n, const double* e_true,
                                              const uint8_t* flags, const double* weight,
                                              const double* e_reco, const uint16_t* bins,
                                              const double* value, double* p_out)
{
    const int nb = int(n * sizeof(double));
    TileBufs b;
    b.e = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(MODE == kHist ? value : e_true), 0, nb, kBufDword3);
    b.f = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(flags), 0, int(n), kBufDword3);
    b.w = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(weight), 0, nb, kBufDword3);
    if constexpr (reads_bins(MODE))
        b.x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(bins), 0,
                                                int(n * sizeof(uint16_t)), kBufDword3);
    else
        b.x = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(e_reco), 0, nb, kBufDword3);
    b.p = __builtin_amdgcn_make_buffer_rsrc(p_out, 0, nb, kBufDword3);
    return b;
}

__device__ __forceinline__ double buf_load_f64(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

// The same arrays as plain pointers (global loads with 64-bit addresses):
// the batched kernel keeps this form, where the resources' SGPRs cost more
// than the address arithmetic they save.
struct TilePtrs {
    const double* e;
    const uint8_t* f;
    const double* w;
    const double* x;
    const uint16_t* s;
};

template <int MODE, bool FULL>
__device__ __forceinline__ EventIn load_event(const TilePtrs& b, uint32_t l, uint32_t g0,
                                              uint32_t n)
{
    EventIn v;
    const uint32_t i = l + g0;
    const bool in = FULL || i < n;
    v.e = in ? b.e[i] : 1.0;
    v.f = (MODE != kHist && in) ? uint32_t(b.f[i]) : 0u;
    v.w = (has_hist(MODE) && in) ? b.w[i] : 0.0;
    v.x = (has_hist(MODE) && !reads_bins(MODE) && in) ? b.x[i] : 0.0;
    v.slot = (reads_bins(MODE) && in) ? uint32_t(b.s[i]) : 0u;
    return v;
}

// Event g0 + l of a tile (0 <= g0 + l < kTileEvents); n = the tile's events
// (kTileEvents when FULL).  g0 is the same for the whole wave.
template <int MODE, bool FULL, bool FILL>
__device__ __forceinline__ EventIn load_event(const TileBufs& b, uint32_t l, uint32_t g0,
                                              uint32_t n)
{
    EventIn v;
    // a ragged tile's offset goes through the VGPR, which the resource's
    // bound covers: lanes past the end read 0 without a branch.  Where they
    // take part in the wave's decisions (FILL), and so in its bits, their energy
    // is 1 GeV, as in the batched kernel's load.
    const uint32_t lv = FULL ? l : l + g0, gs = FULL ? g0 : 0u;
    const uint32_t l8 = lv * 8u, g8 = gs * 8u;
    v.e = buf_load_f64(b.e, l8, g8);
    if (FILL && !FULL && MODE != kHist) v.e = lv < n ? v.e : 1.0;
    v.f = MODE != kHist ? uint32_t(__builtin_amdgcn_raw_buffer_load_b8(b.f, lv, gs, 0)) : 0u;
    v.w = has_hist(MODE) ? buf_load_f64(b.w, l8, g8) : 0.0;
    v.x = has_hist(MODE) && !reads_bins(MODE) ? buf_load_f64(b.x, l8, g8) : 0.0;
    v.slot = reads_bins(MODE)
                 ? uint32_t(__builtin_amdgcn_raw_buffer_load_b16(b.x, lv * 2u, gs * 2u, 0))
                 : 0u;
    return v;
}

__device__ __forceinline__ void store_p(const TileBufs& b, uint32_t l, uint32_t g0, double P)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(BufU2, P), b.p, l * 8u, g0 * 8u,
                                          kBufNonTemporal);
}

// Adds cval of every active lane into its accumulator.  The lanes sharing an
// accumulator add in ascending lane order: one masked LDS atomic add per lane
// group, group after group.  Within a group the lanes hit distinct
// accumulators, and the DS instructions of a wave execute in issue order, so
// every accumulator receives its additions in the contract's order (the LDS
// adder rounds like v_add_f64: round to nearest even).  The empty asm with a
// memory clobber keeps the compiler from merging or reordering the groups.
__device__ __forceinline__ void add_in_lane_order(double* slot, double cval, int lane)
{
#pragma unroll
    for (int p = 0; p < kLaneShare; ++p) {
        if (lane / kHistLanes == p)
            __hip_atomic_fetch_add(slot, cval, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
    }
}

// One group of kGroup events of a lane: the probabilities are computed in
// one straight-line block (no guards: lanes past the end of the sample hold
// dummy inputs), then stored, binned and accumulated in ascending m.
template <int MODE, bool WRITE_P, bool FULL, class PROB, class ARR>
__device__ __forceinline__ void tile_group(const PROB& prob, const BinConsts& bc, double* hist,
                                           int lane, uint32_t l, uint32_t g0, uint32_t n,
                                           const EventIn (&ev)[kGroup], const ARR& arr)
{
    constexpr bool kComputeBins = has_hist(MODE) && !reads_bins(MODE);
    double P[kGroup], k[kGroup];
    bool edge[kGroup];
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
        P[j] = (MODE != kHist) ? prob(ev[j].e, ev[j].f) : ev[j].e;
        edge[j] = false;
        k[j] = kComputeBins ? bin_floor_fast(ev[j].x, bc, edge[j]) : 0.0;
    }
    if (WRITE_P) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const uint32_t gj = g0 + j * kTileLanes;
            // streaming store (nt): P is not read again by this kernel, and
            // letting it allocate in L2 cost ~10 % of the kernel's time
            if (FULL || l + gj < n) store_p(arr, l, gj, P[j]);
        }
    }
    if (MODE == kReweight) return;
    bool any_edge = false;
#pragma unroll
    for (int j = 0; j < kGroup; ++j) any_edge |= edge[j];
    if (kComputeBins && __builtin_expect(any_edge, 0)) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (edge[j]) k[j] = bin_floor_exact(ev[j].x, bc);
    }
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
        if (FULL || l + g0 + j * kTileLanes < n) {
#pragma clang fp contract(off)
            const double cval = ev[j].w * P[j];            // rounded, never fused
            const int slot = reads_bins(MODE) ? int(ev[j].slot)
                                              : hslot(lds_bin(k[j], bc), lane & (kHistLanes - 1));
            add_in_lane_order(hist + slot, cval, lane);
        }
    }
}

// The kLaneEvents events of one lane of the tile whose arrays start at the
// tile's first event (n = the tile's events); the loads of group g + 1 are
// issued before group g is computed.  With ROLL the events run in a loop
// that is not unrolled (the last group reloads itself): about 6 KB of code
// instead of 60 KB and fewer live registers.  The callers choose it per
// kernel from measurements: rolled for the kernels that write P (both
// tiers) and for the batched kernel, fully unrolled for the kernels that
// write no P.
template <int MODE, bool WRITE_P, bool FULL, bool ROLL, class PROB>
__device__ __forceinline__ void tile_events(const PROB& prob, const BinConsts& bc, double* hist,
                                            int lane, uint32_t n, const double* e_true,
                                            const uint8_t* flags, const double* weight,
                                            const double* e_reco, const uint16_t* bins,
                                            const double* value, double* p_out)
{
    constexpr int kGroups = kLaneEvents / kGroup;
    const uint32_t l = uint32_t(lane);
    const TileBufs bufs = tile_bufs<MODE>(n, e_true, flags, weight, e_reco, bins, value, p_out);
    const auto load = [&](int m) {
        return load_event<MODE, FULL, PROB::kDecidesByWave>(bufs, l, m * kTileLanes, n);
    };
    if constexpr (ROLL) {
        EventIn cur[kGroup], nxt[kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) cur[j] = load(j);
#pragma unroll 1
        for (int g = 0; g < kGroups; ++g) {
            const int gn = g + 1 < kGroups ? g + 1 : g;   // the last group reloads itself
#pragma unroll
            for (int j = 0; j < kGroup; ++j) nxt[j] = load(gn * kGroup + j);
            tile_group<MODE, WRITE_P, FULL>(prob, bc, hist, lane, l, g * kGroup * kTileLanes, n,
                                            cur, bufs);
#pragma unroll
            for (int j = 0; j < kGroup; ++j) cur[j] = nxt[j];
        }
    } else {
        EventIn ev[kGroups][kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) ev[0][j] = load(j);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (g + 1 < kGroups) {
#pragma unroll
                for (int j = 0; j < kGroup; ++j) ev[g + 1][j] = load((g + 1) * kGroup + j);
            }
            tile_group<MODE, WRITE_P, FULL>(prob, bc, hist, lane, l, g * kGroup * kTileLanes,
                                            n, ev[g], bufs);
        }
    }
}

// The events of one tile of a binned sample under NS parameter sets, each with
// its own histogram (hist + k * stride): every event is loaded once for all of
// them (plain pointers, the next event's loads ahead).
template <bool MIXED, bool FULL, int NS>
__device__ __forceinline__ void tile_events_sets(const SetConsts* const (&sc)[NS],
                                                 const Tables<MIXED>* const (&T)[NS], double kA,
                                                 double kL, double* hist, int stride, int lane,
                                                 uint32_t n, const TilePtrs& arr)
{
    const uint32_t l = uint32_t(lane);
    EventIn cur = load_event<kPdfBinned, FULL>(arr, l, 0, n);
    MixedRegs regs[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
        regs[k] = NS > 1 ? MixedRegs::in_vgprs(*sc[k]) : MixedRegs::of(*sc[k]);
#pragma unroll 1
    for (int m = 0; m < kLaneEvents; ++m) {
        const uint32_t next = uint32_t(m + 1 < kLaneEvents ? m + 1 : m) * kTileLanes;
        const EventIn nxt = load_event<kPdfBinned, FULL>(arr, l, next, n);
        double P[NS];
        if constexpr (MIXED) {
            event_probs_mixed<NS>(sc, T, regs, kA, kL, cur.e, cur.f, P);
        } else {
#pragma unroll
            for (int k = 0; k < NS; ++k) P[k] = event_prob(*sc[k], *T[k], kA, kL, cur.e, cur.f);
        }
        if (FULL || l + uint32_t(m) * kTileLanes < n) {
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const double c = cur.w * P[k];   // an operand of an LDS addition: never fused
                add_in_lane_order(hist + k * stride + int(cur.slot), c, lane);
            }
        }
        cur = nxt;
    }
}

// A tile shared by the SPLIT waves of a workgroup: wave v computes events m =
// v K / SPLIT .. (v + 1) K / SPLIT - 1 of every lane (all their loads in flight
// at once), then the waves add their contributions one after the other, so
// that every accumulator still takes its additions in ascending m.  (Issuing
// the loads before the workgroup builds its tables delayed the tables: 16.2
// against 14.8 us at 2e6 events.)
template <int MODE, bool WRITE_P, int SPLIT, class PROB>
__device__ __forceinline__ void split_tile_events(const PROB& prob, const BinConsts& bc,
                                                  double* hist, const TileBufs& bufs, int wave,
                                                  int lane, uint32_t n)
{
    constexpr int kShare = kLaneEvents / SPLIT;
    constexpr bool kComputeBins = has_hist(MODE) && !reads_bins(MODE);
    const uint32_t l = uint32_t(lane);
    EventIn ev[kShare];
#pragma unroll
    for (int j = 0; j < kShare; ++j)
        ev[j] = load_event<MODE, false, PROB::kDecidesByWave>(
            bufs, l, uint32_t(wave * kShare + j) * kTileLanes, n);
    double c[kShare];
    int slot[kShare];
#pragma unroll
    for (int j = 0; j < kShare; ++j) {
        const uint32_t g0 = uint32_t(wave * kShare + j) * kTileLanes;
        const double P = (MODE != kHist) ? prob(ev[j].e, ev[j].f) : ev[j].e;
        if (WRITE_P && l + g0 < n) store_p(bufs, l, g0, P);
        c[j] = ev[j].w * P;   // only ever an operand of an LDS addition: never fused
        // the correctly rounded division at once: the short cut of
        // bin_floor_fast with its rare branch kept these arrays in scratch
        slot[j] = kComputeBins ? hslot(lds_bin(bin_floor_exact(ev[j].x, bc), bc),
                                       lane & (kHistLanes - 1))
                               : int(ev[j].slot);
    }
    if constexpr (has_hist(MODE)) {
#pragma unroll 1
        for (int v = 0; v < SPLIT; ++v) {
            if (v == wave) {
#pragma unroll
                for (int j = 0; j < kShare; ++j)
                    if (l + uint32_t(wave * kShare + j) * kTileLanes < n)
                        add_in_lane_order(hist + slot[j], c[j], lane);
            }
            __syncthreads();
        }
    }
}

// Tile of workgroup b of nb: workgroups are dispatched round-robin over the
// 8 XCDs (each with its own L2), so XCD x = b mod 8 is given the contiguous
// tile range that starts at x q + min(x, r) (q = nb / 8, r = nb mod 8); a
// bijection of [0, nb).  Neighbouring tiles then write their per-bin
// results into the same cache lines from one L2.
constexpr int64_t kXcds = 8;
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nb)
{
    const int64_t q = nb / kXcds, r = nb % kXcds, x = b % kXcds;
    return x * q + (x < r ? x : r) + b / kXcds;
}

// The arrays of one tile: the sample's arrays advanced to the tile's first
// event (absent arrays stay null) and the tile's event count.
struct TileArrays {
    const double* e_true;
    const uint8_t* flags;
    const double* weight;
    const double* e_reco;
    const uint16_t* bins;
    const double* value;
    double* p_out;
    uint32_t n;
};

__device__ __forceinline__ TileArrays tile_arrays(int64_t tile, int64_t n, const double* e_true,
                                                  const uint8_t* flags, const double* weight,
                                                  const double* e_reco, const uint16_t* bins,
                                                  const double* value, double* p_out)
{
    const int64_t t0 = tile * kTileEvents;
    TileArrays a;
    a.e_true = e_true ? e_true + t0 : nullptr;
    a.flags = flags ? flags + t0 : nullptr;
    a.weight = weight ? weight + t0 : nullptr;
    a.e_reco = e_reco ? e_reco + t0 : nullptr;
    a.bins = bins ? bins + t0 : nullptr;
    a.value = value ? value + t0 : nullptr;
    a.p_out = p_out ? p_out + t0 : nullptr;
    a.n = uint32_t(min(n - t0, int64_t(kTileEvents)));
    return a;
}

// Build the channel (and flag) tables of a parameter set in LDS (lanes 0-31
// of the block's first wave; the caller's barrier publishes them).
__device__ __forceinline__ void load_tab(const SetConsts& sc, TileTables& T, int lane)
{
    if (lane >= kFlagEntries) return;
    const uint32_t f = uint32_t(lane);
    const bool valid = (kValidFlags >> f) & 1u;
    const uint32_t a = f & 3u, b = (f >> 2) & 3u;
    const Chan c = sc.ch[valid ? 3u * b + a : 0u];
    const double re = valid ? 1.0 : 0.0, im = (f & 16u) ? -re : re;
    const int slot = lane + (lane >> 4);
    T.m[slot] = {re * c.m_re, im * c.m_im};
    T.m2[slot] = {re * c.m2_re, im * c.m2_im};
    T.g[slot] = {re * c.g_re, im * c.g_im};
    T.d[slot] = {re * c.dee, valid ? (a == b ? 1.0 : 0.0) : __builtin_nan("")};
}

__device__ __forceinline__ void load_tab(const LayerPath& lp, LayeredTables& T, int lane)
{
    if (lane < 20) {
        const int row = lane / 5, col = lane % 5;
        T.w[row][col] = row < 3 ? lp.tri.w[row][col] : __builtin_nan("");
    }
}

__device__ __forceinline__ void load_tab(const SetConsts& sc, TileTablesMixed& T, int lane)
{
    if (lane < kMixedChannels) {
        ChanF e;
        if (lane < kInvalidChannel) {
            const int k = lane % kChannels;
            const Chan c = sc.ch[k];
            const bool conj = lane >= kChannels;
            e.m_re = float(c.m_re);
            e.m_im = float(conj ? -c.m_im : c.m_im);
            e.m2_re = float(c.m2_re);
            e.m2_im = float(conj ? -c.m2_im : c.m2_im);
            e.g_re = float(c.g_re);
            e.g_im = float(conj ? -c.g_im : c.g_im);
            e.dee = float(c.dee);
            e.dba = (k % 3 == k / 3) ? 1.0f : 0.0f;
        } else {
            e.m_re = e.m_im = e.m2_re = e.m2_im = e.g_re = e.g_im = e.dee = 0.0f;
            e.dba = __builtin_nanf("");
        }
        T.ch[lane] = e;
    }
    if (lane < kMixedFlags) {
        const uint32_t f = uint32_t(lane);
        const bool valid = (kValidFlags >> f) & 1u;
        const uint32_t anti = (f >> 4) & 1u;
        const uint32_t entry =
            valid ? (f & 3u) + 3u * ((f >> 2) & 3u) + anti * uint32_t(kChannels)
                  : uint32_t(kInvalidChannel);
        T.flag[lane] = FlagInfo{entry * uint32_t(sizeof(ChanF)), valid && anti ? 0x80000000u : 0u};
    }
}

template <int THREADS = kTileLanes>
__device__ __forceinline__ void hist_zero(double* hist, int thread, int nbt)
{
    for (int i = thread; i < nbt * kHistLanes; i += THREADS) hist[i] = 0.0;
}

// Tree over the 64 lanes of every bin of a finished tile, written as row
// `row` of the tile results at `out` (chunked bin-major layout).
// With `only` it is the histogram itself, bin after bin.
template <int THREADS = kTileLanes>
__device__ __forceinline__ void tile_write(const double* hist, int thread, int nbt, int64_t row,
                                           double* out, bool only = false)
{
    for (int bin = thread; bin < nbt; bin += THREADS)
        out[only ? bin : partial_index(row, bin, nbt)] =
            lane_tree<kHistLanes, 0>(hist, lds_row_of_output(bin, nbt - 2));
}

// Adjacent-pair tree across the 64 lanes of a wave (xor butterfly: both
// partners of a pair form the same sum), result in every lane.
__device__ __forceinline__ double wave_tree(double v)
{
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) v = v + __shfl_xor(v, s, 64);
    return v;
}

// One merge level (see MergeLevel): block (gc, bin, set) reduces chunk gc
// of the set's input rows for one bin.  Thread t adds its ROWS contiguous
// rows (+0.0 beyond the sample's rows) as a binary tree in registers; the 64
// lanes of a wave meet in the butterfly tree and the block's waves in a last
// binary tree.
// The block's total is handed to emit(set, sample, chunk, bin, total) by
// thread 0.
template <int WAVES, int ROWS, class EMIT>
__device__ __forceinline__ void merge_level_block(const MergeLevel& L, const double* __restrict__ in,
                                                  EMIT&& emit)
{
    __shared__ double wave_sum[WAVES];
    const int nbt = L.nbt;
    const int bin = int(blockIdx.y);
    const int64_t gc = blockIdx.x, set = blockIdx.z;
    int s = 0;
    while (s + 1 < L.n_samples && gc >= L.chunk0[s + 1]) ++s;
    const int64_t c = gc - L.chunk0[s];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t first = c * (WAVES * 64 * ROWS) + int64_t(t) * ROWS;
    const int64_t count = L.rows[s] - first;
    const double* src = in + set * L.set_stride_in + partial_index(L.in_row0[s] + first, bin, nbt);
    double v[ROWS];
    if (count >= ROWS) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) v[i] = src[i];
    } else {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) v[i] = i < count ? src[i] : 0.0;
    }
#pragma unroll
    for (int w = ROWS / 2; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) v[i] = v[2 * i] + v[2 * i + 1];
    double total = wave_tree(v[0]);
    if constexpr (WAVES > 1) {
        if (lane == 0) wave_sum[wave] = total;
        __syncthreads();
        if (t == 0) {
            // binary tree over the waves' sums, in wave order
            double w[WAVES];
#pragma unroll
            for (int i = 0; i < WAVES; ++i) w[i] = wave_sum[i];
#pragma unroll
            for (int h = WAVES / 2; h >= 1; h >>= 1)
#pragma unroll
                for (int i = 0; i < h; ++i) w[i] = w[2 * i] + w[2 * i + 1];
            total = w[0];
        }
    }
    if (t == 0) emit(set, s, c, bin, total);
}

// -2 ln L of one histogram by a whole wave: 2 sum_b (mu_b - d_b ln mu_b +
// lgamma(d_b + 1)), mu_b = scale hist_b.  Lane l adds bins l, l + 64, ... in
// ascending order, then the lanes meet in the wave's butterfly tree (a fixed
// order).  mu(b) gives hist_b.
template <class MU>
__device__ __forceinline__ double poisson_nll(MU&& mu, const double* __restrict__ d, double scale,
                                              int nbins, int lane)
{
    double acc = 0.0;
    for (int b = lane; b < nbins; b += 64) {
        const double m = scale * mu(b), x = d[b];
        const double term = m == 0.0 ? (x == 0.0 ? 0.0 : __builtin_inf())
                                     : m - x * log(m) + lgamma(x + 1.0);
        acc = acc + term;
    }
    return 2.0 * wave_tree(acc);
}

}  // namespace dev
}  // namespace osc
