"""The FP64 tier's accuracy statement (include/osc.h, osc_reweight) checked
over random configurations: parameter sets near the measured values and
with arbitrary angles and either mass ordering, baselines 0-13000 km,
densities 0 or 0.5-13 g/cm^3, every channel of neutrinos and
antineutrinos, E log-uniform on [0.05, 100] GeV.

Per event the bound is 1e-12 + 4 u phi (1 + spread / gap) + u |A| / gap
(u = 2^-53, phi the largest phase difference, spread and gap the largest
and smallest distances between the eigenvalues of M): the FP64 rounding of
a phase of phi radians, amplified by the conditioning of the eigenvalues,
and the amplitude's cancellation at large matter terms.  The oracle carries
the same rounding, so the bound covers both sides."""
import math

import numpy as np
import pytest

import oracle
from paper_1311_7579_amd import workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U53 = 2.0 ** -53


@pytest.fixture(scope="module")
def osc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1311_7579_amd import osc as _osc
    _osc.load()
    return _osc


@pytest.fixture(scope="module")
def ctx(osc):
    c = osc.Context(0)
    yield c
    c.close()


def eigen_spread_gap(p, A, anti):
    m2 = np.array([0.0, p["dm2_21"], p["dm2_21"] + p["dm2_32"]])
    lam = np.empty((A.size, 3))
    for a in (0, 1):
        U = oracle.pmns(p, anti=bool(a))
        H = (U * m2) @ U.conj().T
        sel = anti == a
        M = np.broadcast_to(H, (int(sel.sum()), 3, 3)).copy()
        M[:, 0, 0] += A[sel]
        lam[sel] = np.linalg.eigvalsh(M)
    return lam[:, 2] - lam[:, 0], np.min(np.diff(lam, axis=1), axis=1)


def fp64_bound(p, L, rho, ye, e, f):
    """The FP64 tier's per-event error bound (module docstring)."""
    anti = (f >> 4) & 1
    A = oracle.k_matter() * ye * rho * e * np.where(anti == 1, -1.0, 1.0)
    spread, gap = eigen_spread_gap(p, A, anti)
    phase = oracle.k_phase() * spread * L / e
    return 1e-12 + 4 * U53 * phase * (1.0 + spread / gap) + U53 * np.abs(A) / gap


@pytest.mark.parametrize("seed", [7, 11])
def test_random_configurations_within_bound(osc, ctx, seed):
    rng = np.random.default_rng(seed)
    n = 100_000
    worst = 0.0
    for k in range(60):
        seed_k = int(rng.integers(1 << 30))
        p = (workload.make_param_sets(1, seed_k)[0] if k % 2 == 0
             else workload.make_random_physics_sets(1, seed_k)[0])
        L = float(rng.uniform(0.0, 13000.0))
        rho = float(rng.choice([0.0, rng.uniform(0.5, 13.0)]))
        ye = float(rng.uniform(0.45, 0.5))
        e = 10 ** rng.uniform(math.log10(0.05), 2.0, n)
        f = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), rng.random(n) < 0.5)
        s = workload.Sample(e, f, np.ones(n), e.copy(), L_km=L, rho_gcc=rho, Ye=ye)
        ctx.osc_set_params([p])
        ds = osc.DeviceSample.from_host(s)
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        ctx.osc_reweight(ds, 0, out)
        got = out.cpu().numpy()
        want = oracle.prob_batch(p, L, rho, ye, e, f)
        ratio = np.abs(got - want) / fp64_bound(p, L, rho, ye, e, f)
        assert ratio.max() <= 1.0, (k, p, L, rho, float(ratio.max()))
        worst = max(worst, float(ratio.max()))
    print(f"worst error / bound over 60 configurations: {worst:.3g}")


def test_near_level_crossings_within_bound(osc, ctx):
    """Matter terms where two eigenvalues come within 0.1-3 % of the
    spread (level crossings of sets with arbitrary angles, and large |A|
    for near-measured sets): there the FP32 seeds are coarsest relative to
    the smallest root distance, and below about 0.85 % the roots need
    their second refinement step.  Such matter terms are found on a fine
    grid of A, events are drawn around them and sorted by A (so that waves
    fall on either side of that threshold, and near it), and every event
    must stay within the FP64 bound, at a short baseline (small phases, so
    the bound is about 1e-12) and a long one."""
    rng = np.random.default_rng(21)
    rho, ye = 13.0, 0.5
    ka = oracle.k_matter() * ye * rho
    sets = ([(workload.make_random_physics_sets(1, sd)[0], 0.1)
             for sd in (1050, 1079, 31, 33, 35, 40, 44, 47)]
            + [(workload.make_param_sets(1, sd)[0], 1.0) for sd in (35, 36)])
    n = 20_000
    checked = 0
    for p, a_max in sets:
        grid = np.linspace(-a_max, a_max, 100_001)
        grid = grid[grid != 0.0]
        spread, gap = eigen_spread_gap(p, grid, (grid < 0).astype(np.int64))
        band = grid[(gap / spread >= 1e-3) & (gap / spread <= 3e-2)]
        if band.size == 0:
            continue
        step = grid[1] - grid[0]
        A = np.sort(rng.choice(band, n) + rng.uniform(-0.5, 0.5, n) * step)
        e = np.abs(A) / ka
        f = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), A < 0)
        for L in (300.0, 6000.0):
            s = workload.Sample(e, f, np.ones(n), e.copy(), L_km=L, rho_gcc=rho, Ye=ye)
            ctx.osc_set_params([p])
            ds = osc.DeviceSample.from_host(s)
            out = torch.empty(n, dtype=torch.float64, device="cuda")
            ctx.osc_reweight(ds, 0, out)
            got = out.cpu().numpy()
            want = oracle.prob_batch(p, L, rho, ye, e, f)
            ratio = np.abs(got - want) / fp64_bound(p, L, rho, ye, e, f)
            assert ratio.max() <= 1.0, (p, L, float(ratio.max()))
        checked += 1
    assert checked == len(sets)


@pytest.mark.parametrize("ordering", [1, -1], ids=["normal", "inverted"])
def test_equally_spaced_eigenvalues(osc, ctx, ordering):
    """Where the middle eigenvalue lies halfway between the others, the
    eigenvalue that the solver treats as isolated changes from the highest to
    the lowest.  Events at matter terms within 1e-12..1e-1 relative of such
    points, on both sides, stay within the FP64 bound in every channel."""
    p = dict(workload.TABLE1, dm2_32=ordering * workload.TABLE1["dm2_32"], delta_cp=0.7)
    rho, ye = 3.0, 0.5
    U = oracle.pmns(p)
    H = (U * np.array([0.0, p["dm2_21"], p["dm2_21"] + p["dm2_32"]])) @ U.conj().T
    lopsided = lambda A: np.dot(np.linalg.eigvalsh(H + np.diag([A, 0, 0])), [1.0, -2.0, 1.0])
    grid = np.concatenate([-np.geomspace(1e-1, 1e-6, 2001), np.geomspace(1e-6, 1e-1, 2001)])
    f = np.array([lopsided(A) for A in grid])
    roots = []
    for k in np.nonzero(np.sign(f[1:]) != np.sign(f[:-1]))[0]:
        lo, hi = grid[k], grid[k + 1]
        if lo * hi < 0:
            continue
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if np.sign(lopsided(mid)) == np.sign(lopsided(lo)) else (lo, mid)
        roots.append(lo)
    assert roots
    rng = np.random.default_rng(17)
    n = 4000
    ctx.osc_set_params([p])
    for a0 in roots:
        A = a0 * (1 + 10 ** rng.uniform(-12, -1, n) * np.where(rng.random(n) < 0.5, -1, 1))
        e = np.abs(A) / (oracle.k_matter() * ye * rho)
        fl = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), A < 0)
        for L in (295.0, 2500.0):
            ds = osc.DeviceSample.from_host(
                workload.Sample(e, fl, np.ones(n), e.copy(), L_km=L, rho_gcc=rho, Ye=ye))
            out = torch.empty(n, dtype=torch.float64, device="cuda")
            ctx.osc_reweight(ds, 0, out)
            want = oracle.prob_batch(p, L, rho, ye, e, fl)
            ratio = np.abs(out.cpu().numpy() - want) / fp64_bound(p, L, rho, ye, e, fl)
            assert ratio.max() <= 1.0, (a0, L, float(ratio.max()))


def brute_force_prob(p, L, rho, ye, e, f):
    """P from an eigendecomposition of the flavour-basis matrix (numpy
    eigh, accurate however close the eigenvalues are)."""
    anti = (f >> 4) & 1
    a, b = f & 3, (f >> 2) & 3
    out = np.empty(e.size)
    m2 = np.array([0.0, p["dm2_21"], p["dm2_21"] + p["dm2_32"]])
    for s in (0, 1):
        sel = np.nonzero(anti == s)[0]
        if sel.size == 0:
            continue
        U = oracle.pmns(p, anti=bool(s))
        H = (U * m2) @ U.conj().T
        M = np.broadcast_to(H, (sel.size, 3, 3)).copy()
        M[:, 0, 0] += oracle.k_matter() * ye * rho * e[sel] * (-1.0 if s else 1.0)
        lam, V = np.linalg.eigh(M)
        ph = np.exp(-1j * oracle.k_phase() * L * lam / e[sel][:, None])
        amp = np.einsum("nk,nk,nk->n", V[np.arange(sel.size), b[sel], :], ph,
                        V[np.arange(sel.size), a[sel], :].conj())
        out[sel] = np.abs(amp) ** 2
    return out


@pytest.mark.parametrize("angles", [(0.0, 0.311), (0.0251, 0.0)], ids=["th13=0", "th12=0"])
def test_exact_level_crossings(osc, ctx, angles):
    """A zero mixing angle decouples a mass state from nu_e, and its
    eigenvalue then crosses another one exactly at one matter term.  The
    analytic method cannot resolve eigenvalues that close (the oracle, which
    follows it, gives NaN or errors up to ~1e-3 there), so the reference is
    a brute-force eigendecomposition.  Events are drawn at relative
    distances 1e-12..1e-1 from the crossing: the FP64 and layered paths give
    NaN only where the two closest eigenvalues are within 1e-3 of the
    spread, and elsewhere stay within the stated bound; the FP32-mixed tier
    gives NaN on the same events and stays within 3e-4 elsewhere (its FP32
    projector numerators cancel next to a crossing)."""
    s13, s12 = angles
    p = dict(workload.TABLE1, sin2_th13=s13, sin2_th12=s12)
    rho, ye = 13.0, 0.5
    grid = np.linspace(1e-5, 0.05, 400_001)
    spread_g, gap_g = eigen_spread_gap(p, grid, np.zeros(grid.size, dtype=np.int64))
    a_cross = grid[int(np.argmin(gap_g / spread_g))]
    rng = np.random.default_rng(13)
    n = 20_000
    A = np.sort(a_cross * (1 + 10 ** rng.uniform(-12, -1, n) * np.where(rng.random(n) < 0.5, -1, 1)))
    e = A / (oracle.k_matter() * ye * rho)
    f = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), np.zeros(n, bool))
    spread, gap = eigen_spread_gap(p, A, np.zeros(n, dtype=np.int64))
    ctx.osc_set_params([p])
    try:
        for L in (300.0, 6000.0):
            s = workload.Sample(e, f, np.ones(n), e.copy(), L_km=L, rho_gcc=rho, Ye=ye)
            ds = osc.DeviceSample.from_host(s)
            want = brute_force_prob(p, L, rho, ye, e, f)
            bound = fp64_bound(p, L, rho, ye, e, f)
            h = torch.empty(52, dtype=torch.float64, device="cuda")
            results = {}
            for tier in ("fp64", "layered", "mixed"):
                out = torch.empty(n, dtype=torch.float64, device="cuda")
                if tier == "fp64":
                    ctx.osc_reweight(ds, 0, out)
                elif tier == "layered":
                    ctx.osc_reweight_layered(ds, [(L, rho, ye)], 0, out)
                else:
                    ctx.osc_fill_pdf(ds, 0, 50, 0.0, 3.0, h, out, precision=osc.OSC_FP32_MIXED)
                results[tier] = out.cpu().numpy()
            nan = np.isnan(results["fp64"])
            assert nan.any() and (~nan).any()
            assert (gap / spread)[nan].max() < 1e-3, (L, float((gap / spread)[nan].max()))
            for tier, got in results.items():
                np.testing.assert_array_equal(np.isnan(got), nan, err_msg=tier)
                d = np.abs(got[~nan] - want[~nan])
                if tier == "mixed":
                    assert d.max() <= 3e-4, (L, tier, float(d.max()))
                else:
                    assert (d / bound[~nan]).max() <= 1.0, (L, tier, float((d / bound[~nan]).max()))
    finally:
        ctx.osc_set_params([workload.TABLE1])


def test_mixed_tier_envelope(osc, ctx):
    """The FP32-mixed tier over the same random domain stays within the
    envelope the header states: about 5e-5 at worst (arbitrary angles,
    long L/E near the solar resonance), checked with a factor 3 of margin,
    and within
    4e-5 wherever E <= 20 GeV, rho <= 3 g/cm^3 and L <= 2500 km."""
    rng = np.random.default_rng(5)
    n = 100_000
    h = torch.empty(52, dtype=torch.float64, device="cuda")
    for k in range(60):
        seed_k = int(rng.integers(1 << 30))
        p = (workload.make_param_sets(1, seed_k)[0] if k % 2 == 0
             else workload.make_random_physics_sets(1, seed_k)[0])
        L = float(rng.uniform(0.0, 13000.0))
        rho = float(rng.choice([0.0, rng.uniform(0.5, 13.0)]))
        ye = float(rng.uniform(0.45, 0.5))
        e = 10 ** rng.uniform(math.log10(0.05), 2.0, n)
        f = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), rng.random(n) < 0.5)
        s = workload.Sample(e, f, np.ones(n), e.copy(), L_km=L, rho_gcc=rho, Ye=ye)
        ctx.osc_set_params([p])
        ds = osc.DeviceSample.from_host(s)
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        ctx.osc_fill_pdf(ds, 0, 50, 0.0, 3.0, h, out, precision=osc.OSC_FP32_MIXED)
        d = np.abs(out.cpu().numpy() - oracle.prob_batch(p, L, rho, ye, e, f))
        assert d.max() <= 1.5e-4, (k, p, L, rho, float(d.max()))
        if rho <= 3.0 and L <= 2500.0:
            assert d[e <= 20.0].max() <= 4e-5, (k, p, L, rho, float(d[e <= 20.0].max()))


@pytest.mark.parametrize("precision", [0, 1])
def test_energies_far_from_one(osc, ctx, precision):
    """Energies whose square is outside FP64: without matter a phase of (next
    to) zero leaves every flavour as it is, at any energy above, and over no
    distance at any energy below."""
    p = [workload.TABLE1, dict(workload.TABLE1, dm2_32=-2.4e-3, delta_cp=1.1)]
    ctx.osc_set_params(p)
    for L, e in ((295.0, (1e100, 1e155, 1e200, 1e290)), (0.0, (1e-100, 1e-155, 1e-200, 1e-280))):
        ev = [(x, a, b, anti) for x in e for a in range(3) for b in range(3) for anti in (0, 1)]
        e_true = np.array([v[0] for v in ev])
        a, b, anti = (np.array([v[k] for v in ev]) for k in (1, 2, 3))
        s = workload.Sample(e_true, workload.make_flags(a, b, anti), np.ones(len(ev)),
                            np.ones(len(ev)), L_km=L, rho_gcc=0.0, Ye=0.5)
        ds = osc.DeviceSample.from_host(s)
        h = torch.empty(3, dtype=torch.float64, device="cuda")
        out = torch.empty(len(ev), dtype=torch.float64, device="cuda")
        for k in range(len(p)):
            ctx.osc_fill_pdf(ds, k, 1, 0.0, 2.0, h, out, precision=precision)
            assert np.abs(out.cpu().numpy() - (a == b)).max() <= (1e-12, 3e-6)[precision]
