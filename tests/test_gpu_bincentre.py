"""GPU parity of the bin-centre reweighting (Sec. 1.1.1) through the C ABI.

  * the migration template: bit-exact against the oracle (each cell's
    weights are added in ascending event order on both sides);
  * P at the true-bin centres: 1e-12 absolute against the oracle;
  * the PDF: bit-exact against the oracle's contraction applied to the
    GPU's own centre probabilities, and within the P tolerance carried
    through the template against the oracle's PDF;
  * the binning effect of Sec. 1.1.1 (a 25 MeV bin at 0.600-0.625 GeV):
    event-by-event against bin-centre, GPU against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1311_7579_amd import workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P_TOL = 1e-12


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
    c.osc_set_params([workload.TABLE1] + workload.make_param_sets(3, 3))
    yield c
    c.close()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def mixed_sample(n, seed, L=810.0, rho=2.84):
    """Every channel, 3 % invalid flag bytes, energies partly outside the
    true binning, integer and fractional weights."""
    rng = np.random.default_rng(seed)
    e = 10 ** rng.uniform(-1.3, 1.1, n)
    f = workload.make_flags(rng.integers(0, 3, n), rng.integers(0, 3, n), rng.random(n) < 0.25)
    bad = rng.random(n) < 0.03
    f[bad] = rng.choice(np.array([3, 7, 13, 44, 255], np.uint8), bad.sum())
    w = rng.uniform(0.5, 1.5, n)
    x = np.maximum(e * rng.normal(1.0, 0.12, n), 1e-12)
    return workload.Sample(e, f, w, x, L_km=L, rho_gcc=rho)


def run_bincentre(osc, ctx, s, nt, lo_t, hi_t, nr, lo_r, hi_r, set_index=0, e_scale=0.0):
    ds = osc.DeviceSample.from_host(s)
    tp = osc.Template(ctx, ds, nt, lo_t, hi_t, nr, lo_r, hi_r, e_scale=e_scale)
    try:
        h = torch.full((nr + 2,), -1.0, dtype=torch.float64, device="cuda")
        P = torch.full((18, nt), -1.0, dtype=torch.float64, device="cuda")
        tp.fill_pdf(set_index, h, P)
        return tp.n_used, host(tp.copy()), host(P), host(h)
    finally:
        tp.close()


@pytest.mark.parametrize("n,nt,nr", [(0, 8, 5), (1, 8, 5), (777, 40, 20), (300_000, 100, 50)])
def test_template_and_pdf_against_oracle(osc, ctx, n, nt, nr):
    s = mixed_sample(n, 11 + n)
    lo_t, hi_t, lo_r, hi_r = 0.1, 6.1, 0.0, 5.0
    used, T, P, h = run_bincentre(osc, ctx, s, nt, lo_t, hi_t, nr, lo_r, hi_r)
    T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, nt, lo_t, hi_t,
                                  nr, lo_r, hi_r)
    assert used == used_o
    np.testing.assert_array_equal(T, T_o)
    P_o = oracle.centre_probs(workload.TABLE1, s.L_km, s.rho_gcc, s.Ye, nt, lo_t, hi_t)
    assert np.abs(P - P_o).max() <= P_TOL
    np.testing.assert_array_equal(h, oracle.bincentre_contract(T, P))
    h_o = oracle.bincentre_contract(T_o, P_o)
    tol = P_TOL * T_o.reshape(nr + 2, -1).sum(axis=1) + 1e-15 * np.abs(h_o)
    assert np.all(np.abs(h - h_o) <= tol)


def hard_weights(kind, n):
    """Weights whose sum in order is easy to get wrong in blocks."""
    rng = np.random.default_rng(4)
    w = rng.uniform(0.5, 1.5, n)
    if kind == "ties":            # every third value halfway between two sums
        w[::3] = 2.0 ** -40 * (2 * rng.integers(0, 1 << 20, w[::3].size) + 1)
    elif kind == "signs":
        w *= np.where(rng.random(n) < 0.3, -1.0, 1.0)
    elif kind == "binades":       # 80 orders of magnitude, ascending
        w = np.sort(10.0 ** rng.uniform(-40, 40, n))
    elif kind == "special":
        w[n // 2], w[n // 3] = np.inf, 0.0
        w[n // 5] = -0.0
    elif kind == "nan":
        w[n // 2] = np.nan
    elif kind == "tiny":          # subnormal sums
        w *= 2.0 ** -1074 * 1000
    elif kind == "huge":          # overflows to infinity
        w *= 2.0 ** 1022
    elif kind == "ones":
        w[:] = 1.0
    return w


@pytest.mark.parametrize("kind", ["plain", "ones", "ties", "signs", "binades", "special", "nan",
                                  "tiny", "huge"])
@pytest.mark.parametrize("n", [31, 32, 33, 65, 1024, 1025, 16384, 16385, 70_001])
def test_cell_sums_are_the_sums_in_order(osc, ctx, kind, n):
    """All events in one cell: the template's entry has the bits of adding
    the weights one after the other (rows added by a lane, a wave and a
    workgroup, whole and ragged blocks)."""
    w = hard_weights(kind, n)
    e = np.full(n, 0.6)
    s = workload.Sample(e, workload.make_flags(np.ones(n, int), np.ones(n, int),
                                               np.zeros(n, bool)), w, e.copy())
    tp = osc.Template(ctx, osc.DeviceSample.from_host(s), 1, 0.5, 1.0, 1, 0.5, 1.0)
    try:
        got = host(tp.copy())[0, 4, 0]
    finally:
        tp.close()
    with np.errstate(all="ignore"):
        want = np.add.accumulate(np.concatenate([[0.0], w]))[-1]
    assert tp.n_used == n
    assert np.array_equal(np.array([got]).view(np.uint64), np.array([want]).view(np.uint64)) or (
        np.isnan(got) and np.isnan(want)), (got, want)


def test_energy_scale_and_other_sets(osc, ctx):
    s = mixed_sample(50_000, 5, L=1300.0, rho=3.0)
    for k, e_scale in ((1, 0.02), (2, -0.015), (3, 0.0)):
        used, T, P, h = run_bincentre(osc, ctx, s, 64, 0.05, 12.85, 30, 0.0, 6.0, set_index=k,
                                      e_scale=e_scale)
        T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, 64, 0.05, 12.85,
                                      30, 0.0, 6.0, e_scale)
        np.testing.assert_array_equal(T, T_o)
        p = (workload.TABLE1 if k == 0 else workload.make_param_sets(3, 3)[k - 1])
        P_o = oracle.centre_probs(p, s.L_km, s.rho_gcc, s.Ye, 64, 0.05, 12.85)
        assert np.abs(P - P_o).max() <= P_TOL
        np.testing.assert_array_equal(h, oracle.bincentre_contract(T, P))


def test_internal_table_and_determinism(osc, ctx):
    s = mixed_sample(20_000, 9)
    ds = osc.DeviceSample.from_host(s)
    tp = osc.Template(ctx, ds, 50, 0.1, 5.1, 25, 0.0, 5.0)
    try:
        h1 = torch.empty(27, dtype=torch.float64, device="cuda")
        h2 = torch.empty(27, dtype=torch.float64, device="cuda")
        P = torch.empty((18, 50), dtype=torch.float64, device="cuda")
        tp.fill_pdf(0, h1)
        tp.fill_pdf(0, h2, P)
        a, b = host(h1), host(h2)
        np.testing.assert_array_equal(a, b)
        tp2 = osc.Template(ctx, ds, 50, 0.1, 5.1, 25, 0.0, 5.0)
        np.testing.assert_array_equal(host(tp.copy()), host(tp2.copy()))
        tp2.close()
    finally:
        tp.close()


def test_invalid_arguments(osc, ctx):
    s = mixed_sample(100, 1)
    ds = osc.DeviceSample.from_host(s)
    bad = [dict(nt=0, lo_t=0.1, hi_t=1.0), dict(nt=10, lo_t=-0.1, hi_t=1.0),
           dict(nt=10, lo_t=1.0, hi_t=1.0), dict(nt=70000, lo_t=0.1, hi_t=1.0)]
    for b in bad:
        with pytest.raises(osc.OscError):
            osc.Template(ctx, ds, b["nt"], b["lo_t"], b["hi_t"], 10, 0.0, 1.0)
    with pytest.raises(osc.OscError):
        osc.Template(ctx, ds, 10, 0.1, 1.0, 0, 0.0, 1.0)
    tp = osc.Template(ctx, ds, 10, 0.1, 1.0, 10, 0.0, 1.0)
    try:
        h = torch.empty(12, dtype=torch.float64, device="cuda")
        with pytest.raises(osc.OscError):
            tp.fill_pdf(99, h)
    finally:
        tp.close()


def test_binning_effect_against_oracle(osc, ctx):
    """Sec. 1.1.1: one 25 MeV true bin at 0.600-0.625 GeV, nu_mu -> nu_mu at
    295 km, flat flux (events at the midpoints of 200000 equal slices).
    Event-by-event: osc_fill_pdf with the reco energy equal to the true one
    and that single bin.  Bin-centre: the template path."""
    n = 200_000
    e = 0.600 + (np.arange(n) + 0.5) * (0.025 / n)
    f = workload.make_flags(np.ones(n, int), np.ones(n, int), np.zeros(n, bool))
    s = workload.Sample(e, f, np.ones(n), e.copy(), L_km=295.0, rho_gcc=2.6)
    ds = osc.DeviceSample.from_host(s)
    h = torch.empty(3, dtype=torch.float64, device="cuda")
    ctx.osc_fill_pdf(ds, 0, 1, 0.600, 0.625, h)
    ebe = host(h)[0]
    used, T, P, hb = run_bincentre(osc, ctx, s, 1, 0.600, 0.625, 1, 0.600, 0.625)
    assert used == n
    bc = hb[0]
    effect = ebe / bc - 1.0
    P_o = oracle.prob_batch(workload.TABLE1, 295.0, 2.6, 0.5, e, f)
    ebe_o = float(np.sum(P_o))
    bc_o = n * oracle.prob(workload.TABLE1, 295.0, 2.6, 0.5, 0.6125, 1, 1, 0)
    assert ebe == pytest.approx(ebe_o, rel=1e-10)
    assert bc == pytest.approx(bc_o, rel=1e-10)
    assert effect == pytest.approx(ebe_o / bc_o - 1.0, abs=1e-9)
    assert 0.02 < effect < 0.05


def test_full_size_template(osc, ctx):
    """The 1e7-event workload: 200 true bins on [0.1, 10.1] GeV, 50 reco
    bins on [0, 3] GeV."""
    s = workload.make_sample(10_000_000, 1)
    used, T, P, h = run_bincentre(osc, ctx, s, 200, 0.1, 10.1, 50, 0.0, 3.0)
    T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, 200, 0.1, 10.1,
                                  50, 0.0, 3.0)
    assert used == used_o
    np.testing.assert_array_equal(T, T_o)
    np.testing.assert_array_equal(h, oracle.bincentre_contract(T, P))
    P_o = oracle.centre_probs(workload.TABLE1, s.L_km, s.rho_gcc, s.Ye, 200, 0.1, 10.1)
    assert np.abs(P - P_o).max() <= P_TOL


@pytest.mark.parametrize("nt", [2, 3, 28, 29, 227, 228, 455, 456, 2731])
def test_contraction_rounds(osc, ctx, nt):
    """Both sides of one and two rounds of terms (4096 each), of one group of
    rows (512) and of the first rows, and many rounds: the fixed order's bits,
    with NaN and infinite terms of a bad event kept in their own bin."""
    s = mixed_sample(20_000, 5 + nt)
    s.weight[::500] = np.inf
    used, T, P, h = run_bincentre(osc, ctx, s, nt, 0.1, 6.1, 4, 0.0, 5.0)
    np.testing.assert_array_equal(h, oracle.bincentre_contract(T, P))


@pytest.mark.parametrize("nt,lengths", [(5, (8191, 8192, 8193, 16385, 0)),
                                        (530, (8193,)),               # more than the workgroups
                                        (5000, (33, 0, 32, 64, 1100)),
                                        (40_000, (1, 31, 0, 34))])
def test_cells_listed_by_length(osc, ctx, nt, lengths):
    """Short, middling and long cells next to one another, and more of a kind
    than there are waves or workgroups to add them: every entry has the bits
    of adding its weights in event order."""
    cell = np.repeat(np.arange(nt), np.resize(lengths, nt))
    rng = np.random.default_rng(nt)
    rng.shuffle(cell)
    w = rng.uniform(0.5, 1.5, cell.size)
    w[::5] = 2.0 ** -40 * (2 * rng.integers(0, 1 << 20, w[::5].size) + 1)   # ties
    e = 1.0 + (cell + 0.5) / nt
    flags = workload.make_flags(np.ones(cell.size, int), np.ones(cell.size, int),
                                np.zeros(cell.size, bool))
    s = workload.Sample(e, flags, w, e.copy())
    used, T, P, h = run_bincentre(osc, ctx, s, nt, 1.0, 2.0, 1, 0.0, 3.0)
    T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, nt, 1.0, 2.0, 1, 0.0, 3.0)
    assert used == used_o == cell.size
    np.testing.assert_array_equal(T, T_o)


@pytest.mark.parametrize("nt,nr", [(200, 50), (333, 120)])     # keys of 18 and 20 bits
@pytest.mark.parametrize("n", [1 << 18, (1 << 18) + 1, 1 << 20, (1 << 20) + 1])
def test_sorts_by_size_and_key_width(osc, ctx, n, nt, nr):
    """Both sides of every size at which the sort of the cells changes: the
    template's bits, event order kept within every cell."""
    s = mixed_sample(n, 3)
    used, T, P, h = run_bincentre(osc, ctx, s, nt, 0.1, 6.1, nr, 0.0, 5.0)
    T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, nt, 0.1, 6.1, nr, 0.0, 5.0)
    assert used == used_o
    np.testing.assert_array_equal(T, T_o)


@pytest.mark.parametrize("nt,nr,bits", [(1, 20, 9), (20_000, 90, 25), (20_000, 100, 26),
                                        (40_000, 100, 27)])
def test_sorts_of_every_key_width_that_saves_a_pass(osc, ctx, nt, nr, bits):
    """Above 2^20 events keys of 9, and of 25 to 27 bits, also take 9 bits a
    pass: the template's bits, event order kept within every cell."""
    assert ((nr + 2) * 18 * nt).bit_length() == bits
    s = mixed_sample((1 << 20) + 1, 3)
    tp = osc.Template(ctx, osc.DeviceSample.from_host(s), nt, 0.1, 6.1, nr, 0.0, 5.0)
    try:
        T, used = host(tp.copy()), tp.n_used
    finally:
        tp.close()
    T_o, used_o = oracle.template(s.e_true, s.flags, s.weight, s.e_reco, nt, 0.1, 6.1, nr, 0.0, 5.0)
    assert used == used_o
    assert np.array_equal(T.reshape(-1), T_o.reshape(-1))
