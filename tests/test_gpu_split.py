"""A tile shared by several waves (one, four or eight, by the number of tiles)
gives the bits of the reduction contract: sizes on both sides of every rule,
whole and ragged last tiles, every form that takes a histogram."""
import numpy as np
import pytest

import oracle
from helpers import P_TOL, assert_bits_equal
from paper_1311_7579_amd import workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NB, HI = 37, 4.0
TILE = 1024


@pytest.fixture(scope="module")
def osc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1311_7579_amd import osc as _osc
    _osc.load()
    return _osc


def hist_of(s, P, hist):
    """hist has the bits of the contract on this P."""
    bins = oracle.bin_indices(s.e_reco, 0.0, HI, NB)
    assert_bits_equal(hist.cpu().numpy(), oracle.hist_contract(s.weight * P, bins, NB + 2))


@pytest.mark.parametrize("n", [1, 64, 257, TILE, TILE + 1, 768 * TILE, 768 * TILE + 1,
                               2048 * TILE, 2048 * TILE + 65, 6144 * TILE, 6144 * TILE + 1])
def test_constant_density_splits(osc, n):
    s = workload.make_sample(n, 5)
    s.flags[::97] = 15                      # invalid bytes: NaN in their bins
    with osc.Context(0) as ctx:
        ctx.osc_set_params([workload.TABLE1])
        ds = osc.DeviceSample.from_host(s)
        new = lambda m: torch.empty(m, dtype=torch.float64, device="cuda")
        p0 = new(n)
        ctx.osc_reweight(ds, 0, p0)
        P = p0.cpu().numpy()
        few = np.arange(0, n, max(1, n // 20000))
        want = oracle.prob_batch(workload.TABLE1, s.L_km, s.rho_gcc, s.Ye, s.e_true[few],
                                 s.flags[few])
        ok = s.flags[few] != 15
        assert np.isnan(P[few][~ok]).all()
        assert np.abs(P[few] - want)[ok].max(initial=0.0) <= P_TOL
        value = new(n).copy_(torch.from_numpy(np.nan_to_num(P)))
        h = new(NB + 2)
        ctx.osc_fill_hist(value, ds.weight, ds.e_reco, NB, 0.0, HI, h)
        hist_of(s, np.nan_to_num(P), h)
        with ctx.osc_binned_create(ds, NB, 0.0, HI) as binned:
            for tier in (osc.OSC_FP64, osc.OSC_FP32_MIXED):
                p, h1 = new(n), new(NB + 2)
                ctx.osc_fill_pdf(ds, 0, NB, 0.0, HI, h1, p, precision=tier)
                if tier == osc.OSC_FP64:
                    assert_bits_equal(p.cpu().numpy(), P)
                hist_of(s, p.cpu().numpy(), h1)
                for fill in (lambda q: ctx.osc_fill_pdf(ds, 0, NB, 0.0, HI, h, q, precision=tier),
                             lambda q: ctx.osc_fill_pdf_binned(binned, 0, h, q, precision=tier)):
                    q = new(n)
                    for out in (None, q):
                        fill(out)
                        assert_bits_equal(h.cpu().numpy(), h1.cpu().numpy())
                    assert_bits_equal(q.cpu().numpy(), p.cpu().numpy())


@pytest.mark.parametrize("n", [1, 257, TILE + 1, 4096 * TILE, 4096 * TILE + 3])
def test_layered_splits(osc, n):
    s = workload.make_sample(n, 6)
    s.flags[::89] = 32
    path = [(500.0, 3.0, 0.5), (1200.0, 5.0, 0.49), (300.0, 4.0, 0.5)]
    with osc.Context(0) as ctx:
        ctx.osc_set_params([workload.TABLE1])
        ds = osc.DeviceSample.from_host(s)
        new = lambda m: torch.empty(m, dtype=torch.float64, device="cuda")
        p0, p1, h0, h1 = new(n), new(n), new(NB + 2), new(NB + 2)
        ctx.osc_reweight_layered(ds, path, 0, p0)
        ctx.osc_fill_pdf_layered(ds, path, 0, NB, 0.0, HI, h0, p1)
        ctx.osc_fill_pdf_layered(ds, path, 0, NB, 0.0, HI, h1)
        P = p0.cpu().numpy()
        few = np.nonzero(s.flags != 32)[0][::max(1, n // 5000)]
        want = oracle.prob_layered_batch(workload.TABLE1, path, s.e_true[few], s.flags[few])
        assert np.abs(P[few] - want).max(initial=0.0) <= P_TOL
        assert np.isnan(P[s.flags == 32]).all()
        assert_bits_equal(p1.cpu().numpy(), P)
        assert_bits_equal(h1.cpu().numpy(), h0.cpu().numpy())
        hist_of(s, P, h0)


@pytest.mark.parametrize("tiles", [2, 1024, 1025, 4096, 4097, 16384, 16385, 32769, 65537])
def test_merge_shapes(osc, tiles):
    """Both sides of every merge shape's row count (one launch up to 65536
    tiles, two above), with a ragged last tile: the contract's bits."""
    n = tiles * TILE - 700
    rng = np.random.default_rng(tiles)
    value = rng.random(n, dtype=np.float32).astype(np.float64)
    x = rng.integers(0, 5, n).astype(np.float64)
    with osc.Context(0) as ctx:
        d = lambda a: torch.from_numpy(a).cuda()
        h = torch.empty(6, dtype=torch.float64, device="cuda")
        w = torch.full((n,), 1.0 / 3.0, dtype=torch.float64, device="cuda")
        ctx.osc_fill_hist(d(value), w, d(x), 4, 0.0, 4.0, h)
        want = oracle.hist_contract((1.0 / 3.0) * value, np.where(x < 4, x, 5).astype(np.int32), 6)
        assert_bits_equal(h.cpu().numpy(), want)


@pytest.mark.parametrize("nbins", [62, 63])          # two sets side by side, or one
@pytest.mark.parametrize("n_sets,spi", [(1, 1), (2, 2), (3, 2), (5, 4), (5, 8)])
def test_sets_side_by_side(osc, nbins, n_sets, spi):
    """Batched FP32-mixed histograms with whole and odd groups of sets equal
    the plain call's bits, also where only some waves, and only one of two
    sets, take the eigenvalues' Newton step (a set with a level crossing) or
    the FP64 assembly (matter terms above 0.01 eV^2)."""
    n = 30_001
    s = workload.make_sample(n, 8, L_km=2500.0, rho_gcc=11.0, e_range=(0.1, 60.0))
    order = np.argsort(s.e_true)
    for a in ("e_true", "flags", "weight", "e_reco"):
        setattr(s, a, np.ascontiguousarray(getattr(s, a)[order]))
    sets = workload.make_param_sets(n_sets, 9)
    for k in range(1, n_sets, 2):
        sets[k]["sin2_th13"] = 0.0
    with osc.Context(0) as ctx:
        ds = osc.DeviceSample.from_host(s)
        batch = osc.Batch(ctx, [ds], nbins, 0.0, 20.0, osc.OSC_FP32_MIXED, max_sets=n_sets)
        ctx.osc_set_params(sets)
        try:
            for schedule in (0, 2):
                batch.config = dict(sets_per_item=spi, schedule=schedule)
                got = batch.run(sets).cpu().numpy()
                for k in range(n_sets):
                    h = torch.empty(nbins + 2, dtype=torch.float64, device="cuda")
                    ctx.osc_fill_pdf(ds, k, nbins, 0.0, 20.0, h, precision=osc.OSC_FP32_MIXED)
                    assert_bits_equal(got[k, 0], h.cpu().numpy(), (k, schedule))
        finally:
            batch.close()


@pytest.mark.parametrize("tail", [1, 17, 63])
@pytest.mark.parametrize("rho,ye,e_range,th12", [(1.0, 0.5, (3.0, 30.0), 1e-3),
                                                 (1.1, 0.5, (3.0, 30.0), 1e-4),
                                                 (1.0, 0.5, (3.0, 30.0), 0.0),
                                                 (150.0, 0.67, (0.05, 0.4), 0.307)])
def test_ragged_wave_decides_alike_in_every_form(osc, rho, ye, e_range, th12, tail):
    """In the FP32-mixed tier a wave decides as a whole on the roots' second
    refinement (near a level crossing) and on the FP64 assembly (|A| > 0.01
    eV^2).  The lanes past the end of a sample count as 1 GeV nu_e -> nu_e
    events in the plain, binned and batched forms: with parameters and
    densities where that event alone tips the wave, P has the bits it has in
    the sample filled up with such events, and all three forms sum that P."""
    n = 5 * 64 + tail
    full = 1024
    p = dict(workload.TABLE1, sin2_th12=th12)
    with osc.Context(0) as ctx:
        ctx.osc_set_params([p])
        for k, L in enumerate((3000.0, 40_000.0, 400_000.0)):
            s = workload.make_sample(full, 31 + k, L_km=L, rho_gcc=rho, e_range=e_range)
            s.Ye = ye
            s.e_true[n:], s.flags[n:] = 1.0, 0
            filled = osc.DeviceSample.from_host(s)
            cut = lambda t: t[:n].clone()
            ds = osc.DeviceSample(cut(filled.e_true), cut(filled.flags), cut(filled.weight),
                                  cut(filled.e_reco), L, rho, ye)
            new = lambda m: torch.empty(m, dtype=torch.float64, device="cuda")
            h, q, want_p = new(NB + 2), new(n), new(full)
            ctx.osc_fill_pdf(filled, 0, NB, 0.0, HI, h, want_p, precision=osc.OSC_FP32_MIXED)
            ctx.osc_fill_hist(cut(want_p), ds.weight, ds.e_reco, NB, 0.0, HI, h)
            want_h, want_p = h.cpu().numpy(), want_p.cpu().numpy()[:n]
            ctx.osc_fill_pdf(ds, 0, NB, 0.0, HI, h, q, precision=osc.OSC_FP32_MIXED)
            assert_bits_equal(q.cpu().numpy(), want_p, ("plain P", L))
            assert_bits_equal(h.cpu().numpy(), want_h, ("plain", L))
            with ctx.osc_binned_create(ds, NB, 0.0, HI) as binned:
                ctx.osc_fill_pdf_binned(binned, 0, h, q, precision=osc.OSC_FP32_MIXED)
            assert_bits_equal(q.cpu().numpy(), want_p, ("binned P", L))
            assert_bits_equal(h.cpu().numpy(), want_h, ("binned", L))
            batch = osc.Batch(ctx, [ds], NB, 0.0, HI, osc.OSC_FP32_MIXED, max_sets=2)
            try:
                got = batch.run([p, p]).cpu().numpy()
            finally:
                batch.close()
            for j in range(2):
                assert_bits_equal(got[j, 0], want_h, ("batched", L, j))


@pytest.mark.parametrize("tiles,nbins", [(768, 20), (769, 20), (1024, 20), (1025, 20),
                                         (2040, 206), (2050, 206), (2050, 20), (6144, 100),
                                         (6145, 100)])
def test_given_values_split(osc, tiles, nbins):
    """Both sides of every line of the rule for given values (tiles, and tiles
    times the histogram's LDS), with a ragged last tile: the contract's bits."""
    n = tiles * TILE - 300
    rng = np.random.default_rng(tiles)
    value, w = rng.random(n), rng.uniform(-0.5, 1.5, n)
    x = rng.uniform(-0.02, 1.02, n)
    with osc.Context(0) as ctx:
        d = lambda a: torch.from_numpy(a).cuda()
        h = torch.empty(nbins + 2, dtype=torch.float64, device="cuda")
        ctx.osc_fill_hist(d(value), d(w), d(x), nbins, 0.0, 1.0, h)
        bins = oracle.bin_indices(x, 0.0, 1.0, nbins)
        assert_bits_equal(h.cpu().numpy(), oracle.hist_contract(w * value, bins, nbins + 2))


@pytest.mark.parametrize("tiles", [32767, 32768, 49152])
def test_merge_lines(osc, tiles):
    """Up to 32768 tile rows one merge level, above it two: the contract's bits
    with a ragged last tile."""
    n = tiles * TILE - 1
    value = np.tile(np.random.default_rng(tiles).random(1 << 20), -(-n // (1 << 20)))[:n]
    with osc.Context(0) as ctx:
        v = torch.from_numpy(value).cuda()
        h = torch.empty(4, dtype=torch.float64, device="cuda")
        ctx.osc_fill_hist(v, torch.full_like(v, 1.0 / 3.0), 4.0 * v, 2, 0.0, 3.0, h)
        bins = oracle.bin_indices(4.0 * value, 0.0, 3.0, 2)
        assert_bits_equal(h.cpu().numpy(), oracle.hist_contract((1.0 / 3.0) * value, bins, 4))


@pytest.mark.parametrize("n", [1600 * TILE, 1600 * TILE + 1])
@pytest.mark.parametrize("path", [[(1300.0, 3.0, 0.5)], [(650.0, 3.0, 0.5)] * 2])
def test_one_solved_layer_splits(osc, n, path):
    """Both sides of the line for paths with one layer to solve: P as without a
    histogram, and the contract's bits on it."""
    s = workload.make_sample(n, 8)
    with osc.Context(0) as ctx:
        ctx.osc_set_params([workload.TABLE1])
        ds = osc.DeviceSample.from_host(s)
        new = lambda m: torch.empty(m, dtype=torch.float64, device="cuda")
        p0, p1, h = new(n), new(n), new(NB + 2)
        ctx.osc_reweight_layered(ds, path, 0, p0)
        ctx.osc_fill_pdf_layered(ds, path, 0, NB, 0.0, HI, h, p1)
        assert_bits_equal(p1.cpu().numpy(), p0.cpu().numpy())
        hist_of(s, p0.cpu().numpy(), h)
        ctx.osc_fill_pdf_layered(ds, path, 0, NB, 0.0, HI, h)
        hist_of(s, p0.cpu().numpy(), h)


@pytest.mark.parametrize("n_sets,spi", [(15, 8), (16, 1), (16, 2), (17, 2), (17, 8), (19, 3)])
def test_paired_sets_from_sixteen(osc, n_sets, spi):
    """The FP32-mixed batch pairs sets from 16 sets on, with more than one set
    per item: whole groups, odd groups and a short last one have the plain
    call's bits, with level crossings and large matter terms in some sets."""
    n = 5 * TILE + 333
    s = workload.make_sample(n, 8, L_km=2500.0, rho_gcc=11.0, e_range=(0.1, 60.0))
    sets = workload.make_param_sets(n_sets, 9)
    for k in range(1, n_sets, 3):
        sets[k]["sin2_th13"] = 0.0
    with osc.Context(0) as ctx:
        ds = osc.DeviceSample.from_host(s)
        batch = osc.Batch(ctx, [ds], NB, 0.0, 20.0, osc.OSC_FP32_MIXED, max_sets=n_sets)
        ctx.osc_set_params(sets)
        try:
            for schedule in (0, 1, 2):
                batch.config = dict(sets_per_item=spi, schedule=schedule)
                got = batch.run(sets).cpu().numpy()
                for k in range(n_sets):
                    h = torch.empty(NB + 2, dtype=torch.float64, device="cuda")
                    ctx.osc_fill_pdf(ds, k, NB, 0.0, 20.0, h, precision=osc.OSC_FP32_MIXED)
                    assert_bits_equal(got[k, 0], h.cpu().numpy(), (k, schedule))
        finally:
            batch.close()
