"""Kernels at the sizes where they can go wrong: remainders, edges of tiles and
the smallest and largest of their ranges, against the FP64 oracle or an exact
reference of the same operation, through the C ABI."""
import numpy as np
import pytest

from oracle import fstat_oracle as O
from oracle import fstat_oracle_grad as G
from paper_2201_00451_amd import synth

pytestmark = pytest.mark.gpu

# the forward path's bar against the oracle
RTOL, ATOL = 1e-4, 1e-3
# the gradients' bar (that of the finite differences)
GRAD_RTOL = 1e-3


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_2201_00451_amd import binding
    binding.load_library()
    return torch


def check_2f(gpu, ref):
    gpu = gpu.cpu().numpy().astype(np.float64)
    strong = ref >= 10.0
    assert np.all(np.isfinite(gpu))
    assert np.max(np.abs(gpu - ref)[strong] / ref[strong]) <= RTOL
    assert np.max(np.abs(gpu - ref)[~strong]) <= ATOL


@pytest.mark.parametrize("ndet,kepler", [(1, False), (4, False), (4, True)])
def test_parameter_blocks_of_every_detector_count(torch_dev, ndet, kepler):
    """The parameter kernel's lanes at one detector and at the maximum (four),
    with isolated and eccentric rows, in the plain and the grouped path."""
    from paper_2201_00451_amd import binding
    extra = dict(binary=True, ecc=0.2, argp=0.7) if kepler else {}
    ds = synth.small_case(seed=90 + ndet, n=3001, n_fft=1 << 13, ndet=ndet, ntmpl=3, gaps=True,
                          noise_vars=[1.0, 0.7, 1.4, 0.9][:ndet], **extra)
    ref = O.oracle_twoF(ds)
    dd = binding.DeviceData(ds, batch=3)
    plain = binding.compute_2f(dd, ds.templates)
    grouped = binding.Search(dd, ds.templates, slots=2).run()
    binding.sync_check()
    assert torch_dev.equal(plain, grouped)
    check_2f(plain, ref)


@pytest.mark.parametrize("ndet,D,porb_d,log_g", [(1, 8, 0.5, 6), (2, 8, 0.2, 5), (2, 16, 0.1, 4),
                                                 (3, 4, 0.2, 5), (4, 12, 0.5, 6)])
def test_resampling_spans(torch_dev, ndet, D, porb_d, log_g):
    """Blocks of two tiles (a launch of many tiles) against blocks of one (one
    template at a time), bit for bit, at every knot spacing solved ahead, with
    an odd number of tiles, gaps and a ragged end; one template against the
    oracle."""
    from paper_2201_00451_amd import binding
    ds = synth.small_case(seed=95, n=35801, n_fft=1 << 16, ndet=ndet, D=D, binary=True, gaps=True,
                          ntmpl=32, noise_vars=[1.0, 0.7, 1.4, 0.9][:ndet])
    ds.templates[:, 5] = 0.3 + 1e-4 * np.arange(32)
    ds.templates[:, 6] = porb_d * synth.DAY
    ds = synth.finish(ds)
    # the knot spacing the library's rule gives these orbits
    om = 2 * np.pi / (porb_d * synth.DAY)
    budget = min(2e-7 / ds.f_het, 1e-7 * ds.dt)
    fits = [(2.0 ** l * ds.dt) ** 4 / 384 * (0.3031 * om ** 4 + 1e-16) <= budget for l in (4, 5, 6)]
    assert sum(fits) + 3 == log_g
    dd = binding.DeviceData(ds)
    k_pad, _, _ = dd.plan.info()
    assert (k_pad // 512) % 2 == 1 and (k_pad // 512) * 32 >= 2048
    many = binding.Search(dd, ds.templates, slots=32).run()
    one = binding.compute_2f(dd, ds.templates)
    binding.sync_check()
    assert torch_dev.equal(many, one)
    check_2f(many[17:18], O.oracle_twoF(ds, ds.templates[17:18]))


def orbit_case(porb_d, asini, ndet, D, n, ecc=None):
    """A search whose injection has the given orbit, and a row off it in every
    parameter."""
    extra = dict(ecc=ecc, argp=0.6) if ecc is not None else {}
    ds = synth.small_case(seed=97, n=n, n_fft=1 << 13, ndet=ndet, D=D, binary=True, gaps=True,
                          ntmpl=1, rho=25, noise_vars=[1.0, 0.7, 1.4, 0.9][:ndet], **extra)
    inj = ds.injections[0]
    inj.update(asini=asini, porb=porb_d * synth.DAY)
    ds.x, _ = synth.make_data(ds.detectors, ds.dt, ds.f_het, 0.0, [inj], 97, gaps=ds.valid)
    ds.templates[:, 5], ds.templates[:, 6] = asini, inj["porb"]
    ds = synth.finish(ds)
    row = ds.templates[0].copy()
    T = n * ds.dt
    row[0] += 0.002
    row[1] -= 0.0015
    row[2] += 0.3 / T
    row[3] += 0.5 / T ** 2
    row[5] *= 1.001
    row[6] *= 1.0 + 2e-5
    row[7] += 1.0
    return ds, row


@pytest.mark.parametrize("porb_d,asini,ndet,D,n,ecc,smooth,log_g",
                         [(0.5, 0.05, 2, 8, 3000, None, True, 6),    # spans of two tiles
                          (0.14, 0.05, 4, 16, 2700, None, True, 5),  # G = 32, every detector
                          (0.13, 0.6, 2, 4, 3300, None, True, 4),    # G = 16: tile by tile
                          (0.5, 0.1, 3, 8, 3000, 0.3, True, 6),      # eccentric, three detectors
                          (0.05, 0.004, 2, 8, 3000, None, False, 5)])  # solved point by point
def test_gradients_by_tile_smoothness(torch_dev, porb_d, asini, ndet, D, n, ecc, smooth, log_g):
    """Both gradient forms against the FP64 oracle for orbits on either side of
    the rule that decides between quintics per tile and per-point solves, at
    each knot spacing."""
    from paper_2201_00451_amd import binding
    ds, row = orbit_case(porb_d, asini, ndet, D, n, ecc)
    om = 2 * np.pi / (porb_d * synth.DAY)
    e2 = (1 - (ecc or 0.0)) ** 2
    budget = min(2e-7 / ds.f_het, 1e-7 * ds.dt)
    fits = [(2.0 ** l * ds.dt) ** 4 / 384 * (row[5] * (om / e2) ** 4 + 1e-16) <= budget
            for l in (2, 3, 4, 5, 6)]
    assert sum(fits) + 1 == log_g
    assert (om * 256 * ds.dt <= 0.3 * e2) == smooth
    dd = binding.DeviceData(ds)
    tf = O.oracle_twoF(ds, row[None])[0]
    m = int(np.argmax(tf))
    w = np.zeros(ds.n_bins)
    w[m - 2:m + 3] = [0.2, 0.5, 1.0, 0.7, 0.1]
    one = np.zeros(ds.n_bins)
    one[m] = 1.0
    g_bin, tf_bin = binding.compute_2f_grad_bin(dd, row[None], [m])
    g_gen, tf_gen = binding.compute_2f_grad(dd, row[None], w[None], want_twoF=True)
    plain = binding.compute_2f(dd, row[None])
    binding.sync_check()
    assert torch_dev.equal(tf_gen, plain)
    check_2f(plain, tf[None])
    assert abs(float(tf_bin[0]) - tf[m]) <= RTOL * tf[m]
    for got, weights in ((g_bin, one), (g_gen, w)):
        _, ref = G.oracle_grad(ds, row, weights)
        got = got.cpu().numpy()[0]
        for i, name in enumerate(G.PARAMS):
            print(f"  {name:6s} gpu {got[i]: .9e} oracle {ref[i]: .9e} "
                  f"rel {abs(got[i] - ref[i]) / abs(ref[i]):.1e}", flush=True)
            assert abs(got[i] - ref[i]) <= GRAD_RTOL * abs(ref[i]), name


@pytest.mark.parametrize("log_n", [12, 15, 17, 18, 19, 21])
def test_fft_items_of_small_and_large_launches(torch_dev, log_n):
    """The passes' small-launch items, the default ones and the largest line
    counts give the same bits in every epilogue (plain, Fa and Fb, summed,
    the adjoint's 2F) on a ragged band, at row lengths 2^6 to 2^11; one template
    against the oracle."""
    from paper_2201_00451_amd import binding
    n_fft = 1 << log_n
    lo, nb = n_fft // 5 + 1, n_fft // 2 + 3
    ds = synth.small_case(seed=98, n=2500, n_fft=n_fft, ndet=2, gaps=True, ntmpl=32, rho=20,
                          bin_lo=lo, n_bins=nb)
    dd = binding.DeviceData(ds, batch=32)
    one, ab = binding.compute_2f(dd, ds.templates, fafb=True)
    many, ab_many = binding.compute_2f_batched(dd, ds.templates, fafb=True)
    plain = binding.compute_2f_batched(dd, ds.templates)
    search = binding.Search(dd, ds.templates, slots=32, accumulate=True)
    total = torch_dev.full((32, nb), 3.0, device="cuda:0")
    search.run(out=total)
    w = torch_dev.linspace(0.0, 1.0, nb, device="cuda:0")[None].repeat(3, 1)
    g1, tf1 = binding.compute_2f_grad(dd, ds.templates[:3], w, want_twoF=True, batch=1)
    g3, tf3 = binding.compute_2f_grad(dd, ds.templates[:3], w, want_twoF=True, batch=3)
    lr = log_n // 2
    wide = binding.DeviceData(ds, batch=32, tune=dict(
        tune_col_lines=min(64, 16384 >> lr), tune_row_lines=min(32, 8192 >> (log_n - lr))))
    full, ab_full = binding.compute_2f_batched(wide, ds.templates, fafb=True)
    binding.sync_check()
    for a, b in ((one, many), (one, plain), (one, full), (ab, ab_many), (ab, ab_full),
                 (one + 3.0, total), (one[:3], tf1), (one[:3], tf3), (g1, g3)):
        assert torch_dev.equal(a, b)
    check_2f(one[5:6], O.oracle_twoF(ds, ds.templates[5:6]))


@pytest.mark.parametrize("log_n,col,row_lines", [(20, 10, 0), (21, 10, 0), (21, 10, 2),
                                                 (22, 11, 0), (22, 11, 2), (23, 11, 0),
                                                 (23, 11, 1)])
def test_fft_intermediate_in_column_blocks(torch_dev, log_n, col, row_lines):
    """Searches whose column pass writes blocks of eight columns (and, at 2^20,
    the shortest plan that does not) give the bits of the in-place transforms
    with a row-major intermediate: plain, summed, and candidates with the
    loudest bin, on a ragged band, every row kernel that reads blocks; one
    template against the oracle."""
    from paper_2201_00451_amd import binding
    n_fft = 1 << log_n
    lo, nb = n_fft // 5 + 1, n_fft // 2 + 3
    ds = synth.small_case(seed=97, n=2500, n_fft=n_fft, ndet=2, gaps=True, ntmpl=5, rho=20,
                          bin_lo=lo, n_bins=nb)
    dd = binding.DeviceData(ds, batch=5, tune=dict(tune_col_log_len=col, tune_col_lines=8,
                                                   tune_row_lines=row_lines))
    want = binding.compute_2f_batched(dd, ds.templates)
    got = torch_dev.empty_like(want)
    binding.Search(dd, ds.templates, slots=5).run(out=got)
    total = torch_dev.full_like(want, 3.0)
    binding.Search(dd, ds.templates, slots=5, accumulate=True).run(out=total)
    level = float(want.max()) * 0.9
    rep = binding.Search(dd, ds.templates, slots=5).run_candidates(level)
    binding.sync_check()
    assert torch_dev.equal(got, want) and torch_dev.equal(total, want + 3.0)
    assert rep["count"] == int((want > level).sum()) > 0
    assert torch_dev.equal(rep["best_twoF"], want.max(dim=1).values)
    check_2f(want[1:2], O.oracle_twoF(ds, ds.templates[1:2]))


@pytest.mark.parametrize("D,share", [(8, 0.46), (16, 0.46), (16, 0.49)])
def test_gradients_near_the_band_edge(torch_dev, D, share):
    """The orbit's gradients of a signal at 0.46 and 0.49 of the sampling rate,
    where the interpolation's response falls off and the sums over its taps
    feel the curvature of the delay derivatives, for an orbit at the limit of
    the quintics per tile (0.297 rad per half tile), against the FP64 oracle.
    Tolerance: ten FP32 roundings (6e-8) per term, times 16 for terms that
    cancel."""
    from paper_2201_00451_amd import binding
    dt, n = 2.0, 3300
    ds = synth.small_case(seed=304, n=n, dt=dt, n_fft=1 << 13, ndet=2, D=D, binary=True, gaps=True,
                          ntmpl=1, rho=25, f_inj=share / dt, noise_vars=[1.0, 0.7])
    inj = ds.injections[0]
    inj.update(asini=0.6, porb=2 * np.pi * 256 * dt / 0.297)
    ds.x, _ = synth.make_data(ds.detectors, dt, ds.f_het, 0.0, [inj], 304, gaps=ds.valid)
    ds.templates[:, 5], ds.templates[:, 6] = inj["asini"], inj["porb"]
    ds = synth.finish(ds)
    row = ds.templates[0] + np.array([0.002, -0.0015, 0.3 / (n * dt), 0.5 / (n * dt) ** 2, 0, 6e-4,
                                      0.2, 1.0])
    dd = binding.DeviceData(ds)
    m = int(np.argmax(O.oracle_twoF(ds, row[None])[0]))
    w = np.zeros(ds.n_bins)
    w[m] = 1.0
    _, ref = G.oracle_grad(ds, row, w)
    g_bin, _ = binding.compute_2f_grad_bin(dd, row[None], [m])
    g_gen = binding.compute_2f_grad(dd, row[None], w[None])
    binding.sync_check()
    for got in (g_bin, g_gen):
        err = np.abs(got.cpu().numpy()[0] - ref) / np.abs(ref)
        print("  ", dict(zip(G.PARAMS, err)), flush=True)
        assert np.all(err[4:] <= 10 * 6e-8 * 16)


def test_point_by_point_launches(torch_dev):
    """Single-bin gradients of templates solved point by point (an orbit of 24
    minutes): a launch of many templates, whose blocks walk the tiles, gives the
    bits of one template at a time, a block per tile."""
    from paper_2201_00451_amd import binding
    ds = synth.small_case(seed=61, n=530001, dt=2.0, n_fft=1 << 20, ndet=2, binary=True, ntmpl=32,
                          n_bins=4096, bin_lo=1 << 19)
    ds.templates[:, 5] = 0.001 * (1 + 1e-4 * np.arange(32))
    ds.templates[:, 6] = 1440.0
    ds = synth.finish(ds)
    assert 2 * np.pi / 1440.0 * 256 * ds.dt > 0.3
    dd = binding.DeviceData(ds)
    assert dd.plan.info()[0] // 512 > 32768 // 32
    bins = [100 * i for i in range(32)]
    many, tf_many = binding.compute_2f_grad_bin(dd, ds.templates, bins, batch=32)
    one, tf_one = binding.compute_2f_grad_bin(dd, ds.templates, bins, batch=1)
    binding.sync_check()
    assert torch_dev.isfinite(many).all()
    assert torch_dev.equal(many, one) and torch_dev.equal(tf_many, tf_one)


def test_parameter_blocks_of_a_large_bank(torch_dev):
    """A bank of more templates than the first dimension of the parameter launch
    holds: every template's loudest bin is the one of a search of its own few
    neighbours."""
    from paper_2201_00451_amd import binding
    ds = synth.small_case(seed=71, n=2000, n_fft=1 << 12, ndet=1, ntmpl=1, f1dot=0.0)
    n = (1 << 16) + 300
    rows = np.repeat(ds.templates, n, axis=0)
    rows[:, 3] = 1e-9 * (np.arange(n) - n // 2) / n
    dd = binding.DeviceData(ds)
    many = binding.Search(dd, rows, slots=32).run_candidates(60.0, capacity=16)
    binding.sync_check()
    assert many["best_twoF"].numel() == n and torch_dev.isfinite(many["best_twoF"]).all()
    for lo, hi in ((0, 64), ((1 << 16) - 32, (1 << 16) + 32), (n - 33, n)):
        few = binding.Search(dd, rows[lo:hi], slots=32).run_candidates(60.0, capacity=16)
        binding.sync_check()
        assert torch_dev.equal(many["best_twoF"][lo:hi], few["best_twoF"])
        assert torch_dev.equal(many["best_bin"][lo:hi], few["best_bin"])


@pytest.mark.parametrize("log_n,col,row_lines", [(21, 10, 0), (22, 11, 0), (23, 11, 1)])
def test_flagged_template_and_fafb_with_column_blocks(torch_dev, log_n, col, row_lines):
    """Searches with a blocked intermediate, plain and with its rows split: a
    template with a spin-down that is no number is NaN in every bin of 2F, Fa
    and Fb, counted once, and leaves its neighbours' bits alone."""
    from paper_2201_00451_amd import binding
    n_fft = 1 << log_n
    lo, nb = n_fft // 3 + 1, n_fft // 3 + 7
    ds = synth.small_case(seed=96, n=2500, n_fft=n_fft, ndet=2, gaps=True, ntmpl=5, rho=20,
                          bin_lo=lo, n_bins=nb)
    ds.templates[3, 3] = np.nan
    dd = binding.DeviceData(ds, batch=5, tune=dict(tune_col_log_len=col, tune_col_lines=8,
                                                   tune_row_lines=row_lines))
    search = binding.Search(dd, ds.templates, slots=5)
    got, ab = search.run(fafb=True)
    plain = search.run()
    flagged = binding.flagged_count(search.ws)
    rep = search.run_candidates(1e9)
    want, ab_want = binding.compute_2f_batched(dd, ds.templates, fafb=True)
    binding.sync_check()
    ok = [0, 1, 2, 4]
    assert flagged == 1
    for x, y in ((got, want), (plain, want), (ab, ab_want)):
        assert torch_dev.equal(x[ok], y[ok]) and torch_dev.isfinite(torch_dev.abs(x[ok])).all()
        assert torch_dev.isnan(torch_dev.abs(x[3])).all()
    assert torch_dev.equal(rep["best_twoF"][ok], want[ok].max(dim=1).values)
    assert torch_dev.isnan(rep["best_twoF"][3]) and rep["count"] == 0


def test_spans_flag_windows_and_pass_bad_samples(torch_dev):
    """The gradient kernels' spans: an orbit whose delay drifts by a fifth of a
    tile, more than a tile's 616 staged samples hold (512 (1 + 0.2) + 2 D), is
    flagged (NaN 2F and gradients), a neighbour is not touched by it; an infinite
    and a NaN sample reach the results."""
    from paper_2201_00451_amd import binding
    ds = synth.small_case(seed=62, n=4001, n_fft=1 << 13, ndet=2, f_het=1.0, binary=True, ntmpl=2)
    om = 5.5e-4
    ds.templates[:, 5], ds.templates[:, 6] = [0.05, 0.2 / om], 2 * np.pi / om
    ds.templates[:, 7] = 4000.0  # the largest rate in the middle of the data
    ds = synth.finish(ds)
    # the spans' conditions: knots at least 16 points apart, 0.3 rad per half tile
    assert 32.0 ** 4 / 384 * (0.2 / om) * om ** 4 <= 2e-7 and om * 512 <= 0.3
    ds.tau0 = synth.grid_origin(0.0, ds.dt, ds.max_delay)
    dd = binding.DeviceData(ds)
    bins = [4000, 4000]
    w = np.zeros((2, ds.n_bins))
    w[:, 4000] = 1.0
    plain = binding.compute_2f(dd, ds.templates)
    g_bin, tf_bin = binding.compute_2f_grad_bin(dd, ds.templates, bins)
    g_gen = binding.compute_2f_grad(dd, ds.templates, w)
    binding.sync_check()
    for x in (plain, g_bin, tf_bin, g_gen):
        assert torch_dev.isfinite(x[0]).all() and torch_dev.isnan(x[1]).all()
    for bad in (np.nan, np.inf):
        ds.x[1][1500] = bad
        dd = binding.DeviceData(ds)
        plain = binding.compute_2f(dd, ds.templates[:1])
        g_bin, tf_bin = binding.compute_2f_grad_bin(dd, ds.templates[:1], bins[:1])
        binding.sync_check()
        for x in (plain, g_bin, tf_bin):
            assert not torch_dev.isfinite(x).any()


@pytest.mark.parametrize("porb_d", [0.5, 0.016])  # spans; solved point by point
def test_gradients_refuse_delays_beyond_the_bound(torch_dev, porb_d):
    """Single-bin gradients of a template whose delays exceed max_delay by 145 s,
    more than the taps (20 s at D = 8 and 2 s a sample) and two intervals of the
    trajectory (60 s): NaN, in both forms of the kernels; at the bound: finite."""
    from paper_2201_00451_amd import binding
    ds = synth.small_case(seed=12, n=3000, n_fft=1 << 13, ndet=1, binary=True, ntmpl=1)
    ds.templates[:, 5], ds.templates[:, 6] = 0.001, porb_d * synth.DAY
    for excess in (0.0, 145.0):
        ds = synth.finish(ds)
        det = ds.detectors[0]
        pos = synth.detector_pos_vel(ds.ephem_model, det, np.arange(-600.0, 7000.0, 10.0))[0]
        # the sky position of the longest delays, opposite the Earth
        mid = -pos[:, pos.shape[1] // 2]
        row = ds.templates[0].copy()
        row[0] = np.arctan2(mid[1], mid[0])
        row[1] = np.arcsin(mid[2] / np.linalg.norm(mid))
        longest = np.abs(synth.sky_unit(row[0], row[1]) @ pos).max() + row[5]
        ds.max_delay = longest + 1.0 - excess
        dd = binding.DeviceData(ds)
        g, _ = binding.compute_2f_grad_bin(dd, row[None], [4000])
        binding.sync_check()
        assert bool(torch_dev.isfinite(g).all()) == (excess == 0.0)
        assert bool(torch_dev.isnan(g).all()) == (excess > 0.0)


@pytest.mark.parametrize("half_tile", [0.178, 0.19])
def test_eccentric_gradients_at_the_spans_limit(torch_dev, half_tile):
    """Single-bin gradients of an eccentric orbit (0.4) on either side of the
    limit of the quintics per tile, 0.18 rad of phase at periapsis per half tile,
    against the FP64 oracle."""
    from paper_2201_00451_amd import binding
    ecc, dt = 0.4, 2.0
    porb_d = 2 * np.pi * 256 * dt / (half_tile * (1 - ecc) ** 2) / synth.DAY
    ds, row = orbit_case(porb_d, 0.1, 2, 8, 3000, ecc)
    dd = binding.DeviceData(ds)
    m = int(np.argmax(O.oracle_twoF(ds, row[None])[0]))
    w = np.zeros(ds.n_bins)
    w[m] = 1.0
    _, ref = G.oracle_grad(ds, row, w)
    got, _ = binding.compute_2f_grad_bin(dd, row[None], [m])
    binding.sync_check()
    assert np.all(np.abs(got.cpu().numpy()[0] - ref) <= GRAD_RTOL * np.abs(ref))
