"""Kernels at the sizes where they can go wrong: remainders, edges of tiles and
the smallest and largest of their ranges, against the FP64 oracle or an exact
reference of the same operation, through the C ABI."""
import numpy as np
import pytest

from oracle import fstat_oracle as O
from paper_2201_00451_amd import synth

pytestmark = pytest.mark.gpu

# the forward path's bar against the oracle
RTOL, ATOL = 1e-4, 1e-3


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
