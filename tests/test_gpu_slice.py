"""The FP64 tile on wave-private slices (Nq = 8), which calls that name no tile
shape take, against the general tile (a named shape) of the same call: every
form the call accepts, and states at which the pressure's power is special.

Tolerance of the finite values: both tiles sum the same products in another
order, 3 Nq of them per value, with pressures good to a few ulp, so they differ
by at most about 50 units of 2^-53 of the largest term of a sum; the terms of
a line exceed the rate by up to three orders of magnitude (D's entries against
their cancelling sum), 1e-12 of the field's largest rate."""
import numpy as np
import pytest
import torch

from paper_1604_08501_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1604_08501_amd as m
    m.lib()
    return m


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("Ne", [1, 2, 5])
@pytest.mark.parametrize("ref", [False, True])
@pytest.mark.parametrize("acc", [False, True])
def test_slice_tile_equals_the_general_tile(sv, Ne, ref, acc):
    w = I.warped_workload(N=7, n_elements=Ne, k=300 + Ne)
    base = np.random.default_rng(Ne).standard_normal(w.q.shape)
    got = []
    for tile in ({}, dict(elems_per_block=1, layout="full")):
        out = dev(base)
        sv.volume_rhs(dev(w.q), dev(w.geo), dev(w.D), dev(w.rho_ref) if ref else None,
                      dev(w.theta_ref) if ref else None, w.phys.as_tuple(), out=out,
                      accumulate=acc, **tile)
        got.append(out.cpu().numpy())
    assert I.rel_err_per_field(got[0], got[1]).max() <= 1e-12


@pytest.mark.parametrize("theta", [0.0, -1.0, 5e-324, 1e-310, np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("ref", [False, True])
def test_special_pressures_as_the_general_tile(sv, theta, ref):
    w = I.warped_workload(N=7, n_elements=2, k=310)
    w.q[1, 4, 8 * 8 * 3 + 8 * 2 + 5] = theta
    got = []
    for tile in ({}, dict(elems_per_block=1, layout="full")):
        out = sv.volume_rhs(dev(w.q), dev(w.geo), dev(w.D), dev(w.rho_ref) if ref else None,
                            dev(w.theta_ref) if ref else None, w.phys.as_tuple(), **tile)
        got.append(out.cpu().numpy())
    a, b = got
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(a[np.isinf(b)], b[np.isinf(b)]) and np.array_equal(np.isinf(a), np.isinf(b))
    ok = np.isfinite(b)
    assert ok[0].all()
    scale = np.broadcast_to(np.where(ok, np.abs(b), 0.0).max(axis=(0, 2))[None, :, None], b.shape)
    assert np.all(np.abs(a[ok] - b[ok]) <= 1e-12 * scale[ok])
