"""Volume tiles on line transforms at the edges of their rule: the numbers of
elements at which they take over from the tile that contracts node by node,
and workgroups whose last elements are missing.  Against the FP64 oracle with
the forward tolerances."""
import numpy as np
import pytest
import torch

from paper_1604_08501_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {False: 1e-12, True: 2e-5}


@pytest.fixture(scope="module")
def sv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1604_08501_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def first(w, n):
    for name in ("geo", "q", "rho_ref", "theta_ref"):
        setattr(w, name, getattr(w, name)[:n])
    return w


def check(call, oracle, w, fp32):
    if fp32:
        w = I.to_fp32(w)
    u = I.upcast(w) if fp32 else w
    ref = oracle(u)
    base = np.random.default_rng(w.Nq).standard_normal(w.q.shape).astype(w.q.dtype)
    args = (dev(w.q), dev(call.geo(w)), dev(w.D), dev(w.rho_ref), dev(w.theta_ref),
            w.phys.as_tuple())
    out = call.run(*args).cpu().numpy().astype(np.float64)
    assert I.rel_err_per_field(out, ref).max() <= TOL[fp32]
    acc = dev(base.copy())
    call.run(*args, out=acc, accumulate=True)
    acc = acc.cpu().numpy().astype(np.float64)
    assert I.rel_err_per_field(acc, base + ref).max() <= TOL[fp32]


class Call:
    def __init__(self, run, geo=lambda w: w.geo):
        self.run, self.geo = run, geo


@pytest.mark.parametrize("fp32,Nq,Ne", [(False, 2, 17), (False, 4, 1), (False, 9, 640),
                                        (False, 9, 641), (False, 12, 320), (False, 12, 321),
                                        (True, 3, 15), (True, 3, 17), (True, 4, 9), (True, 8, 1)])
def test_per_element_metric_terms(sv, oracle_mod, fp32, Nq, Ne):
    w = first(I.affine_workload(N=Nq - 1, n_side=9, k=500 + Nq, with_adjoint=False), Ne)
    check(Call(sv.volume_rhs_affine, lambda w: I.element_geo(w.geo)),
          lambda u: oracle_mod.volume_rhs(u.D, u.geo, u.q, u.rho_ref, u.theta_ref,
                                          u.phys.as_tuple()), w, fp32)


@pytest.mark.parametrize("fp32,Nq,nf,dirs,Ne", [(False, 10, 5, 3, 384), (False, 10, 5, 3, 385),
                                                (False, 10, 8, 3, 385), (False, 3, 8, 7, 3),
                                                (False, 12, 8, 7, 2), (False, 7, 5, 7, 1280),
                                                (False, 7, 5, 7, 1281), (True, 9, 5, 7, 1),
                                                (True, 9, 8, 7, 2), (True, 5, 8, 7, 1)])
def test_fields_and_directions(sv, oracle_mod, fp32, Nq, nf, dirs, Ne):
    w = I.warped_workload(N=Nq - 1, n_side=16, n_elements=Ne, k=520 + Nq)
    if nf == 8:
        w = I.add_tracers(w)
    check(Call(lambda *a, **k: sv.volume_rhs_ext(*a, dirs=dirs, **k)),
          lambda u: oracle_mod.volume_rhs_ext(u.D, u.geo, u.q, u.rho_ref, u.theta_ref,
                                              u.phys.as_tuple(), dirs=dirs), w, fp32)


@pytest.mark.parametrize("Nq", [6, 7, 9])
@pytest.mark.parametrize("theta", [0.0, -1.0, 1e-310, np.inf, np.nan])
def test_special_pressures_stay_in_their_lines(sv, Nq, theta):
    """Against a named tile shape: what is not finite is so at the same nodes."""
    w = I.warped_workload(N=Nq - 1, n_elements=1400, k=540 + Nq)
    w.q[1, 4, Nq * Nq + 2 * Nq + 1] = theta
    a, b = (sv.volume_rhs(dev(w.q), dev(w.geo), dev(w.D), dev(w.rho_ref), dev(w.theta_ref),
                          w.phys.as_tuple(), **tile).cpu().numpy()
            for tile in ({}, dict(elems_per_block=1, layout="full")))
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
    ok = np.isfinite(b)
    scale = np.broadcast_to(np.where(ok, np.abs(b), 0.0).max(axis=(0, 2))[None, :, None], b.shape)
    assert np.all(np.abs(a[ok] - b[ok]) <= 1e-12 * scale[ok])


@pytest.mark.parametrize("fp32,Nq,n_side,Ne", [
    (False, 2, 44, 80000), (False, 2, 44, 80001), (False, 5, 14, 2200), (False, 5, 14, 2201),
    (False, 6, 11, 1024), (False, 6, 11, 1025), (False, 7, 9, 600), (False, 7, 9, 601),
    (True, 3, 32, 30000), (True, 3, 32, 30001), (True, 4, 22, 9500), (True, 4, 22, 9501),
    (True, 6, 11, 1200), (True, 6, 11, 1201), (True, 7, 9, 700), (True, 7, 9, 701),
    (True, 8, 16, 3500), (True, 8, 16, 3501), (True, 9, 9, 600), (True, 9, 9, 601)])
def test_per_element_metric_terms_few_elements(sv, oracle_mod, fp32, Nq, n_side, Ne):
    w = first(I.affine_workload(N=Nq - 1, n_side=n_side, k=560 + Nq, with_adjoint=False), Ne)
    check(Call(sv.volume_rhs_affine, lambda w: I.element_geo(w.geo)),
          lambda u: oracle_mod.volume_rhs(u.D, u.geo, u.q, u.rho_ref, u.theta_ref,
                                          u.phys.as_tuple()), w, fp32)


@pytest.mark.parametrize("fp32,Nq,nf,dirs,Ne", [
    (False, 3, 8, 3, 12), (False, 3, 8, 3, 13), (False, 3, 8, 3, 3500), (False, 3, 8, 3, 3501),
    (False, 5, 8, 3, 3), (False, 5, 8, 3, 4), (False, 5, 8, 3, 2200), (False, 5, 8, 3, 2201),
    (False, 3, 8, 7, 8), (False, 3, 8, 7, 9), (False, 3, 8, 7, 3500), (False, 3, 8, 7, 3501),
    (False, 5, 8, 7, 3), (False, 5, 8, 7, 4), (False, 5, 8, 7, 600), (False, 5, 8, 7, 601),
    (False, 6, 8, 7, 1), (False, 6, 8, 7, 2), (False, 7, 8, 7, 256), (False, 7, 8, 7, 257),
    (False, 6, 5, 7, 1), (False, 6, 5, 7, 2), (True, 6, 5, 3, 2), (True, 6, 5, 3, 3),
    (True, 6, 5, 3, 512), (True, 6, 5, 3, 513), (True, 6, 8, 7, 1), (True, 6, 8, 7, 2)])
def test_fields_and_directions_few_elements(sv, oracle_mod, fp32, Nq, nf, dirs, Ne):
    w = I.warped_workload(N=Nq - 1, n_side=16, n_elements=Ne, k=580 + Nq)
    if nf == 8:
        w = I.add_tracers(w)
    check(Call(lambda *a, **k: sv.volume_rhs_ext(*a, dirs=dirs, **k)),
          lambda u: oracle_mod.volume_rhs_ext(u.D, u.geo, u.q, u.rho_ref, u.theta_ref,
                                              u.phys.as_tuple(), dirs=dirs), w, fp32)
