"""Field, order-statistic, point and given-moduli kernels at the sizes where
they can go wrong: every truncation order, grids below and just past a tile,
ranks at both ends, many equal distances, point counts around a workgroup."""
import numpy as np
import pytest

from gpu_helpers import torch
from oracle import field as fld
from paper_2511_04025_amd import workloads as wl

pytestmark = pytest.mark.gpu


# FP64 sums of at most 13^3 terms per charge: 1e-12 of the largest value, as the
# existing comparisons with the oracle
@pytest.mark.parametrize("K,n", [(1, 2), (2, 3), (3, 17), (3, 64), (4, 16), (5, 33), (6, 15), (6, 65)])
def test_field_every_order(K, n):
    from paper_2511_04025_amd import api
    rng = np.random.default_rng(100 * K + n)
    d = wl.random_design(40 + K, n, N=5 + 60 * (n == 17), vf=0.3).with_(K=K, alpha=rng.uniform(0.5, 1.5, (K + 1,) * 3))
    print(f"field K {K} n {n}", flush=True)
    r = api.field(d)
    F, G = fld.field_and_gradient(d.pos, d.q, n, K=K, alpha=d.alpha)
    assert np.max(np.abs(r["F"].cpu().numpy().ravel() - np.ravel(F))) <= 1e-12 * np.abs(F).max()
    pts = (np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3)[:, ::-1] + 0.5) / n
    Fp, Gp = api.field_points(d, pts[:777].copy(), gradient=True)
    m = min(777, n ** 3)
    assert np.max(np.abs(Fp.cpu().numpy() - r["F"].cpu().numpy().ravel()[:m])) <= 1e-12 * np.abs(F).max()
    g = r["G"].cpu().numpy().reshape(3, -1)
    assert np.max(np.abs(Gp.cpu().numpy() - g[:, :m])) <= 1e-12 * np.abs(g).max()


@pytest.mark.parametrize("n,vf", [(2, 0.5), (3, 0.99), (17, 1e-5), (17, 0.99999), (16, 0.5), (64, 0.137), (101, 0.05)])
def test_thickness_is_the_midpoint_of_two_order_statistics(n, vf):
    # exact: the rule on the distances that the call returns; mirrored charges
    # make many of them equal
    from paper_2511_04025_amd import api
    d = wl.random_design(50 + n, n, N=4, vf=vf).with_(symmetry="mirror" if n == 16 else 0)
    print(f"thickness n {n} vf {vf}", flush=True)
    r = api.field(d)
    s = np.sort(r["d"].cpu().numpy().ravel())
    k = int(np.floor(vf * n ** 3 + 0.5))
    t = 0.5 * s[0] if k <= 0 else (2.0 * s[-1] + 1.0 if k >= n ** 3 else 0.5 * (s[k - 1] + s[k]))
    assert r["t"] == t
    assert np.array_equal(r["beta"].cpu().numpy(), (r["d"].cpu().numpy() < t).astype(float))


@pytest.mark.parametrize("q", [2e307, 8e307, 1.7e308])
@pytest.mark.parametrize("vf", [0.02, 0.5, 0.98])
def test_thickness_counts_a_nan_distance_as_infinite(q, vf):
    # charges whose field overflows: some distances are infinite and some, from
    # the difference of infinities, no numbers; a rank among those means t = inf
    from paper_2511_04025_amd import api
    n = 12
    d = wl.Design(pos=np.array([[0.1, 0.2, 0.3], [0.6, 0.55, 0.9]]), q=np.array([q, -q]), n=n, dist_mode=1, target_vf=vf)
    print(f"overflowing field q {q} vf {vf}", flush=True)
    r = api.field(d)
    dist = r["d"].cpu().numpy()
    s = np.sort(np.where(np.isnan(dist), np.inf, dist).ravel())
    k = int(np.floor(vf * n ** 3 + 0.5))
    with np.errstate(over="ignore"):
        t = 0.5 * (s[k - 1] + s[k])
    assert r["t"] == t
    assert np.array_equal(r["beta"].cpu().numpy(), (dist < t).astype(float))


@pytest.mark.parametrize("n,vf,kappa", [(2, 0.4, 1e7), (3, 0.5, 30.0), (17, 0.01, 50.0), (33, 0.97, 400.0),
                                        (128, 0.3, 256.0), (130, 0.3, 256.0)])
def test_logistic_thickness_is_the_bisection(n, vf, kappa):
    # three steps a pass and, past 128^3, one; (2, 1e7): a step too steep to meet
    # the target, all 200 steps.  The volume fractions differ from the oracle's by
    # rounding (1e-15), which can move the end of a bisection that passes 1e-12 by
    # a step: t to 1e-9, V to the criterion
    from paper_2511_04025_amd import api
    d = wl.random_design(70 + n, n, N=6, vf=vf).with_(kappa=kappa)
    print(f"logistic thickness n {n} vf {vf} kappa {kappa}", flush=True)
    r = api.field(d)
    dist = r["d"].cpu().numpy()
    t = fld.thickness_for_volume(dist, vf, kappa)
    assert abs(r["t"] - t) <= 1e-9 * max(1.0, abs(t))
    if n > 2:
        assert abs(r["V"] - vf) <= 1e-12 + 1e-14
    assert np.max(np.abs(r["beta"].cpu().numpy() - fld.occupancy(dist, r["t"], kappa))) <= 1e-13


@pytest.mark.parametrize("M", [1, 31, 32, 33, 257])
@pytest.mark.parametrize("K", [2, 3, 4, 6])
def test_points_around_a_workgroup(M, K):
    from paper_2511_04025_amd import api
    d = wl.random_design(60 + K, 8, N=70, vf=0.2).with_(K=K)
    rng = np.random.default_rng(M)
    pts, w = rng.random((M, 3)), rng.standard_normal(M)
    print(f"points {M} K {K}", flush=True)
    F = api.field_points(d, pts)
    Fo = fld.field_at_points(pts, d.pos, d.q, K=K)
    assert np.max(np.abs(F.cpu().numpy() - Fo)) <= 1e-12 * np.abs(Fo).max()
    # F is linear in q and in alpha: sum_j q_j dL/dq_j = sum alpha dL/dalpha = L
    dpos, dq, dal = api.field_points_grad(d, pts, w)
    L = float(w @ Fo)
    scale = float(np.abs(w) @ np.abs(Fo)) + np.abs(dq).sum() + np.abs(dal).sum()
    assert abs(dq @ d.q - L) <= 1e-12 * scale and abs(dal.sum() - L) <= 1e-12 * scale


@pytest.mark.parametrize("n", [2, 5, 33])
@pytest.mark.parametrize("dtype", ["uint8", "float32", "float64"])
def test_given_moduli(n, dtype):
    # volume fraction and validity from the one pass over the moduli
    from paper_2511_04025_amd import api
    rng = np.random.default_rng(n)
    E = rng.uniform(0.2, 3.0, (n, n, n))
    E[0, 0, 0] = 0.0
    print(f"moduli n {n} {dtype}", flush=True)
    if dtype == "uint8":
        u = (E > 1.0).astype(np.uint8)
        r = api.homogenize_field(torch.tensor(u, device="cuda"), 0.3, E_solid=2.0, E_void=0.5, precision="fp64")
        assert abs(r["V"] - u.mean()) <= 1e-14
        return
    Et = torch.tensor(E, dtype=getattr(torch, dtype), device="cuda")
    r = api.homogenize_field(Et, 0.3, precision="fp64")
    e = Et.double().cpu().numpy()
    assert abs(r["V"] - e.mean() / e.max()) <= 1e-14
    for bad in (torch.zeros_like(Et), -Et, torch.full_like(Et, float("inf"))):
        with pytest.raises(Exception):
            api.homogenize_field(bad.contiguous(), 0.3, precision="fp64")


def test_operator_refuses_invalid_moduli():
    from paper_2511_04025_amd import api
    n = 9
    p = torch.randn((2, 3, n, n, n), dtype=torch.float64, device="cuda")
    for v in (0.0, -1.0, float("inf"), float("nan")):
        E = torch.full((n, n, n), v, dtype=torch.float64, device="cuda")
        with pytest.raises(Exception):
            api.apply_stiffness(E, p, 0.3)
    E = torch.ones((n, n, n), dtype=torch.float64, device="cuda")
    q = api.apply_stiffness(E, p, 0.3)
    assert torch.isfinite(q).all()


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 0.0])
def test_refused_moduli_leave_the_output_alone(bad):
    # the moduli are checked on the device, after the pass has been launched
    import torch
    from ctypes import c_double, c_size_t
    from paper_2511_04025_amd import api, binding as B
    n = 10
    E = torch.ones((n, n, n), dtype=torch.float64, device="cuda")
    if np.isinf(bad):
        E[3, 4, 5] = bad
    else:
        E.fill_(bad)  # no modulus above 0
    for prec, dt in (("fp64", torch.float64), ("mixed", torch.float32)):
        p = torch.ones((6, 3, n, n, n), dtype=dt, device="cuda")
        q = torch.full_like(p, 7.0)
        ws = api.Workspace(api.operator_workspace_bytes(n, prec))
        code = B.PREC_FP64 if prec == "fp64" else B.PREC_MIXED
        rc = B.lib().shh_apply_stiffness(n, code, api._ptr(E), c_double(0.3), 6, api._ptr(p), api._ptr(q), ws.ptr,
                                         c_size_t(ws.nbytes), api._stream())
        assert rc != 0 and bool((q == 7.0).all())
    f = torch.full((6, 3, n, n, n), 7.0, dtype=torch.float64, device="cuda")
    ws = api.Workspace(api.operator_workspace_bytes(n, "fp64"))
    rc = B.lib().shh_load_vectors(n, api._ptr(E), c_double(0.3), api._ptr(f), ws.ptr, c_size_t(ws.nbytes), api._stream())
    assert rc != 0 and bool((f == 7.0).all())
