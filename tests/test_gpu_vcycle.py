"""The V-cycle's fused passes at the sizes where their tiles can go wrong: one
tile with more nodes than the grid, remainders in x and y, runs of two planes,
hierarchies that end after one level.  A pass that drops or doubles a node at a
tile edge leaves C^H right and only slows CG down, so the iteration counts are
what is checked: the expected sums over the six load cases are those of the
unfused passes (one kernel per vector update and transfer), and a rounding of
the last digits can move a load case's count by one."""
import numpy as np
import pytest

from gpu_helpers import assert_ch_close
from paper_2511_04025_amd import workloads as wl

pytestmark = pytest.mark.gpu

# n: (FP64 at 1e-10, mixed at 1e-6)
COUNTS = {6: (290, 174), 10: (289, 174), 12: (283, 164), 14: (280, 163), 16: (240, 147), 20: (302, 180),
          24: (217, 132), 28: (221, 133), 40: (218, 141), 48: (257, 170), 56: (210, 133), 64: (196, 122),
          80: (242, 153), 96: (190, 126), 112: (183, 123), 128: (225, 151), 160: (192, 128)}


def design(n):
    return wl.random_design(7000 + n, n, N=16, vf=0.2, E_void=1e-2)


@pytest.mark.parametrize("n", sorted(COUNTS))
def test_iteration_counts(n):
    from paper_2511_04025_amd import api
    C = {}
    for k, (precision, rtol) in enumerate((("fp64", 1e-10), ("mixed", 1e-6))):
        print(f"vcycle {n}^3 {precision}", flush=True)
        r = api.homogenize(design(n), precision=precision, rtol=rtol, solver="mg")
        assert r["status"] == 0
        assert abs(int(np.sum(r["iters"])) - COUNTS[n][k]) <= 6, (r["iters"], COUNTS[n][k])
        C[precision] = r["C"]
    assert_ch_close(C["mixed"], C["fp64"], 1e-4)


def test_mixed_batch_equals_single_designs():
    # different z-run lengths and uneven shares of the launch in one batch
    from paper_2511_04025_amd import api
    designs = [design(n) for n in (96, 16, 64, 6, 128, 40)]
    print("vcycle mixed batch", flush=True)
    batch = api.homogenize_batch(designs, precision="mixed", rtol=1e-6, solver="mg")
    for d, rb in zip(designs, batch):
        rs = api.homogenize(d, precision="mixed", rtol=1e-6, solver="mg")
        assert np.array_equal(rs["C"], rb["C"]) and np.array_equal(rs["iters"], rb["iters"])


# n: the largest FP64 iteration count with the coarsest grid inverted by plain
# sequential elimination
INVERSE = {6: 45, 8: 47, 10: 40, 14: 42, 28: 39, 40: 53}


@pytest.mark.parametrize("n", sorted(INVERSE))
def test_coarsest_inverse_block_edges(n):
    # coarsest grids of 3^3, 4^3, 5^3 and 7^3 nodes: 81, 192, 375 and 1029 rows
    # in blocks of 32.  A wrong block shows in the iteration count, which
    # rounding can move by one; C^H within the usual FP64 bar of the Jacobi path
    from paper_2511_04025_amd import api
    d = wl.random_design(7100 + n, n, N=12, vf=0.25, E_void=1e-2)
    print(f"coarsest inverse {n}^3", flush=True)
    mg = api.homogenize(d, precision="fp64", rtol=1e-10, solver="mg")
    ja = api.homogenize(d, precision="fp64", rtol=1e-10, solver="jacobi")
    assert mg["status"] == 0 and ja["status"] == 0
    assert_ch_close(mg["C"], ja["C"], 1e-7)
    assert abs(int(mg["iters"].max()) - INVERSE[n]) <= 1


@pytest.mark.parametrize("n", [80, 96, 112, 128, 160])
def test_level_one_from_moduli_matches_the_stored_stencil(n):
    # coarse grids of 40^3 to 80^3: both tile shapes, with and without a
    # remainder in x, y and z.  FP64 keeps the stored stencil (held to the
    # oracle's Galerkin product elsewhere); in FP32 a row sums 8 elements of 24
    # terms after two 3-level transforms, at most ~100 roundings of 6e-8 of the
    # largest term
    import torch
    from paper_2511_04025_amd import api
    m = n // 2
    g = torch.Generator(device="cuda").manual_seed(n)
    E = torch.where(torch.rand(n, n, n, device="cuda", generator=g) < 0.3, 1.0, 1e-3).double()
    V = torch.randn(6, 3, m, m, m, device="cuda", generator=g)
    print(f"level one {n}^3", flush=True)
    ref = api.mg_operator(E, V.double(), 0.3, 1, "fp64")
    got = api.mg_operator(E, V, 0.3, 1, "mixed").double()
    assert float((got - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


# (n, nu): rms and largest error of the FP32 product A_1 v with a stencil stored in
# FP32 (element matrices summed in FP64, rounded once), in units of the largest
# modulus times the largest entry of v: moduli 0.1 + U[0, 1), v normal
STORED = {(80, 0.3): (5.69e-8, 7.97e-7), (96, -0.5): (7.69e-8, 1.23e-6), (96, 0.0): (4.56e-8, 7.54e-7),
          (96, 0.45): (1.28e-7, 1.51e-6), (96, 0.49): (5.58e-7, 6.28e-6), (160, 0.3): (4.85e-8, 7.56e-7)}


@pytest.mark.parametrize("n,nu", sorted(STORED))
def test_level_one_from_moduli_is_no_further_off_than_the_stored_stencil(n, nu):
    # the moduli enter in FP32 and the element is formed in FP32
    import torch
    from paper_2511_04025_amd import api
    m = n // 2
    E = (0.1 + torch.rand(n, n, n, generator=torch.Generator().manual_seed(n), dtype=torch.float64)).cuda()
    V = torch.randn(6, 3, m, m, m, generator=torch.Generator().manual_seed(n + 1), dtype=torch.float64).float().cuda()
    print(f"level one error {n}^3 nu {nu}", flush=True)
    d = api.mg_operator(E, V, nu, 1, "mixed").double() - api.mg_operator(E, V.double(), nu, 1, "fp64")
    d /= float(E.max()) * float(V.abs().max())
    assert float(d.pow(2).mean().sqrt()) <= STORED[n, nu][0] and float(d.abs().max()) <= STORED[n, nu][1]


@pytest.mark.parametrize("n", [32, 40, 48, 64])
def test_one_step_smoothing_beside_two(n):
    # hierarchies of different depths and operator forms in one batch: the passes
    # of a cycle split by design, and each design's result is that of its own solve
    from paper_2511_04025_amd import api
    designs = [design(n), design(80 if n < 48 else 40), design(24)]
    print(f"one step beside two {n}^3", flush=True)
    for precision, rtol in (("fp64", 1e-8), ("mixed", 1e-6)):
        batch = api.homogenize_batch(designs, precision=precision, rtol=rtol, solver="mg")
        for d, rb in zip(designs, batch):
            rs = api.homogenize(d, precision=precision, rtol=rtol, solver="mg")
            assert rs["status"] == 0 and np.array_equal(rs["C"], rb["C"]) and np.array_equal(rs["iters"], rb["iters"])


# (n, precision): the most iterations a load case of a thin shell (5 % volume, void
# 1e-6) takes with every pass a kernel of its own and two smoothing steps each side
# on every coarse level
LIMITS = {(48, "fp64"): 202, (48, "mixed"): 129, (64, "fp64"): 324, (64, "mixed"): 160}


@pytest.mark.parametrize("n,precision", sorted(LIMITS))
def test_thin_shell_converges_within_its_iteration_limit(n, precision):
    # rounding can move a count of hundreds by one or two
    from paper_2511_04025_amd import api
    d = wl.random_design(5000 + n, n, N=24, vf=0.05, E_void=1e-6)
    print(f"iteration limit {n}^3 {precision}", flush=True)
    r = api.homogenize(d, precision=precision, rtol=1e-10 if precision == "fp64" else 1e-6, solver="mg",
                       max_iter=LIMITS[n, precision] + 2)
    assert r["status"] == 0, r["iters"]


@pytest.mark.parametrize("precision,rtol", [("fp64", 1e-10), ("mixed", 3e-6)])
@pytest.mark.parametrize("solver", ["mg", "selective"])
@pytest.mark.parametrize("n", [12, 24, 48])
def test_last_levels_in_one_launch(n, solver, precision, rtol):
    # 3 x 2^k grids: the 6^3 and 3^3 levels run in one launch, as level 1 (fed
    # and read by the voxel level, 12^3) or below it; the V-cycle must stay a
    # symmetric preconditioner that converges to the Jacobi solution
    from paper_2511_04025_amd import api
    d = wl.random_design(7200 + n, n, N=12, vf=0.25, E_void=0.0 if solver != "mg" else 1e-2)
    print(f"last levels {n}^3 {solver} {precision}", flush=True)
    mg = api.homogenize(d, precision=precision, rtol=rtol, solver=solver)
    ja = api.homogenize(d, precision="fp64", rtol=1e-10, solver="selective-jacobi" if solver != "mg" else "jacobi")
    assert mg["status"] == 0 and ja["status"] == 0
    assert_ch_close(mg["C"], ja["C"], 1e-7 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("n", [25, 28, 29, 42, 64])
def test_tall_fp64_tiles(n):
    # tiles of 32 x 14 nodes from 25^3: remainders of 11, 0, 1 and 8 rows and of
    # the 32 columns; K p against the oracle's element sum at nodes around the
    # tile edges (FP64 sums of 8 x 24 terms: 1e-12 of the largest), and flat and
    # tall slots in one Jacobi batch
    import torch
    from oracle import fem
    from paper_2511_04025_amd import api
    rng = np.random.default_rng(n)
    E, p = rng.uniform(0.1, 1.0, (n, n, n)), rng.standard_normal((6, 3, n, n, n))
    print(f"tall tiles {n}^3", flush=True)
    q = api.apply_stiffness(torch.tensor(E, device="cuda"), torch.tensor(p, device="cuda"), 0.3, "fp64").cpu().numpy()
    edge = [i for i in (0, 1, 12, 13, 14, 15, 27, 28, 31, 32, 33, n - 2, n - 1) if i < n]
    nodes = np.unique([(z * n + y) * n + x for z in (0, n // 2, n - 1) for y in edge for x in edge])
    U = p.reshape(6, 3, -1).transpose(2, 1, 0)
    ref = fem.stiffness_rows(E.ravel(), 0.3, n, lambda ids: U[ids], nodes)
    got = q.reshape(6, 3, -1)[:, :, nodes].transpose(2, 1, 0)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.abs(ref).max()
    if n > 28:
        return
    designs = [wl.random_design(7300 + k, k, N=8, vf=0.3, E_void=1e-1) for k in (n, 24, 10)]
    batch = api.homogenize_batch(designs, precision="fp64", rtol=1e-8, solver="jacobi")
    for d, rb in zip(designs, batch):
        rs = api.homogenize(d, precision="fp64", rtol=1e-8, solver="jacobi")
        assert rs["status"] == 0 and np.array_equal(rs["C"], rb["C"]) and np.array_equal(rs["iters"], rb["iters"])


@pytest.mark.parametrize("sizes", [(48, 24, 28), (24, 20), (28, 48)])
def test_flat_and_tall_fp64_multigrid_batch(sizes):
    # the two FP64 tilings make a launch each from one table of segments: 24^3 and
    # 20^3 flat, 28^3 and 48^3 tall, in batches of both, of one, and of the other
    from paper_2511_04025_amd import api
    print(f"FP64 batch {sizes}", flush=True)
    designs = [wl.random_design(7400 + n, n, N=8, vf=0.3, E_void=1e-4) for n in sizes]
    batch = api.homogenize_batch(designs, precision="fp64", rtol=1e-8, solver="mg")
    for d, rb in zip(designs, batch):
        rs = api.homogenize(d, precision="fp64", rtol=1e-8, solver="mg")
        assert rs["status"] == 0 and np.array_equal(rs["C"], rb["C"]) and np.array_equal(rs["iters"], rb["iters"])
