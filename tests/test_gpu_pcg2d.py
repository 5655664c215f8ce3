"""The 2D Jacobi-PCG preconditioners (one launch per step on regions in registers; meshes of at most 64 x 64 nodes by
one workgroup per system) against the oracle's conjugate gradients.  Needs an MI355X."""
import numpy as np
import pytest

from oracle.apfc_oracle import tri_k
from paper_1902_09761_amd import apfc, inputs
from tests.gpu_util import H_TRI, from_dev, families_of_a_step, oracle_for, solver_for, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(n):
    return inputs.Mesh(2, (n[0], n[1], 1), (n[0] * H_TRI, n[1] * H_TRI, 1.0))


def _pinv(meshes, pairs, its, mass="iter", dt=0.7, precision=apfc.APFC_FP64):
    s = solver_for(meshes, apfc.APFC_TRI2D, [0.02] * len(meshes), inner_kind=apfc.APFC_INNER_PCG, mass_iters=its[0],
                   diff_iters=its[1], precision=precision,
                   mass_kind=apfc.APFC_MASS_SEPARABLE if mass == "sep" else apfc.APFC_MASS_ITER)
    zo = [torch.zeros((3, 2, m.N), dtype=torch.float64, device="cuda") for m in meshes]
    eo = [torch.zeros_like(t) for t in zo]
    s.apply(apfc.APFC_OP_PINV, [to_dev(z) for z, _ in pairs], [to_dev(e) for _, e in pairs], zo, eo, dt)
    return [(from_dev(z), from_dev(e)) for z, e in zip(zo, eo)]


def _half_step_launches(meshes, its, mass="iter", precision=apfc.APFC_FP64):
    """Whether P^{-1} takes a launch per half of a CG step (the updates of x and r are launches of their own)."""
    s = solver_for(meshes, apfc.APFC_TRI2D, [0.02] * len(meshes), rtol=1e-4, inner_kind=apfc.APFC_INNER_PCG, restart=6,
                   mass_iters=its[0], diff_iters=its[1], precision=precision,
                   mass_kind=apfc.APFC_MASS_SEPARABLE if mass == "sep" else apfc.APFC_MASS_ITER)
    n = families_of_a_step(s, meshes)
    assert n["pcg_spmv"] > 0
    return n["pcg_update"] > 0


def _worst(meshes, pairs, got, its, mass="iter", dt=0.7):
    worst = 0.0
    for m, (z, e), (gz, ge) in zip(meshes, pairs, got):
        o = oracle_for(m, tri_k(), 0.02)
        for j in range(3):
            ref = np.concatenate(o.precond_apply(j, z[j], e[j], dt, inner="pcg", mass_iters=its[0], diff_iters=its[1],
                                                 mass=mass))
            worst = max(worst, float(np.max(np.abs(np.concatenate([gz[j], ge[j]]) - ref)) / np.max(np.abs(ref))))
    return worst


def _random(meshes, seed):
    r = np.random.default_rng(seed)
    return [tuple(r.normal(size=(3, m.N)) + 1j * r.normal(size=(3, m.N)) for _ in range(2)) for m in meshes]


TOL = 1e-12          # FP64 rounding, as for the step-by-step kernels


@pytest.mark.parametrize("n,its,mass", [
    ((4, 65), (3, 5), "iter"),         # every x neighbour a wrap onto the mesh itself
    ((65, 13), (1, 1), "iter"),        # one iteration per solve
    ((44, 72), (3, 5), "iter"),        # regions filled exactly
    ((89, 73), (3, 5), "iter"),        # one node more in each direction
    ((133, 64), (5, 5), "iter"),       # the longest solves
    ((96, 80), (2, 4), "iter"),
    ((130, 70), (3, 5), "sep"),
    ((530, 500), (3, 5), "iter"),      # more regions than CUs: eight rows per wave
])
def test_matches_oracle(n, its, mass):
    m = [_mesh(n)]
    pairs = _random(m, 41)
    assert _worst(m, pairs, _pinv(m, pairs, its, mass), its, mass) <= TOL


@pytest.mark.parametrize("precision,tol", [(apfc.APFC_FP64, TOL), (apfc.APFC_MIXED, 2e-5)])
@pytest.mark.parametrize("n,its,mass", [
    ((4, 4), (3, 5), "iter"), ((5, 13), (1, 1), "iter"), ((64, 64), (3, 5), "iter"), ((63, 17), (4, 9), "iter"),
    ((33, 61), (2, 5), "sep"),
])
def test_one_workgroup_per_system(precision, tol, n, its, mass):
    m = [_mesh(n), _mesh((40, 28))]
    pairs = _random(m, 44)
    assert _worst(m, pairs, _pinv(m, pairs, its, mass, precision=precision), its, mass) <= tol


@pytest.mark.parametrize("n", [(40, 64), (63, 64), (4, 64)])
def test_one_workgroup_narrow_and_tall(n):
    m = [_mesh(n)]
    pairs = _random(m, 48)
    assert _worst(m, pairs, _pinv(m, pairs, (3, 5)), (3, 5)) <= TOL


@pytest.mark.parametrize("n,count,its,small", [
    ((8, 8), 256, (3, 5), True),       # three systems per CU
    ((8, 8), 300, (3, 5), False), ((4, 5), 400, (1, 1), False), ((16, 16), 300, (1, 1), False),
    ((16, 16), 300, (3, 5), True), ((7, 17), 300, (1, 1), True),
])
@pytest.mark.parametrize("precision,tol", [(apfc.APFC_FP64, TOL), (apfc.APFC_MIXED, 2e-5)])
def test_many_tiny_meshes(n, count, its, small, precision, tol):
    """One workgroup per system up to three of them per CU and where a mesh has enough rows and steps; else launches
    over all of them."""
    m = [_mesh(n)] * count
    pairs = (_random(m[:4], 50) * count)[:count]
    assert _half_step_launches(m, its, precision=precision) != small
    got = _pinv(m, pairs, its, precision=precision)
    for q in (0, count - 2):
        assert _worst(m[:2], pairs[q:q + 2], got[q:q + 2], its) <= tol


def test_batch_of_uneven_meshes():
    m = [_mesh(n) for n in ((40, 28), (64, 64), (7, 90), (200, 33))]
    pairs = _random(m, 42)
    assert _worst(m, pairs, _pinv(m, pairs, (3, 5)), (3, 5)) <= TOL


@pytest.mark.parametrize("kind", ["zero", "constant", "mode", "mode+noise"])
def test_small_invariant_spaces(kind):
    """Right-hand sides that CG solves in fewer steps than it is given: the coefficients stay finite and the
    result accurate to the square root of the dropped pivots (1e-14 of H_00, times the condition of OP)."""
    m = _mesh((72, 50))
    X, Y = np.meshgrid(np.arange(72), np.arange(50))
    mode = (np.exp(2j * np.pi * X / 72) + 0.5 * np.exp(-4j * np.pi * Y / 50)).ravel()
    f = {"zero": 0 * mode, "constant": np.ones_like(mode), "mode": mode,
         "mode+noise": mode + 1e-6 * np.random.default_rng(5).normal(size=mode.size)}[kind]
    pairs = [(np.stack([f, 2 * f, 1j * f]), np.stack([f, -f, f]))]
    got = _pinv([m], pairs, (3, 5))
    if kind == "zero":
        assert not np.any(got[0][0]) and not np.any(got[0][1])
    else:
        assert _worst([m], pairs, got, (3, 5)) <= 1e-6


@pytest.mark.parametrize("n,its,dt", [((250, 234), (3, 5), 1.0), ((250, 234), (3, 5), 10.0), ((96, 80), (2, 4), 0.1)])
@pytest.mark.parametrize("kind", ["grain", "mode+1e-4", "mode+1e-6"])
def test_smooth_right_hand_sides(kind, n, its, dt):
    """Right-hand sides as amplitude fields are: a few CG steps solve for most of them, and the later steps work on
    what is left.  CG keeps those steps' digits (5e-16 to 2e-15 per solve against 80-bit arithmetic), so the bound
    is that of rough right-hand sides."""
    m = _mesh(n)
    X, Y = np.meshgrid(np.arange(n[0]), np.arange(n[1]))
    r = np.random.default_rng(45)
    mode = (np.exp(2j * np.pi * X / n[0]) + 0.5 * np.exp(-4j * np.pi * Y / n[1])).ravel()
    w = 0.5 * (1 - np.tanh((np.hypot(X - n[0] / 2, Y - n[1] / 2) - 0.2 * min(n)) / 1.5)).ravel()
    noise = r.normal(size=mode.size) + 1j * r.normal(size=mode.size)
    f = {"grain": 0.16 * (w * np.exp(0.03j * (X - Y)).ravel() + 1 - w), "mode+1e-4": mode + 1e-4 * noise,
         "mode+1e-6": mode + 1e-6 * noise}[kind]
    pairs = [(np.stack([f, 2 * f, 1j * f]), np.stack([f, -f, f[::-1]]))]
    assert _worst([m], pairs, _pinv([m], pairs, its, dt=dt), its, dt=dt) <= TOL


@pytest.mark.parametrize("mass", ["iter", "sep"])
@pytest.mark.parametrize("its", [(1, 1), (2, 1), (1, 2), (2, 2)])
@pytest.mark.parametrize("n", [(121, 25), (250, 234), (530, 500)])    # regions of 16, 16 and 32 rows
def test_shapes_of_the_step_sequence(n, its, mass):
    """Solves of one and two steps, whose first and last steps take other vectors than those between."""
    m = [_mesh(n)]
    pairs = _random(m, 46)
    assert _worst(m, pairs, _pinv(m, pairs, its, mass), its, mass) <= TOL


def test_more_than_a_million_nodes():
    """Regions of 64 rows."""
    m = [_mesh((1040, 1012))]
    pairs = _random(m, 51)
    assert _worst(m, pairs, _pinv(m, pairs, (2, 3)), (2, 3)) <= TOL


def test_large_meshes_in_a_batch():
    """Many regions, uneven systems (regions of 32 rows)."""
    m = [_mesh(n) for n in ((250, 234), (40, 28), (300, 260), (256, 512), (190, 310), (64, 64), (380, 220), (301, 299))]
    pairs = _random(m, 47)
    assert _worst(m, pairs, _pinv(m, pairs, (3, 5)), (3, 5)) <= TOL


@pytest.mark.parametrize("n,its,mass", [((96, 80), (6, 7), "iter"), ((70, 65), (5, 6), "iter"), ((130, 70), (3, 8), "sep")])
def test_longer_solves(n, its, mass):
    """More than five iterations per solve: two launches per step."""
    m = [_mesh(n)]
    pairs = _random(m, 49)
    assert _half_step_launches(m, its, mass)
    assert _worst(m, pairs, _pinv(m, pairs, its, mass), its, mass) <= TOL


def test_step_on_the_static_scratch():
    """The region table also reaches the scratch of step_noalloc: the same step as on a workspace."""
    m = _mesh((50, 67))
    eta = 0.2 * np.ones((3, m.N)) + 1e-2 * _random([m], 43)[0][0]
    out = []
    for entry in ("step", "step_noalloc"):
        s = solver_for([m], apfc.APFC_TRI2D, [0.02], rtol=1e-10, restart=8)
        et, zt = to_dev(eta), torch.zeros((3, 2, m.N), dtype=torch.float64, device="cuda")
        getattr(s, entry)([et], [zt], 1.0)
        out.append((from_dev(et), from_dev(zt)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
