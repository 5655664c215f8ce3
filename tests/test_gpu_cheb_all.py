"""The 2D Chebyshev preconditioner in one launch (meshes whose regions all fit on the chip at once) and, just
above that size, in three, against the oracle's four steps, element by element.  Needs an MI355X."""
import re

import numpy as np
import pytest

from oracle.apfc_oracle import tri_k
from paper_1902_09761_amd import apfc, inputs
from tests.gpu_util import H_TRI, from_dev, families_of_a_step, kernels_of, oracle_for, rel_l2, solver_for, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(n):
    return inputs.Mesh(2, (n[0], n[1], 1), (n[0] * H_TRI, n[1] * H_TRI, 1.0))


def _worst(meshes, precision, its, sep, region=0, dt=0.7):
    r = np.random.default_rng(51)
    ins = [tuple(r.normal(size=(3, m.N)) + 1j * r.normal(size=(3, m.N)) for _ in range(2)) for m in meshes]
    s = solver_for(meshes, apfc.APFC_TRI2D, [0.02] * len(meshes), inner_kind=apfc.APFC_INNER_CHEB, precision=precision,
                   mass_iters=its[0], diff_iters=its[1],
                   mass_kind=apfc.APFC_MASS_SEPARABLE if sep else apfc.APFC_MASS_ITER)
    s.set_tiles(16, region)
    zo = [torch.zeros((3, 2, m.N), dtype=torch.float64, device="cuda") for m in meshes]
    eo = [torch.zeros_like(z) for z in zo]
    s.apply(apfc.APFC_OP_PINV, [to_dev(z) for z, _ in ins], [to_dev(e) for _, e in ins], zo, eo, dt)
    worst = 0.0
    for m, (z, e), gz, ge in zip(meshes, ins, map(from_dev, zo), map(from_dev, eo)):
        o = oracle_for(m, tri_k(), 0.02)
        for j in range(3):
            ref = np.concatenate(o.precond_apply(j, z[j], e[j], dt, inner="cheb", mass_iters=its[0], diff_iters=its[1],
                                                 mass="sep" if sep else "iter"))
            worst = max(worst, float(np.max(np.abs(np.concatenate([gz[j], ge[j]]) - ref)) / np.max(np.abs(ref))))
    return worst


@pytest.mark.parametrize("precision,tol", [(apfc.APFC_FP64, 1e-12), (apfc.APFC_MIXED, 2e-5)])
@pytest.mark.parametrize("n,its,sep", [
    ((4, 4), (3, 3), True),        # every neighbour a wrap onto the mesh itself
    ((46, 14), (3, 3), True),      # one region, filled exactly
    ((47, 15), (3, 3), True),      # one node more in each direction
    ((130, 118), (4, 3), True),    # the longest filter, the largest halo
    ((61, 90), (1, 1), True),
    ((96, 80), (5, 3), False),     # Chebyshev mass solve
    ((50, 33), (1, 1), False),     # no stencil in the L solves
    ((320, 250), (3, 3), True),    # more regions than CUs: three launches
])
def test_matches_oracle(n, its, sep, precision, tol):
    assert _worst([_mesh(n)], precision, its, sep, region=1) <= tol


def test_batch_of_uneven_meshes():
    assert _worst([_mesh(n) for n in ((40, 28), (130, 9), (7, 90))], apfc.APFC_FP64, (3, 3), True) <= 1e-12


def test_forms_the_basis_vectors():
    """Inside FGMRES the launch also forms and stores both halves of every basis vector: steps against the
    oracle's direct solve."""
    m = _mesh((50, 45))
    r = np.random.default_rng(52)
    eta = 0.2 + 1e-2 * (r.normal(size=(3, m.N)) + 1j * r.normal(size=(3, m.N)))
    o = oracle_for(m, tri_k(), 0.02)
    s = solver_for([m], apfc.APFC_TRI2D, [0.02], rtol=1e-12, inner_kind=apfc.APFC_INNER_CHEB, precision=apfc.APFC_MIXED,
                   mass_kind=apfc.APFC_MASS_SEPARABLE, mass_iters=3, diff_iters=3, restart=4, x0_order=3)
    et, zt = to_dev(eta), torch.zeros((3, 2, m.N), dtype=torch.float64, device="cuda")
    s.init_zeta([et], [zt])
    ref = eta
    for _ in range(2):
        _, ref = o.step(ref, 1.0)
        s.step([et], [zt], 1.0)
    assert rel_l2(from_dev(et), ref) <= 1e-9


def _shapes(names):
    """Region shapes (columns, rows) of the three-launch kernel among kernel names."""
    return {tuple(map(int, m)) for n in names for m in re.findall(r"k_cheb2d<\w+, \d+, (\d+), (\d+),", n)}


SHAPES = [(128, 32), (64, 32), (64, 64), (128, 36), (128, 64), (256, 32)]


def test_autotune_times_the_region_shapes():
    """On a mesh that takes one launch the search still runs every region shape: Krylov indices above 8 use it."""
    s = solver_for([_mesh((96, 80))], apfc.APFC_TRI2D, [0.02], inner_kind=apfc.APFC_INNER_CHEB, mass_iters=3, diff_iters=3,
                   mass_kind=apfc.APFC_MASS_SEPARABLE)
    seen = set()
    for _ in range(4):      # the profiler may miss a kernel
        seen |= _shapes(kernels_of(s.autotune))
        if len(seen) == len(SHAPES):
            break
    assert seen == set(SHAPES)


@pytest.mark.parametrize("precision,tol", [(apfc.APFC_FP64, 1e-12), (apfc.APFC_MIXED, 2e-5)])
@pytest.mark.parametrize("region,taps", [(0, 1), (1, 2), (2, 4), (3, 3), (4, 1), (5, 2), (0, 3), (4, 4)])
def test_three_launches_with_the_separable_stage(region, taps, precision, tol):
    """Every region shape and tap count on a mesh of more regions than CUs: three launches per application."""
    m = [_mesh((331, 257))]
    s = solver_for(m, apfc.APFC_TRI2D, [0.02], rtol=1e-4, inner_kind=apfc.APFC_INNER_CHEB, precision=precision, restart=4,
                   mass_iters=taps, diff_iters=3, mass_kind=apfc.APFC_MASS_SEPARABLE)
    s.set_tiles(16, region)
    n = families_of_a_step(s, m)
    assert n["cheb"] == 3 * n["apply"] > 0
    assert _worst(m, precision, (taps, 3), True, region=region) <= tol
