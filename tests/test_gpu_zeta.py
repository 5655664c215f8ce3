"""zeta = M^{-1} G eta by one line filter per direction (apfc_init_zeta; the energy and its gradient use the same
field) against the oracle's direct mass solve.  Needs an MI355X."""
import ctypes
import time

import numpy as np
import pytest

from oracle.apfc_oracle import bcc_k, fcc_k, tri_k
from paper_1902_09761_amd import apfc, inputs
from tests.gpu_util import H_TRI, from_dev, oracle_for, rel_l2, solver_for, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(n):
    return inputs.Mesh(len(n), tuple(n) + (1,) * (3 - len(n)), tuple(m * H_TRI for m in n) + (1.0,) * (3 - len(n)))


# lines shorter than the recursions' start (32 nodes, wrapped several times), ends of the 8-node blocks, of the
# 32-node segments and of the 448-node segments of an x line
@pytest.mark.parametrize("n", [(4, 4), (5, 33), (31, 32), (64, 65), (447, 4), (448, 31), (449, 8), (897, 5),
                               (4, 5, 6), (9, 33, 4), (70, 4, 65)])
def test_zeta_matches_direct_mass_solve(n):
    """Random amplitudes (no smoothness): the condition of M (9 in 2D, 27 in 3D) times FP64 rounding, with room for
    the direct solve's own error: 1e-13 relative."""
    mesh = _mesh(n)
    kind, k = (apfc.APFC_TRI2D, tri_k()) if len(n) == 2 else (apfc.APFC_BCC3D, bcc_k())
    rng = np.random.default_rng(17)
    eta = rng.normal(size=(len(k), mesh.N)) + 1j * rng.normal(size=(len(k), mesh.N))
    s = solver_for([mesh], kind, [0.02])
    z = torch.full((len(k), 2, mesh.N), float("nan"), dtype=torch.float64, device="cuda")
    s.init_zeta([to_dev(eta)], [z])
    ref = oracle_for(mesh, k, 0.02).zeta_of(eta)
    assert rel_l2(from_dev(z), ref) <= 1e-13


def test_zeta_energy_gradient_of_an_uneven_batch():
    """Instances of different sizes share the launches; a NaN in one stays there.  Energy 1e-12 and gradient 1e-12
    (sums of a few thousand terms of like size)."""
    meshes = [_mesh(n) for n in ((12, 40), (70, 9), (33, 33))]
    k = tri_k()
    rng = np.random.default_rng(3)
    etas = [0.2 * (rng.normal(size=(3, m.N)) + 1j * rng.normal(size=(3, m.N))) for m in meshes]
    dev = [to_dev(e) for e in etas]
    dev[1][0, 0, 5] = float("nan")
    s = solver_for(meshes, apfc.APFC_TRI2D, [0.02, 0.03, 0.04])
    grads = [torch.empty_like(e) for e in dev]
    E = s.energy(dev)
    ddB = s.energy_grad(dev, grads)
    assert np.isnan(E[1]) and np.isnan(ddB[1])
    for b, dB in ((0, 0.02), (2, 0.04)):
        o = oracle_for(meshes[b], k, dB)
        assert abs(E[b] - o.energy(etas[b])) <= 1e-12 * abs(o.energy(etas[b]))
        assert rel_l2(from_dev(grads[b]), o.energy_grad(etas[b])) <= 1e-12
        assert abs(ddB[b] - o.energy_ddB(etas[b])) <= 1e-12 * abs(o.energy_ddB(etas[b]))


@pytest.mark.parametrize("rows", [4, 32])
@pytest.mark.parametrize("ns", [((200, 150), (6, 5), (4, 70), (5, 4), (11, 9)), ((70, 4, 8), (4, 4, 4), (5, 9, 4), (4, 6, 5))])
def test_zeta_of_one_large_and_several_small_meshes(ns, rows):
    """Meshes of very different sizes share out each system's lines over its tiles, also where tiles are fewer than
    the workgroups that the lines would fill (70 x 4 x 8 by tiles of 32 rows)."""
    meshes = [_mesh(n) for n in ns]
    kind, k = (apfc.APFC_TRI2D, tri_k()) if len(ns[0]) == 2 else (apfc.APFC_BCC3D, bcc_k())
    rng = np.random.default_rng(19)
    etas = [rng.normal(size=(len(k), m.N)) + 1j * rng.normal(size=(len(k), m.N)) for m in meshes]
    s = solver_for(meshes, kind, [0.02] * len(meshes))
    s.set_tiles(rows)
    zs = [torch.full((len(k), 2, m.N), float("nan"), dtype=torch.float64, device="cuda") for m in meshes]
    s.init_zeta([to_dev(e) for e in etas], zs)
    for m, e, z in zip(meshes, etas, zs):
        assert rel_l2(from_dev(z), oracle_for(m, k, 0.02).zeta_of(e)) <= 1e-13


def test_time_of_a_batch_follows_its_nodes():
    """One 1024^2 and 511 meshes of 16^2 (an eighth more nodes) in at most four times the time of the large one alone;
    as many workgroups for a small mesh as for the large one made the kernels take thirty times as long.  Calls of the C
    entry point (the binding checks 512 tensors per call)."""
    large, small = _mesh((1024, 1024)), _mesh((16, 16))
    stream = torch.cuda.current_stream().cuda_stream

    def best(meshes):
        s = solver_for(meshes, apfc.APFC_TRI2D, [0.02] * len(meshes))
        etas = [torch.zeros((3, 2, m.N), dtype=torch.float64, device="cuda") for m in meshes]
        zs = [torch.zeros_like(e) for e in etas]
        states = s._states(etas, zs)
        torch.cuda.synchronize()
        t = []
        for _ in range(8):
            t0 = time.perf_counter()
            assert apfc.lib().apfc_init_zeta(s.ctx, states, ctypes.c_void_p(stream)) == 0
            t.append(time.perf_counter() - t0)
        return min(t)

    alone, batch = best([large]), best([large] + [small] * 511)
    print("1024^2:", 1e6 * alone, "with 511 of 16^2:", 1e6 * batch, "us")
    assert batch <= 4 * alone


def test_fcc_energy_gradient():
    """Seven amplitudes: the nodal part's eight-slot instance, rows shared by more tiles than a tile has rows."""
    mesh = _mesh((9, 6, 11))
    k = fcc_k()
    rng = np.random.default_rng(5)
    eta = 0.2 * (rng.normal(size=(7, mesh.N)) + 1j * rng.normal(size=(7, mesh.N)))
    s = solver_for([mesh], apfc.APFC_FCC3D, [0.02])
    g = torch.empty((7, 2, mesh.N), dtype=torch.float64, device="cuda")
    o = oracle_for(mesh, k, 0.02)
    for rows in (4, 16):
        s.set_tiles(rows)
        assert abs(s.energy([to_dev(eta)])[0] - o.energy(eta)) <= 1e-12 * abs(o.energy(eta))
        ddB = s.energy_grad([to_dev(eta)], [g])[0]
        assert rel_l2(from_dev(g), o.energy_grad(eta)) <= 1e-12
        assert abs(ddB - o.energy_ddB(eta)) <= 1e-12 * abs(o.energy_ddB(eta))
