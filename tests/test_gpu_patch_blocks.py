"""The contact patch kernel and the node import/export kernels at the edges of
their blocks of 256 (runs on an MI355X): 4, 256 and 257 contact-eligible
nodes and several blocks with a remainder; nothing, some nodes and every node
in contact; against the FP64 oracle.

Bounds: the device evaluates the contact law in FP64 on both paths, at u
rounded to the path's type. A depth is a difference of lengths up to L, a few
operations of it rounded: 16 eps L; a force is k times that, or 1e-12 of
itself; the resultant adds at most 1e3 entries: 1e-12 of the sum of their
sizes on top. Uploaded displacements come back as they were rounded.
"""
import numpy as np
import pytest

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps
MESHES = {"nodes_4": ((1, 1, 1), 4), "nodes_256": ((5, 9, 8), 256), "nodes_257": ((4, 12, 7), 257),
          "blocks_3": ((13, 12, 9), None)}


@pytest.mark.parametrize("name", list(MESHES))
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_patch_at_block_edges(oracle_lib, name, precision):
    cells, eligible = MESHES[name]
    mesh = W.block_mesh(cells, (0.01, 0.01, 0.01))
    dev = fem.FemMesh(mesh.X, mesh.tets, mesh.fixed, precision=precision)
    orc = oracle_lib.Solver(mesh.X, mesh.tets, mesh.fixed, E=0.3e6, nu=0.45)
    assert eligible in (None, dev.info()["n_eligible"])
    u = W.random_displacement(mesh, 3, 0.01)
    if precision == "fp32":
        u = u.astype(np.float32).astype(np.float64)
    dev.set_displacements(u)
    np.testing.assert_array_equal(dev.displacements(), u)
    far, near, over = (3e-3, [5e-3, 5e-3, 50e-3]), (6e-3, [5e-3, 5e-3, 12e-3]), (100e-3, [5e-3, 4e-3, 6e-3])
    for r, c in (far, near, over):
        print("case", name, precision, r, flush=True)
        k = W.Indentation(W.SPHERE, np.array([r]), np.eye(3), np.array(c), np.array([0.0, 0.0, -1.0]), 0.0, 1).k_penalty
        for s in (dev, orc):
            s.set_indenter(W.SPHERE, np.array([r]), np.eye(3), np.array(c), k)
        ids, f, phi, F = dev.contact_patch()
        ids_r, f_r, phi_r, F_r = orc.contact_patch(u)
        np.testing.assert_array_equal(ids, ids_r)
        depth = 16 * EPS * max(r, 0.05)
        sizes = np.abs(f_r).sum() if len(ids) else 0.0
        np.testing.assert_allclose(phi, phi_r, rtol=0, atol=depth)
        np.testing.assert_allclose(f, f_r, rtol=1e-12, atol=k * depth)
        np.testing.assert_allclose(F, F_r, rtol=0, atol=len(ids) * k * depth + 2e-12 * sizes)
        assert len(ids) == {far[0]: 0, over[0]: dev.info()["n_eligible"]}.get(r, len(ids))
