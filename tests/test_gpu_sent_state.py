"""Calls in a row on one handle and one batch, each with parameters, a pose or
states of its own (runs on an MI355X): parameters are sent to the device only
when they differ from those there, and states without a wait, so every call is
held against a handle that made no other call.

Bound: FP64 evaluations that differ in the order of LDS additions alone, 24
contributions a node: 1e-12 of the largest entry.
"""
import numpy as np
import pytest

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu


def handle(mesh, u):
    d = fem.FemMesh(mesh.X, mesh.tets, mesh.fixed, precision="fp64")
    d.set_material(0.3e6, 0.45, 1100.0)
    d.set_displacements(u)
    return d


def pose(d, z):
    d.set_indenter(W.SPHERE, np.array([3e-3]), np.eye(3), np.array([5e-3, 5e-3, 13e-3 - z]), 1e3)


@pytest.mark.parametrize("order", [(0, 1, 0), (1, 1, 0)])
def test_calls_in_a_row_equal_calls_alone(order):
    mesh = W.cube_block_mesh()
    u = W.random_displacement(mesh, 5, 0.005)
    v = np.random.default_rng(6).uniform(-1.0, 1.0, size=mesh.X.shape)
    row = handle(mesh, u)
    for k, full in enumerate(order):
        print("case", order, k, flush=True)
        alone = handle(mesh, u)
        for d in (row, alone):
            pose(d, 4e-4 * (k + 1))
        got, want = ([d.hessvec(v, d.default_params(contact_hessian=full)), d.gradient()[0], d.contact_patch()[1],
                      d.tet_stress()[0], d.hessvec(v, d.default_params(contact_hessian=1 - full))]
                     for d in (row, alone))
        for a, b in zip(got, want):
            assert a.shape == b.shape and np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
        assert not np.allclose(got[0], got[4], rtol=1e-9, atol=0)   # the parameter matters here
        alone.close()
    row.close()


def test_jobs_restarted_twice_before_a_run():
    """The second restart replaces the first before any kernel ran the job."""
    mesh = W.cube_block_mesh()

    def ind(depth):
        return W.Indentation(W.SPHERE, np.array([3e-3]), np.eye(3), np.array([5e-3, 5e-3, 13e-3]),
                             np.array([0.0, 0.0, -1.0]), depth, 2)

    def solved(depths):
        b = fem.FemBatch(2, "fp64")
        P = b.default_params(newton_rtol=1e-10, cg_rtol=1e-10)
        mid = b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
        ids = [b.add_job(mid, ind(1e-4)) for _ in range(2)]
        for depth in depths:
            for j in ids:
                b.restart_job(j, ind(depth), 0.3e6, 0.45)
        assert b.run(P) == 0
        out = [b.displacements(j) for j in ids]
        b.close()
        return out

    for a, b in zip(solved((1e-4, 2e-4)), solved((2e-4,))):
        assert np.abs(a - b).max() <= 1e-9 * np.abs(b).max()
