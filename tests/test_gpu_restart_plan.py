"""Jobs restarted after the launch plan was made for fewer of them (runs on an
MI355X): a run advances every unfinished job, whichever of them the plan of the
last launch held. Each case ends some jobs of a batch so that the teams are
planned anew for the rest, restarts them in their slots and holds every job to
the solver steps of the rounds that follow: 16 a round, of which a Newton
iteration's init and a load step's start take none of the counted passes.
"""
import numpy as np
import pytest

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu


def press(mesh, steps, depth=4e-5, **kw):
    if mesh.name.startswith("fingertip"):
        ind = W.seat_on_mesh(W.random_indentation(5000, steps=steps), mesh)
    else:
        top, c = mesh.X[:, 2].max(), mesh.X.mean(axis=0)
        ind = W.Indentation(W.SPHERE, np.array([3e-3]), np.eye(3), np.array([c[0], c[1], top + 3e-3]),
                            np.array([0.0, 0.0, -1.0]), 0.0, steps)
    ind.depth = depth * steps
    for k, v in kw.items():
        setattr(ind, k, v)
    return ind


def passes(b, j):
    info = b.job_info(j)
    return info["hv_products"] + info["grad_passes"], info["newton_iters"], info["step"]


def run_all_advance(b, ids, rounds):
    """`rounds` rounds, in which every job of ids runs from start to end."""
    before = [passes(b, j) for j in ids]
    assert b.run(max_rounds=rounds) == len(ids)
    for j, old in zip(ids, before):
        new = passes(b, j)
        newton, steps = new[1] - old[1], new[2] - old[2]
        assert 16 * rounds - 2 * newton - 2 * steps - 2 <= new[0] - old[0] <= 16 * rounds, (j, old, new)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_one_of_five_large_jobs(precision):
    """One of five jobs on 50k tets ends: the other four's teams are planned
    over two XCDs each, and the fifth slot is used again."""
    mesh = W.fingertip_mesh(50000)
    b = fem.FemBatch(5, precision)
    mid = b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
    ids = [b.add_job(mid, press(mesh, steps)) for steps in (1, 40, 40, 40, 40)]
    while b.run(max_rounds=4) == 5:
        pass
    print("one ended", precision, flush=True)
    run_all_advance(b, ids[1:], 2)
    b.restart_job(ids[0], press(mesh, 40))
    # a restarted job's counters start from zero
    before = [passes(b, j) for j in ids[1:]]
    assert b.run(max_rounds=2) == 5
    assert passes(b, ids[0])[0] > 16
    assert all(passes(b, j)[0] > old[0] for j, old in zip(ids[1:], before))
    run_all_advance(b, ids, 2)
    b.close()


def test_small_job_beside_a_large_one():
    """Run to the end (the large job's team is planned over all XCDs once the
    small one is done), then both restarted."""
    large, small = W.fingertip_mesh(50000), W.cube_block_mesh()
    b = fem.FemBatch(2, "fp32")
    ml, ms = (b.add_mesh(m.X, m.tets, m.fixed) for m in (large, small))
    ids = [b.add_job(ml, press(large, 3)), b.add_job(ms, press(small, 1))]
    assert b.run() == 0
    print("ended", flush=True)
    b.restart_job(ids[0], press(large, 40))
    b.restart_job(ids[1], press(small, 40))
    assert b.run(max_rounds=2) == 2
    assert all(passes(b, j)[0] > 16 for j in ids)
    run_all_advance(b, ids, 2)
    b.close()


def test_slot_whose_law_changes():
    """The only co-rotational job ends, and its slot takes a Neo-Hookean one."""
    mesh = W.cube_block_mesh()
    b = fem.FemBatch(5, "fp64")
    mid = b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
    ids = [b.add_job(mid, press(mesh, 1, model=1))] + [b.add_job(mid, press(mesh, 40)) for _ in range(4)]
    while b.run(max_rounds=4) == 5:
        pass
    print("co-rotational job ended", flush=True)
    run_all_advance(b, ids[1:], 2)
    b.restart_job(ids[0], press(mesh, 40))
    assert b.run(max_rounds=2) == 5
    assert all(passes(b, j)[0] > 16 for j in ids)
    run_all_advance(b, ids, 2)
    b.close()
