"""Which kernels take a run, and the counters that decide it (runs on an MI355X).

Results are held to the step kernels' as in the team kernel's own tests: 1e-9
of the largest displacement in FP64.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu


def block_jobs(count, steps):
    mesh = W.cube_block_mesh()
    return mesh, [W.Indentation(W.SPHERE, np.array([3e-3]), np.eye(3), np.array([5e-3, 5e-3, 13e-3]),
                                np.array([0.0, 0.0, -1.0]), 4e-5 * steps * (1 + i % 3), steps) for i in range(count)]


class Batch:
    def __init__(self, mesh, inds, graphs=1):
        self.b = fem.FemBatch(len(inds), "fp64")
        self.b.set_graphs(graphs)
        self.P = self.b.default_params(newton_rtol=1e-10, cg_rtol=1e-10)
        mid = self.b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
        self.inds, self.ids = inds, [self.b.add_job(mid, ind) for ind in inds]

    def restart(self):
        for j, ind in zip(self.ids, self.inds):
            self.b.restart_job(j, ind)

    def launches(self):
        t, s = C.c_int64(), C.c_int64()
        assert fem.load().fem_debug_team_launches(self.b.h, C.byref(t), C.byref(s)) == 0
        return t.value, s.value

    def displacements(self):
        return [self.b.displacements(j) for j in self.ids]


def reference(mesh, inds):
    r = Batch(mesh, inds, graphs=0)
    assert r.b.run(r.P) == 0
    u = r.displacements()
    r.b.close()
    return u


def close_to(us, refs):
    for u, ref in zip(us, refs):
        assert np.abs(u - ref).max() <= 1e-9 * np.abs(ref).max()


@pytest.mark.parametrize("jobs", [1, 12])
def test_counters_that_wrap(jobs):
    """Counters just below 2^32 wrap in the first run; it and the next are
    taken by the team kernel alone and give what the step kernels give."""
    mesh, inds = block_jobs(jobs, 2)
    ref = reference(mesh, inds)
    t = Batch(mesh, inds)
    assert fem.load().fem_debug_team_counters(t.b.h, C.c_uint32(2**32 - 1 - jobs // 2)) == 0
    for k in range(3):
        print("case", jobs, k, flush=True)
        before = t.launches()
        assert t.b.run(t.P) == 0
        close_to(t.displacements(), ref)
        after = t.launches()
        assert after[0] > before[0] and after[1] == before[1]
        t.restart()
    t.b.close()


def test_round_of_a_single_job():
    """One job's round has the expected length of its Newton iteration: 16 CG
    iterations before the first solve, then those of the solve before, and
    three steps more at the start of an iteration, rounded up to the lengths of
    captured rounds, 4 to 64 solver steps. At the FP64 tolerance solves take
    more than 40 iterations on this mesh, so such rounds are among them. A round
    that ends between a trial and its init is counted one off."""
    mesh, inds = block_jobs(1, 3)
    t = Batch(mesh, inds)

    def steps():   # CG iterations, gradients and trials, and the inits behind accepted trials
        info = t.b.job_info(t.ids[0])
        return info["hv_products"] + info["grad_passes"] + info["newton_iters"]

    took, last = [], 0
    while t.b.run(t.P, max_rounds=1):
        took.append(steps() - last)
        last = steps()
    print("rounds", took, flush=True)
    assert abs(took[0] - 20) <= 1
    assert min(took) >= 3 and 40 <= max(took) <= 65
    t.b.close()


def absent(t, workgroups):
    assert fem.load().fem_debug_team_absent(t.b.h, C.c_int32(workgroups)) == 0


def test_teams_that_do_not_meet_in_a_run_of_rounds():
    """Twelve jobs, two teams on four of the XCDs, one on the others; launches
    leave out one workgroup per XCD, so that the second team of an XCD does not
    meet. Every job still takes the solver steps of its rounds, no fewer and no
    more, and ends as the step kernels end it."""
    mesh, inds = block_jobs(12, 3)
    ref = reference(mesh, inds)
    t = Batch(mesh, inds)
    absent(t, 1)

    def steps(j):
        info = t.b.job_info(j)
        return info["hv_products"] + info["grad_passes"], info["newton_iters"], info["step"]

    for rounds in (2, 3):
        before = [steps(j) for j in t.ids]
        assert t.b.run(t.P, max_rounds=rounds) == 12
        print("rounds", rounds, t.launches(), flush=True)
        for j, old in zip(t.ids, before):
            new = steps(j)
            assert 16 * rounds - 2 * (new[1] - old[1]) - 2 * (new[2] - old[2]) - 2 <= new[0] - old[0] <= 16 * rounds
    assert t.b.run(t.P) == 0
    close_to(t.displacements(), ref)
    t.b.close()


def test_teams_that_never_meet_are_left_alone():
    """The only team of a job lacks a member: the step kernels take the job,
    teams are not tried again for a number of rounds, and then they are."""
    mesh, inds = block_jobs(1, 2)
    ref = reference(mesh, inds)
    t = Batch(mesh, inds)
    absent(t, 1)
    for k in range(40):   # short runs, each of which would wait for the meeting
        assert t.b.run(t.P, max_rounds=1) == 1
        t.restart()
    tries, rounds = t.launches()
    print("tries", tries, "rounds", rounds, flush=True)
    assert tries == 1 and rounds == 40
    assert t.b.run(t.P) == 0
    close_to(t.displacements(), ref)
    t.restart()
    tries = t.launches()[0]
    absent(t, 0)
    for k in range(200):
        assert t.b.run(t.P) == 0
        close_to(t.displacements(), ref)
        t.restart()
        if t.launches()[0] > tries:
            break
    before = t.launches()
    assert before[0] > tries
    assert t.b.run(t.P) == 0
    close_to(t.displacements(), ref)
    assert t.launches()[0] > before[0] and t.launches()[1] == before[1]
    t.b.close()


def test_streams_of_the_caller():
    """Two batches on streams that the program made, one after another."""
    mesh, inds = block_jobs(3, 2)
    ref = reference(mesh, inds)
    for stream in (torch.cuda.Stream(), torch.cuda.current_stream()):
        b = fem.FemBatch(len(inds), "fp64", stream=stream)
        P = b.default_params(newton_rtol=1e-10, cg_rtol=1e-10)
        mid = b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
        ids = [b.add_job(mid, ind) for ind in inds]
        for _ in range(2):
            assert b.run(P) == 0
            close_to([b.displacements(j) for j in ids], ref)
            for j, ind in zip(ids, inds):
                b.restart_job(j, ind)
        b.close()
