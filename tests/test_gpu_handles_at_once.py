"""Several handles in use at a time on one device (runs on an MI355X): results
as alone, and nobody waits for another's whole run or launch. The host's calls
release the interpreter lock, so threads overlap as a program's would.

Time bounds: a launch of teams ends within 16 solver steps (3 ms of the batch
here) of another handle's call, and within 20 ms anyway; the batch's run to the
end takes more than half a second. 60 ms leaves room for the host.
"""
import ctypes as C
import threading
import time

import numpy as np
import pytest
import torch

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu

SOON = 0.06


def launches(h):
    t, s = C.c_int64(), C.c_int64()
    assert fem.load().fem_debug_team_launches(h, C.byref(t), C.byref(s)) == 0
    return t.value, s.value


class BigBatch:
    """256 jobs on the 50k fingertip, which hold every XCD, in a thread."""

    def __init__(self, steps=8):
        mesh = W.fingertip_mesh(50000)
        self.b = fem.FemBatch(256, "fp32")
        mid = self.b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
        self.inds = [W.seat_on_mesh(W.random_indentation(3000 + i, steps=steps), mesh) for i in range(256)]
        for ind in self.inds:
            ind.depth = max(ind.depth, 0.5e-3) * steps / 100.0
        self.ids = [self.b.add_job(mid, ind) for ind in self.inds]
        assert self.b.run(max_rounds=1) == 256   # tables and plan made

    def start(self):
        for j, ind in zip(self.ids, self.inds):
            self.b.restart_job(j, ind)
        self.thread = threading.Thread(target=self.b.run)
        self.thread.start()
        time.sleep(0.05)

    def join(self):
        self.thread.join()
        return [self.b.displacements(j) for j in self.ids]


def evaluation(mesh, u):
    d = fem.FemMesh(mesh.X, mesh.tets, mesh.fixed, precision="fp64")
    d.set_material(0.3e6, 0.45, 1100.0)
    d.set_indenter(W.SPHERE, np.array([3e-3]), np.eye(3), np.array([5e-3, 5e-3, 13e-3 - 4e-4]), 1e3)
    d.set_displacements(u)
    return d


def test_evaluations_beside_a_batch():
    mesh = W.cube_block_mesh()
    u = W.random_displacement(mesh, 5, 0.005)
    d = evaluation(mesh, u)
    g0 = d.gradient()[0]
    big = BigBatch()
    big.start()
    alone = big.join()
    big.start()
    took = []
    while big.thread.is_alive() and len(took) < 12:
        t = time.perf_counter()
        g = d.gradient()[0]
        took.append(time.perf_counter() - t)
        assert np.abs(g - g0).max() <= 1e-12 * np.abs(g0).max()
        time.sleep(0.01)
    print("gradients beside the batch, ms:", [round(1e3 * t, 2) for t in took], flush=True)
    beside = big.join()
    print("batch launches", launches(big.b.h), flush=True)
    assert len(took) >= 5 and max(took) < SOON
    for a, b in zip(alone, beside):
        assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()
    big.b.close()
    d.close()


def test_other_streams_beside_a_batch():
    """Work that is not the library's, on a stream of its own: a matrix
    product, whose blocks don't fit beside the batch's."""
    x = torch.ones(2048, 2048, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        y = x @ x
        s.synchronize()
    big = BigBatch()
    big.start()
    took = []
    with torch.cuda.stream(s):
        while big.thread.is_alive() and len(took) < 12:
            t = time.perf_counter()
            y = x @ x
            s.synchronize()
            took.append(time.perf_counter() - t)
            time.sleep(0.01)
    print("kernels beside the batch, ms:", [round(1e3 * t, 2) for t in took], flush=True)
    big.join()
    assert len(took) >= 5 and max(took) < SOON
    assert float(y[0, 0]) == 2048.0
    big.b.close()


@pytest.mark.parametrize("count", [2, 4, 8])
def test_single_jobs_at_once(count):
    """Batches of one job that takes most of an XCD (20k tets in FP64), in
    threads: each has an XCD of its own, so the teams take them to the end, and
    results are those of the batch alone (1e-9: both end below 1e-10)."""
    mesh = W.fingertip_mesh(20000)
    inds = [W.seat_on_mesh(W.random_indentation(5000 + i, steps=2), mesh) for i in range(count)]
    for ind in inds:
        ind.depth = 8e-5
    batches = []
    for ind in inds:
        b = fem.FemBatch(1, "fp64")
        b.add_job(b.add_mesh(mesh.X, mesh.tets, mesh.fixed), ind)
        batches.append((b, b.default_params(newton_rtol=1e-10, cg_rtol=1e-10)))
    alone = []
    for b, P in batches:
        assert b.run(P) == 0
        alone.append(b.displacements(0))
    print("alone done", flush=True)
    gate = threading.Barrier(count)

    def again(k):
        b, P = batches[k]
        gate.wait()
        for _ in range(4):
            b.restart_job(0, inds[k])
            b.run(P)

    threads = [threading.Thread(target=again, args=(k,)) for k in range(count)]
    t = time.perf_counter()
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    print("at once", count, round(1e3 * (time.perf_counter() - t), 1), "ms", [launches(b.h) for b, _ in batches], flush=True)
    for (b, _), u in zip(batches, alone):
        assert np.abs(b.displacements(0) - u).max() <= 1e-9 * np.abs(u).max()
        assert launches(b.h)[1] == 0
        b.close()


def test_handles_made_beside_a_batch():
    """Making and closing a handle allocates and frees, which waits for the
    device several times; each of them takes little longer than alone."""
    mesh = W.cube_block_mesh()
    u = W.random_displacement(mesh, 5, 0.005)

    def life():
        t = [time.perf_counter()]
        d = evaluation(mesh, u)
        t.append(time.perf_counter())
        d.close()
        return t[1] - t[0], time.perf_counter() - t[1]

    life()
    alone = life()
    big = BigBatch()
    big.start()
    took = [life()]
    while big.thread.is_alive():
        took.append(life())
    big.join()
    print("made and closed, ms: alone", [round(1e3 * t, 1) for t in alone], "beside",
          [[round(1e3 * t, 1) for t in x] for x in took], flush=True)
    for made, closed in took:
        assert made < alone[0] + SOON and closed < alone[1] + SOON
    big.b.close()
