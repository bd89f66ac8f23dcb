"""One job on meshes around the line from which its team spans several XCDs (56
tile and contact blocks in FP64, 64 in FP32), against the step kernels (runs on
an MI355X). Bounds: 1e-9 of the largest displacement in FP64, 1e-5 in FP32, as
for the team kernel at the other sizes."""
import numpy as np
import pytest

from paper_2103_16747_amd import fem, workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("h_mm", [1.06, 1.0, 0.95, 0.92])
def test_either_side_of_the_line(h_mm, precision):
    mesh = W.fingertip_mesh(h=h_mm * 1e-3)
    ind = W.seat_on_mesh(W.random_indentation(5000, steps=1), mesh)
    ind.depth = 6e-5
    out = []
    for graphs in (1, 0):
        b = fem.FemBatch(1, precision)
        b.set_graphs(graphs)
        P = b.default_params(newton_rtol=1e-10, cg_rtol=1e-10) if precision == "fp64" else b.default_params()
        mid = b.add_mesh(mesh.X, mesh.tets, mesh.fixed)
        info = b.mesh_info(mid)
        j = b.add_job(mid, ind)
        assert b.run(P) == 0 and b.job_info(j)["steps_failed"] == 0
        out.append(b.displacements(j))
        b.close()
    print(precision, "blocks", info["n_tiles"] + (info["n_eligible"] + 255) // 256, flush=True)
    assert np.abs(out[0] - out[1]).max() <= {"fp64": 1e-9, "fp32": 1e-5}[precision] * np.abs(out[1]).max()
