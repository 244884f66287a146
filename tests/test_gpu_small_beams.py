"""Float64 beams on both sides of the sizes from which they take the element rows
(four damped elements, of a mesh or of a batch in all, or eight undamped ones)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd.api import TLBatch
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu

PLAIN = W.Material(W.SVK, (7e8, 0.33, 0.0))
DAMPED = W.Material(W.SVK, (7e8, 0.33, 0.0), 1e4, 7e3)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 8, 9, 10])
def test_beam_records_and_rows(n):
    print(f"[gpu] small beams {n}", flush=True)
    wl = W.beam_3243(n, 340 + n, "small", material=PLAIN)
    om = oracle.Mesh.of(wl.mesh)
    m = make_mesh(wl, "fp64")
    q, qd = cuda(wl.q), cuda(wl.qdot)
    for mat in (DAMPED, PLAIN, DAMPED):  # one handle: its buffer serves both
        m.set_material(mat)
        f_ref, v_ref = oracle.assemble(om, oracle.material_of(mat), wl.q, wl.qdot, 1e-3, 1.0)
        f, v = m.assemble(q, qd, 1e-3, 1.0)
        torch.cuda.synchronize()
        assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
        assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    m.close()


@pytest.mark.parametrize("sizes", [(1,), (1, 2), (1, 3), (2, 1, 1), (1, 6, 1)])
def test_beam_batch_records_and_rows(sizes):
    print(f"[gpu] small beam batch {sizes}", flush=True)
    wls = [W.beam_3243(n, 350 + i, "small", material=DAMPED if i % 2 else PLAIN) for i, n in enumerate(sizes)]
    handles = [make_mesh(wl, "fp64") for wl in wls]
    b = TLBatch(handles)
    q, qd = (cuda(np.concatenate([getattr(wl, k) for wl in wls])) for k in ("q", "qdot"))
    f, v = b.assemble(q, qd, torch.full((len(wls),), 1e-3, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    for i, wl in enumerate(wls):
        f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material), wl.q, wl.qdot, 1e-3, 1.0)
        assert rel_err(f[b.dof_off[i]:b.dof_off[i + 1]].cpu().numpy(), f_ref)[0] <= TOL["fp64"]
        assert rel_err(v[b.nnz_off[i]:b.nnz_off[i + 1]].cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    b.close()
    for m in handles:
        m.close()
