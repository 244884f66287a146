"""T10 element rows in mixed precision on both sides of the sizes where their launch
changes: from 24,576 damped or 32,768 undamped elements on the stores pass the
caches (a mesh, a batch per item and a batch with the persistent schedule), up to
682 damped tiles each row component has a workgroup of its own."""
import dataclasses

import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd.api import TLBatch
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("damped,n", [(True, 24576), (True, 24577), (False, 32768), (False, 32769)])
def test_rows_through_and_past_the_caches(damped, n):
    print(f"[gpu] row stores damped={damped} {n}", flush=True)
    mat = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), *((1e3, 7e2) if damped else ()))
    wl = W.t10_beam(1366, 2, 2, 330, "stores", lx=17.075, ly=0.025, lz=0.025, material=mat)
    wl = dataclasses.replace(wl, mesh=dataclasses.replace(wl.mesh, conn=wl.mesh.conn[:n].copy()))
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(mat), wl.q, wl.qdot, 1e-3, 1.0)
    m = make_mesh(wl, "mixed")
    q, qd = cuda(wl.q), cuda(wl.qdot)
    b = TLBatch([m])
    h = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    outs = [m.assemble(q, qd, 1e-3, 1.0), b.assemble(q, qd, h)]
    for tile in (25, 16):
        b.set_schedule(True, tile)
        outs.append(b.assemble(q, qd, h))
    torch.cuda.synchronize()
    for f, v in outs:
        assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["mixed"]
        assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["mixed"]
    b.close()
    m.close()


@pytest.mark.parametrize("n", [1, 681, 682, 683])
def test_row_components_split_over_workgroups(n):
    print(f"[gpu] split rows {n}", flush=True)
    mat = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), 1e3, 7e2)
    wl = W.t10_beam(29, 2, 2, 331, "split", lx=0.3625, ly=0.025, lz=0.025, material=mat)
    wl = dataclasses.replace(wl, mesh=dataclasses.replace(wl.mesh, conn=wl.mesh.conn[:n].copy()))
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(mat), wl.q, wl.qdot, 1e-3, 1.0)
    m = make_mesh(wl, "mixed")
    f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), 1e-3, 1.0)
    f_only = torch.empty_like(f)
    m.assemble_nodes(f_only)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["mixed"]
    assert rel_err(f_only.cpu().numpy(), f_ref)[0] <= TOL["mixed"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["mixed"]
    m.close()
