"""Float64 point records of shell and beam meshes created in mixed precision, whose
default launch shape has eight waves: few ranges, more ranges than CUs, a shape set
by the caller, and a batch; and the force alone from mixed row blocks."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd.api import TLBatch
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu


def shell(n):
    mat = W.Material(W.SVK, (7e8, 0.33, 0.0), 1e4, 7e3)
    wl = W.shell_plate(n, 380 + n, "waves")
    return dataclasses.replace(wl, material=mat, qdot=np.random.default_rng(n).normal(0.0, 0.05, wl.q.shape))


@pytest.mark.parametrize("n,shape", [(4, None), (27, None), (30, None), (30, (8, 768, 4096)), (30, (1, 768, 4096))])
def test_records_of_a_mesh_created_mixed(n, shape):
    print(f"[gpu] record waves {n} {shape}", flush=True)
    wl = shell(n)
    m = make_mesh(wl, "mixed")
    if shape:
        m.set_gather_shape(*shape)
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material), wl.q, wl.qdot, 1e-3, 1.0)
    q, qd = cuda(wl.q), cuda(wl.qdot)
    for precision in ("mixed", "fp64"):
        m.set_precision(precision)
        f, v = m.assemble(q, qd, 1e-3, 1.0)
        f_only = torch.empty_like(f)
        m.assemble_nodes(f_only)
        torch.cuda.synchronize()
        for got, ref in ((f, f_ref), (v, v_ref), (f_only, f_ref)):
            assert rel_err(got.cpu().numpy(), ref)[0] <= TOL[precision]
    b = TLBatch([m])
    f, v = b.assemble(q, qd, torch.full((1,), 1e-3, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    b.close()
    m.close()
