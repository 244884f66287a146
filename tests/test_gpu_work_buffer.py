"""The work buffer of a large float64 T10 mesh across changes of the material and
the precision: no call allocates where the handle held what the form before it
needed, and work captured on the handle stays valid."""
import dataclasses

import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu

PLAIN = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8))
DAMPED = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), 1e3, 7e2)


def big_body(material, n=49153):  # above the line of the float64 element rows
    wl = W.t10_beam(2049, 2, 2, 300, "work", lx=25.6, ly=0.025, lz=0.025, material=material)
    return dataclasses.replace(wl, mesh=dataclasses.replace(wl.mesh, conn=wl.mesh.conn[:n].copy()))


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("first", ["undamped", "mixed"])
def test_material_and_precision_keep_the_buffer(first):
    print(f"[gpu] work buffer {first}", flush=True)
    wl = big_body(PLAIN if first == "undamped" else DAMPED)
    precision = "fp64" if first == "undamped" else "mixed"
    m = make_mesh(wl, precision)
    om = oracle.Mesh.of(wl.mesh)
    q, qd = cuda(wl.q), cuda(wl.qdot)
    f, v = m.assemble(q, qd, 1e-3, 1.0)
    f0, v0 = f.clone(), v.clone()
    before = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(before):
        m.assemble(q, qd, 1e-3, 1.0, f=f, vals=v)
    free = free_bytes()
    if first == "undamped":
        m.set_material(DAMPED)
    else:
        m.set_precision("fp64")
    m.assemble(q, qd, 1e-3, 1.0, f=f, vals=v)
    assert free_bytes() == free  # the second form found its buffer
    f_ref, v_ref = oracle.assemble(om, oracle.material_of(DAMPED), wl.q, wl.qdot, 1e-3, 1.0)
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"] and rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    after = torch.cuda.CUDAGraph()
    with torch.cuda.graph(after):
        m.assemble(q, qd, 1e-3, 1.0, f=f, vals=v)
    for _ in range(3):
        f.zero_(), v.zero_()
        before.replay()
        torch.cuda.synchronize()
        assert rel_err(f.cpu().numpy(), f0.cpu().numpy())[0] <= TOL[precision]
        assert rel_err(v.cpu().numpy(), v0.cpu().numpy())[0] <= TOL[precision]
        f.zero_(), v.zero_()
        after.replay()
        torch.cuda.synchronize()
        assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"] and rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    m.close()


def test_a_damped_mesh_of_its_own_takes_the_rows():
    """A handle whose first tangent is damped float64 sizes its buffer for the rows
    (7,680 bytes an element; the records take 3,840)."""
    print("[gpu] work buffer rows", flush=True)
    wl = big_body(DAMPED)
    m = make_mesh(wl, "fp64")
    q, qd = cuda(wl.q), cuda(wl.qdot)
    m.internal_force(q, qd)  # a force-sized buffer first
    f = torch.empty(m.n_dof, dtype=torch.float64, device="cuda")
    v = torch.empty(m.nnz, dtype=torch.float64, device="cuda")
    free = free_bytes()
    m.assemble(q, qd, 1e-3, 1.0, f=f, vals=v)
    taken = free - free_bytes()
    assert taken > 0.9 * wl.mesh.n_elem * 10 * (96 * 8 - 3 * 8)
    m.close()
