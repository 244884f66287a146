"""Parity with the oracle at the edges of the kernels' element tiles: one
element, one less than a tile, a whole one, one more (the meshes are the first
n elements of a larger one, so some of their nodes have no element)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu


def first_elements(wl, n):
    return dataclasses.replace(wl, mesh=dataclasses.replace(wl.mesh, conn=wl.mesh.conn[:n].copy()))


# force and backward kernels: 51 elements a workgroup
@pytest.mark.parametrize("n", [1, 50, 51, 52, 103])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_t10_force_and_vjp_tiles(precision, n):
    print(f"[gpu] force tile {precision} {n}", flush=True)
    wl = first_elements(W.t10_beam(5, 2, 2, 140 + n, "tile"), n)
    m = make_mesh(wl, precision)
    om, mat = oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material)
    f_ref, _ = oracle.assemble(om, mat, wl.q, wl.qdot, 1.0, 0.0)
    f = m.internal_force(cuda(wl.q), cuda(wl.qdot))
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL[precision]
    gq, gqd, gp = m.vjp(cuda(wl.q), cuda(wl.qdot), cuda(wl.w))
    refs = oracle.vjp(om, mat, wl.q, wl.qdot, wl.w)
    for got, ref in zip((gq, gqd), refs):
        assert rel_err(got.cpu().numpy(), ref)[0] <= TOL["fp64"]
    assert np.abs(gp.cpu().numpy() - refs[2]).max() <= 1e-12 * np.abs(refs[2]).max()
    m.close()


# element rows: 12 elements a wave (damped), 25 a workgroup (undamped), four at a time
@pytest.mark.parametrize("n", [1, 3, 4, 5, 11, 12, 13, 24, 25, 26, 37])
@pytest.mark.parametrize("damped", [True, False])
def test_t10_row_tiles(damped, n):
    print(f"[gpu] rows tile damped={damped} {n}", flush=True)
    mat = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), *((1e3, 7e2) if damped else ()))
    wl = first_elements(W.t10_beam(3, 2, 2, 160 + n, "tile", material=mat), n)
    m = make_mesh(wl, "mixed")
    om = oracle.Mesh.of(wl.mesh)
    f_ref, v_ref = oracle.assemble(om, oracle.material_of(mat), wl.q, wl.qdot, 1e-3, 1.0)
    f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), 1e-3, 1.0)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["mixed"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["mixed"]
    m.close()
