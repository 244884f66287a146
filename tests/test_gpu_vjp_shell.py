"""Backward products of damped shells with and without the velocity product: the
two forms read the gradient table differently."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2604_10357_amd import workloads as W
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want", [(True, False, False), (True, False, True), (True, True, False), (False, True, False)])
@pytest.mark.parametrize("gl", [(3, 3, 2), (4, 4, 3)])
def test_shell_vjp_subsets(gl, want):
    print(f"[gpu] shell vjp {gl} {want}", flush=True)
    mat = W.Material(W.SVK, (7e8, 0.33, 0.0), 1e4, 7e3)
    wl = W.shell_plate(4, 360, "vjp", gl=gl)
    rng = np.random.default_rng(361)
    wl = dataclasses.replace(wl, material=mat, qdot=rng.normal(0.0, 0.05, wl.q.shape), w=rng.normal(0.0, 1.0, wl.q.shape))
    m = make_mesh(wl, "fp64")
    refs = oracle.vjp(oracle.Mesh.of(wl.mesh), oracle.material_of(mat), wl.q, wl.qdot, wl.w)
    got = m.vjp(cuda(wl.q), cuda(wl.qdot), cuda(wl.w), *want)
    for x, ref, on in zip(got[:2], refs, want):
        assert (x is not None) == on
        if on:
            assert rel_err(x.cpu().numpy(), ref)[0] <= TOL["fp64"]
    if want[2]:
        assert np.abs(got[2].cpu().numpy() - refs[2]).max() <= 1e-12 * np.abs(refs[2]).max()
    m.close()
