"""Every form of a float64 pass 2 over element rows (force alone, K alone,
accumulating, with the mass, upper triangle) against the oracle, and Mooney-Rivlin
shells and beams on the rows."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from tests.gpu_util import TOL, cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu

RHO, H = 1200.0, 1e-3


def body(kind, damped, mr=False):
    kv = (1e3, 7e2) if damped else ()
    if kind == "t10":  # above the line of the rows, which damped meshes take
        mat = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), *kv)
        wl = W.t10_beam(21, 20, 20, 390, "forms", lx=0.2625, ly=0.25, lz=0.25, material=mat)  # affine: it has a mass
        return dataclasses.replace(wl, mesh=dataclasses.replace(wl.mesh, conn=wl.mesh.conn[:49153].copy()))
    mat = W.Material(W.MOONEY_RIVLIN, (2e7, 5e6, 1e9), *kv) if mr else W.Material(W.SVK, (7e8, 0.33, 0.0), *kv)
    if kind == "beam":
        return W.beam_3243(13, 391, "forms", material=mat)
    n = 64 if kind == "332" else 4  # 4,096 and 16 elements
    wl = W.shell_plate(n, 392, "forms", gl=tuple(int(c) for c in kind))
    return dataclasses.replace(wl, material=mat, qdot=np.random.default_rng(393).normal(0.0, 0.05, wl.q.shape))


@pytest.mark.parametrize("kind,damped", [("t10", True), ("beam", True), ("beam", False), ("443", True), ("443", False),
                                         ("332", True), ("332", False)])
def test_forms_of_pass_2(kind, damped):
    print(f"[gpu] rows64 forms {kind} damped={damped}", flush=True)
    wl = body(kind, damped)
    om, mat = oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material)
    pat = oracle.csr_pattern(om)
    f_ref, v_ref = oracle.assemble(om, mat, wl.q, wl.qdot, H, 1.0, pattern=pat)
    m = make_mesh(wl, "fp64")
    q, qd = cuda(wl.q), cuda(wl.qdot)
    tol = TOL["fp64"]

    def check(got, ref, t=tol):
        torch.cuda.synchronize()
        assert rel_err(got.cpu().numpy(), ref)[0] <= t

    check(m.tangent(q, qd, h=H), v_ref)  # K alone, fused
    m.assemble_points(q, qd, H, 1.0, want_tangent=True)
    f, v = torch.empty(m.n_dof, dtype=torch.float64, device="cuda"), torch.empty(m.nnz, dtype=torch.float64, device="cuda")
    m.assemble_nodes(f, None)
    check(f, f_ref)
    m.assemble_nodes(None, v)
    check(v, v_ref)
    # accumulating onto values of the results' own size: the sum loses no digits
    f0, v0 = cuda(np.roll(f_ref, 5)), cuda(np.roll(v_ref, 7))
    for f_on, v_on in ((True, True), (True, False), (False, True)):
        fa, va = f0.clone(), v0.clone()
        m.assemble_nodes(fa if f_on else None, va if v_on else None, accumulate=True)
        check(fa, np.roll(f_ref, 5) + f_ref if f_on else np.roll(f_ref, 5))
        check(va, np.roll(v_ref, 7) + v_ref if v_on else np.roll(v_ref, 7))
    fa, va = f0.clone(), v0.clone()
    m.assemble_accumulate(q, qd, H, 1.0, fa, va)
    check(fa, np.roll(f_ref, 5) + f_ref)
    check(va, np.roll(v_ref, 7) + v_ref)
    # the Newton matrix
    m.build_mass(RHO)
    h_ref = v_ref + oracle.mass_csr(om, RHO, pat) / H
    fn, hn = m.assemble_newton(q, qd, H)
    check(fn, f_ref)
    check(hn, h_ref)
    if not damped:
        m.build_upper_pattern()
        rows = np.repeat(np.arange(m.n_dof), np.diff(pat[0]))
        up = pat[1] >= rows
        fu, vu = m.assemble_upper(q, qd, H, 1.0)
        check(fu, f_ref)
        check(vu, v_ref[up])
        fu, hu = m.assemble_newton_upper(q, qd, H)
        check(fu, f_ref)
        check(hu, h_ref[up])
    m.close()


@pytest.mark.parametrize("damped", [True, False])
@pytest.mark.parametrize("kind", ["beam", "332", "443"])
def test_mooney_rivlin_rows(kind, damped):
    print(f"[gpu] rows64 mooney-rivlin {kind} damped={damped}", flush=True)
    wl = body(kind, damped, mr=True)
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material), wl.q, wl.qdot, H, 1.0)
    m = make_mesh(wl, "fp64")
    f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), H, 1.0)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    m.close()
