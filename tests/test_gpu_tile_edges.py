"""Parity with the oracle at the edges of the kernels' element tiles: one
element, one less than a tile, a whole one, one more (the meshes are the first
n elements of a larger one, so some of their nodes have no element)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd._native import TlfeaError
from paper_2604_10357_amd.api import TLBatch
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


def test_t10_float64_rows_and_records():
    """float64 meshes above 49,152 damped elements take the element rows: a mesh
    just above the line and its undamped form (point records) against the oracle,
    in one batch with a small mesh and alone."""
    print("[gpu] float64 rows", flush=True)
    kv = W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), 1e3, 7e2)
    big = W.t10_beam(2049, 2, 2, 180, "rows64", lx=25.6, ly=0.025, lz=0.025, material=kv)
    big = first_elements(big, 49153)
    small = W.t10_beam(3, 2, 2, 181, "rows64_small", material=kv)
    refs, handles = [], []
    for wl in (big, small):
        om, mat = oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material)
        refs.append(oracle.assemble(om, mat, wl.q, wl.qdot, 1e-3, 1.0))
        handles.append(make_mesh(wl, "fp64"))
    for wl, m, (f_ref, v_ref) in zip((big, small), handles, refs):
        f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), 1e-3, 1.0)
        f_only = torch.empty_like(f)
        m.assemble_nodes(f_only)  # the force alone from the blocks
        torch.cuda.synchronize()
        assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
        assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
        assert rel_err(f_only.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
    b = TLBatch(handles)
    q, qd = (cuda(np.concatenate([getattr(wl, k) for wl in (big, small)])) for k in ("q", "qdot"))
    f, v = b.assemble(q, qd, torch.full((2,), 1e-3, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    for i, (f_ref, v_ref) in enumerate(refs):
        assert rel_err(f[b.dof_off[i]:b.dof_off[i + 1]].cpu().numpy(), f_ref)[0] <= TOL["fp64"]
        assert rel_err(v[b.nnz_off[i]:b.nnz_off[i + 1]].cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    with pytest.raises(TlfeaError):  # the persistent schedule is for mixed batches
        b.set_schedule(True, 25)
    b.close()
    handles[0].set_material(W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8)))
    om = oracle.Mesh.of(big.mesh)
    f_ref, v_ref = oracle.assemble(om, oracle.material_of(handles[0].material), big.q, big.qdot, 1e-3, 1.0)
    f, v = handles[0].assemble(cuda(big.q), cuda(big.qdot), 1e-3, 1.0)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"] and rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    for m in handles:
        m.close()


# float64 element rows of the beam (five elements a wave) and of the shells (five
# a workgroup of the 4x4x3 rule, seven of the 3x3x2 rule from 3,000 elements on)
@pytest.mark.parametrize("damped", [True, False])
@pytest.mark.parametrize("kind,n", [("beam", n) for n in (1, 4, 5, 6, 11)] + [("443", n) for n in (1, 4, 5, 6, 11)]
                         + [("332", n) for n in (2999, 3000, 3001, 3003)])
def test_float64_ancf_row_tiles(kind, n, damped):
    print(f"[gpu] float64 ANCF rows {kind} {n} damped={damped}", flush=True)
    mat = W.Material(W.SVK, (7e8, 0.33, 0.0), *((1e4, 7e3) if damped else ()))
    if kind == "beam":
        wl = W.beam_3243(12, 190 + n, "tile", material=mat)
    else:
        wl = W.shell_plate(4 if kind == "443" else 55, 190 + n, "tile", gl=tuple(int(c) for c in kind))
        rng = np.random.default_rng(n)
        wl = dataclasses.replace(wl, material=mat, qdot=rng.normal(0.0, 0.05, wl.q.shape))
    wl = first_elements(wl, n)
    m = make_mesh(wl, "fp64")
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(mat), wl.q, wl.qdot, 1e-3, 1.0)
    f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), 1e-3, 1.0)
    f_only = torch.empty_like(f)
    m.assemble_nodes(f_only)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["fp64"]
    assert rel_err(f_only.cpu().numpy(), f_ref)[0] <= TOL["fp64"]
    m.close()


# mixed element rows of undamped ANCF meshes: ten beams a workgroup, two
# coefficients a lane; seven and two shells
@pytest.mark.parametrize("kind,n", [("beam", n) for n in (1, 2, 9, 10, 11, 21)] + [("332", n) for n in (1, 6, 7, 8)]
                         + [("443", n) for n in (1, 2, 3)])
def test_mixed_ancf_row_tiles(kind, n):
    print(f"[gpu] mixed ANCF rows {kind} {n}", flush=True)
    if kind == "beam":
        wl = W.beam_3243(22, 230 + n, "tile")
    else:
        wl = W.shell_plate(3, 230 + n, "tile", gl=tuple(int(c) for c in kind))
    wl = first_elements(wl, n)
    m = make_mesh(wl, "mixed")
    f_ref, v_ref = oracle.assemble(oracle.Mesh.of(wl.mesh), oracle.material_of(wl.material), wl.q, wl.qdot, 1e-3, 1.0)
    f, v = m.assemble(cuda(wl.q), cuda(wl.qdot), 1e-3, 1.0)
    torch.cuda.synchronize()
    assert rel_err(f.cpu().numpy(), f_ref)[0] <= TOL["mixed"]
    assert rel_err(v.cpu().numpy(), v_ref)[0] <= TOL["mixed"]
    m.close()


# ANCF gradient: four lanes a node (64 nodes a workgroup), three neighbours a step;
# shell nodes have 4, 6 or 9
@pytest.mark.parametrize("kind,n", [("beam", 1), ("beam", 62), ("beam", 63), ("beam", 64), ("332", 1), ("332", 9)])
def test_ancf_gradient_nodes(kind, n):
    print(f"[gpu] ANCF gradient {kind} {n}", flush=True)
    wl = W.beam_3243(n, 260, "grad") if kind == "beam" else W.shell_plate(n, 261, "grad")
    m = make_mesh(wl, "fp64")
    m.build_mass(1200.0)
    om = oracle.Mesh.of(wl.mesh)
    pat = oracle.csr_pattern(om)
    rng = np.random.default_rng(262)
    v, v_prev, f, f_ext = (rng.normal(0, 1.0, wl.mesh.n_dof) for _ in range(4))
    g_ref = oracle.gradient(pat, oracle.mass_csr(om, 1200.0, pat), v, v_prev, f, f_ext, 1e-3)
    g = m.newton_gradient(cuda(v), cuda(v_prev), cuda(f), cuda(f_ext), 1e-3)
    assert rel_err(g.cpu().numpy(), g_ref)[0] <= 1e-12
    m.close()


# the backward product's sums: 1,024 rows a workgroup, one more workgroup for the
# parameters; every subset of the three gradients
@pytest.mark.parametrize("want", [(True, False, False), (False, True, False), (False, False, True),
                                  (True, True, False), (True, False, True), (False, True, True)])
@pytest.mark.parametrize("kind", ["t10", "beam"])
def test_vjp_subsets(kind, want):
    print(f"[gpu] vjp subset {kind} {want}", flush=True)
    kv = W.Material(W.SVK, (7e8, 0.33, 0.0), 1e4, 7e3)
    wl = W.t10_beam(6, 3, 2, 270, "sub", material=kv) if kind == "t10" else W.beam_3243(85, 271, "sub", material=kv)
    m = make_mesh(wl, "fp64")
    refs = oracle.vjp(oracle.Mesh.of(wl.mesh), oracle.material_of(kv), wl.q, wl.qdot, wl.w)
    got = m.vjp(cuda(wl.q), cuda(wl.qdot), cuda(wl.w), *want)
    for x, ref, on in zip(got[:2], refs, want):
        assert (x is not None) == on
        if on:
            assert rel_err(x.cpu().numpy(), ref)[0] <= TOL["fp64"]
    if want[2]:
        assert np.abs(got[2].cpu().numpy() - refs[2]).max() <= 1e-12 * np.abs(refs[2]).max()
    m.close()


# float64 ANCF batches: bodies of less than a tile, more than one, a large one (the
# 3x3x2 shells' line of 3,000 elements counts the batch's total); materials differ
@pytest.mark.parametrize("kind,sizes", [("beam", (1, 11, 5)), ("443", (1, 3, 2)), ("332", (2, 55, 1))])
def test_float64_ancf_batch(kind, sizes):
    print(f"[gpu] float64 ANCF batch {kind}", flush=True)
    wls = []
    for i, n in enumerate(sizes):
        mat = W.Material(W.SVK, (7e8, 0.33, 0.0), *((1e4, 7e3) if i % 2 else ()))
        if kind == "beam":
            wl = W.beam_3243(n, 280 + i, "batch", material=mat)
        else:
            wl = W.shell_plate(n, 280 + i, "batch", gl=tuple(int(c) for c in kind))
            qdot = np.random.default_rng(i).normal(0.0, 0.05, wl.q.shape)
            wl = dataclasses.replace(wl, material=mat, qdot=qdot)
        wls.append(wl)
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
