"""The first-order solver's table of bias corrections: bounded however rarely the
caller checks, and right across its end (4,096 iterations)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import cuda, make_mesh, rel_err
from tests.test_gpu_adamw import H, RHO, problem

pytestmark = pytest.mark.gpu


def solve(m, wl, v_n, f_ext, **kw):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        out = m.adamw_solve(cuda(wl.q), cuda(v_n), cuda(v_n.copy()), H, 1e-4, 0.9, 0.9999, 1e-8, 0.0,
                            f_ext=cuda(f_ext), **kw)
    s.synchronize()
    return out


def test_a_solve_that_never_checks_takes_no_memory():
    print("[gpu] adamw table", flush=True)
    wl, v_n, f_ext = problem(320)
    m = make_mesh(wl, "fp64")
    m.build_mass(RHO)
    solve(m, wl, v_n, f_ext, max_iters=2)  # torch's own buffers and the mesh's
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    # converges at the check after the first iteration
    _, _, done, _, _ = solve(m, wl, v_n, f_ext, eps_in=1e10, max_iters=2**31 - 1, check_every=2**31 - 1)
    assert done == 1
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    m.close()


@pytest.mark.parametrize("iters", [4096, 4097, 4098, 8200])
def test_more_iterations_than_the_table_holds(iters):
    print(f"[gpu] adamw table {iters}", flush=True)
    wl, v_n, f_ext = problem(321, "beam")
    m = make_mesh(wl, "fp64")
    m.build_mass(RHO)
    v, q, done, _, g = solve(m, wl, v_n, f_ext, max_iters=iters, check_every=iters)
    v2, q2, done2, _, g2 = solve(m, wl, v_n, f_ext, max_iters=iters, check_every=400)
    assert done == done2 == iters
    for x, y in ((v, v2), (q, q2), (g, g2)):  # the same sums in the same order
        assert np.isfinite(x.cpu().numpy()).all()
        assert rel_err(x.cpu().numpy(), y.cpu().numpy())[0] <= 1e-12
    m.close()
