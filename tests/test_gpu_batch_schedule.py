"""The schedule that a batch reports is one that it can be set to."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd._native import TlfeaError
from paper_2604_10357_amd.api import TLBatch
from tests.gpu_util import cuda, make_mesh, rel_err

pytestmark = pytest.mark.gpu

KV = W.Material(W.SVK, (1e7, 0.3, 0.0), 1e3, 7e2)


def body(kind, i):
    if kind == "t10":
        return W.t10_beam(2 + i, 2, 1, 310 + i, "schedule", material=KV)
    if kind == "beam":
        return W.beam_3243(3 + 4 * i, 310 + i, "schedule", material=KV)
    return dataclasses.replace(W.shell_plate(2 + i, 310 + i, "schedule", gl=tuple(int(c) for c in kind)), material=KV)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("kind,tile", [("t10", 25), ("beam", 10), ("332", 7), ("443", 2)])
def test_reported_tile_can_be_set(kind, tile, precision):
    print(f"[gpu] batch schedule {kind} {precision}", flush=True)
    wls = [body(kind, i) for i in range(3)]
    handles = [make_mesh(wl, precision) for wl in wls]
    b = TLBatch(handles)
    q, qd = (cuda(np.concatenate([getattr(wl, k) for wl in wls])) for k in ("q", "qdot"))
    h = torch.full((3,), 1e-3, dtype=torch.float64, device="cuda")
    f0, v0 = b.assemble(q, qd, h)
    reported = b.schedule()
    assert reported["persistent"] == 0 and reported["tile_elems"] == tile
    if kind == "t10" and precision == "mixed":
        b.set_schedule(True, reported["tile_elems"])
        assert b.schedule()["tile_elems"] == tile
        f, v = b.assemble(q, qd, h)
        torch.cuda.synchronize()
        assert rel_err(f.cpu().numpy(), f0.cpu().numpy())[0] <= 1e-13
        assert rel_err(v.cpu().numpy(), v0.cpu().numpy())[0] <= 1e-13
    else:
        with pytest.raises(TlfeaError) as e:
            b.set_schedule(True, reported["tile_elems"])
        assert e.value.status == -2
    b.set_schedule(False)
    b.close()
    for m in handles:
        m.close()
