"""The backward's time on layers with hard-decaying key channels, whose blocks
are evaluated 16-token tile by tile, against the same layer without them.

Bar: 1.65.  A walk in 16-token tiles whose data is loaded ahead takes 1.3 to 1.4
times as long as blocks of 32 or 64 tokens; with every tile's loads waited for
where they are used it takes 1.7 to 2.2 times.  Times are the least of several
runs of ten calls each.
"""
import pytest
import torch

from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs
from tests.gpu_util import to_gpu

pytestmark = pytest.mark.gpu


def _us(f):
    for _ in range(3):
        f()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 100)
    return best


@pytest.mark.parametrize("D,L", [(128, 64), (128, 32), (64, 64)])
def test_hard_decay_time(D, L):
    print(f"case hard decay time D={D} L={L}", flush=True)
    w = Workload("hard", B=1, H=16, T=1024, Dk=D, Dv=D, L=L, R=32, dtype="bf16", mu=3.0)
    x = to_gpu(make_inputs(w, seed=3), torch.bfloat16)
    dims = carve.make_dims(w.B, w.T, w.H, D, D, w.R, L, torch.bfloat16)
    ws = torch.empty(carve.workspace_size(dims, True), dtype=torch.uint8, device="cuda")
    us = []
    for rate in (0.0, 5.5):
        if rate:
            x["g"][..., ::9] = -rate
        args = (x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"])
        _, _, sc = carve.chunk_fwd(*args, L=L)
        us.append(_us(lambda: carve.chunk_bwd(*args, sc, x["dO"], None, L=L, workspace=ws)))
    print("us without and with: %.1f %.1f" % tuple(us), flush=True)
    assert us[1] <= 1.65 * us[0], us
