"""Backward calls on two streams at once, with separate workspaces: results are
bitwise those of calls made one after another, and no wait ran out.  Each call's
grid alone fits the device, the two together do not, so workgroups of one wait
for a place while the other's recompute already runs.
"""
import pytest
import torch

from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs
from tests.gpu_util import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L", [(2, 16, 64), (6, 16, 32), (1, 8, 16)])
def test_two_streams(B, H, L):
    print(f"case two streams B={B} H={H} L={L}", flush=True)
    w = Workload("streams", B=B, H=H, T=1024, Dk=128, Dv=128, L=L, R=32, dtype="bf16", mu=3.0)
    calls = []
    for seed in (1, 2):
        x = to_gpu(make_inputs(w, seed=seed), torch.bfloat16)
        args = (x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"])
        _, _, sc = carve.chunk_fwd(*args, L=L)
        dims = carve.make_dims(B, w.T, H, 128, 128, 32, L, torch.bfloat16)
        ws = torch.empty(carve.workspace_size(dims, True), dtype=torch.uint8, device="cuda")
        calls.append((args, sc, x["dO"], ws, dims, torch.cuda.Stream()))
    torch.cuda.synchronize()
    one = [carve.chunk_bwd(*a, sc, dO, L=L, workspace=ws) for a, sc, dO, ws, _, _ in calls]
    torch.cuda.synchronize()
    for _ in range(3):
        both = []
        for a, sc, dO, ws, _, st in calls:
            with torch.cuda.stream(st):
                both.append(carve.chunk_bwd(*a, sc, dO, L=L, workspace=ws))
        torch.cuda.synchronize()
        for i, (ref, got) in enumerate(zip(one, both)):
            assert not carve.bwd_wait_status(calls[i][4], calls[i][3])
            for k in ref:
                assert torch.equal(ref[k], got[k]), (i, k)
