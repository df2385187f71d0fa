"""Parameter gradients of the backward at the edges of the split rule: 16 chunk
(token) splits per (batch, head) up to 32 of them, then as many as give 512
workgroups of a kind, one from 512 on; with fewer chunks than splits, and chunk
counts that do not divide.

Every other gradient is compared too, and every one of a second call: with this
many workgroups on the card the recompute's records once lost single lanes.

Bars against the CPU oracle's exact reverse mode: f32 inputs 1e-4, bf16 2e-2
(max-rel per tensor, the bars of the backward's other tests).
"""
import pytest
import torch

from oracle import oracle as orc
from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs
from tests.gpu_util import host, max_rel, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("B,H,T,L", [
    (1, 1, 16, 16),       # 16 splits, one chunk
    (2, 16, 304, 16),     # 16 splits of 19 chunks
    (3, 11, 304, 16),     # 33 (batch, head): still 16
    (5, 13, 144, 16),     # 65: 8 splits of 9 chunks
    (10, 13, 64, 32),     # 130: 4 splits, two chunks of two tiles
    (1, 511, 32, 16),     # 2 splits, one chunk each
    (2, 257, 32, 16),     # 514: no split
])
def test_param_splits(dtype, tol, B, H, T, L):
    print(f"case param splits {dtype} B={B} H={H} T={T} L={L}", flush=True)
    w = Workload("splits", B=B, H=H, T=T, Dk=32, Dv=32, L=L, R=7, dtype=dtype, mu=3.0, s0=0.1, u_std=0.3)
    inp = make_inputs(w, seed=B * H)
    x = to_gpu(inp, torch.float32 if dtype == "f32" else torch.bfloat16)
    args = (x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"])
    _, _, sc = carve.chunk_fwd(*args, x["S0"], L=L)
    gr = carve.chunk_bwd(*args, sc, x["dO"], None, L=L)
    again = carve.chunk_bwd(*args, sc, x["dO"], None, L=L)
    torch.cuda.synchronize()
    ref = orc.bwd(inp, L, inp["dO"], None)
    errs = {k: max_rel(host(gr[k]), ref[k]) for k in gr}
    assert {"dq", "dk", "dv", "dbeta", "dg", "dbx", "dwx", "dUb", "dUw", "dVb", "dVw", "dS0"} <= set(errs)
    print("max-rel errors:", {k: float("%.3g" % e) for k, e in errs.items()}, flush=True)
    assert max(errs.values()) <= tol, errs
    for k in gr:
        assert torch.equal(gr[k], again[k]), k
