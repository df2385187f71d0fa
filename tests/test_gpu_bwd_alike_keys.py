"""The f32 backward on keys that are alike (repeated tokens, padding): the unit
triangular systems of a tile are then far from the identity, and their
inverses are what carries the error.  The chunk-start states come from the
oracle, so this checks the recompute and the adjoint alone.

Bars against the oracle's exact reverse mode: dv, dwx and dS0, which meet only
the triangular inverses and f32 products, 3e-6 (2-norm): f32's rounding (6e-8)
times the about fifty dependent sums of a tile's chain; every gradient 1e-4
(max-rel, the bar of the other f32 tests).
"""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs
from tests.gpu_util import host, max_rel, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("cosine", [0.9, 1.0])
def test_f32_backward_on_alike_keys(D, cosine):
    print(f"case f32 alike keys D={D} cosine={cosine}", flush=True)
    w = Workload("alike", B=1, H=2, T=256, Dk=D, Dv=D, L=64, R=16, dtype="f32", mu=2.0, s0=0.1)
    inp = make_inputs(w, seed=D, dS_T=True)
    k = inp["k"]
    base = k[:, :1]
    rest = k - (k * base).sum(-1, keepdims=True) * base
    rest /= np.maximum(np.linalg.norm(rest, axis=-1, keepdims=True), 1e-6)
    inp["k"] = (cosine * base + np.sqrt(1.0 - cosine ** 2) * rest).astype(np.float32)
    inp["beta"] = np.full_like(inp["beta"], 0.95)
    rf = orc.fwd_serial(inp, w.L, want_chunks=True)
    ref = orc.bwd(inp, w.L, inp["dO"], inp["dS_T"])
    x = to_gpu(inp, torch.float32)
    sc = torch.from_numpy(np.ascontiguousarray(rf["S_chunks"], dtype=np.float32)).cuda()
    gr = carve.chunk_bwd(x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"],
                         sc, x["dO"], x["dS_T"], L=w.L)
    torch.cuda.synchronize()
    got = {n: host(t).astype(np.float64) for n, t in gr.items()}
    two = {n: float(np.linalg.norm(got[n] - ref[n]) / np.linalg.norm(ref[n])) for n in ("dv", "dwx", "dS0")}
    errs = {n: max_rel(got[n], ref[n]) for n in got}
    print("2-norm errors:", two, "max-rel errors:", {n: float("%.3g" % e) for n, e in errs.items()}, flush=True)
    assert max(two.values()) <= 3e-6, two
    assert max(errs.values()) <= 1e-4, errs
