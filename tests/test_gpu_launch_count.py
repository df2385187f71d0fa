"""The launches of each backward as the measurement hook's header lists them:
four, and a fifth with the decay formed in the kernels or the input activations.
"""
import pytest
import torch

from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs
from tests.gpu_util import to_gpu

pytestmark = pytest.mark.gpu


def _recorded(call):
    """Events the hook records during one call: those after a marker recorded first."""
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
    mark = torch.cuda.Event(enable_timing=True)
    for e in ev:
        e.record()
    mark.record()
    torch.cuda.synchronize()
    carve.profile_events(ev)
    call()
    torch.cuda.synchronize()
    return sum(mark.elapsed_time(e) > 0 for e in ev)


@pytest.mark.parametrize("variant,launches", [("plain", 4), ("gated", 5), ("sw", 4), ("sw_gated", 5), ("act", 5)])
def test_backward_launches(variant, launches):
    print(f"case launches {variant}", flush=True)
    w = Workload("launches", B=1, H=2, T=128, Dk=64, Dv=64, L=32, R=8, dtype="bf16", mu=3.0)
    sw, gated = variant.startswith("sw"), variant.endswith("gated")
    x = to_gpu(make_inputs(w, seed=1, gated=gated, scalar_write=sw, act=variant == "act"), torch.bfloat16)
    if sw:
        args = (x["q"], x["k"], x["v"], x["beta"], x["bx"], x["wx"], x["Ub"], x["Vb"])
        kw = {"f": x["f"], "A": x["A"], "tau_f": x["tau_f"]} if gated else {"g": x["g"]}
        fwd, bwd = carve.chunk_fwd_sw, carve.chunk_bwd_sw
    else:
        dec = (x["f"], x["A"], x["tau_f"]) if gated else (x["g"],)
        args = (x["q"], x["k"], x["v"], x["beta"], *dec, x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"])
        kw = {"act": True} if variant == "act" else {}
        fwd, bwd = (carve.chunk_fwd_gated, carve.chunk_bwd_gated) if gated else (carve.chunk_fwd, carve.chunk_bwd)
    _, _, sc = fwd(*args, L=w.L, **kw)
    assert _recorded(lambda: fwd(*args, L=w.L, **kw)) == 1 + 1
    assert _recorded(lambda: bwd(*args, sc, x["dO"], None, L=w.L, **kw)) == launches + 1
