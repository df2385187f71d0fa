"""The backward's two evaluations of a WY block, mixed within one call, against
the CPU oracle's exact reverse mode.

A block of up to 64 tokens takes one log-retention reference per key channel
while every channel stays above -80 over the block, and is evaluated 16-token
tile by tile otherwise.  Blocks of both kinds follow each other here in every
order: first and last of the call, alternating, several in a row, different
kinds inside one 128-token chunk (two blocks) and in different heads at the same
place, with 32- and 64-token blocks, both padded ranks and every layer variant.
(16-token blocks, of 16-token chunks, are one tile and have one evaluation; they
get the same decays here.)

Bar: bf16 inputs with f32 state and accumulation, max-rel <= 2e-2 per tensor
(the bar of the erase-heavy cases).
"""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import Workload, make_inputs, round_bf16
from tests.gpu_util import host, max_rel, to_gpu

pytestmark = pytest.mark.gpu

TOL = 2e-2


def _inputs(w, pattern, seed, **kw):
    """Erase gates saturated (about -8 of log retention per token) on eight key
    channels in the blocks marked 1; a pattern per (batch, head), or one for all."""
    inp = make_inputs(w, seed=seed, dS_T=True, **kw)
    rng = np.random.default_rng(seed)
    block = min(w.L, 64)
    marks = np.broadcast_to(np.asarray(pattern), (w.B, w.H, np.shape(pattern)[-1]))
    for b, h, i in zip(*np.nonzero(marks)):
        ch = rng.choice(w.Dk, size=8, replace=False)
        t = slice(i * block, (i + 1) * block)
        inp["bx"][b, t, h][:, ch] = round_bf16(8.0 + 0.5 * rng.standard_normal((block, 8)).astype(np.float32))
    return inp


@pytest.mark.parametrize("variant,D,L,R,pattern", [
    ("plain", 128, 64, 20, (1, 0, 0, 1, 1, 0)),
    ("plain", 128, 64, 20, (0, 1, 0, 1, 0, 1)),
    ("plain", 128, 128, 20, (1, 0, 0, 1, 0, 0, 1, 1)),
    ("plain", 128, 32, 20, (0, 1, 1, 0, 1)),
    ("plain", 128, 16, 20, (0, 1, 1, 0, 1)),
    ("plain", 64, 64, 20, (1, 0, 1)),
    ("plain", 32, 64, 20, (0, 1, 0)),
    # heads that differ: in the kind of the block, in the first and last one
    ("plain", 128, 64, 20, (((0, 1, 1, 0), (1, 0, 1, 0)), ((0, 0, 0, 1), (0, 0, 0, 0)))),
    ("plain", 64, 128, 20, (((0, 1, 1, 0), (1, 0, 1, 1)), ((1, 1, 0, 0), (0, 0, 0, 0)))),
    # 64 padded fold rows
    ("plain", 64, 64, 40, (1, 0, 1, 1)),
    ("plain", 64, 32, 64, (0, 1, 0, 1)),
    ("plain", 32, 64, 33, (0, 1, 1, 0)),
    ("sw", 32, 128, 64, (0, 1, 1, 0)),
    ("gated", 128, 64, 20, (0, 1, 0, 0)),
    ("sw", 128, 64, 20, (0, 1, 0, 1)),
    ("sw_gated", 128, 64, 20, (1, 0, 1, 0)),
    ("sw_gated", 64, 32, 20, (0, 1, 1, 0)),
    ("act", 128, 128, 20, (0, 1, 0, 0)),
])
def test_mixed_blocks(variant, D, L, R, pattern):
    shape = np.shape(pattern)
    B, H = shape[:2] if len(shape) == 3 else (1, 2)
    w = Workload("blocks", B=B, H=H, T=min(L, 64) * shape[-1], Dk=D, Dv=D, L=L, R=R, dtype="bf16", mu=3.0, s0=0.2,
                 u_std=0.3)
    print(f"case mixed blocks {variant} D={D} L={L} R={R} {pattern}", flush=True)
    sw, gated = variant.startswith("sw"), variant.endswith("gated")
    inp = _inputs(w, pattern, seed=D + L + shape[-1], gated=gated, scalar_write=sw, act=variant == "act")
    x = to_gpu(inp, torch.bfloat16)
    if sw:
        args = (x["q"], x["k"], x["v"], x["beta"], x["bx"], x["wx"], x["Ub"], x["Vb"])
        decay = {"f": x["f"], "A": x["A"], "tau_f": x["tau_f"]} if gated else {"g": x["g"]}
        _, _, sc = carve.chunk_fwd_sw(*args, x["S0"], L=L, **decay)
        gr = carve.chunk_bwd_sw(*args, sc, x["dO"], x["dS_T"], L=L, **decay)
        ref = orc.bwd_sw(inp, L, inp["dO"], inp["dS_T"])
    elif gated:
        args = (x["q"], x["k"], x["v"], x["beta"], x["f"], x["A"], x["tau_f"], x["bx"], x["wx"], x["Ub"], x["Uw"],
                x["Vb"], x["Vw"])
        _, _, sc = carve.chunk_fwd_gated(*args, x["S0"], L=L)
        gr = carve.chunk_bwd_gated(*args, sc, x["dO"], x["dS_T"], L=L)
        ref = orc.bwd_gated(inp, L, inp["dO"], inp["dS_T"])
    else:
        act = variant == "act"
        args = (x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"], x["Vb"], x["Vw"])
        _, _, sc = carve.chunk_fwd(*args, x["S0"], L=L, act=act)
        gr = carve.chunk_bwd(*args, sc, x["dO"], x["dS_T"], L=L, act=act)
        ref = (orc.bwd_act if act else orc.bwd)(inp, L, inp["dO"], inp["dS_T"])
    torch.cuda.synchronize()
    errs = {}
    for key, val in gr.items():
        got = host(val)
        assert np.all(np.isfinite(got)), key
        errs[key] = max_rel(got, ref[key])
    print("max-rel errors:", {k: float("%.3g" % e) for k, e in errs.items()}, flush=True)
    bad = {k: e for k, e in errs.items() if not e <= TOL}
    assert not bad, bad
