"""Parity of the output RMS normalisation (carve_rmsnorm_fwd / _bwd: the step
that closes Alg. carve_fwd, y = W_O RMSNorm(reshape(o)), without W_O) through
the C ABI against the oracle's double-precision definition and its reverse mode.

Rows are the H*Dv values of a token.  Bars: f32 max-rel <= 1e-5; bf16 (f32
arithmetic, bf16 in and out) max-rel <= 2e-2; dweight is a fixed-order
reduction, bitwise identical on reruns.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2606_27229_amd import carve
from paper_2606_27229_amd.inputs import WORKLOADS, make_inputs, round_bf16
from tests.gpu_util import host, max_rel, to_gpu

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


def _inputs(B, T, H, Dv, dtype, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    o = rng.standard_normal((B, T, H, Dv), dtype=np.float32) * rng.uniform(0.2, 5.0, size=(B, T, 1, 1)).astype(np.float32)
    dy = rng.standard_normal((B, T, H, Dv), dtype=np.float32)
    w = (1.0 + 0.1 * rng.standard_normal(H * Dv)).astype(np.float32)
    if dtype == "bf16":
        o, dy = round_bf16(o), round_bf16(dy)
    return o, dy, w


def _run(o, dy, w, dtype, eps=1e-6):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    og = torch.from_numpy(o).to(dt).cuda()
    dyg = torch.from_numpy(dy).to(dt).cuda()
    wg = torch.from_numpy(w).cuda()
    y = carve.rmsnorm_fwd(og, wg, eps=eps)
    d_o, dw = carve.rmsnorm_bwd(og, wg, dyg, eps=eps)
    torch.cuda.synchronize()
    return host(y), host(d_o), host(dw)


@pytest.mark.parametrize("dtype,B,T,H,Dv", [
    ("f32", 1, 16, 1, 32), ("f32", 3, 37, 2, 64), ("f32", 2, 50, 16, 128),
    ("bf16", 1, 16, 1, 32), ("bf16", 3, 37, 4, 64), ("bf16", 2, 129, 16, 128), ("bf16", 1, 64, 32, 128),
])
def test_rmsnorm_parity(dtype, B, T, H, Dv):
    print(f"case rmsnorm {dtype} B={B} T={T} H={H} Dv={Dv}", flush=True)
    o, dy, w = _inputs(B, T, H, Dv, dtype, seed=B * 1000 + T + H + Dv)
    y, d_o, dw = _run(o, dy, w, dtype)
    ry = orc.rmsnorm(o, w)
    rdo, rdw = orc.rmsnorm_bwd(o, w, dy)
    errs = {"y": max_rel(y, ry), "d_o": max_rel(d_o, rdo), "dweight": max_rel(dw, rdw)}
    print("max-rel errors:", {k: float("%.3g" % e) for k, e in errs.items()}, flush=True)
    assert all(np.all(np.isfinite(a)) for a in (y, d_o, dw))
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype,N", [("bf16", 2048), ("bf16", 1544), ("f32", 2048), ("f32", 1028)])
@pytest.mark.parametrize("rows", [1, 5, 2047, 2049, 4097, 6150])
def test_rmsnorm_rows_per_wave(dtype, N, rows):
    """Row lengths of 32 columns per lane (whole, and with idle lanes) over the
    512 workgroups of four waves: fewer rows than waves, one more than a wave
    each, and ragged counts of two and four.  dweight is an f32 sum of the rows'
    f32 products for both dtypes: 1e-5 of its largest value."""
    print(f"case rmsnorm rows {dtype} N={N} rows={rows}", flush=True)
    o, dy, w = _inputs(1, rows, 1, N, dtype, seed=rows + N)
    _, d_o, dw = _run(o, dy, w, dtype)
    rdo, rdw = orc.rmsnorm_bwd(o, w, dy)
    errs = {"d_o": max_rel(d_o, rdo), "dweight": max_rel(dw, rdw)}
    print("max-rel errors:", {k: float("%.3g" % e) for k, e in errs.items()}, flush=True)
    assert errs["d_o"] <= TOL[dtype] and errs["dweight"] <= 1e-5, errs


def test_rmsnorm_headline_layer_output():
    """The norm of the headline layer's own output (B=4 H=16 T=4096 d=128, bf16),
    in the configuration the benchmark times: every row against the oracle."""
    w_ = WORKLOADS["layer_1p3b_T4096"]
    print("case rmsnorm on the headline layer output", flush=True)
    inp = make_inputs(w_, seed=4)
    x = to_gpu(inp, torch.bfloat16)
    o, _, _ = carve.chunk_fwd(x["q"], x["k"], x["v"], x["beta"], x["g"], x["bx"], x["wx"], x["Ub"], x["Uw"],
                              x["Vb"], x["Vw"], x["S0"], L=w_.L, want_chunks=False, want_state=False)
    del x
    rng = np.random.Generator(np.random.PCG64(9))
    N = w_.H * w_.Dv
    wt = torch.from_numpy((1.0 + 0.1 * rng.standard_normal(N)).astype(np.float32)).cuda()
    dy = torch.from_numpy(round_bf16(rng.standard_normal(tuple(o.shape), dtype=np.float32))).to(torch.bfloat16).cuda()
    y = carve.rmsnorm_fwd(o, wt)
    d_o, dw = carve.rmsnorm_bwd(o, wt, dy)
    d_o2, dw2 = carve.rmsnorm_bwd(o, wt, dy)
    torch.cuda.synchronize()
    oh, wh, dyh = host(o), host(wt), host(dy)
    errs = {"y": max_rel(host(y), orc.rmsnorm(oh, wh))}
    rdo, rdw = orc.rmsnorm_bwd(oh, wh, dyh)
    errs["d_o"] = max_rel(host(d_o), rdo)
    errs["dweight"] = max_rel(host(dw), rdw)
    print("max-rel errors:", {k: float("%.3g" % e) for k, e in errs.items()}, flush=True)
    assert max(errs.values()) <= TOL["bf16"], errs
    assert torch.equal(dw, dw2) and torch.equal(d_o, d_o2)


def test_rmsnorm_rejections():
    lib = carve.load_library()
    o = torch.zeros((1, 4, 64, 128), dtype=torch.bfloat16, device="cuda")   # N = 8192 > 4096
    with pytest.raises(carve.CarveError) as err:
        carve.rmsnorm_fwd(o, torch.ones(64 * 128, device="cuda"))
    assert err.value.status == -3
    o = torch.zeros((1, 4, 2, 32), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(carve.CarveError) as err:
        carve.rmsnorm_fwd(o, torch.ones(64, device="cuda"), eps=-1.0)
    assert err.value.status == -7
    d = carve.make_dims(1, 4, 2, 32, 32, 1, 1, torch.bfloat16)
    assert lib.carve_rmsnorm_workspace_size(d) > 0
