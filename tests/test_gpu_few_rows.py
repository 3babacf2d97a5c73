"""Projections of 1 to 49 rows, on either side of the row counts at which the
few-row GEMM takes another number of row blocks or hands over to the tiled
kernels, against the oracle at the bounds of the layer tests; then the tiles
that the library picks for more rows against a forced tile that those tests
compare with the oracle."""
import numpy as np
import pytest

from harness import log
from oracle import proj_oracle as PO
import paper_2607_02043_amd as mla
from paper_2607_02043_amd import workloads as W
import test_gpu_layer as layer

pytestmark = pytest.mark.gpu
weights = layer.weights


@pytest.mark.parametrize("rows", [1, 2, 15, 16, 17, 32, 33, 48, 49])
def test_pre_attn_few_rows(rows, weights, monkeypatch):
    rng = np.random.default_rng(rows)
    decodes = max(0, rows - 9)
    case = (list(rng.integers(0, 9000, decodes)) + [100], [1] * decodes + [rows - decodes], 16)
    monkeypatch.setitem(layer.PRE_CASES, "few", case)
    layer.test_pre_attn_parity("few", None, weights)


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 32, 33, 48, 49])
@pytest.mark.parametrize("attn_bf16,out_bf16", [(False, False), (True, False), (True, True)])
def test_post_attn_few_rows(rows, attn_bf16, out_bf16, weights):
    import torch
    _, wo, dw = weights
    log(f"[gpu] post_attn T={rows} attn_bf16={attn_bf16} out_bf16={out_bf16}")
    a = W.random_attn_out(rows, seed=31)
    a_dev = torch.from_numpy(a).cuda()
    if attn_bf16:
        a_dev = a_dev.to(torch.bfloat16)
    out = torch.full((rows, 2048), float("nan"), dtype=torch.bfloat16 if out_bf16 else torch.float32, device="cuda")
    ws = torch.empty(mla.mla_proj_workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    mla.mla_post_attn(a_dev, dw, out, ws)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    ab = PO.through_bf16(a.astype(np.float64))  # what the value up-projection reads
    o_exact = np.concatenate([ab[:, h] @ wo.w_uv[h].T for h in range(16)], axis=1)
    up, mags = layer._gemm_bound(o_exact, wo.w_o)
    exact = o_exact @ wo.w_o.T
    tol = up + 2.0 ** -16 * mags + (layer._ulp_bf16(exact) if out_bf16 else 0.0)
    d = np.abs(got - exact)
    log(f"  out: max |d|/tol = {float((d / tol).max()):.3f}")
    assert np.isfinite(got).all() and (d <= tol).all()


@pytest.mark.parametrize("rows", [49, 64, 65, 130, 257, 300, 512, 545, 1024, 3700])
def test_picked_tiles_equal_forced_tiles(rows, weights):
    """Both accumulate the same products in fp32 in another order, so a stored
    bf16 value moves by one step where it lies next to a rounding boundary.
    With at most 1 % of the values moving (the bound of the layer tests), by at
    most 2^-7 of themselves, the 2-norm of the difference stays below 2^-7
    sqrt(0.01) = 8e-4 of the result's, and so do the sums over moved inputs."""
    import torch
    _, _, dw = weights
    log(f"[gpu] picked against forced tiles, {rows} rows")
    batch = W.make_batch([17, 100], [1, rows - 1], 64, 3)
    db = mla.DeviceBatch.from_batch(batch)
    hidden = layer.to_dev(W.random_hidden(rows, seed=5))
    attn = torch.from_numpy(W.random_attn_out(rows, seed=6)).cuda()
    ws = torch.empty(mla.mla_proj_workspace_bytes(rows), dtype=torch.uint8, device="cuda")

    def run():
        q = torch.empty((rows, 16, 576), dtype=torch.bfloat16, device="cuda")
        lat = torch.empty((rows, 576), dtype=torch.bfloat16, device="cuda")
        outs = [torch.empty((rows, 2048), dtype=dt, device="cuda") for dt in (torch.float32, torch.bfloat16, torch.float32)]
        mla.mla_pre_attn(db, hidden, dw, q, lat, ws)
        for a, o in zip((attn, attn, attn.to(torch.bfloat16)), outs):
            mla.mla_post_attn(a, dw, o, ws)
        torch.cuda.synchronize()
        return [q, lat, *outs]

    picked = run()
    with mla.tuned({mla.TUNE_GEMM_BM: 64, mla.TUNE_GEMM_BN: 64, mla.TUNE_GEMM_DEPTH: 4}):
        forced = run()
    for k, (x, y) in enumerate(zip(picked, forced)):
        assert torch.isfinite(x).all()
        d = float((x.double() - y.double()).norm() / y.double().norm())
        log(f"  output {k}: {d:.2e}")
        assert d <= 8e-4
