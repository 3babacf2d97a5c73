"""Projections of enough rows for 256 x 256 tiles (from 3585 rows before the
attention and 6913 after it): the smallest row counts that take them, with one
row in the last row tile, and grids of more than one round of workgroups.
Rows sampled over the tiles' edges against the oracle at the bounds of the
layer tests; nothing is written past the last row."""
import numpy as np
import pytest

from harness import log, to_dev
from oracle import proj_oracle as PO
import paper_2607_02043_amd as mla
from paper_2607_02043_amd import workloads as W
import test_gpu_layer as layer

pytestmark = pytest.mark.gpu
weights = layer.weights


def _sample(rows):
    rng = np.random.default_rng(rows)
    edges = [0, 1, 15, 16, 127, 128, 255, 256, 257, rows // 2, rows - 258, rows - 257, rows - 2, rows - 1]
    return np.unique(np.concatenate([edges, rng.integers(0, rows, 40)]))


@pytest.mark.parametrize("rows", [6913, 8193])
@pytest.mark.parametrize("out_bf16", [False, True])
def test_post_attn_many_rows(rows, out_bf16, weights):
    import torch
    _, wo, dw = weights
    log(f"[gpu] post_attn T={rows} out_bf16={out_bf16}")
    gen = torch.Generator(device="cuda").manual_seed(rows)
    a = torch.randn((rows, 16, 512), device="cuda", generator=gen)
    whole = torch.full((rows + 2, 2048), 7.0, dtype=torch.bfloat16 if out_bf16 else torch.float32, device="cuda")
    whole[:rows] = float("nan")
    ws = torch.empty(mla.mla_proj_workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    mla.mla_post_attn(a, dw, whole[:rows], ws)
    torch.cuda.synchronize()
    assert torch.isfinite(whole).all() and (whole[rows:] == 7.0).all()
    s = _sample(rows)
    got = whole[torch.from_numpy(s).cuda()].double().cpu().numpy()
    ab = PO.through_bf16(a[torch.from_numpy(s).cuda()].double().cpu().numpy())  # what the value up-projection reads
    o_exact = np.concatenate([ab[:, h] @ wo.w_uv[h].T for h in range(16)], axis=1)
    up, mags = layer._gemm_bound(o_exact, wo.w_o)
    exact = o_exact @ wo.w_o.T
    tol = up + 2.0 ** -16 * mags + (layer._ulp_bf16(exact) if out_bf16 else 0.0)
    d = np.abs(got - exact)
    log(f"  out: max |d|/tol = {float((d / tol).max()):.3f}")
    assert (d <= tol).all()


@pytest.mark.parametrize("rows", [3585, 8193])
def test_pre_attn_many_rows(rows, weights):
    import torch
    _, wo, dw = weights
    log(f"[gpu] pre_attn T={rows}")
    b = W.make_batch([17, 3000, 0], [1, rows - 2, 1], 64, 3)
    hidden = W.random_hidden(rows, seed=rows)
    q = torch.full((rows + 1, 16, 576), 7.0, dtype=torch.bfloat16, device="cuda")
    lat = torch.full((rows + 1, 576), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(mla.mla_proj_workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    mla.mla_pre_attn(mla.DeviceBatch.from_batch(b), to_dev(hidden), dw, q[:rows], lat[:rows], ws)
    torch.cuda.synchronize()
    assert torch.isfinite(q).all() and torch.isfinite(lat).all()
    assert (q[rows:] == 7.0).all() and (lat[rows:] == 7.0).all()
    s = _sample(rows)
    bits = lambda t: t[torch.from_numpy(s).cuda()].view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    x = PO.bf16_value(hidden[s])
    pos = PO.positions(b.q_lens, b.prefix_lens)[s]
    q_ref, lat_ref = PO.pre_attn(pos, x, wo, rounded=True)
    q_exact, lat_exact = PO.pre_attn(pos, x, wo, rounded=False)
    q_nope = (x @ wo.w_q.T).reshape(-1, 16, 192)[:, :, :128]
    up, mags = (np.stack(t, axis=1) for t in zip(*(layer._gemm_bound(q_nope[:, h], wo.w_uk_t[h]) for h in range(16))))
    layer.check_bf16(bits(q)[:, :, :512], q_ref[:, :, :512], q_exact[:, :, :512], "q_abs latent part", up, mags)
    m_q = (np.abs(x) @ np.abs(wo.w_q).T).reshape(-1, 16, 192)[:, :, 128:]
    layer.check_bf16(bits(q)[:, :, 512:], q_ref[:, :, 512:], q_exact[:, :, 512:], "q_abs rope part",
                     mags=np.repeat(m_q[..., 0::2] + m_q[..., 1::2], 2, axis=-1))
    m_kv = np.abs(x) @ np.abs(wo.w_dkv).T
    kv = x @ wo.w_dkv.T
    inv = 1.0 / np.sqrt(np.mean(kv[:, :512] ** 2, axis=1, keepdims=True) + wo.eps)
    m_lat = np.concatenate([m_kv[:, :512] * inv * np.abs(wo.kv_gain) + np.abs(lat_exact[:, :512]),
                            np.repeat(m_kv[:, 512::2] + m_kv[:, 513::2], 2, axis=-1)], axis=1)
    layer.check_bf16(bits(lat), lat_ref, lat_exact, "new latents", mags=m_lat)
