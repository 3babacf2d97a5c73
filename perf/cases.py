"""The work that a decode node of this framework does, as cases to time: mixed
steps (append + attention), the two-call form of a step, whole attention
layers and the projections around the attention.

A case is a dict of plain values: `kind` (the entry points it calls, see
run()), the request lengths (a seeded list of decode contexts and a text of
prefix:length chunks), the page size and the output type.  The lengths belong
to the case and the values and page tables to the seed: a serving step calls
each of these entry points once per layer with the same lengths.
"""
import math

import numpy as np
import torch

import paper_2607_02043_amd as mla
from paper_2607_02043_amd import workloads as W

HEADS, DQK, DV, HIDDEN, NOPE, ROPE, VHEAD = 16, 576, 512, 2048, 128, 64, 128
LATENT = DQK - ROPE
EPS, BASE = 1e-6, 10000.0
PROJ_FLOPS_PER_ROW = {
    "pre": 2 * (HIDDEN * (HEADS * (NOPE + ROPE) + DQK) + HEADS * NOPE * LATENT),
    "post": 2 * (HEADS * LATENT * VHEAD + HEADS * VHEAD * HIDDEN),
}
WEIGHT_BYTES = 2 * (HIDDEN * (HEADS * (NOPE + ROPE) + DQK) + LATENT + 2 * HEADS * LATENT * NOPE + HEADS * VHEAD * HIDDEN)


def _case(name, kind, decodes, lo, hi, chunks, *, median=0.0, sigma=0.0, lens=0, page=64, out="f32"):
    """median 0: decode contexts uniform in [lo, hi]; else lognormal, clipped to it."""
    return dict(name=name, kind=kind, decodes=decodes, median=float(median), sigma=float(sigma), lo=lo, hi=hi, lens=lens,
                chunks=chunks, page=page, out=out)


def listed():
    return [
        # a nearly idle decode node: four requests of the paper's microbenchmark contexts, latency and launches count
        _case("step decode x4", "step", 4, 842, 3569, ""),
        # the smallest mixed step: a few short requests and one short chunk, small pages
        _case("step 5 + 32 rows, page 16", "step", 5, 17, 256, "0:32", page=16),
        # a lightly loaded node that takes its first deflected chunk
        _case("step 32 + 512", "step", 32, 16, 8192, "0:512", median=1024, sigma=1.0, lens=1),
        # a busy node with a long prompt's later chunk: matrix-bound
        _case("step 128 + 2048 at 6144", "step", 128, 16, 32768, "6144:2048", median=2048, sigma=1.2, lens=2),
        # the largest decode batch without a chunk: bound by memory
        _case("step decode x256", "step", 256, 512, 16384, "", lens=3),
        # the same batch beside a first chunk, in bf16: both bounds at once
        _case("step 256 + 2048, bf16", "step", 256, 512, 16384, "0:2048", lens=3, out="bf16"),
        # four deflected prompts at different progress beside 64 requests: one layer of the headline benchmark
        _case("step 64 + 4 x 1024", "step", 64, 1, 32768, "0:1024,1024:1024,3072:1024,8192:1024", median=4096, sigma=1.0, lens=4),
        # ragged chunks at unaligned prefixes on small pages, append and attention as two calls
        _case("two calls, ragged, page 16", "two", 37, 1, 3001, "0:2,517:131,1999:333,60:601", page=16, lens=5),
        # the whole attention layer of a small decode step: reading the weights and launches count
        _case("layer decode x19", "layer", 19, 100, 4099, "", lens=6),
        # the whole layer of the lightly loaded mixed step
        _case("layer 32 + 512", "layer", 32, 16, 8192, "0:512", median=1024, sigma=1.0, lens=1),
        # the whole layer of the largest mixed step, bf16 output
        _case("layer 64 + 4 x 1024, bf16", "layer", 64, 1, 32768, "0:1024,1024:1024,3072:1024,8192:1024", median=4096, sigma=1.0, lens=4, out="bf16"),
        # the projections by themselves, as a program with its own attention calls them: odd rows, fp32 attention output
        _case("projections 301 + 700 rows", "proj", 301, 1, 2000, "1000:700", lens=7),
    ]


def draw(rng):
    """A step, layer or projection call of the same ranges: 1 to 256 decode
    requests of up to 32768 keys and up to four chunks of 2 to 2048 rows."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    while True:
        kind = rng.choice(["step", "step", "step", "two", "layer", "layer", "proj"])
        decodes = log(1, 256)
        chunks = ["%d:%d" % (rng.choice([0, rng.randint(1, 8192)]), log(2, 2048)) for _ in range(rng.choice([0, 1, 1, 2, 3, 4]))]
        median, hi = (0, log(64, 16384)) if rng.random() < 0.5 else (log(64, 8192), 32768)
        c = _case("", kind, decodes, rng.randint(1, 64), hi, ",".join(chunks), median=median, sigma=rng.choice([0.5, 1.0, 1.2]),
                  lens=rng.randrange(1 << 20), page=rng.choice([16, 32, 64, 64, 128]), out=rng.choice(["f32", "bf16"]))
        del c["name"]
        w = work(c)
        if w["bytes"] <= 2.5e9 and w["flops"] <= 4.9e11:
            return c


def _lengths(case):
    """(prefix, new rows) of every request: decodes, then chunks."""
    rng = np.random.default_rng(case["lens"])
    n, lo, hi = case["decodes"], case["lo"], case["hi"]
    ctx = W.lognormal_lengths(rng, n, case["median"], case["sigma"], lo, hi) if case["median"] else rng.integers(lo, hi, n, endpoint=True)
    chunks = [tuple(int(x) for x in t.split(":")) for t in case["chunks"].split(",") if t]
    return [int(x) - 1 for x in ctx] + [p for p, _ in chunks], [1] * n + [c for _, c in chunks]


def _bf16(gen, shape, scale=1.0):
    """scale * N(0, 1) as bf16."""
    x = torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=gen)
    return x if scale == 1.0 else x.mul_(scale)


def _bits(x):
    return x.view(torch.int16)


class _Weights:
    """Projection weights of one layer at 1/sqrt(fan-in), as the C ABI lays them out."""

    def __init__(self, gen):
        self.t = {
            "w_q": _bf16(gen, (HEADS * (NOPE + ROPE), HIDDEN), HIDDEN ** -0.5),
            "w_dkv": _bf16(gen, (DQK, HIDDEN), HIDDEN ** -0.5),
            "kv_gain": (1.0 + 0.1 * torch.randn(LATENT, device="cuda", generator=gen)).to(torch.bfloat16),
            "w_uk": _bf16(gen, (HEADS, NOPE, LATENT), NOPE ** -0.5),
            "w_uv": _bf16(gen, (HEADS, VHEAD, LATENT), LATENT ** -0.5),
            "w_o": _bf16(gen, (HIDDEN, HEADS * VHEAD), (HEADS * VHEAD) ** -0.5),
        }
        self.t["w_uk_t"] = self.t["w_uk"].transpose(1, 2).contiguous()
        self.rms_eps, self.rope_base = EPS, BASE
        for k, v in self.t.items():
            setattr(self, k, _bits(v).cpu().numpy().view(np.uint16))


def _values(case, seed):
    """The batch and its random tensors."""
    prefix, rows = _lengths(case)
    b = W.make_batch(prefix, rows, case["page"], seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    T, kind = b.num_rows, case["kind"]
    v = {"batch": b}
    if kind != "proj":  # free slots hold the latents of requests that have left
        v["cache"] = _bf16(gen, (b.num_pages, b.page_size, DQK))
    if kind in ("step", "two"):
        v["q"] = _bf16(gen, (T, HEADS, DQK))
        v["new"] = _bf16(gen, (T, DQK))
    else:
        v["hidden"] = _bf16(gen, (T, HIDDEN))
        v["weights"] = _Weights(gen)
    if kind == "proj":
        v["attn"] = torch.randn((T, HEADS, DV), device="cuda", generator=gen)
    return v


def prepare(case, seed):
    v = _values(case, seed)
    b, kind = v["batch"], case["kind"]
    T, dt = b.num_rows, torch.float32 if case["out"] == "f32" else torch.bfloat16
    s = {"kind": kind, "batch": mla.DeviceBatch.from_batch(b)}
    if kind != "proj":
        s["cache"] = v["cache"]
    if kind in ("step", "two"):
        s["q"], s["new"] = v["q"], v["new"]
        s["out"] = torch.empty((T, HEADS, DV), dtype=dt, device="cuda")
        s["lse"] = torch.empty((T, HEADS), dtype=torch.float32, device="cuda")
        s["ws"] = mla.workspace_for(s["batch"])
    else:
        s["hidden"], s["weights"] = v["hidden"], mla.DeviceProjWeights(v["weights"])
        s["out"] = torch.empty((T, HIDDEN), dtype=dt, device="cuda")
    if kind == "layer":
        s["ws"] = mla.layer_workspace_for(s["batch"])
    if kind == "proj":
        s["attn"] = v["attn"]
        s["q_abs"] = torch.empty((T, HEADS, DQK), dtype=torch.bfloat16, device="cuda")
        s["new"] = torch.empty((T, DQK), dtype=torch.bfloat16, device="cuda")
        s["ws"] = torch.zeros(mla.mla_proj_workspace_bytes(T), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    b, kind = s["batch"], s["kind"]
    if kind == "step":
        mla.mixed_step(b, s["q"], s["new"], s["cache"], W.SOFTMAX_SCALE, s["out"], s["lse"], s["ws"])
        return {"out": s["out"], "lse": s["lse"], "cache": s["cache"]}
    if kind == "two":
        mla.append_latent_kv(b, s["new"], s["cache"])
        mla.mixed_step_attn(b, s["q"], s["cache"], W.SOFTMAX_SCALE, s["out"], s["lse"], s["ws"])
        return {"out": s["out"], "lse": s["lse"], "cache": s["cache"]}
    if kind == "layer":
        mla.mla_attention_layer(b, s["hidden"], s["weights"], s["cache"], W.SOFTMAX_SCALE, s["out"], s["ws"])
        return {"out": s["out"], "cache": s["cache"]}
    mla.mla_pre_attn(b, s["hidden"], s["weights"], s["q_abs"], s["new"], s["ws"])
    mla.mla_post_attn(s["attn"], s["weights"], s["out"], s["ws"])
    return {"q_abs": s["q_abs"], "new": s["new"], "out": s["out"]}


def work(case):
    prefix, rows = (np.asarray(x, dtype=np.int64) for x in _lengths(case))
    T, out_b, kind = int(rows.sum()), 4 if case["out"] == "f32" else 2, case["kind"]
    pages = int((-(-(prefix + rows) // case["page"])).sum())
    pairs = int((rows * prefix + rows * (rows + 1) // 2).sum())
    attn_flops = 2 * HEADS * (DQK + DV) * pairs
    if kind in ("step", "two"):
        # cached keys read; new latents read and written; queries read; outputs and lse written; tables read
        return {"bytes": 2 * DQK * int(prefix.sum()) + 4 * DQK * T + 2 * HEADS * DQK * T + HEADS * DV * out_b * T +
                4 * HEADS * T + 4 * pages + 12 * len(rows), "flops": attn_flops}
    proj = (PROJ_FLOPS_PER_ROW["pre"] + PROJ_FLOPS_PER_ROW["post"]) * T
    if kind == "layer":
        # cached keys, weights and hidden rows read; latents and the output written
        return {"bytes": 2 * DQK * int(prefix.sum()) + 2 * DQK * T + WEIGHT_BYTES + 2 * HIDDEN * T + HIDDEN * out_b * T +
                4 * pages + 12 * len(rows), "flops": attn_flops + proj}
    return {"bytes": WEIGHT_BYTES + 2 * HIDDEN * T + 2 * (HEADS + 1) * DQK * T + 4 * HEADS * DV * T + HIDDEN * out_b * T,
            "flops": proj}


def tolerance(case):
    """The 2-norm bar of the least exact output.  Rows of a chunk carry their
    probabilities in fp16 and decode rows theirs in 16 bits split in two;
    bf16 outputs round once, a layer at each of its stored intermediates."""
    if case["kind"] in ("layer", "proj"):
        return {"rel": 1e-2, "max": 0.1}
    if case["out"] == "bf16":
        return {"rel": 5e-3, "max": 2e-2}
    return {"rel": 1e-3, "max": 2e-2} if case["chunks"] else {"rel": 1e-5, "max": 2e-4}


# ------------------------------------------------------------- in 64 bits
def _rope(x, pos):
    """Rotate pairs (2i, 2i + 1) of the last axis (64 dims) by pos base^(-2i/64)."""
    i = torch.arange(ROPE // 2, dtype=torch.float64, device=x.device)
    ang = pos.double().reshape(-1, *([1] * (x.dim() - 1))) * BASE ** (-2.0 * i / ROPE)
    c, s = torch.cos(ang), torch.sin(ang)
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * c - x1 * s, x0 * s + x1 * c), dim=-1).reshape(x.shape)


def _pre(v, pos):
    """Absorbed queries [T][16][576] and new latents [T][576]."""
    w = {k: t.double() for k, t in v["weights"].t.items()}
    x = v["hidden"].double()
    q = (x @ w["w_q"].T).reshape(-1, HEADS, NOPE + ROPE)
    kv = x @ w["w_dkv"].T
    c = kv[:, :LATENT]
    c = c / torch.sqrt((c * c).mean(dim=1, keepdim=True) + EPS) * w["kv_gain"]
    new = torch.cat((c, _rope(kv[:, LATENT:], pos)), dim=1)
    q_abs = torch.cat((torch.matmul(q[:, :, :NOPE].transpose(0, 1).contiguous(), w["w_uk"]).transpose(0, 1),
                       _rope(q[:, :, NOPE:], pos)), dim=2)
    return q_abs, new


def _post(v, o):
    """[T][16][512] attention output -> [T][2048]."""
    w = {k: t.double() for k, t in v["weights"].t.items()}
    h = torch.matmul(o.transpose(0, 1).contiguous(), w["w_uv"].transpose(1, 2).contiguous()).transpose(0, 1)
    return h.reshape(-1, HEADS * VHEAD) @ w["w_o"].T


def _attend(b, q, cache, bt, fresh):
    """out [T][16][512] and lse [T][16]; keys from `cache` (whole pool, any type) and a request's new rows from `fresh`."""
    T = b.num_rows
    out = torch.empty((T, HEADS, DV), dtype=torch.float64, device="cuda")
    lse = torch.empty((T, HEADS), dtype=torch.float64, device="cuda")
    flat, row0 = cache.reshape(-1, DQK), 0
    for r in range(b.num_reqs):
        p, c = int(b.prefix_lens[r]), int(b.q_lens[r])
        t = torch.arange(p, device="cuda")
        keys = torch.cat((flat[bt[r, t // b.page_size] * b.page_size + t % b.page_size].double(), fresh[row0:row0 + c].double()))
        step = max(1, (1 << 26) // (HEADS * (p + c)))
        for i in range(0, c, step):
            n = min(step, c - i)
            x = (q[row0 + i:row0 + i + n].double().reshape(n * HEADS, DQK) @ keys.T).reshape(n, HEADS, p + c) * W.SOFTMAX_SCALE
            hidden = torch.arange(p + c, device="cuda")[None, :] > p + i + torch.arange(n, device="cuda")[:, None]
            x.masked_fill_(hidden[:, None, :], -math.inf)
            l = torch.logsumexp(x, dim=2)
            lse[row0 + i:row0 + i + n] = l
            x = torch.exp(x - l[:, :, None])
            out[row0 + i:row0 + i + n] = (x.reshape(n * HEADS, p + c) @ keys[:, :DV]).reshape(n, HEADS, DV)
        row0 += c
    return out, lse


def exact(case, seed):
    v = _values(case, seed)
    b, kind = v["batch"], case["kind"]
    first = torch.from_numpy(b.cu_q[:-1].copy()).cuda().long()
    rows = torch.from_numpy(b.q_lens.copy()).cuda().long()
    req = torch.repeat_interleave(torch.arange(b.num_reqs, device="cuda"), rows)
    pos = torch.from_numpy(b.prefix_lens.copy()).cuda().long()[req] + torch.arange(b.num_rows, device="cuda") - first[req]
    bt = torch.from_numpy(b.block_table.copy()).cuda().long()
    if kind in ("step", "two"):
        out, lse = _attend(b, v["q"], v["cache"], bt, v["new"])
        return {"out": out, "lse": lse, "cache": None}
    q_abs, new = _pre(v, pos)
    if kind == "proj":
        return {"q_abs": q_abs, "new": new, "out": _post(v, v["attn"].double())}
    out, _ = _attend(b, q_abs, v["cache"], bt, new)
    cache = v["cache"].double().reshape(-1, DQK)
    cache[bt[req, pos // b.page_size] * b.page_size + pos % b.page_size] = new
    return {"out": _post(v, out), "cache": cache.reshape(b.num_pages, b.page_size, DQK)}
