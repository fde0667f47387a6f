"""Performance cases: the calls a program that serves EG-MLA layers makes, over the sizes it makes them at.

A case is a dict of plain values.  Its "kind" names the entry points it runs:

  decode    one eg_mla_decode call over a latent cache
  step      eg_mla_append_ws of one new token per sequence, then eg_mla_decode: a layer's whole decode step
  unfolded  eg_mla_gate_table of the step's ids, then eg_mla_decode with that table (the gate from the embedding)
  prefill   one eg_mla_prefill_varlen call over packed sequences
  append    one eg_mla_append_ws call of many tokens (the cache rows of a prompt)
  literal   one eg_mla_decode_literal call (the gate and LayerNorm after the up-projection)

and "layer" one of LAYERS.  Sequence lengths are spread evenly over [min_len, max_len] and handed to the
sequences in a random order, so that a case's work does not depend on the seed.
"""
import math

import torch

from paper_2509_16686_amd import binding as B

# heads, head dim (queries and values), latent, RoPE, vocabulary, model width, storage
LAYERS = {
    "tiny": dict(h=4, dh=32, dc=32, dr=0, vocab=1000, hidden=128, dtype="fp32"),       # the fp32 test layer
    "kv16": dict(h=12, dh=64, dc=16, dr=64, vocab=50304, hidden=768, dtype="bf16"),    # the paper's 12-layer
    "kv64": dict(h=12, dh=64, dc=64, dr=64, vocab=50304, hidden=768, dtype="bf16"),    # models: 12 heads of
    "kv128": dict(h=12, dh=64, dc=128, dr=64, vocab=50304, hidden=768, dtype="bf16"),  # 64, cache widths
    "kv256": dict(h=12, dh=64, dc=256, dr=64, vocab=50304, hidden=768, dtype="bf16"),  # 16 to 256
    "h16": dict(h=16, dh=128, dc=128, dr=64, vocab=50304, hidden=2048, dtype="bf16"),  # the 1.2B-class layer
    "mla320": dict(h=16, dh=128, dc=320, dr=64, vocab=50304, hidden=2048, dtype="bf16", ones=True),  # plain MLA
    "h128": dict(h=128, dh=128, dc=512, dr=64, vocab=129280, hidden=7168, dtype="bf16"),  # the 128-head layer
}

EMB = 512  # embedding width of the unfolded gate


def listed():
    return [
        # the smallest call: one sequence of a small fp32 layer, launches and latency only
        dict(name="decode_tiny_fp32", kind="decode", layer="tiny", batch=1, min_len=128, max_len=128, page=64, paged=False),
        # one layer's decode step of a lightly loaded server: few sequences of mixed length, paged cache
        dict(name="step_b8", kind="step", layer="h16", batch=8, min_len=203, max_len=2000, page=64, paged=True),
        # the ordinary throughput batch (the benchmark's default workload)
        dict(name="decode_b32_l4096", kind="decode", layer="h16", batch=32, min_len=4096, max_len=4096, page=64, paged=False),
        # long contexts, few sequences
        dict(name="decode_b4_l32768", kind="decode", layer="h16", batch=4, min_len=32768, max_len=32768, page=64, paged=False),
        # a large batch of mixed lengths whose gate rows come from the embedding at every step
        dict(name="unfolded_b256", kind="unfolded", layer="h16", batch=256, min_len=250, max_len=3901, page=64, paged=True),
        # the 128-head layer under load: paged, lengths from 512 to 16384
        dict(name="decode_h128_b64", kind="decode", layer="h128", batch=64, min_len=512, max_len=16384, page=64, paged=True),
        # plain MLA (all-ones gate, latent 320), the model EG-MLA is compared with, large batch
        dict(name="decode_mla320_b256", kind="decode", layer="mla320", batch=256, min_len=2048, max_len=2048, page=64, paged=False),
        # the paper's small model (12 heads of 64, latent 64), a mid-size batch of mixed lengths
        dict(name="decode_kv64_b64", kind="decode", layer="kv64", batch=64, min_len=100, max_len=3003, page=64, paged=True),
        # prompts of mixed length packed into one prefill call
        dict(name="prefill_h16_b8", kind="prefill", layer="h16", batch=8, min_len=1001, max_len=4096),
        # the same of the 128-head layer (another form: explicit keys and values per head)
        dict(name="prefill_h128_b2", kind="prefill", layer="h128", batch=2, min_len=1111, max_len=2985),
        # the cache rows of a prompt of the 128-head layer
        dict(name="append_h128_n4096", kind="append", layer="h128", batch=4096, norm=True),
        # the gate as the paper prints it (after the up-projection, with the LayerNorm)
        dict(name="literal_b8", kind="literal", layer="h16", batch=8, min_len=1000, max_len=4096, page=64, paged=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lens(rng, batch, lo, hi, total):
    """A length range within [lo, hi] whose sum over the batch stays below `total`."""
    top = max(lo, min(_log(rng, lo, hi), total // batch))
    return (top if rng.random() < 0.3 else rng.randint(max(1, top // 16), top)), top


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "step", "unfolded", "prefill", "prefill", "append", "literal"])
    if kind == "decode":
        layer = rng.choice(["h16", "h16", "h128", "mla320", "kv16", "kv64", "kv128", "kv256", "tiny"])
        if layer == "tiny":
            b, (lo, hi) = rng.randint(1, 4), (rng.randint(1, 64), rng.randint(65, 512))
        elif layer == "h128":
            b = _log(rng, 1, 64)
            lo, hi = _lens(rng, b, 32, 16384, 400000)
        elif layer in ("h16", "mla320"):
            b = _log(rng, 1, 256)
            lo, hi = _lens(rng, b, 32, 32768, 500000)
        else:
            b = _log(rng, 1, 64)
            lo, hi = _lens(rng, b, 32, 4096, 100000)
        return dict(kind=kind, layer=layer, batch=b, min_len=lo, max_len=hi, page=rng.choice([16, 64]),
                    paged=rng.random() < 0.6)
    if kind in ("step", "unfolded"):
        layer = "h16" if kind == "unfolded" else rng.choice(["h16", "h128"])
        b = _log(rng, 1, 64)
        lo, hi = _lens(rng, b, 32, 8192, 200000)
        return dict(kind=kind, layer=layer, batch=b, min_len=lo, max_len=hi, page=rng.choice([16, 64]), paged=True)
    if kind == "prefill":
        layer = rng.choice(["h16", "h128"])
        b = rng.randint(1, 8)
        lo, hi = _lens(rng, b, 16, 4096 if layer == "h16" else 2800, 16384 if layer == "h16" else 4000)
        return dict(kind=kind, layer=layer, batch=b, min_len=lo, max_len=hi)
    if kind == "append":
        return dict(kind=kind, layer=rng.choice(["h16", "h128"]), batch=_log(rng, 1, 8192), norm=rng.random() < 0.7)
    b = _log(rng, 1, 8)
    lo, hi = _lens(rng, b, 32, 4096, 20000)
    return dict(kind=kind, layer="h16", batch=b, min_len=lo, max_len=hi, page=64, paged=rng.random() < 0.5)


def _lengths(case):
    n, lo, hi = case["batch"], case["min_len"], case["max_len"]
    return [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in range(n)]


class _Draw:
    """Seeded values on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, dtype, std=1.0, mean=0.0):
        x = torch.randn(shape, generator=self.g, device="cuda")
        if std != 1.0 or mean != 0.0:
            x.mul_(std).add_(mean)
        return x.to(dtype)

    def ints(self, hi, n):
        return torch.randint(0, hi, (n,), generator=self.g, device="cuda", dtype=torch.int32)

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device="cuda").to(torch.int32)


def _inputs(case, seed):
    """Every input of a case, as a program holds them before the call."""
    L = LAYERS[case["layer"]]
    r = _Draw(seed)
    dt = torch.bfloat16 if L["dtype"] == "bf16" else torch.float32
    h, dh, dc, dr = L["h"], L["dh"], L["dc"], L["dr"]
    tiny = case["layer"] == "tiny"
    kind = case["kind"]
    s = dict(L=L, kind=kind, case=case, dt=dt)
    s["dims"] = B.make_dims(num_heads=h, head_dim=dh, v_head_dim=dh, latent_dim=dc, rope_dim=dr,
                            vocab_size=L["vocab"], page_size=case.get("page", 64),
                            dtype=B.BF16 if L["dtype"] == "bf16" else B.FP32)
    if kind in ("append", "step"):
        n = case["batch"]
        s["x"] = r.normal((n, L["hidden"]), dt)
        s["w_dkv"] = r.normal((dc + dr, L["hidden"]), dt, 1 / math.sqrt(L["hidden"]))
        s["norm_w"] = r.normal((dc,), dt, 0.1, 1.0) if case.get("norm", True) else None
        s["new_ids"] = r.ints(L["vocab"], n)
    if kind == "append":
        s["positions"] = r.ints(32768, n)
        s["slots"] = r.perm(n)
        s["cache"] = torch.zeros((n, dc + dr), dtype=dt, device="cuda")
        s["ids"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        return s
    lens = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")[r.perm(case["batch"]).long()].contiguous()
    total = sum(_lengths(case))
    std = 1 / math.sqrt(dc)
    s["w_uk"], s["w_uv"] = r.normal((h, dh, dc), dt, std), r.normal((h, dh, dc), dt, std)
    if kind == "literal":
        s["gate"] = r.normal((L["vocab"], h * 2 * dh), dt, 0.1, 1.0)
        s["ln_w"], s["ln_b"] = r.normal((h * 2 * dh,), dt, 0.1, 1.0), r.normal((h * 2 * dh,), dt, 0.1)
    elif kind == "unfolded":
        s["emb"], s["w_ue"] = r.normal((L["vocab"], EMB), dt), r.normal((dc, EMB), dt, 1 / math.sqrt(EMB))
        s["gate"] = torch.zeros((L["vocab"], dc), dtype=dt, device="cuda")
    elif L.get("ones"):
        s["gate"] = torch.ones((L["vocab"], dc), dtype=dt, device="cuda")
    else:
        s["gate"] = r.normal((L["vocab"], dc), dt, 0.1, 1.0)
    if kind == "prefill":
        s["cu"] = torch.cat([torch.zeros(1, dtype=torch.int32, device="cuda"), lens.cumsum(0).to(torch.int32)])
        s["cache"], s["ids"] = r.normal((total, dc + dr), dt), r.ints(L["vocab"], total)
        s["q"] = r.normal((total, h, dh + dr), dt)
        s["out"] = torch.empty((total, h, dh), dtype=dt, device="cuda")
        return s
    page = case["page"]
    pages = -(-case["max_len"] // page)
    s["lens"], s["max_pages"] = lens, pages
    if case["paged"]:
        n_pages = sum(-(-n // page) for n in _lengths(case))
        per = (lens + (page - 1)) // page
        table = torch.zeros((case["batch"], pages), dtype=torch.int32, device="cuda")
        table[torch.arange(pages, device="cuda")[None, :] < per[:, None]] = r.perm(n_pages)
        s["table"] = table
    else:
        n_pages = case["batch"] * pages
        s["table"] = None
    rows = n_pages * page
    if tiny:  # the fp32 layer's values are scaled by their width
        s["cache"], s["q"] = r.normal((rows, dc + dr), dt, std), r.normal((case["batch"], h, dh + dr), dt, 1 / math.sqrt(dh))
    else:
        s["cache"], s["q"] = r.normal((rows, dc + dr), dt), r.normal((case["batch"], h, dh + dr), dt)
    s["ids"] = r.ints(L["vocab"], rows)
    s["out"] = torch.empty((case["batch"], h, dh), dtype=dt, device="cuda")
    if kind == "unfolded":
        s["step_ids"] = s["ids"]
    if kind == "step":
        last = (lens - 1).long()
        pg = torch.gather(s["table"], 1, (last // page)[:, None])[:, 0].long()
        s["slots"] = (pg * page + last % page).to(torch.int32)
        s["positions"] = last.to(torch.int32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    d, kind = s["dims"], s["kind"]
    if kind in ("append", "step"):
        s["ws_append"] = B.alloc_workspace(B.append_workspace_size(d, case["batch"], s["L"]["hidden"]))
    if kind in ("decode", "step", "unfolded"):
        s["ws"] = B.alloc_workspace(B.decode_workspace_size(d, case["batch"], s["max_pages"]))
    if kind == "unfolded":
        s["marks"] = torch.zeros(B.gate_table_marks_size(d, EMB, s["L"]["vocab"]), dtype=torch.uint8, device="cuda")
        s["stamp"] = 0
    if kind == "prefill":
        s["ws"] = B.alloc_workspace(B.prefill_varlen_workspace_size(d, int(s["q"].shape[0])))
    if kind == "literal":
        s["ws"] = B.alloc_workspace(B.decode_literal_workspace_size(d, case["batch"], s["max_pages"]))
        s["dd"] = B.DeviceDecode(dims=d, q=s["q"], cache=s["cache"], ids=s["ids"], gate=None, w_uk=s["w_uk"],
                                 w_uv=s["w_uv"], seq_lens=s["lens"], page_table=s["table"],
                                 max_pages=s["max_pages"], out=s["out"])
    return s


def _decode(s):
    B.decode(s["dims"], s["q"], s["cache"], s["ids"], s["gate"], s["w_uk"], s["w_uv"], s["lens"], s["table"],
             s["max_pages"], s["ws"], s["out"])
    return s["out"]


def _append(s):
    B.append_ws(s["dims"], s["x"], s["new_ids"], s["positions"], s["slots"], s["w_dkv"], s["norm_w"], s["cache"],
                s["ids"], s["ws_append"])
    return [s["cache"], s["ids"]]


def run(s):
    kind = s["kind"]
    if kind == "decode":
        return _decode(s)
    if kind == "append":
        return _append(s)
    if kind == "step":
        rows = _append(s)
        return [_decode(s)] + rows
    if kind == "unfolded":
        s["stamp"] += 1
        B.gate_table(s["dims"], s["step_ids"], s["emb"], s["w_ue"], s["gate"], s["marks"], s["stamp"])
        return [_decode(s), s["gate"]]
    if kind == "prefill":
        B.prefill_varlen(s["dims"], s["cu"], s["q"], s["cache"], s["ids"], s["gate"], s["w_uk"], s["w_uv"], s["ws"],
                         s["out"])
        return s["out"]
    B.decode_literal(s["dd"], s["gate"], s["ln_w"], s["ln_b"], 0, s["ws"])
    return s["out"]


def _append_work(L, n):
    eb = 2 if L["dtype"] == "bf16" else 4
    row = L["dc"] + L["dr"]
    return (n * (L["hidden"] + row) + L["hidden"] * row + L["dc"]) * eb + n * 16, 2 * n * L["hidden"] * row


def work(case):
    L, kind = LAYERS[case["layer"]], case["kind"]
    h, dh, dc, dr, v = L["h"], L["dh"], L["dc"], L["dr"], L["vocab"]
    eb = 2 if L["dtype"] == "bf16" else 4
    if kind == "append":
        by, fl = _append_work(L, case["batch"])
        return {"bytes": by, "flops": fl}
    lens = _lengths(case)
    n = sum(lens)
    distinct = v * (1 - (1 - 1 / v) ** n)  # gate rows that uniform ids touch
    rows = case["batch"] if kind != "prefill" else n
    by = n * ((dc + dr) * eb + 4) + rows * h * (2 * dh + dr) * eb + 2 * h * dh * dc * eb
    pairs = n if kind != "prefill" else sum(x * (x + 1) // 2 for x in lens)
    if kind == "literal":
        by += distinct * h * 2 * dh * eb
        fl = n * h * (2 * dc * 2 * dh + 2 * (dh + dr) + 2 * dh)
    elif kind == "prefill":
        by += distinct * dc * eb
        fl = pairs * h * 2 * (2 * dh + dr) + n * h * 2 * dc * 2 * dh
    else:
        by += distinct * dc * eb
        fl = pairs * h * 2 * (2 * dc + dr) + rows * h * 2 * dc * 2 * dh
    if kind == "step":
        b2, f2 = _append_work(L, case["batch"])
        by, fl = by + b2, fl + f2
    if kind == "unfolded":
        by += distinct * EMB * eb + dc * EMB * eb
        fl += distinct * 2 * EMB * dc
    return {"bytes": int(by), "flops": int(fl)}


def tolerance(case):
    if case["layer"] == "tiny":  # fp32 sums in another order
        return {"rel": 2e-6, "max": 1e-5}
    # bf16 outputs: their own rounding is 1.7e-3 (2-norm) and up to 2^-8 of an element
    return {"rel": 7e-3, "max": 4e-2}


def _exact_append(s):
    L = s["L"]
    dc, dr = L["dc"], L["dr"]
    y = s["x"].double() @ s["w_dkv"].double().T
    c, k = y[:, :dc], y[:, dc:]
    if s["norm_w"] is not None:
        c = c / torch.sqrt((c * c).mean(1, keepdim=True) + 1e-6) * s["norm_w"].double()
    ang = s["positions"].double()[:, None] * 10000.0 ** (-2.0 * torch.arange(dr // 2, device="cuda").double() / dr)
    a, b = k[:, 0::2], k[:, 1::2]
    k = torch.stack([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], 2).reshape(-1, dr)
    cache, ids = s["cache"].double(), s["ids"].clone()
    cache[s["slots"].long()] = torch.cat([c, k], 1)
    ids[s["slots"].long()] = s["new_ids"]
    return cache, ids


def _seq_rows(s, b, n):
    if s["table"] is None:
        at = b * s["max_pages"] * s["case"]["page"]
        return torch.arange(at, at + n, device="cuda")
    page = s["case"]["page"]
    j = torch.arange(n, device="cuda")
    return s["table"][b].long()[j // page] * page + j % page


def _exact_decode(s, cache, gate, ids):
    L = s["L"]
    dh, dc = L["dh"], L["dc"]
    tau = 1 / math.sqrt(dh + L["dr"])
    out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
    w_uk, w_uv = s["w_uk"].double(), s["w_uv"].double()
    for b, n in enumerate(s["lens"].tolist()):
        rows = _seq_rows(s, b, n)
        row = cache[rows].double()
        c = row[:, :dc] * gate[ids[rows].long()].double()
        q = s["q"][b].double()
        ql = (q[:, None, :dh] @ w_uk)[:, 0]
        p = torch.softmax(tau * (ql @ c.T + q[:, dh:] @ row[:, dc:].T), 1)
        out[b] = (w_uv @ (p @ c)[:, :, None])[:, :, 0]
    return out


def _exact_prefill(s):
    L = s["L"]
    dh, dc = L["dh"], L["dc"]
    tau = 1 / math.sqrt(dh + L["dr"])
    out = torch.empty(s["out"].shape, dtype=torch.float64, device="cuda")
    cu = s["cu"].tolist()
    for a, e in zip(cu[:-1], cu[1:]):
        c = s["cache"][a:e, :dc].double() * s["gate"][s["ids"][a:e].long()].double()
        kr = s["cache"][a:e, dc:].double()
        late = torch.ones((e - a, e - a), dtype=torch.bool, device="cuda").triu(1)
        for h in range(L["h"]):
            q = s["q"][a:e, h].double()
            k = torch.cat([c @ s["w_uk"][h].double().T, kr], 1)
            sc = (tau * (q @ k.T)).masked_fill_(late, -math.inf)
            out[a:e, h] = torch.softmax(sc, 1) @ (c @ s["w_uv"][h].double().T)
    return out


def _exact_literal(s):
    L = s["L"]
    h, dh, dc = L["h"], L["dh"], L["dc"]
    tau = 1 / math.sqrt(dh + L["dr"])
    out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
    w = torch.cat([s["w_uk"], s["w_uv"]], 1).double().reshape(h * 2 * dh, dc)
    lw, lb = s["ln_w"].double(), s["ln_b"].double()
    for b, n in enumerate(s["lens"].tolist()):
        rows = _seq_rows(s, b, n)
        row = s["cache"][rows].double()
        x = (row[:, :dc] @ w.T) * s["gate"][s["ids"][rows].long()].double()
        y = torch.nn.functional.layer_norm(x, (h * 2 * dh,), lw, lb, 1e-5).reshape(n, h, 2 * dh)
        q = s["q"][b].double()
        for i in range(h):
            p = torch.softmax(tau * (y[:, i, :dh] @ q[i, :dh] + row[:, dc:] @ q[i, dh:]), 0)
            out[b, i] = p @ y[:, i, dh:]
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = s["kind"]
    if kind == "append":
        return list(_exact_append(s))
    if kind == "prefill":
        return _exact_prefill(s)
    if kind == "literal":
        return _exact_literal(s)
    if kind == "step":  # the cache holds the new rows in its storage type
        cache, ids = _exact_append(s)
        return [_exact_decode(s, cache.to(s["dt"]), s["gate"], ids), cache, ids]
    if kind == "unfolded":  # so does the table
        table = torch.zeros(s["gate"].shape, dtype=torch.float64, device="cuda")
        used = torch.unique(s["step_ids"]).long()
        table[used] = s["emb"][used].double() @ s["w_ue"].double().T
        return [_exact_decode(s, s["cache"], table.to(s["dt"]), s["ids"]), table]
    return _exact_decode(s, s["cache"], s["gate"], s["ids"])
