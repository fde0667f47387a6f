"""The distinct-id passes of eg_mla_gate_table (a claim per row, a bitmap) against eg_mla_gate_rows, bit for bit."""
import numpy as np
import pytest

from paper_2509_16686_amd import binding as B
from paper_2509_16686_amd import workloads as W
from parity import say


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [1, 2, 31, 33, 1000, 50304])
@pytest.mark.parametrize("n", [1, 2049, 9000, 70000])
def test_gate_table_bitmap(gpu, vocab, n):
    """Words at the vocabulary's end, few rows (claims) and many (the bitmap), three calls on the same marks."""
    import torch
    wl = W.WORKLOADS[1].replace(latent_dim=32, gate_dim=32, vocab=vocab, seed=9)
    ge = W.generate_gate_embedding(wl, 128)
    d = B.dims_for(wl)
    emb, wue = B.to_device_tensor(ge.emb, "bf16"), B.to_device_tensor(ge.w_ue, "bf16")
    marks = torch.zeros(B.gate_table_marks_size(d, 128, vocab), dtype=torch.uint8, device="cuda")
    for stamp in (1, 2, 3):
        ids_h = np.random.default_rng(stamp).integers(-2, vocab + 2, n).astype(np.int32)
        ids = torch.from_numpy(ids_h).cuda()
        table = torch.full((vocab, 32), 0x7bcd, dtype=torch.int16, device="cuda").view(torch.bfloat16)
        say(f"gate table vocab={vocab} n={n} stamp={stamp}")
        B.gate_table(d, ids, emb, wue, table, marks, stamp)
        rows = torch.empty((n, 32), dtype=torch.bfloat16, device="cuda")
        B.gate_rows(d, ids, emb, wue, rows)
        torch.cuda.synchronize()
        got = table.view(torch.int16).cpu().numpy()
        cid = np.clip(ids_h, 0, vocab - 1)
        assert np.array_equal(got[cid], rows.view(torch.int16).cpu().numpy())
        rest = np.ones(vocab, dtype=bool)
        rest[cid] = False
        assert np.all(got[rest] == 0x7bcd)


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [2, 33, 1000, 32767, 32768, 50304, 522240, 522241])
def test_gate_table_passes_alternate(gpu, vocab):
    """Calls of many rows (bitmap, up to 522240 ids) and of few (a claim per row) on the same marks, in every order of
    the two and of the stamp's parity."""
    import torch
    d_c, e = 32, 128
    wl = W.WORKLOADS[1].replace(latent_dim=d_c, gate_dim=d_c, vocab=vocab)
    d = B.dims_for(wl)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    emb = torch.randn(vocab, e, generator=g, device="cuda").to(torch.bfloat16)
    wue = torch.randn(d_c, e, generator=g, device="cuda").to(torch.bfloat16)
    marks = torch.zeros(B.gate_table_marks_size(d, e, vocab), dtype=torch.uint8, device="cuda")
    many, few = max(65536, vocab), 300
    for stamp, n in enumerate([many, few, many, many + 1, few, few, many, few, few, few, many, few, many - 1], 1):
        # ids of a part of the vocabulary that moves from call to call, some out of range
        lo = vocab * (stamp % 3) // 4
        ids = torch.randint(lo - 2, lo + vocab // 2 + 2, (n,), generator=g, device="cuda", dtype=torch.int32)
        table = torch.full((vocab, d_c), 0x7bcd, dtype=torch.int16, device="cuda").view(torch.bfloat16)
        say(f"gate table vocab={vocab} n={n} stamp={stamp}")
        B.gate_table(d, ids, emb, wue, table, marks, stamp)
        rows = torch.empty((n, d_c), dtype=torch.bfloat16, device="cuda")
        B.gate_rows(d, ids, emb, wue, rows)
        torch.cuda.synchronize()
        at = ids.long().clamp(0, vocab - 1)
        want = torch.full((vocab, d_c), 0x7bcd, dtype=torch.int16, device="cuda")
        want[at] = rows.view(torch.int16)
        assert torch.equal(table.view(torch.int16), want), (n, stamp)
