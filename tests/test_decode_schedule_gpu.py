"""The d_c 128 decode's work distribution: the balanced schedule of larger batches, short splits and the shared
absorption of small ones."""
import numpy as np
import pytest

from paper_2509_16686_amd import binding as B
from paper_2509_16686_amd import workloads as W
from parity import assert_close, oracle_decode, say


def decode(inp, plan=None):
    import torch
    dd = B.stage_decode(inp)
    B.run_decode(dd, plan=plan)
    torch.cuda.synchronize()
    return B.out_to_f64(dd.out)


def lens_mix(batch, top, seed):
    """Empty, single-token, unit-edge and piece-edge lengths among random ones, one sequence at the top."""
    lens = np.random.default_rng(seed).integers(1, top // 4, batch)
    edges = [0, 1, 16, 17, 255, 256, 257, 512, 513, 0]
    lens[:len(edges)] = edges
    lens[-1] = top
    return lens.astype(np.int32)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,top,balanced", [
    (33, 16, 1024, False),   # short items: (sequence, split) ones
    (40, 32, 4100, True),    # two head groups share each piece
    (64, 16, 9000, True),    # one long sequence among short ones
    (384, 16, 1100, True),   # the largest balanced batch
    (385, 16, 1100, False),  # past it: one item per sequence
])
def test_balanced_schedule(gpu, tok_pieces, batch, heads, top, balanced):
    assert tok_pieces("plan", heads, batch, -(-top // 16) * 16)[0][0] == balanced
    wl = W.WORKLOADS[1].replace(name="balanced", batch=batch, heads=heads, vocab=3000, seq_len=None,
                                seq_len_range=(0, top), page_size=16, paged=True, seed=5)
    inp = W.generate(wl, seq_lens=lens_mix(batch, top, batch))
    say(f"decode balanced B={batch} H={heads} top={top}")
    got = decode(inp)
    assert_close(got, oracle_decode(inp), "bf16", "balanced")
    assert not got[inp.seq_lens == 0].any()
    # all of one length: every sequence the same number of pieces
    inp = W.generate(wl, seq_lens=np.full(batch, 1024, dtype=np.int32))
    got = decode(inp)
    d = got - decode(inp, B.make_plan(B.PATH_MFMA, 256))  # (sequence, split) items
    assert np.linalg.norm(d) <= 5e-3 * np.linalg.norm(got)  # two bf16 outputs of sums in another order


@pytest.mark.gpu
@pytest.mark.parametrize("batch,top,balanced", [
    (72, 1600, True),     # 288 items of 480 tokens
    (64, 1728, False),    # 256 items of 448
    (256, 1920, True),    # 256 items of 1920
])
def test_balanced_rule(gpu, tok_pieces, batch, top, balanced):
    assert tok_pieces("plan", 16, batch, top)[0][0] == balanced
    wl = W.WORKLOADS[1].replace(name="balanced", batch=batch, vocab=3000, seq_len=None, seq_len_range=(0, top),
                                page_size=16, paged=True, seed=7)
    inp = W.generate(wl, seq_lens=lens_mix(batch, top, batch))
    say(f"decode balanced rule B={batch} top={top}")
    got = decode(inp)
    d = got - decode(inp, B.make_plan(B.PATH_MFMA, 256))  # (sequence, split) items
    assert np.linalg.norm(d) <= 5e-3 * np.linalg.norm(got)  # two bf16 outputs of sums in another order


@pytest.mark.gpu
@pytest.mark.parametrize("batch,length,spread", [
    (60, 20000, 1),      # an even cut into one piece per compute unit would pass the 4096-token list
    (128, 10000, 1),
    (48, 24000, 1536),   # lengths 1536 apart at most
])
def test_balanced_schedule_long(gpu, tok_pieces, batch, length, spread):
    """Balanced pieces near the token list's end against (sequence, split) items of 4096 tokens."""
    import torch
    lens = length - np.random.default_rng(batch).integers(0, spread, batch)
    lens[0] = length
    balanced = tok_pieces("plan", 16, batch, length)[0][0]
    cut = tok_pieces("cut", 16, batch, length, text=" ".join(map(str, lens)))
    assert balanced and 1800 < max(t for _, _, t in cut) <= 4096
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    dims = B.make_dims(num_heads=16, head_dim=128, v_head_dim=128, latent_dim=128, rope_dim=64, vocab_size=5000,
                       page_size=8)
    pages = length // 8
    q, cache = rnd(batch, 16, 192), rnd(batch * length, 192)
    ids = torch.randint(0, 5000, (batch * length,), generator=g, device="cuda", dtype=torch.int32)
    gate, w_uk, w_uv = rnd(5000, 128), rnd(16, 128, 128) / 11, rnd(16, 128, 128) / 11
    seq = torch.from_numpy(lens.astype(np.int32)).cuda()
    outs = []
    for plan in (None, B.make_plan(B.PATH_MFMA, 4096)):
        out = torch.full((batch, 16, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        dd = B.DeviceDecode(dims=dims, q=q, cache=cache, ids=ids, gate=gate, w_uk=w_uk, w_uv=w_uv, seq_lens=seq,
                            page_table=None, max_pages=pages, out=out)
        say(f"decode balanced long B={batch} L={length} plan={'balanced' if plan is None else 4096}")
        B.run_decode(dd, plan=plan)
        torch.cuda.synchronize()
        outs.append(out.double().cpu().numpy())
    assert np.isfinite(outs[0]).all()
    # two bf16 outputs of sums in another order: an absorbed query one fp32 sum of 128 products each way
    assert np.linalg.norm(outs[0] - outs[1]) <= 5e-3 * np.linalg.norm(outs[1])


@pytest.mark.gpu
def test_balanced_schedule_no_tokens(gpu):
    wl = W.WORKLOADS[1].replace(batch=40, vocab=100, seq_len=None, seq_len_range=(0, 1024), page_size=64, paged=True)
    inp = W.generate(wl, seq_lens=np.zeros(40, dtype=np.int32))
    assert not decode(inp).any()


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1, 64, 65, 0, 129, 2000], [3, 300], [16384]])
def test_short_splits(gpu, lens):
    """Few sequences: 64-token splits, most of them empty for the short ones."""
    wl = W.WORKLOADS[1].replace(batch=len(lens), vocab=500, seq_len=None, seq_len_range=(0, max(lens)), page_size=16,
                                paged=True, seed=6)
    inp = W.generate(wl, seq_lens=np.array(lens, dtype=np.int32))
    say(f"decode short splits {lens}")
    assert_close(decode(inp), oracle_decode(inp), "bf16", f"short splits {lens}")


@pytest.mark.gpu
@pytest.mark.parametrize("batch,n", [(1, 300), (8, 2000), (40, 4100)])  # short splits, shared absorption, balanced
def test_tokens_of_infinitely_low_score(gpu, batch, n):
    """A unit of 16 tokens whose RoPE scores overflow to -inf weighs nothing, wherever a split or piece has it; the
    vector kernel is the reference."""
    import torch
    wl = W.WORKLOADS[1].replace(batch=batch, vocab=700, seq_len=n, page_size=4, paged=False, seed=4)
    dd = B.stage_decode(W.generate(wl, seq_lens=np.full(batch, n, dtype=np.int32)))
    dd.q[..., -64:] = dd.q[..., -64:].abs() + 2
    rows = dd.cache.view(batch, n, -1)
    for at in (64, 160, 256):
        rows[:, at:at + 16, -64:] = -3e38
    say(f"decode -inf scores B={batch} n={n}")
    got = B.run_decode(dd).double()
    dd.out = torch.empty_like(dd.out)
    ref = B.run_decode(dd, plan=B.make_plan(B.PATH_VALU)).double()
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all() and torch.isfinite(got).all()
    assert (got - ref).norm() <= 5e-3 * ref.norm()  # bf16 outputs, fp16 latent operands on one side


@pytest.mark.gpu
@pytest.mark.parametrize("wl,most,batch,top", [
    (W.WORKLOADS[1], 256, 100, 4096),           # balanced pieces do not fit the workspace of 256 sequences
    (W.WORKLOADS[1], 64, 40, 4096),
    (W.MLA_DC320_BIGBATCH, 64, 50, 1024),       # whole-row kernel
])
def test_workspace_of_a_larger_batch(gpu, wl, most, batch, top):
    wl = wl.replace(batch=batch, vocab=900, seq_len=None, seq_len_range=(0, top), page_size=64, paged=True, seed=12)
    lens = np.random.default_rng(3).integers(0, top + 1, batch).astype(np.int32)
    dd = B.stage_decode(W.generate(wl, seq_lens=lens))
    import torch
    say(f"decode d_c {wl.latent_dim} B={batch} in the workspace of B={most}")
    want = B.run_decode(dd).double()
    dd.out = torch.full_like(dd.out, float("nan"))
    got = B.run_decode(dd, workspace=B.alloc_workspace(B.decode_workspace_size(dd.dims, most, top // 64))).double()
    torch.cuda.synchronize()
    # two bf16 outputs of sums in another order
    assert torch.isfinite(got).all() and (got - want).norm() <= 5e-3 * want.norm()


def test_balanced_workspace_fits_the_scratch_as_before():
    """A batch whose (sequence, split) plan fits the 32 MiB scratch fits it with the plan it gets."""
    d = B.make_dims(num_heads=16, head_dim=128, v_head_dim=128, latent_dim=128, rope_dim=64, vocab_size=50304)
    rows = lambda b, r: b * 16 * 192 * 4 + r * 16 * 130 * 4
    for b in list(range(1, 400, 7)) + [1000, 1500]:
        for pages in (1, 4, 16, 40, 64, 200, 512, 2048):
            cap = 64 * pages
            split = min(4096, max(256, -(-(b * cap // 256) // 32) * 32))
            before = rows(b, b * -(-cap // split))
            if before < (32 << 20) - 65536:
                assert B.decode_workspace_size(d, b, pages) <= 32 << 20, (b, pages)
