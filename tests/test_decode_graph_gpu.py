"""Decode calls replayed from a captured graph: every replay against the eager result for the same inputs."""
import numpy as np
import pytest

from paper_2509_16686_amd import binding as B
from paper_2509_16686_amd import workloads as W
from parity import say


@pytest.mark.gpu
@pytest.mark.parametrize("layer,v_dim,lens", [
    ("h16", 128, [1024, 700, 3, 0]),             # the split kernel absorbs the query (16 splits, most of them empty)
    ("h16", 128, [512] * 3),                     # ... 8 splits: the small merge
    ("h16", 64, [1024, 1000]),                   # ... the merge of other value dims
    ("h16", 128, [300, 2000, 64]),               # ... 32 splits: the first 16 absorb it
    ("h16", 128, [300, 5000, 64]),               # a separate absorption
    ("h16", 128, list(range(100, 1999, 50))),    # balanced schedule
    ("kv64", 64, [900, 5]),                      # fp32 matrix-core kernel
    ("kv64", 64, [300, 5]),                      # ... in one launch
])
def test_replays_follow_the_inputs(gpu, layer, v_dim, lens):
    import torch
    over = dict(heads=12, head_dim=64, latent_dim=64, gate_dim=64) if layer == "kv64" else {}
    wl = W.WORKLOADS[1].replace(batch=len(lens), v_head_dim=v_dim, vocab=700, seq_len=None,
                                seq_len_range=(0, max(lens)), page_size=16, paged=True, seed=8, **over)
    dd = B.stage_decode(W.generate(wl, seq_lens=np.array(lens, dtype=np.int32)))
    ws = B.alloc_workspace(B.decode_workspace_size(dd.dims, len(lens), dd.max_pages))
    queries = [torch.randn(dd.q.shape, generator=torch.Generator().manual_seed(i)).to(dd.q) for i in range(4)]
    out = torch.empty_like(dd.out)
    entries = {"decode": lambda o: B.decode(dd.dims, dd.q, dd.cache, dd.ids, dd.gate, dd.w_uk, dd.w_uv, dd.seq_lens,
                                            dd.page_table, dd.max_pages, ws, o),
               "noalloc": lambda o: B.decode_noalloc(dd.dims, dd.q, dd.cache, dd.ids, dd.gate, dd.w_uk, dd.w_uv,
                                                     dd.seq_lens, dd.page_table, dd.max_pages, o)}
    for name, call in entries.items():
        say(f"decode graph {layer} {lens[:4]} {name}")
        refs = []
        for q in queries:
            dd.q.copy_(q)
            call(out)
            torch.cuda.synchronize()
            refs.append(out.clone())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(out)
        for n, i in enumerate((0, 1, 2, 3, 0, 2, 1)):
            if n == 4:
                call(out)  # an eager call on the same workspace between the replays
            dd.q.copy_(queries[i])
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), refs[i].view(torch.int16)), (name, n, i)


@pytest.mark.gpu
@pytest.mark.parametrize("v_dim,lens", [(128, [1024, 700, 3, 0]), (128, [512] * 3), (128, [2048] * 33), (64, [1024, 1000]),
                                        (128, [70, 2000])])
def test_no_stamp_outlives_the_call(gpu, v_dim, lens):
    """A replay's stamp is the captured one: had the call left its stamps (the last words of the workspace), a replay's
    work-groups would take the previous replay's absorbed query for its own."""
    import torch
    wl = W.WORKLOADS[1].replace(batch=len(lens), v_head_dim=v_dim, vocab=700, seq_len=None,
                                seq_len_range=(0, max(lens)), page_size=16, paged=True, seed=8)
    dd = B.stage_decode(W.generate(wl, seq_lens=np.array(lens, dtype=np.int32)))
    ws = B.alloc_workspace(B.decode_workspace_size(dd.dims, len(lens), dd.max_pages)).fill_(0xff)
    say(f"decode stamps d_v {v_dim} lens {lens[:4]}")
    B.run_decode(dd, workspace=ws)
    torch.cuda.synchronize()
    splits = {512: 8, 2048: 8, 2000: 32}.get(max(lens), 16)  # per sequence, each with a stamp
    n = len(lens) * splits
    at = ws.numel() - (n * 8 + 255) // 256 * 256
    assert not ws[at:at + n * 8].any()
    assert ws[at - 256:at].any()  # (the partial rows before them hold results)
