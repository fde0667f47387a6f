"""The whole-row decode kernel (d_c 320): unit, wave-round and split edges, head groups, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2509_16686_amd import binding as B
from paper_2509_16686_amd import workloads as W
from parity import assert_close, oracle_decode, say


@pytest.mark.gpu
@pytest.mark.parametrize("heads,paged", [(16, False), (32, True)])
@pytest.mark.parametrize("split", [0, 32, 2048])
def test_rows_kernel(gpu, heads, paged, split):
    lens = np.array([1, 15, 16, 17, 63, 64, 65, 0, 2047, 2049, 300], dtype=np.int32)
    wl = W.MLA_DC320_BIGBATCH.replace(batch=len(lens), heads=heads, vocab=700, seq_len=None, seq_len_range=(0, 2112),
                                      page_size=32, paged=paged, gate_all_ones=False, seed=3)
    inp = W.generate(wl, seq_lens=lens)
    say(f"decode d_c 320 H={heads} paged={paged} split={split}")
    import torch
    dd = B.stage_decode(inp)
    B.run_decode(dd, B.make_plan(B.PATH_MFMA, split))
    torch.cuda.synchronize()
    got = B.out_to_f64(dd.out)
    assert_close(got, oracle_decode(inp), "bf16", "whole rows")
    assert not got[lens == 0].any()


@pytest.mark.gpu
def test_rows_kernel_tokens_of_infinitely_low_score(gpu):
    """16 tokens (a whole unit of a wave) whose RoPE scores overflow to -inf weigh nothing; the vector kernel, which
    looks at 32 at a time, is the reference."""
    import torch
    n = 300
    wl = W.MLA_DC320_BIGBATCH.replace(batch=1, vocab=700, seq_len=n, seq_len_range=None, page_size=4, paged=False,
                                      gate_all_ones=False, seed=4)
    dd = B.stage_decode(W.generate(wl, seq_lens=np.array([n], dtype=np.int32)))
    dd.q[..., -64:] = dd.q[..., -64:].abs() + 2
    dd.cache[:16, -64:] = -3e38
    dd.cache[80:96, -64:] = -3e38
    say("decode d_c 320 -inf scores")
    got = B.run_decode(dd).double()
    dd.out = torch.empty_like(dd.out)
    ref = B.run_decode(dd, plan=B.make_plan(B.PATH_VALU)).double()
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all() and torch.isfinite(got).all()
    assert (got - ref).norm() <= 5e-3 * ref.norm()  # bf16 outputs, fp16 latent operands on one side
