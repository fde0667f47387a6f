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
