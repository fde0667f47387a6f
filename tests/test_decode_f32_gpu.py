"""eg_mla_decode on the shapes without a 16-bit fast path (fp32 storage, head counts off 16, small
heads and latents): the fp32 matrix-core kernel, in one launch and in three, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2509_16686_amd import binding as B
from paper_2509_16686_amd import workloads as W
from parity import assert_close, oracle_decode, say

# (dtype, heads, d_h, d_v, d_c, d_r): the paper's 12-head models, then edges of the latent buckets (64, 128, 256, 320),
# columns off 16, a second partly filled block of heads, no RoPE part
SHAPES = [("bf16", 12, 64, 64, 16, 64), ("bf16", 12, 64, 64, 64, 64), ("bf16", 12, 64, 64, 128, 64),
          ("bf16", 12, 64, 64, 256, 64), ("bf16", 17, 40, 24, 24, 8), ("bf16", 3, 128, 128, 320, 64),
          ("fp32", 4, 32, 32, 32, 0), ("fp32", 33, 20, 48, 132, 12), ("fp32", 2, 64, 64, 300, 64),
          ("fp32", 1, 4, 4, 4, 4)]
# contexts around a unit (16), a round of the waves (64, 128), one-launch limit (512) and list chunk
LENS = [np.array([1, 16, 17, 65, 128, 0, 129, 300]), np.array([512, 511, 3]), np.array([513, 64, 0, 1]),
        np.array([1500, 2049])]


def workload(shape, lens, paged):
    dt, h, dh, dv, dc, dr = shape
    base = W.WORKLOADS[0] if dt == "fp32" else W.WORKLOADS[1]
    return base.replace(name="f32_shapes", batch=len(lens), heads=h, head_dim=dh, v_head_dim=dv, latent_dim=dc,
                        gate_dim=dc, rope_dim=dr, vocab=500, seq_len=None, seq_len_range=(0, int(lens.max())),
                        page_size=16, paged=paged, seed=77)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("li", range(len(LENS)))
def test_f32_kernel_against_oracle(gpu, shape, li):
    import torch
    wl = workload(shape, LENS[li], paged=li % 2 == 0)
    inp = W.generate(wl, seq_lens=LENS[li])
    say(f"decode {shape} lens {LENS[li].tolist()}")
    dd = B.stage_decode(inp)
    ref = oracle_decode(inp)
    for split in (0, 96):
        got = B.out_to_f64(B.run_decode(dd, B.make_plan(B.PATH_AUTO, split)))
        torch.cuda.synchronize()
        # fp32 storage: the stated 1e-5 is for unit-scale outputs; these values are of that scale
        assert_close(got, ref, wl.dtype, f"{shape} split {split}")
        assert not got[LENS[li] == 0].any()


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("batch,cap", [(1, 128), (7, 512), (64, 3008), (300, 640), (2, 40000)])
def test_f32_plan_needs_no_more_workspace(shape, batch, cap):
    """What fitted a workspace (or the 32 MiB scratch) sized for the vector kernel still fits; a forced MFMA plan
    stays refused."""
    d = B.dims_for(workload(shape, np.array([cap]), True))
    pages = -(-cap // d.page_size)
    auto = B.decode_workspace_size(d, batch, pages)
    assert 0 < auto <= B.decode_workspace_size(d, batch, pages, B.make_plan(B.PATH_VALU))
    assert B.decode_workspace_size(d, batch, pages, B.make_plan(B.PATH_MFMA)) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dt,n", [("fp32", 300), ("fp32", 700), ("bf16", 300), ("bf16", 700)])
def test_tokens_of_infinitely_low_score(gpu, dt, n):
    """A block of tokens whose scores overflow to -inf weighs nothing, also where it fills whole units of a wave (and
    not a whole 32-token tile of the vector kernel, which is the reference here)."""
    import torch
    wl = workload((dt, 4, 32, 32, 32, 8), np.array([n]), paged=False)
    dd = B.stage_decode(W.generate(wl, seq_lens=np.array([n])))
    dd.q[..., -8:] = dd.q[..., -8:].abs() + 2
    dd.cache[:16, -8:] = -3e38   # the first unit of the first wave
    dd.cache[80:96, -8:] = -3e38  # a later one
    say(f"decode -inf scores {dt} n={n}")
    got = B.run_decode(dd).double()
    ref_out = torch.empty_like(dd.out)
    dd.out = ref_out
    ref = B.run_decode(dd, plan=B.make_plan(B.PATH_VALU)).double()
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all() and torch.isfinite(got).all()
    # fp32 sums in another order; bf16 outputs also round differently
    assert (got - ref).norm() <= (1e-5 if dt == "fp32" else 5e-3) * ref.norm()
