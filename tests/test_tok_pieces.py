"""Pieces of the d_c 128 decode's balanced schedule, cut on the host by the device's own arithmetic, and workspaces."""
import pytest

TOKEN_LIST = 4096  # tokens a work-group of the split kernel can list


@pytest.mark.parametrize("heads", [16, 32, 48, 64, 96, 128])
def test_pieces_fit_the_token_list(tok_pieces, heads):
    """Over every batch and capacity with a balanced schedule: no piece beyond the token list, no more pieces than
    partial rows, every token in one piece (the program fails otherwise)."""
    plans, cuts, longest = tok_pieces("sweep", heads)[0]
    assert plans > 0 and cuts == 7 * plans and longest <= TOKEN_LIST


def test_piece_counts_are_quotients(tok_pieces):
    """The float piece count equals the integer one for every piece size, around every multiple of it."""
    assert tok_pieces("quotients") == [(0,)]


@pytest.mark.parametrize("batch,length", [(40, 25000), (60, 20000), (64, 20000), (62, 28000), (128, 10000),
                                          (48, 24000), (40, 28672)])
def test_long_batches(tok_pieces, batch, length):
    """Where an even cut into one piece per compute unit would be longer than the list."""
    balanced, pieces = tok_pieces("plan", 16, batch, length)[0][:2]
    assert balanced and pieces == 512
    cut = tok_pieces("cut", 16, batch, length, text=f"{length} " * batch)
    assert len(cut) <= pieces and max(t for _, _, t in cut) <= TOKEN_LIST
    assert sum(t for _, _, t in cut) == batch * length


@pytest.mark.parametrize("batch,cap,v_dim,split", [
    (1, 64, 128, 64), (16, 1024, 128, 64), (1, 32768, 128, 256),   # one unit per wave, at most 128 partials
    (2, 1856, 128, 64), (4, 4096, 128, 128), (3, 2080, 128, 96),   # up to 4 sequences of 4096: 32 splits at most
    (4, 4128, 128, 96), (5, 4096, 128, 96), (1, 8192, 128, 64),    # beyond: as many as fill the chip
    (12, 2048, 128, 128), (14, 2048, 128, 128),                    # 16 splits where 64 to 96 tokens are too many items
    (20, 600, 128, 96), (24, 1500, 128, 192), (32, 1100, 128, 160),  # 8 splits
    (20, 1600, 128, 256), (28, 2048, 128, 256), (48, 1000, 128, 256),
    (1, 1024, 64, 64), (4, 2048, 64, 128), (1, 4096, 64, 256), (1, 32768, 64, 256),  # the general merge: few partials
])
def test_automatic_splits(tok_pieces, batch, cap, v_dim, split):
    balanced, _, got, _ = tok_pieces("plan", 16, batch, cap, v_dim)[0]
    assert not balanced and got == split


@pytest.mark.parametrize("layer", [(16, 128, 128, 128, 64, 1), (32, 128, 128, 128, 64, 1), (16, 128, 128, 320, 64, 1),
                                   (12, 64, 64, 64, 64, 1), (12, 64, 64, 256, 64, 1), (4, 32, 32, 32, 0, 0),
                                   (128, 128, 128, 512, 64, 1)], ids=str)
def test_a_workspace_serves_smaller_batches(tok_pieces, layer):
    """A workspace sized once, at a server's largest batch, holds every smaller batch whose plan of whole splits of 256
    tokens (or the vector kernel's) it holds: balanced pieces and short splits give way where they do not fit."""
    for batch in (8, 64, 128, 256, 384, 512):
        for cap in (512, 1024, 2048, 4096, 32768):
            whole, held, _ = tok_pieces("server", *layer, batch, cap)[0]
            assert whole > 0 and held == whole, (batch, cap)
