"""Every row of the passes of 128 rows and more, bit for bit (test_gpu_pass_tiles.py compares their first 128): the same tiles, those of
contractions of a few K slabs, up to 4096 rows and beyond, and those with a wave that touches the weights ahead."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from test_gpu_pass_tiles import D, F, TILES, V
from test_gpu_tiles import step_of_first
from util import require_gpu

pytestmark = pytest.mark.gpu


def repeating(cfg, n, S, S_max, seed=3, period=127):
    """State and tokens of n sequences, sequence i equal to sequence i % period, which divides no tile: every row of a large pass
    has its value in a pass of 128 rows."""
    st, which = si.make_decode_state(cfg, period, S, S_max, seed=seed), np.arange(n) % period
    st = dict(k=st["k"][:, which], v=st["v"][:, which], seq_len=st["seq_len"][which], x_top=st["x_top"][which], carry=st["carry"][:, which])
    return st, si.make_tokens(cfg.vocab, period, cfg.meta_context, 7)[which], torch.from_numpy(which).cuda()


def check_rows_agree(cfg, w, st, forced, which, batches):
    """Logits, top state and cache of every sequence, bit for bit those of the 128-row pass."""
    ref = None
    for Bt in batches:
        state, trace = step_of_first(cfg, w, st, Bt, forced)
        got = [trace["logits"], state.x_top, state.k.transpose(0, 1), state.v.transpose(0, 1)]
        ref = ref or got
        for a, b in zip(ref, got):
            assert torch.equal(a[which[:Bt]], b), Bt
    return ref


def test_every_row_over_the_tiles_of_a_pass():
    require_gpu()
    cfg = si.PhotonConfig(L=1, C=(2,), R=(1,), D=D, H=13, d_h=64, n_layers=2, d_ff=F, vocab=V, dtype="bf16")
    st, forced, which = repeating(cfg, max(TILES), 20, 64)
    check_rows_agree(cfg, si.make_weights(cfg, 12), st, forced, which, TILES)


# Contractions of one to four K slabs, fewer than the tiles load ahead or no more, and their last row tiles partly empty (128 x 96 and
# 128 x 160 are not taken below three and four slabs).  The last three have more than 4096 rows, where up to three slabs go by the same
# tiles and longer contractions by others.
@pytest.mark.parametrize("D,F,V,Bt,tiles", [
    (64, 64, 1008, 333, dict(qkv=(32, 32), down=(32, 32))),
    (128, 128, 1008, 301, dict(qkv=(32, 32), down=(32, 32))),
    (128, 128, 7008, 3457, dict(logits=(128, 64))),
    (128, 192, 16016, 3081, dict(logits=(256, 256))),
    (192, 2688, 7008, 833, dict(logits=(128, 64))),
    (192, 2688, 1008, 3841, dict(gate_up=(128, 32))),
    (192, 7616, 1008, 1537, dict(gate_up=(256, 128))),
    (192, 2432, 4576, 533, dict(logits=(128, 96), gate_up=(128, 48))),
    (256, 5632, 11296, 333, dict(logits=(128, 160), gate_up=(128, 80))),
    (64, 64, 1008, 4097, dict(qkv=(32, 32), down=(32, 32), gate_up=(64, 16))),
    (192, 192, 1008, 4161, dict(qkv=(128, 64), down=(64, 64), logits=(128, 64))),
    (64, 640, 1008, 4500, dict(qkv=(32, 32), down=(64, 32), gate_up=(128, 32))),
])
def test_every_row_at_few_slabs(D, F, V, Bt, tiles):
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32, PHOTON_CONTRACT_SWIGLU
    tile = lambda N, K, output=PHOTON_CONTRACT_F32: ph.photon_contract_tile(Bt, N, K, output)[:2]
    taken = dict(qkv=tile(3 * D, D), down=tile(D, F), logits=tile(V, D), gate_up=tile(F, D, PHOTON_CONTRACT_SWIGLU))
    assert {k: taken[k] for k in tiles} == tiles
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=D, H=D // 64, d_h=64, n_layers=2, d_ff=F, vocab=V, dtype="bf16")
    st, forced, which = repeating(cfg, Bt, 4, 16)
    check_rows_agree(cfg, si.make_weights(cfg, 12, encoders=False), st, forced, which, (128, Bt))


def test_every_row_with_weights_touched_ahead():
    """A module of 160 MB: 64 x 64 tiles of three row tiles and of nine (a band of eight and one by itself), 128 x 64 tiles of eight, the
    last ones partly empty; 128 rows take neither."""
    require_gpu()
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=1344, H=21, d_h=64, n_layers=4, d_ff=3200, vocab=1008, dtype="bf16")
    st, forced, which = repeating(cfg, 1000, 4, 16)
    check_rows_agree(cfg, si.make_weights(cfg, 12, encoders=False), st, forced, which, (128, 190, 520, 1000))
