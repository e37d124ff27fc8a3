"""Tiles that only the passes of 128 rows and more take (32 x 32, 128 x 96, 128 x 160, gate and up rows eight by eight): a
sequence's step at batches whose passes take different tiles, bit for bit in every row, and the greedy choice from their logits."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from oracle import photon_oracle as po
from test_gpu_tiles import step_of_first
from util import TOL, nerr, require_gpu

pytestmark = pytest.mark.gpu

D, F, V = 832, 2112, 8016
# projections of a pass of `rows` rows: q/k/v, O, gate/up, down, vocabulary
TILES = {128: [(64, 32), (32, 32), (64, 32), (32, 32), (64, 64)],
         300: [(64, 64), (64, 32), (128, 32), (64, 32), (128, 96)],
         600: [(128, 64), (32, 32), (128, 48), (32, 32), (128, 160)],
         1030: [(128, 96), (64, 64), (128, 80), (64, 64), (128, 160)]}


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


def test_steps_agree_over_the_tiles_of_a_pass():
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32, PHOTON_CONTRACT_SWIGLU
    for rows, tiles in TILES.items():
        f32 = lambda N, K: ph.photon_contract_tile(rows, N, K, PHOTON_CONTRACT_F32)[:2]
        assert [f32(3 * D, D), f32(D, D), ph.photon_contract_tile(rows, F, D, PHOTON_CONTRACT_SWIGLU)[:2], f32(D, F), f32(V, D)] == tiles
    cfg = si.PhotonConfig(L=1, C=(2,), R=(1,), D=D, H=13, d_h=64, n_layers=2, d_ff=F, vocab=V, dtype="bf16")
    w = si.make_weights(cfg, 12)
    st, forced, which = repeating(cfg, max(TILES), 20, 64)
    logits, x_top, _, _ = check_rows_agree(cfg, w, st, forced, which, TILES)
    # 16 sequences of them against the oracle
    ost = po.state_to_f64(dict(k=st["k"][:, :16], v=st["v"][:, :16], seq_len=st["seq_len"][:16], x_top=st["x_top"][:16], carry=st["carry"][:, :16]))
    otr = po.decode_step(cfg, po.weights_to_f64(w), ost, forced_tokens=forced[:16])
    assert nerr(logits[:16], otr["logits"]) < TOL["bf16"] and nerr(x_top[:16], otr["x_top"]) < TOL["bf16"]


@pytest.mark.parametrize("Bt", [300, 600])               # logits by 128 x 96 and 128 x 160 tiles, the last one partly empty
def test_greedy_choice_from_wide_stretches(Bt):
    require_gpu()
    import paper_2512_20687_amd as ph
    cfg = si.PhotonConfig(L=2, C=(1, 1), R=(1, 1), D=D, H=13, d_h=64, n_layers=1, d_ff=64, vocab=V, dtype="bf16")
    w = si.make_weights(cfg, 5)
    w["W_lm"][V // 2:] = w["W_lm"][: V - V // 2]         # equal logits: the lower index wins
    st = si.make_decode_state(cfg, Bt, 4, 16, seed=2)
    model = ph.PhotonModel(cfg, w)
    state = ph.PhotonState(model, Bt, 16, k=st["k"], v=st["v"], seq_len=st["seq_len"], x_top=st["x_top"], carry=st["carry"])
    out = torch.full((Bt, 1), -1, dtype=torch.int32, device="cuda")
    logits = torch.full((Bt, 1, V), float("nan"), device="cuda")
    ph.photon_decode_step(model, state, out, trace={"logits": logits})
    torch.cuda.synchronize()
    index = torch.arange(V, device="cuda").expand_as(logits)
    first = torch.where(logits == logits.amax(-1, keepdim=True), index, V).amin(-1)
    assert torch.equal(out.long(), first) and int(out.max()) < V - V // 2


# Contractions of one to four K slabs, fewer than the tiles load ahead or no more, and their last row tiles partly empty (128 x 96 and
# 128 x 160 are not taken below three and four slabs).
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
])
def test_steps_agree_at_few_slabs(D, F, V, Bt, tiles):
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32, PHOTON_CONTRACT_SWIGLU
    tile = lambda N, K, output=PHOTON_CONTRACT_F32: ph.photon_contract_tile(Bt, N, K, output)[:2]
    taken = dict(qkv=tile(3 * D, D), down=tile(D, F), logits=tile(V, D), gate_up=tile(F, D, PHOTON_CONTRACT_SWIGLU))
    assert {k: taken[k] for k in tiles} == tiles
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=D, H=D // 64, d_h=64, n_layers=2, d_ff=F, vocab=V, dtype="bf16")
    st, forced, which = repeating(cfg, Bt, 4, 16)
    check_rows_agree(cfg, si.make_weights(cfg, 12, encoders=False), st, forced, which, (128, Bt))


def test_steps_agree_with_weights_touched_ahead():
    """A module of 160 MB, whose wide tiles have a wave that touches the weights ahead: 64 x 64 tiles of three row tiles and of nine (a band
    of eight and one by itself), 128 x 64 tiles of eight, the last ones partly empty; 128 rows take neither."""
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32
    D, F = 1344, 3200
    assert [ph.photon_contract_tile(r, D, K, PHOTON_CONTRACT_F32)[:2] for r, K in ((128, D), (520, D), (520, F), (1000, D), (1000, F))] == [
        (32, 32), (64, 64), (64, 64), (128, 64), (128, 64)]
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=D, H=21, d_h=64, n_layers=4, d_ff=F, vocab=1008, dtype="bf16")
    st, forced, which = repeating(cfg, 1000, 4, 16)
    check_rows_agree(cfg, si.make_weights(cfg, 12, encoders=False), st, forced, which, (128, 190, 520, 1000))
