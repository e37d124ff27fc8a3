"""Tiles that only the passes of 128 rows and more take (32 x 32, 128 x 96, 128 x 160, gate and up rows eight by eight): a
sequence's step at batches whose passes take different tiles, bit for bit, and the greedy choice from their logits."""
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


def test_steps_agree_over_the_tiles_of_a_pass():
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32, PHOTON_CONTRACT_SWIGLU
    for rows, tiles in TILES.items():
        f32 = lambda N, K: ph.photon_contract_tile(rows, N, K, PHOTON_CONTRACT_F32)[:2]
        assert [f32(3 * D, D), f32(D, D), ph.photon_contract_tile(rows, F, D, PHOTON_CONTRACT_SWIGLU)[:2], f32(D, F), f32(V, D)] == tiles
    cfg = si.PhotonConfig(L=1, C=(2,), R=(1,), D=D, H=13, d_h=64, n_layers=2, d_ff=F, vocab=V, dtype="bf16")
    most = max(TILES)
    w, st = si.make_weights(cfg, 12), si.make_decode_state(cfg, most, 20, 64, seed=3)
    forced = si.make_tokens(cfg.vocab, most, cfg.meta_context, 7)
    ref = None
    for Bt in TILES:
        state, trace = step_of_first(cfg, w, st, Bt, forced)
        got = [trace["logits"][:128], state.x_top[:128], state.k[:, :128], state.v[:, :128]]
        if ref is None:
            # 16 sequences of them against the oracle
            ost = po.state_to_f64(dict(k=st["k"][:, :16], v=st["v"][:, :16], seq_len=st["seq_len"][:16], x_top=st["x_top"][:16], carry=st["carry"][:, :16]))
            otr = po.decode_step(cfg, po.weights_to_f64(w), ost, forced_tokens=forced[:16])
            assert nerr(got[0][:16], otr["logits"]) < TOL["bf16"] and nerr(got[1][:16], otr["x_top"]) < TOL["bf16"]
            ref = got
        for a, b in zip(ref, got):
            assert torch.equal(a, b), Bt


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


def test_steps_agree_with_weights_touched_ahead():
    """A module of 160 MB, whose wide tiles have a wave that touches the weights ahead: 64 x 64 tiles of nine row tiles (a band of
    eight and one by itself), 128 x 64 tiles of eight, the last ones partly empty; 128 rows take neither."""
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32
    D, F = 1344, 3200
    assert [ph.photon_contract_tile(r, D, K, PHOTON_CONTRACT_F32)[:2] for r, K in ((128, D), (520, D), (520, F), (1000, D), (1000, F))] == [
        (32, 32), (64, 64), (64, 64), (128, 64), (128, 64)]
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=D, H=21, d_h=64, n_layers=4, d_ff=F, vocab=1008, dtype="bf16")
    w, st = si.make_weights(cfg, 12, encoders=False), si.make_decode_state(cfg, 1000, 4, 16, seed=3)
    forced = si.make_tokens(cfg.vocab, 1000, cfg.meta_context, 7)
    ref = None
    for Bt in (128, 520, 1000):
        state, trace = step_of_first(cfg, w, st, Bt, forced)
        got = [trace["logits"][:128], state.x_top[:128], state.k[:, :128], state.v[:, :128]]
        ref = ref or got
        for a, b in zip(ref, got):
            assert torch.equal(a, b), Bt
