"""The tiled bf16 contractions: tile edges through photon_chunker_project (Eq. 4) against an fp32 product of the same
bf16 inputs; splits over K and sums in pieces through decode steps against the oracle."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from util import TOL, dev, require_gpu

pytestmark = pytest.mark.gpu


# A row more and a row less than whole row tiles, a last column tile of 16 columns, one to five K slabs (which tile each of
# them takes is left to the time model; test_every_tile_kind names its tiles).
@pytest.mark.parametrize("rows,K,N", [(6144, 64, 2048), (6145, 128, 2048), (6143, 192, 2048), (49409, 64, 256), (6100, 320, 2064)])
def test_tiled_contraction_edges(rows, K, N):
    check_chunker(rows, K, N)


def check_chunker(rows, K, N):
    require_gpu()
    import paper_2512_20687_amd as ph
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    x = torch.randn((rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    b = torch.randn((N,), generator=g, device="cuda")
    out = torch.full((rows + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ph.photon_chunker_project(x, w, b, out[:rows], 1)
    torch.cuda.synchronize()
    assert bool(torch.isnan(out[rows]).all())                       # nothing is stored past the last row
    ref = x.float() @ w.float().t() + b
    # one rounding of the output to bf16 (2^-9 of its value) and fp32 sums of K products in two orders
    err = (out[:rows].float() - ref).abs()
    bound = ref.abs() * 2.0 ** -8 + 1e-5 * K ** 0.5
    assert bool((err <= bound).all()), float((err - bound).max())


# Every tile of the contraction at one, two and three K slabs, fewer and more than it loads ahead: a row more or less than whole
# row tiles, a last column tile of 16 columns, a tile count that is no multiple of the 8 XCDs.
# The narrow ones also at odd and even numbers of slabs above that, in grids of up to 256 tiles and of more (64 x 32: six or four slab buffers).
@pytest.mark.parametrize("tile,rows,K,N", [
    ((64, 32), 63, 64, 48), ((64, 32), 65, 128, 80), ((64, 32), 193, 192, 144), ((64, 32), 1, 704, 80), ((64, 32), 129, 768, 2000),
    ((64, 32), 77, 320, 4944), ((64, 32), 127, 384, 4944),
    ((64, 64), 9473, 64, 592), ((64, 64), 11777, 128, 208), ((64, 64), 9855, 192, 144),
    ((64, 64), 191, 704, 3216), ((64, 64), 255, 768, 3856), ((64, 64), 2369, 768, 336),
    ((128, 64), 62719, 64, 144), ((128, 64), 29697, 128, 144), ((128, 64), 19711, 192, 144),
    ((128, 128), 28927, 64, 1040), ((128, 128), 25855, 128, 528), ((128, 128), 23553, 192, 400),
    ((128, 256), 20481, 64, 4624), ((128, 256), 7425, 128, 6416), ((128, 256), 14337, 192, 2064), ((128, 256), 641, 704, 8208),
    ((256, 256), 42495, 64, 2064), ((256, 256), 13313, 128, 3344), ((256, 256), 25599, 192, 1040), ((256, 256), 1537, 320, 7696),
])
def test_every_tile_kind(tile, rows, K, N):
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_CHUNKER
    assert ph.photon_contract_tile(rows, N, K, PHOTON_CONTRACT_CHUNKER) == (*tile, 1, False)
    assert -(-rows // tile[0]) * -(-N // tile[1]) % 8 != 0
    check_chunker(rows, K, N)


# 16 rows below to hundreds above the switch to the tiled contractions, at every level; a first sub-step that is above it
# while the others are below (12 sequences, two converter rows); split and unsplit K, attention-only blocks, padded heads,
# tile columns partly empty.
@pytest.mark.parametrize("kw,Bt", [
    (dict(), 5),                                                    # level 1: 20 rows
    (dict(D=1024, H=16, d_ff=2560, n_layers=1), 17),                # level 2: 17 rows, level 1: 68 (split K)
    (dict(R=(2, 2)), 12),                                           # level 2: 24 rows, then 12
    (dict(d_ff=0, R=(1, 2)), 18),
    (dict(D=832, H=16, d_h=52, d_ff=1024, R=(2, 1), n_layers=1), 33),
    (dict(D=448, H=8, d_h=56, d_ff=704, n_layers=1, L=3, C=(2, 3, 2), R=(1, 2, 1)), 40),
    (dict(n_layers=1), 65),
])
def test_decode_step_at_many_rows(kw, Bt):
    require_gpu()
    from test_gpu_decode_step import check_against_oracle
    base = dict(L=2, C=(4, 4), R=(1, 1), D=512, H=8, d_h=64, n_layers=2, d_ff=1280, vocab=1008, dtype="bf16")
    base.update(kw)
    cfg = si.PhotonConfig(**base)
    S, S_max = 40, 48
    st = si.make_decode_state(cfg, Bt, S, S_max, seed=3)
    errs, _, _ = check_against_oracle(cfg, si.make_weights(cfg, 12), st, Bt, S_max, si.make_tokens(cfg.vocab, Bt, cfg.meta_context, 7), TOL["bf16"])
    print(errs)


# Attention-only blocks whose first token sub-step has more than 16 rows and whose items are fewer: the last block's result
# comes in pieces, the whole one of which is the buffer the next rows enter through, and is joined for the few-row head.
@pytest.mark.parametrize("kw,Bt", [
    (dict(D=512, H=8, R=(2, 1)), 3),
    (dict(D=1024, H=16, R=(3, 2), n_layers=1), 4),
    (dict(D=256, H=4, R=(9, 1), C=(4, 2)), 2),
])
def test_attention_only_blocks_joined_for_a_few_row_head(kw, Bt):
    require_gpu()
    from test_gpu_decode_step import test_logits_when_the_items_are_not_requested as check
    check(dict(dict(L=2, C=(4, 4), d_ff=0, vocab=1008, dtype="bf16"), **kw), Bt)


# Greedy steps with enough rows that the vocabulary contraction leaves each row's best columns beside the logits: a narrow
# and a wide wave tile, a last stretch of 16 columns, equal logits (the vocabulary's second half repeats the first: the
# lower index wins), logits in the state's own buffer (no trace) as well.
@pytest.mark.parametrize("Bt,vocab", [(5, 1008), (17, 4000), (65, 8016), (256, 16000)])
def test_greedy_choice_at_many_rows(Bt, vocab):
    require_gpu()
    import paper_2512_20687_amd as ph
    cfg = si.PhotonConfig(L=2, C=(4, 4), R=(1, 1), D=256, H=4, d_h=64, n_layers=1, d_ff=640, vocab=vocab, dtype="bf16")
    w = si.make_weights(cfg, 5)
    w["W_lm"][vocab // 2:] = w["W_lm"][: vocab - vocab // 2]
    st = si.make_decode_state(cfg, Bt, 20, 32, seed=2)
    model = ph.PhotonModel(cfg, w)
    tokens = []
    for traced in (True, False):
        state = ph.PhotonState(model, Bt, 32, k=st["k"], v=st["v"], seq_len=st["seq_len"], x_top=st["x_top"], carry=st["carry"])
        out = torch.full((Bt, cfg.meta_context), -1, dtype=torch.int32, device="cuda")
        logits = torch.full((Bt, cfg.meta_context, vocab), float("nan"), device="cuda")
        ph.photon_decode_step(model, state, out, trace={"logits": logits} if traced else None)
        torch.cuda.synchronize()
        tokens.append(out)
        if traced:
            index = torch.arange(vocab, device="cuda").expand_as(logits)
            first = torch.where(logits == logits.amax(-1, keepdim=True), index, vocab).amin(-1)
            assert torch.equal(out.long(), first) and int(out.max()) < vocab - vocab // 2
    assert torch.equal(tokens[0], tokens[1])


def step_of_first(cfg, w, st, Bt, forced):
    """One step of the first Bt sequences of `st`: the state afterwards and the trace."""
    from test_gpu_decode_step import run_step
    part = dict(k=st["k"][:, :Bt], v=st["v"][:, :Bt], seq_len=st["seq_len"][:Bt], x_top=st["x_top"][:Bt], carry=st["carry"][:, :Bt])
    _, state, _, trace = run_step(cfg, w, part, Bt, st["k"].shape[3], forced[:Bt])
    return state, trace


# A sequence's step does not depend on how many others it is decoded with, as long as every level stays on the same side of
# 17 and of 128 rows (where rows are rounded, and where the order of the sums over the width changes): bit for bit, over
# different tiles and splits.  Widths with whole and half chunks of 128, more and fewer than 8 of them.
@pytest.mark.parametrize("kw,batches", [
    (dict(L=1, C=(4,), R=(1,), D=512, d_ff=1280), (17, 64, 127)),
    (dict(L=1, C=(3,), R=(1,), D=1344, H=21, d_ff=2560), (17, 65, 120)),
    (dict(L=1, C=(2,), R=(1,), D=320, H=5, d_ff=704), (128, 300, 1100)),
    (dict(L=2, C=(4, 4), R=(1, 1), D=1024, H=16, d_ff=2560), (128, 257)),
    (dict(L=2, C=(4, 4), R=(1, 1), D=1024, H=16, d_ff=2560), (5, 16)),
])
def test_a_sequence_s_step_does_not_depend_on_the_batch(kw, batches):
    require_gpu()
    base = dict(H=8, d_h=64, n_layers=2, vocab=1008, dtype="bf16")
    base.update(kw)
    cfg = si.PhotonConfig(**base)
    w, st = si.make_weights(cfg, 12), si.make_decode_state(cfg, batches[-1], 20, 64, seed=3)
    forced = si.make_tokens(cfg.vocab, batches[-1], cfg.meta_context, 7)
    ref = None
    for Bt in batches:
        state, trace = step_of_first(cfg, w, st, Bt, forced)
        got = [trace["logits"][:batches[0]], state.x_top[:batches[0]], state.k[:, :batches[0]], state.v[:, :batches[0]]]
        if ref is None:
            ref = got
        for a, b in zip(ref, got):
            assert torch.equal(a, b), Bt


# The order of a contraction's sum: below 128 rows that of the few-row kernel on the same bf16 rows, from 128 on that of the
# chunker entry point (whose result is rounded to bf16): the top chunker of a step against both, bit for bit.
@pytest.mark.parametrize("Bt,C,D,tile", [
    (17, 4, 512, (64, 32, 8)), (64, 3, 448, (64, 32, 8)), (100, 2, 64, (64, 32, 1)), (127, 8, 1024, (64, 64, 8)), (127, 1, 1024, (64, 32, 4)),
    (127, 1, 2048, (64, 64, 4)), (128, 4, 512, (32, 32, 1)), (333, 3, 448, (32, 32, 1)), (333, 2, 1024, (64, 32, 1)), (1000, 3, 448, (64, 32, 1)),
])
def test_order_of_a_contraction_s_sum(Bt, C, D, tile):
    require_gpu()
    import paper_2512_20687_amd as ph
    from paper_2512_20687_amd.binding import PHOTON_CONTRACT_F32
    assert ph.photon_contract_tile(Bt, D, C * D, PHOTON_CONTRACT_F32) == (*tile, False)
    cfg = si.PhotonConfig(L=1, C=(C,), R=(1,), D=D, H=D // 64, d_h=64, n_layers=1, d_ff=64, vocab=1008, dtype="bf16")
    w, st = si.make_weights(cfg, 2), si.make_decode_state(cfg, Bt, 10, 64, seed=1)
    _, trace = step_of_first(cfg, w, st, Bt, si.make_tokens(cfg.vocab, Bt, C, 7))
    rows = trace["new_units"][0].reshape(Bt, C * D).to(torch.bfloat16)
    W, b = dev(w["enc"][0]["chunker"]["w"], "bf16"), dev(w["enc"][0]["chunker"]["b"])
    if Bt < 128:
        out = torch.zeros((Bt, D), device="cuda")
        ph.photon_linear(rows, W, out, bias=b)
        assert torch.equal(out, trace["a_hat"])
    else:
        out = torch.zeros((Bt, D), dtype=torch.bfloat16, device="cuda")
        ph.photon_chunker_project(rows.reshape(Bt * C, D), W, b, out, C)
        assert torch.equal(out, trace["a_hat"].to(torch.bfloat16))


# SwiGLU of many rows against the few-row kernel's on the same bf16 rows.  Identity converter, no attention, a down projection
# that adds up every D-th hidden column: the new unit is the norm of (row of +-1) + those sums.  One hidden value rounded
# to the other side (2^-8 of it) would show at 1e-4; fp32 sums and the norm leave 1e-6.
@pytest.mark.parametrize("Bt", [40, 127])
def test_swiglu_of_many_rows_is_that_of_the_few_row_kernel(Bt):
    require_gpu()
    import paper_2512_20687_amd as ph
    D, F = 1024, 4096
    cfg = si.PhotonConfig(L=1, C=(1,), R=(1,), D=D, H=16, d_h=64, n_layers=1, d_ff=F, vocab=1008, dtype="bf16")
    w, st = si.make_weights(cfg, 6), si.make_decode_state(cfg, Bt, 4, 16, seed=5)
    dec, eye = w["dec"][0], np.eye(D, dtype=np.float32)
    dec["converter"]["w"], dec["converter"]["b"] = eye, np.zeros((D,), np.float32)
    layer = dec["module"]["layers"][0]
    layer["wv"] = np.zeros((D, D), np.float32)
    layer["g2"], dec["module"]["g_final"] = np.ones((D,), np.float32), np.ones((D,), np.float32)
    layer["wd"] = np.tile(eye, (1, F // D))
    st["x_top"] = np.where(st["x_top"] < 0, -1.0, 1.0).astype(np.float32)
    _, trace = step_of_first(cfg, w, st, Bt, si.make_tokens(cfg.vocab, Bt, 1, 7))
    rows = dev(st["x_top"])
    wgu, hidden = dev(np.concatenate([layer["wg"], layer["wu"]]), "bf16"), torch.zeros((Bt, F), dtype=torch.bfloat16, device="cuda")
    for m in range(0, Bt, 16):
        ph.photon_linear(rows[m:m + 16].to(torch.bfloat16), wgu, hidden[m:m + 16], epilogue=2)
    ref = rows.double() + hidden.double().reshape(Bt, F // D, D).sum(1)
    ref = ref / (ref.pow(2).mean(1, keepdim=True) + cfg.rms_eps).sqrt()
    err = (trace["new_units"][0].reshape(Bt, D).double() - ref).abs().max()
    assert float(err) <= 1e-5, float(err)
