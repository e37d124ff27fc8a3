"""Small fp32 models: a decode level, and the chunker with the STEP behind it, as one launch each, against the oracle and against
the separate launches they replace."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from test_gpu_decode_step import check_against_oracle
from util import TOL, nerr, require_gpu

pytestmark = pytest.mark.gpu


def _profiled_launches(cfg, w, st, Bt, S_max, persistent):
    import paper_2512_20687_amd as ph
    ph.photon_set_persistent(persistent)
    try:
        model = ph.PhotonModel(cfg, w)
        state = ph.PhotonState(model, Bt, S_max, k=st["k"], v=st["v"], seq_len=st["seq_len"], x_top=st["x_top"], carry=st["carry"])
        logits = torch.empty((Bt, cfg.meta_context, cfg.vocab), device="cuda")
        toks = torch.empty((Bt, cfg.meta_context), dtype=torch.int32, device="cuda")
        ph.photon_profile_reset()
        ph.photon_profile_enable(True)
        ph.photon_decode_step(model, state, toks, trace={"logits": logits})
        torch.cuda.synchronize()
        ph.photon_profile_enable(False)
        n = sum(launches for launches, _ in ph.photon_profile_get().values())
        ph.photon_profile_reset()
        return state, toks, logits, n
    finally:
        ph.photon_set_persistent(True)
        ph.photon_profile_enable(False)


@pytest.mark.parametrize("kw,Bt,S0,S_max", [
    (dict(), 1, 16, 128),                                        # the tiny configuration
    (dict(D=16, H=1, d_h=16, d_ff=40, vocab=500), 2, 1, 5),      # narrower than a k step, one head, odd cache, one entry
    (dict(D=20, H=5, d_h=4, d_ff=4, vocab=1), 3, 5, 6),          # smallest heads, one column
    (dict(D=96, H=3, d_h=32, d_ff=240, vocab=1000), 8, 37, 40),  # heads that do not divide the waves, several k steps
    (dict(D=128, H=2, d_h=64, d_ff=320, R=(2, 2), C=(4, 3)), 2, 100, 131),
    (dict(D=128, H=1, d_h=128, d_ff=320, vocab=300), 2, 9, 64),  # widest head
    (dict(D=120, H=10, d_h=12, d_ff=0, n_layers=2), 3, 20, 33),  # more heads than waves, no feed-forward
    (dict(n_layers=8, d_ff=64), 1, 3, 7),                        # as many blocks as the arguments hold
    (dict(L=3, C=(2, 3, 2), R=(1, 2, 1), n_layers=2), 3, 9, 24),
    (dict(L=1, C=(4,), R=(2,)), 2, 9, 24),
    (dict(rope_theta=0.0, C=(2, 5)), 2, 9, 24),
    (dict(C=(16, 2)), 2, 9, 24),                                 # windows of 16 positions: every lane of the softmax
    (dict(C=(15, 2), R=(2, 1)), 2, 9, 24),
    (dict(D=16, H=4, d_h=4, d_ff=40, C=(15, 2), R=(2, 1)), 3, 9, 24),
    (dict(D=128, H=4, d_ff=320, n_layers=3, C=(16, 1)), 2, 9, 24),   # 62 of 64 KB of LDS
])
def test_small_step_against_oracle_and_separate_launches(kw, Bt, S0, S_max):
    require_gpu()
    base = dict(L=2, C=(4, 4), R=(1, 1), D=64, H=2, d_h=32, n_layers=1, d_ff=160, vocab=512, dtype="f32")
    base.update(kw)
    cfg = si.PhotonConfig(**base)
    w = si.make_weights(cfg, 21)
    st = si.make_decode_state(cfg, Bt, S0, S_max, seed=5)
    st["seq_len"] = np.array([max(1, S0 - 3 * b) for b in range(Bt)], np.int32)
    if cfg.vocab > 1:
        check_against_oracle(cfg, w, st, Bt, S_max, None, TOL["f32"])
    one, toks1, logits1, n1 = _profiled_launches(cfg, w, st, Bt, S_max, True)
    sep, toks0, logits0, n0 = _profiled_launches(cfg, w, st, Bt, S_max, False)
    assert n1 == 2 * cfg.L + 1 < n0, (n1, n0)                    # begin, levels, conditioning, chunker with STEP
    assert torch.equal(toks1, toks0)
    # the same fp32 sums in another order: a sum of 512 products collects about sqrt(512) roundings of 2^-24 (1.3e-6); four times that for
    # the maps in a row and the items fed back (measured: 5e-7 at most over 221 models)
    for a, b in ((logits1, logits0), (one.x_top, sep.x_top), (one.carry, sep.carry), (one.k, sep.k), (one.v, sep.v)):
        if a.numel():
            assert nerr(a, b.double().cpu().numpy()) < 5e-6


def test_small_step_full_cache():
    """A full cache: the new entry overwrites the last one, as with separate launches, and nothing is written behind it."""
    require_gpu()
    cfg = si.PhotonConfig(L=2, C=(4, 4), R=(1, 1), D=64, H=2, d_h=32, n_layers=2, d_ff=160, vocab=96, dtype="f32")
    w = si.make_weights(cfg, 3)
    S_max = 9
    st = si.make_decode_state(cfg, 2, 9, S_max, seed=5)
    st["seq_len"] = np.array([9, 8], np.int32)
    one, toks1, logits1, _ = _profiled_launches(cfg, w, st, 2, S_max, True)
    sep, toks0, logits0, _ = _profiled_launches(cfg, w, st, 2, S_max, False)
    assert torch.equal(one.seq_len, sep.seq_len) and torch.equal(one.status, sep.status) and int(one.status) == 1
    for a, b in ((logits1, logits0), (one.x_top, sep.x_top), (one.k, sep.k), (one.v, sep.v)):
        assert nerr(a, b.double().cpu().numpy()) < 5e-6


def _greedy(cfg, w, st, Bt, S_max, persistent):
    """Tokens and logits of a greedy step, with one launch a level or with separate launches."""
    state, toks, logits, n = _profiled_launches(cfg, w, st, Bt, S_max, persistent)
    assert (n == 2 * cfg.L + 1) == persistent
    return toks, logits


@pytest.mark.parametrize("vocab,bad", [
    (512, range(512)), (333, range(333)),                        # every logit a NaN
    (512, [0]), (512, [3, 4, 130]), (512, range(256, 512)), (512, [511]), (333, [0]), (333, [1, 64]), (333, range(64, 333)),
    (3000, [2048, 2999]), (3000, range(0, 3000, 7)), (3001, [1030]),
    (512, ()), (333, ()),                                        # none: equal logits alone
])
def test_token_choice_with_equal_logits_and_nan(vocab, bad):
    """The choice of the separate kernel: the lowest of equal columns, and the same token where logits are NaN (columns of
    W_lm that are; 0 where all are)."""
    require_gpu()
    cfg = si.PhotonConfig(L=2, C=(2, 2), R=(1, 1), D=64, H=2, d_h=32, n_layers=1, d_ff=160, vocab=vocab, dtype="f32")
    Bt = 3
    w, st = si.make_weights(cfg, 8), si.make_decode_state(cfg, Bt, 9, 16, seed=4)
    w["W_lm"][vocab // 2: vocab // 2 * 2] = w["W_lm"][: vocab // 2]   # values come twice
    w["W_lm"][list(bad)] = np.nan
    one, logits1 = _greedy(cfg, w, st, Bt, 16, True)
    sep, logits0 = _greedy(cfg, w, st, Bt, 16, False)
    assert torch.equal(one, sep), (one, sep)
    assert torch.equal(logits1.isnan(), logits0.isnan())
    if len(bad) == vocab:
        assert not bool(one.any())
    elif len(bad) == 0:
        index = torch.arange(vocab, device="cuda").expand_as(logits1)
        first = torch.where(logits1 == logits1.amax(-1, keepdim=True), index, vocab).amin(-1)
        assert torch.equal(one.long(), first)


@pytest.mark.parametrize("kw,Bt,S_max,level,step", [
    # a long vocabulary: 558 us with separate launches, 1264 with the level in one
    (dict(D=32, H=1, C=(8,), n_layers=4, d_ff=128, vocab=32000), 1, 64, False, True),
    (dict(D=16, H=1, d_h=16, C=(8,), n_layers=2, d_ff=40, vocab=32000), 2, 32, False, True),     # 353 and 881 us
    # few launches to save: 44 us separate, 61 with the level in one, 78 with STEP in one
    (dict(D=72, H=9, d_h=8, C=(1,), d_ff=288, vocab=4000), 1, 512, False, False),
    (dict(D=120, H=6, d_h=20, C=(2,), n_layers=3, d_ff=0, vocab=16000), 2, 512, False, False),   # STEP 139 and 181 us
    (dict(C=(4,)), 1, 128, True, True),
    # long caches: full, STEP 139 us separate, 210 in one
    (dict(D=8, H=1, d_h=8, C=(1,), n_layers=4, d_ff=32, vocab=100), 3, 4765, True, False),
    (dict(D=16, H=1, d_h=16, C=(2,), d_ff=64, vocab=500), 9, 2049, True, False),
    (dict(D=16, H=1, d_h=16, C=(2,), d_ff=64, vocab=500), 9, 2048, True, True),
])
def test_one_launch_only_where_it_is_faster(kw, Bt, S_max, level, step):
    require_gpu()
    import paper_2512_20687_amd as ph
    cfg = si.PhotonConfig(**dict(dict(L=1, R=(1,), D=64, H=2, d_h=32, n_layers=1, d_ff=160, vocab=512, dtype="f32"), **kw))
    w, st = si.make_weights(cfg, 21), si.make_decode_state(cfg, Bt, 9, S_max, seed=5)
    model = ph.PhotonModel(cfg, w)
    state = ph.PhotonState(model, Bt, S_max, k=st["k"], v=st["v"], seq_len=st["seq_len"], x_top=st["x_top"], carry=st["carry"])
    toks = torch.empty((Bt, cfg.meta_context), dtype=torch.int32, device="cuda")
    ph.photon_profile_reset()
    ph.photon_profile_enable(True)
    try:
        ph.photon_decode_step(model, state, toks)
        torch.cuda.synchronize()
    finally:
        ph.photon_profile_enable(False)
    classes = ph.photon_profile_get()
    ph.photon_profile_reset()
    assert ("local_attn_kernel" not in classes) == level and ("coarse_attn_kernel" not in classes) == step, classes
    assert classes.get("small_model_kernels", (0,))[0] == level + step, classes


@pytest.mark.parametrize("kw,Bt", [(dict(), 2), (dict(L=3, C=(2, 3, 2), R=(1, 2, 1), D=48, H=4, d_h=12, d_ff=124), 3), (dict(L=1, C=(4,), R=(1,)), 4)])
def test_small_steps_joined_pipelined_and_captured(kw, Bt):
    """Steps that leave their lower levels running beside the next one, and steps replayed from a graph, are the joined ones bit for bit
    (the same kernels in all three), with eager work and a synchronisation between the replays."""
    require_gpu()
    import paper_2512_20687_amd as ph
    cfg = si.PhotonConfig(**dict(dict(L=2, C=(4, 4), R=(1, 1), D=64, H=2, d_h=32, n_layers=2, d_ff=160, vocab=500, dtype="f32"), **kw))
    n_steps, S, S_max = 4, 9, 40
    w, st = si.make_weights(cfg, 31), si.make_decode_state(cfg, Bt, S, S_max, seed=6)
    model = ph.PhotonModel(cfg, w)
    names = ("k", "v", "seq_len", "x_top", "carry")
    res = {}
    for mode in ("joined", "pipelined", "graph"):
        state = ph.PhotonState(model, Bt, S_max, k=st["k"], v=st["v"], seq_len=st["seq_len"], x_top=st["x_top"], carry=st["carry"],
                               pipeline=mode != "joined" and cfg.L > 1)
        toks = torch.full((n_steps, Bt, cfg.meta_context), -1, dtype=torch.int32, device="cuda")
        logits = torch.zeros((n_steps, Bt, cfg.meta_context, cfg.vocab), device="cuda")
        keep = {n: getattr(state, n).clone() for n in names}

        def run():
            for i in range(n_steps):
                ph.photon_decode_step(model, state, toks[i], trace={"logits": logits[i]})
            ph.photon_decode_join(state)

        if mode != "graph":
            run()
        else:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                run()
            for _ in range(3):
                toks.fill_(-1)
                logits.zero_()
                for n, t in keep.items():
                    getattr(state, n).copy_(t)
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(toks, res["joined"][0]) and torch.equal(logits, res["joined"][1])
        torch.cuda.synchronize()
        assert int(state.status.item()) == 0 and int(state.c_state.lower_levels_pending) == 0
        res[mode] = (toks, logits, *(getattr(state, n) for n in names))
    for mode in ("pipelined", "graph"):
        for a, b in zip(res["joined"], res[mode]):
            assert torch.equal(a, b), mode


@pytest.mark.parametrize("C,Bt", [((2, 1), 256), ((2, 4), 64), ((1, 2), 128)])
def test_small_step_at_the_most_chunks(C, Bt):
    """256 chunks (sequences) are one launch, one sequence more is not: the same results for those that both decode."""
    require_gpu()
    cfg = si.PhotonConfig(L=2, C=C, R=(1, 2), D=32, H=2, d_h=16, n_layers=2, d_ff=80, vocab=300, dtype="f32")
    assert Bt * C[1] == 256
    w, st = si.make_weights(cfg, 11), si.make_decode_state(cfg, Bt + 1, 5, 12, seed=9)
    part = lambda n: dict(k=st["k"][:, :n], v=st["v"][:, :n], seq_len=st["seq_len"][:n], x_top=st["x_top"][:n], carry=st["carry"][:, :n])
    one, toks1, logits1, n1 = _profiled_launches(cfg, w, part(Bt), Bt, 12, True)
    more, toks2, logits2, n2 = _profiled_launches(cfg, w, part(Bt + 1), Bt + 1, 12, True)
    sep, toks0, logits0, n0 = _profiled_launches(cfg, w, part(Bt + 1), Bt + 1, 12, False)
    assert n1 == 5 < n2 <= n0 and (n2 == n0) == (Bt == 256), (n1, n2, n0)
    for toks, logits, state in ((toks1, logits1, one), (toks2[:Bt], logits2[:Bt], more)):
        assert torch.equal(toks, toks0[:Bt])
        assert nerr(logits, logits0[:Bt].double().cpu().numpy()) < 5e-6
        assert nerr(state.x_top[:Bt], sep.x_top[:Bt].double().cpu().numpy()) < 5e-6


def test_small_step_with_a_long_cache():
    """A cache whose entries a workgroup takes longer for than the launches: the levels stay one launch each, STEP does not."""
    require_gpu()
    cfg = si.PhotonConfig(L=2, C=(2, 2), R=(1, 1), D=64, H=4, d_h=16, n_layers=2, d_ff=160, vocab=300, dtype="f32")
    launches = []
    for S_max in (512, 8192):
        w, st = si.make_weights(cfg, 11), si.make_decode_state(cfg, 2, S_max - 3, S_max, seed=9)
        one, toks1, logits1, n1 = _profiled_launches(cfg, w, st, 2, S_max, True)
        sep, toks0, logits0, n0 = _profiled_launches(cfg, w, st, 2, S_max, False)
        launches.append((n1, n0))
        assert torch.equal(toks1, toks0)
        for a, b in ((logits1, logits0), (one.x_top, sep.x_top), (one.k, sep.k), (one.v, sep.v)):
            assert nerr(a, b.double().cpu().numpy()) < 5e-6
    assert launches[0][0] == 5 and 5 < launches[1][0] < launches[1][1], launches


@pytest.mark.parametrize("S_max,one_launch", [(430, True), (431, False)])
def test_small_step_at_the_most_lds(S_max, one_launch):
    """Scores of 32 heads over the longest cache that fits the 64 KB of LDS (to 96 bytes), and over one entry more: separate launches."""
    require_gpu()
    cfg = si.PhotonConfig(L=1, C=(4,), R=(1,), D=128, H=32, d_h=4, n_layers=1, d_ff=512, vocab=100, dtype="f32")
    Bt = 96
    w, st = si.make_weights(cfg, 17), si.make_decode_state(cfg, Bt, S_max - 1, S_max, seed=2)
    one, toks1, logits1, n1 = _profiled_launches(cfg, w, st, Bt, S_max, True)
    sep, toks0, logits0, n0 = _profiled_launches(cfg, w, st, Bt, S_max, False)
    assert (n1 == 3) == one_launch and n1 < n0, (n1, n0)
    assert torch.equal(toks1, toks0)
    for a, b in ((logits1, logits0), (one.x_top, sep.x_top), (one.k, sep.k), (one.v, sep.v)):
        assert nerr(a, b.double().cpu().numpy()) < 5e-6
