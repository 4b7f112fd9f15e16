"""fp32 contexts against the oracle where their kernels can go wrong: widths
that are no multiple of the 16-wide pieces (loads by element), odd head
dimensions, one-row calls, both tile sizes of the projections, partial last
tiles everywhere, and non-finite rows that other candidates must not see.

Tolerance: 1e-4 per token, the bar of the fp32 path (float32 sums of at most
2112 terms of unit-scale products against float64: measured below 3e-6)."""
import numpy as np
import pytest

import oracle
from paper_2601_01513_amd import workload as W
from test_gpu_drafting import check_draft, run_draft, run_oracle

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _cfg(d, hq, hkv, hd, ff, vocab, p, pv, m, c):
    return W.VerifierConfig(
        name=f"fp32 d{d} {hq}/{hkv}x{hd} F{ff} V{vocab} P{p} M{m}x{c}", n_layers=2, d_model=d,
        n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=ff, vocab=vocab, rope_base=10000.0,
        dtype=W.F32, n_prefix=p, n_visual=pv, n_cands=m, cand_len=c)


CASES = [
    _cfg(100, 3, 3, 36, 70, 333, 1, 0, 1, 1),          # by element; one prefix row
    _cfg(72, 2, 1, 6, 50, 65, 18, 18, 3, 5),           # head dim not a multiple of 4
    _cfg(256, 4, 2, 64, 704, 1000, 33, 7, 3, 17),      # one row past a tile
    _cfg(96, 4, 1, 128, 112, 257, 65, 1, 2, 33),       # 8 pieces of the head dim
    _cfg(128, 2, 2, 200, 144, 500, 100, 50, 4, 20),    # 13 of 16 pieces
    _cfg(64, 4, 4, 16, 2112, 33000, 500, 100, 5, 14),  # 32-row tiles (FFN, LM head)
]


def _inputs(cfg, seed):
    torch = _torch()
    wl = W.make_workload(cfg, seed, device="cuda")
    lens = np.asarray([cfg.cand_len - (m * cfg.cand_len) // (cfg.n_cands + 1)
                       for m in range(cfg.n_cands)], dtype=np.int32)
    for m in range(cfg.n_cands):
        wl.cand_ids[m, lens[m]:] = 0
    wl.cand_len = lens
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda") if cfg.n_text else None
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    return wl, wl.visual if cfg.n_visual else None, ids, cids


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_f32_passes(cfg):
    torch = _torch()
    from paper_2601_01513_amd.binding import Verifier
    wl, vis, ids, cids = _inputs(cfg, 1)
    v = Verifier(cfg, wl.weights, device="cuda", max_new=2)
    ref, _, am = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                            W.to_host_f32(wl.visual), wl.prefix_ids, wl.cand_ids,
                                            wl.cand_len)
    one = v.verify(vis, ids, cids, wl.cand_len)
    v.prefill(vis, ids)
    two = v.score(cids, wl.cand_len)
    tok = run_draft(v, wl.cand_ids, wl.cand_len, 2)
    for out in (one, two):
        assert np.abs(out[0].cpu().numpy() - ref).max() <= 1e-4
        assert int(out[2].cpu()[0]) == am
    # Every greedy token is the oracle's, or within 2e-4 of its largest logit.
    check_draft(cfg, tok, run_oracle(wl, wl.cand_ids, wl.cand_len, tok))


@pytest.mark.parametrize("cfg", [CASES[0], CASES[1], CASES[4]], ids=lambda c: c.name)
def test_f32_greedy_token_in_the_last_partial_chunk(cfg):
    """The head's rows of the greedy token and of the last vocabulary entry
    trade places: the token is the last entry then, from a partial 64-entry
    chunk. With both rows equal it is the lower of the two."""
    torch = _torch()
    from paper_2601_01513_amd.binding import Verifier
    assert cfg.vocab % 64
    wl, vis, ids, _ = _inputs(cfg, 1)
    last = cfg.vocab - 1

    def first_token():
        v = Verifier(cfg, wl.weights, device="cuda", max_new=1)
        v.prefill(vis, ids)
        return int(run_draft(v, wl.cand_ids, wl.cand_len, 1)[0, 0])

    t = first_token()
    assert t != last
    head = wl.weights["lm_head"]
    head[[t, last]] = head[[last, t]].clone()
    assert first_token() == last
    head[t] = head[last]
    assert first_token() == t


def test_f32_candidates_do_not_see_each_others_nan():
    """Candidate 1 reads an embedding row of NaN; candidates 0 and 2, in the
    same row and key tiles, keep their log-probs, and candidate 1 keeps those
    of its earlier tokens. A key tile with a NaN adds its keys in another order:
    32 terms p v with sum p <= 1 and |v| of order 1 differ by at most
    32 eps = 2e-6 per attention output, below 1e-5 in a log-prob after two
    layers."""
    torch = _torch()
    from paper_2601_01513_amd.binding import Verifier
    cfg = _cfg(64, 2, 2, 32, 96, 200, 20, 4, 3, 6)
    wl, vis, ids, cids = _inputs(cfg, 2)
    wl.weights["embed"][7] = float("nan")
    cids[cids == 7] = 8
    if ids is not None:
        ids[ids == 7] = 8
    v = Verifier(cfg, wl.weights, device="cuda")
    lens = [6, 6, 6]
    clean = v.verify(vis, ids, cids, lens)[0].cpu().numpy()
    cids[1, 3] = 7
    got = v.verify(vis, ids, cids, lens)[0].cpu().numpy()
    np.testing.assert_allclose(got[[0, 2]], clean[[0, 2]], rtol=0, atol=1e-5)
    np.testing.assert_allclose(got[1, :3], clean[1, :3], rtol=0, atol=1e-5)
    assert np.isnan(got[1, 4:]).all()


def test_f32_head_past_one_launch():
    """131072 scored rows of a 140000-entry vocabulary: 9 million blocks of the
    LM head, more than one launch takes. A candidate's log-probs do not depend
    on how many others are scored with it."""
    torch = _torch()
    import dataclasses
    from paper_2601_01513_amd.binding import Verifier
    cfg = _cfg(32, 2, 2, 16, 32, 140000, 8, 0, 256, 512)
    small = dataclasses.replace(cfg, n_cands=2)
    wl = W.make_workload(small, 3, device="cuda")
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    few = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    few[:, -1] = cfg.vocab - 1  # a target of the last column tile
    many = few[torch.arange(256, device="cuda") % 2].contiguous()
    v = Verifier(small, wl.weights, device="cuda")
    v.prefill(None, ids)
    ref = v.score(few, [512] * 2)[0]
    v = Verifier(cfg, wl.weights, device="cuda")
    v.prefill(None, ids)
    got = v.score(many, [512] * 256)[0]
    assert torch.isfinite(ref).all()
    assert (got.view(128, 2, 512) - ref).abs().max().item() <= 1e-5
