"""Precise attention on blocks of four and of eight waves: prefixes of 154 and
176 query tiles (the line lies at 176), candidates and draft prompts whose
four-wave blocks are one round of the CUs and more (120 and 140 rows: 242 and
484 blocks), against the oracle at the bar of the fp16-operand path."""
import numpy as np
import pytest

import oracle
from paper_2601_01513_amd import workload as W
from test_gpu_drafting import check_draft, make_verifier, run_draft, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix", [1792, 2048])
@pytest.mark.parametrize("lens", [[60, 60], [70, 70]])
def test_both_block_shapes(prefix, lens):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = W.VerifierConfig(
        name=f"precise blocks P{prefix} {lens}", n_layers=2, d_model=128, n_heads=22,
        n_kv_heads=22, head_dim=128, d_ff=128, vocab=512, rope_base=1e6, dtype=W.BF16,
        n_prefix=prefix, n_visual=0, n_cands=2, cand_len=70)
    wl = W.make_workload(cfg, prefix + lens[0], device="cuda")
    for m in range(2):
        wl.cand_ids[m, lens[m]:] = 0
    lens = np.asarray(lens, dtype=np.int32)
    v = make_verifier(wl, max_new=2, split_layers=2)
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    got = v.score(cids, lens)[0].cpu().numpy()
    ref, _, _ = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                           W.to_host_f32(wl.visual), wl.prefix_ids,
                                           wl.cand_ids, lens)
    assert np.abs(got - ref).max() <= 2e-2
    toks = run_draft(v, wl.cand_ids, lens, 2)
    check_draft(cfg, toks, run_oracle(wl, wl.cand_ids, lens, toks))


def test_block_shape_does_not_show():
    """The same candidate beside a second one of 60 tokens (120 rows: blocks of
    four waves) and of 80 (140 rows: eight): 11 key chunks either way, of the same
    bounds for its rows, and so the same log-probs bit for bit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name="precise blocks, one candidate twice", n_layers=2, d_model=128, n_heads=22,
        n_kv_heads=22, head_dim=128, d_ff=128, vocab=512, rope_base=1e6, dtype=W.BF16,
        n_prefix=1792, n_visual=0, n_cands=2, cand_len=80)
    wl = W.make_workload(cfg, 7, device="cuda")
    v = Verifier(cfg, wl.weights, device="cuda", split_layers=2)
    v.prefill(None, torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda"))
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    four = v.score(cids, [60, 60])[0].cpu().numpy()
    eight = v.score(cids, [60, 80])[0].cpu().numpy()
    np.testing.assert_array_equal(four[0, :60], eight[0, :60])
    np.testing.assert_array_equal(four[1, :60], eight[1, :60])
