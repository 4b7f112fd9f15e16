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
