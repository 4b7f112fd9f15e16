"""Projections on 128 x 128 tiles (few 256 x 256 tiles): row counts around the
tile, a last column tile of 64, one K panel up to more than the ring holds,
prefix lengths that leave value blocks unaligned, plain and split operands,
against the oracle at the bar of the fp16-operand path; both weight storages
must agree bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2601_01513_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d, hq, ff", [(64, 1, 64), (320, 2, 448)])
@pytest.mark.parametrize("prefix, lens", [(127, [30, 9]), (128, [64, 64]), (129, [33, 64]),
                                          (300, [50, 40])])
def test_small_tiles(d, hq, ff, prefix, lens):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name=f"small tiles d{d}", n_layers=2, d_model=d, n_heads=hq, n_kv_heads=1, head_dim=128,
        d_ff=ff, vocab=512, rope_base=1e6, dtype=W.BF16, n_prefix=prefix, n_visual=16, n_cands=2,
        cand_len=64)
    wl = W.make_workload(cfg, prefix, device="cuda")
    for m in range(2):
        wl.cand_ids[m, lens[m]:] = 0
    lens = np.asarray(lens, dtype=np.int32)
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    ref, _, _ = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                           W.to_host_f32(wl.visual), wl.prefix_ids, wl.cand_ids,
                                           lens)
    for split in ((0, 0), (2, 1)):
        out = []
        for storage in ("f16", "bf16"):
            v = Verifier(cfg, wl.weights, device="cuda", gemm_weights=storage,
                         split_layers=split[0], split_mlp_layers=split[1])
            out.append(v.verify(wl.visual, ids, cids, lens)[0].cpu().numpy())
            v.prefill(wl.visual, ids)
            out.append(v.score(cids, lens)[0].cpu().numpy())
        np.testing.assert_array_equal(out[0], out[2])
        np.testing.assert_array_equal(out[1], out[3])
        assert max(np.abs(o - ref).max() for o in out) <= 2e-2, split
